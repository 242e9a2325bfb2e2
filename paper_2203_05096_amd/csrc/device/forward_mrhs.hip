// The product for blocks of right-hand sides by the window walk: one matrix and
// batched launches.
#include "window_mrhs.hpp"

namespace csrk {
namespace dev {

namespace {

template <typename VT, int RL, int VX, bool KEEP>
__global__ void __launch_bounds__(1024) k_spmv_win_mrhs(WinArrays win, int32_t stride, const VT *__restrict__ vals,
                                                        const typename Store<VT>::X *__restrict__ x,
                                                        typename Store<VT>::X *__restrict__ y, int64_t nnz, int nrhs,
                                                        XcdSplit split) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x / kWave);
    const int nw = blockDim.x / kWave;
    unsigned char *lds = smem + size_t(wave) * win_mrhs_lds<VT>(win.cap, false);
    const int32_t t = ssr_of_block(split, int32_t(blockIdx.x));
    if (t < 0) return;
    for (int32_t w = wave; w < stride; w += nw) {
        const WinRec rec = win.rec[int64_t(t) * stride + w];
        if (rec.rows() == 0) break;
        win_forward_mrhs<VT, RL, VX>(rec, win.rend, win.cols, vals, x, y, nnz, nrhs, win.cap,
                                     std::bool_constant<KEEP>{}, lds, lane);
    }
}

// Items and XCD order as in k_batch_forward.
template <typename VT, int RL, int VX>
__global__ void __launch_bounds__(1024) k_batch_forward_win_mrhs(const MatDesc *__restrict__ descs,
                                                                 const int2 *__restrict__ items,
                                                                 const WinRec *__restrict__ wrec, int32_t stride,
                                                                 int32_t nitems, int nrhs, int cap) {
    using X = typename Store<VT>::X;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x / kWave);
    const int nw = blockDim.x / kWave;
    unsigned char *lds = smem + size_t(wave) * win_mrhs_lds<VT>(cap, false);
    const int32_t b = xcd_contiguous(blockIdx.x, gridDim.x);
    const int32_t per = (nitems + gridDim.x - 1) / gridDim.x;
    const int32_t i0 = b * per, i1 = min(nitems, i0 + per);
    for (int32_t it = i0; it < i1; ++it) {
        const MatDesc &d = descs[items[it].x];
        for (int32_t w = wave; w < stride; w += nw) {
            const WinRec rec = wrec[int64_t(it) * stride + w];
            if (rec.rows() == 0) break;
            win_forward_mrhs<VT, RL, VX>(rec, global_ptr(d.wrend), global_ptr(d.wcols),
                                         global_ptr(static_cast<const VT *>(d.vals)),
                                         global_ptr(static_cast<const X *>(d.x)), global_ptr(static_cast<X *>(d.y)),
                                         d.nnz, nrhs, cap, std::false_type{}, lds, lane);
        }
    }
}

template <typename F>
hipError_t by_store_block(csrk_dtype store, int nrhs, F &&f) {
    return by_dtype(store, [&](auto vt) -> hipError_t {
        return by_block<typename Store<decltype(vt)>::X>(nrhs, [&](auto rc, auto vc) { return f(vt, rc, vc); });
    });
}

}  // namespace

hipError_t spmv_win_mrhs(const Arrays &a, csrk_dtype store, const void *vals, const void *x, void *y, int nrhs,
                         Shape s, hipStream_t st) {
    return by_store_block(store, nrhs, [&](auto vt, auto rc, auto vc) -> hipError_t {
        using VT = decltype(vt);
        using X = typename Store<VT>::X;
        constexpr int RL = decltype(rc)::value, VX = decltype(vc)::value;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(a.split_fwd.width * kXcds), dim3(s.waves * kWave),
                               size_t(s.waves) * win_mrhs_lds<VT>(a.win.cap, false), st, a.win, a.srec_stride,
                               static_cast<const VT *>(vals), static_cast<const X *>(x), static_cast<X *>(y), a.nnz,
                               nrhs, a.split_fwd);
            return hipGetLastError();
        };
        return win_keep<VT>(a, nrhs, false) ? go(k_spmv_win_mrhs<VT, RL, VX, true>)
                                            : go(k_spmv_win_mrhs<VT, RL, VX, false>);
    });
}

hipError_t batch_forward_win_mrhs(const MatDesc *descs, const int2 *items, const BatchWin &win, int32_t stride,
                                  int32_t nitems, csrk_dtype store, int nrhs, Shape s, int grid, hipStream_t st) {
    return by_store_block(store, nrhs, [&](auto vt, auto rc, auto vc) -> hipError_t {
        using VT = decltype(vt);
        hipLaunchKernelGGL((k_batch_forward_win_mrhs<VT, decltype(rc)::value, decltype(vc)::value>), dim3(grid),
                           dim3(s.waves * kWave), size_t(s.waves) * win_mrhs_lds<VT>(win.cap, false), st, descs, items,
                           win.rec, stride, nitems, nrhs, win.cap);
        return hipGetLastError();
    });
}

int batch_forward_win_mrhs_occupancy(csrk_dtype store, int nrhs, const BatchWin &win, Shape s) {
    int blocks = 1;
    const hipError_t e = by_store_block(store, nrhs, [&](auto vt, auto rc, auto vc) -> hipError_t {
        using VT = decltype(vt);
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, k_batch_forward_win_mrhs<VT, decltype(rc)::value, decltype(vc)::value>, s.waves * kWave,
            size_t(s.waves) * win_mrhs_lds<VT>(win.cap, false));
    });
    return (e != hipSuccess || blocks < 1) ? 1 : blocks;
}

}  // namespace dev
}  // namespace csrk
