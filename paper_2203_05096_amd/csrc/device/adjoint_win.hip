// The one-pass adjoint by the window walk (single right-hand side, every
// super-row one window of 16-bit columns): one matrix and batched launches.
#include "window.hpp"

namespace csrk {
namespace dev {

namespace {

template <typename VT, bool IND, bool UNI>
__global__ void __launch_bounds__(1024) k_adjoint_win(WinArrays win, int32_t stride, const int32_t *__restrict__ src,
                                                      const VT *__restrict__ vals,
                                                      const typename Store<VT>::X *__restrict__ x,
                                                      const typename Store<VT>::X *__restrict__ g,
                                                      typename Store<VT>::X *__restrict__ gx,
                                                      typename Store<VT>::A *__restrict__ gv, int64_t nnz,
                                                      XcdSplit split) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x / kWave);
    const int nw = blockDim.x / kWave;
    unsigned char *lds = smem + size_t(wave) * win_adjoint_lds<VT>();
    const int32_t t = ssr_of_block(split, int32_t(blockIdx.x));
    if (t < 0) return;
    for (int32_t w = wave; w < stride; w += nw) {
        const int64_t slot = int64_t(t) * stride + w;
        const WinRec rec = win.rec[slot];
        if (rec.rows() == 0) break;
        if constexpr (UNI)
            win_adjoint<VT, IND, true>(rec, win.urec[slot], win.rend, win.xend, win.ucols, src, vals, x, g, gx, gv,
                                       nnz, lds, lane);
        else
            win_adjoint<VT, IND, false>(rec, rec, win.rend, nullptr, win.cols, src, vals, x, g, gx, gv, nnz, lds,
                                        lane);
    }
}

// Batched: items and XCD order as in k_batch_forward.  A matrix takes the
// union form where its pattern is nonsymmetric (its descriptor's uni).
template <typename VT, bool IND>
__global__ void __launch_bounds__(1024) k_batch_adjoint_win(const MatDesc *__restrict__ descs,
                                                            const int2 *__restrict__ items,
                                                            const WinRec *__restrict__ wrec,
                                                            const WinRec *__restrict__ wrec_u, int32_t stride,
                                                            int32_t nitems) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x / kWave);
    const int nw = blockDim.x / kWave;
    unsigned char *lds = smem + size_t(wave) * win_adjoint_lds<VT>();
    const int32_t b = xcd_contiguous(blockIdx.x, gridDim.x);
    const int32_t per = (nitems + gridDim.x - 1) / gridDim.x;
    const int32_t i0 = b * per, i1 = min(nitems, i0 + per);
    for (int32_t it = i0; it < i1; ++it) {
        const MatDesc &d = descs[items[it].x];
        const X *x = global_ptr(static_cast<const X *>(d.x)), *g = global_ptr(static_cast<const X *>(d.g));
        X *gx = global_ptr(static_cast<X *>(d.gx));
        A *gv = global_ptr(static_cast<A *>(d.gv));
        const uint16_t *rend = global_ptr(d.wrend);
        for (int32_t w = wave; w < stride; w += nw) {
            const int64_t slot = int64_t(it) * stride + w;
            const WinRec rec = wrec[slot];
            if (rec.rows() == 0) break;
            if (d.uni)
                win_adjoint<VT, IND, true>(rec, wrec_u[slot], rend, global_ptr(d.wxend), global_ptr(d.wucols),
                                           global_ptr(d.u_src),
                                           global_ptr(static_cast<const VT *>(IND ? d.vals : d.u_vals)), x, g, gx, gv,
                                           d.nu, lds, lane);
            else
                win_adjoint<VT, IND, false>(rec, rec, rend, nullptr, global_ptr(d.wcols), global_ptr(d.t_src),
                                            global_ptr(static_cast<const VT *>(d.vals)), x, g, gx, gv, d.nnz, lds,
                                            lane);
        }
    }
}

template <typename F>
hipError_t by_store_ind(csrk_dtype store, bool ind, F &&f) {
    return by_dtype(store, [&](auto vt) -> hipError_t {
        return ind ? f(vt, std::true_type{}) : f(vt, std::false_type{});
    });
}

}  // namespace

hipError_t adjoint_win(const Arrays &a, csrk_dtype store, const void *vals, const void *x, const void *g, void *gx,
                       void *gv, Shape s, hipStream_t st) {
    if (a.nssr == 0) return hipSuccess;
    return by_store_ind(store, vals != nullptr, [&](auto vt, auto ic) -> hipError_t {
        using VT = decltype(vt);
        using X = typename Store<VT>::X;
        using A = typename Store<VT>::A;
        constexpr bool IND = decltype(ic)::value;
        const dim3 grid(a.split_adj.width * kXcds), block(s.waves * kWave);
        const size_t lds = size_t(s.waves) * win_adjoint_lds<VT>();
        if (a.sym)
            hipLaunchKernelGGL((k_adjoint_win<VT, IND, false>), grid, block, lds, st, a.win, a.srec_stride, a.t_src,
                               static_cast<const VT *>(IND ? vals : a.vals_t), static_cast<const X *>(x),
                               static_cast<const X *>(g), static_cast<X *>(gx), static_cast<A *>(gv), a.nnz,
                               a.split_adj);
        else
            hipLaunchKernelGGL((k_adjoint_win<VT, IND, true>), grid, block, lds, st, a.win, a.srec_stride, a.u_src,
                               static_cast<const VT *>(IND ? vals : a.u_vals), static_cast<const X *>(x),
                               static_cast<const X *>(g), static_cast<X *>(gx), static_cast<A *>(gv), a.nu,
                               a.split_adj);
        return hipGetLastError();
    });
}

hipError_t batch_adjoint_win(const MatDesc *descs, const int2 *items, const WinRec *wrec, const WinRec *wrec_u,
                             int32_t stride, int32_t nitems, csrk_dtype store, Shape s, int grid, bool ind,
                             hipStream_t st) {
    return by_store_ind(store, ind, [&](auto vt, auto ic) -> hipError_t {
        using VT = decltype(vt);
        hipLaunchKernelGGL((k_batch_adjoint_win<VT, decltype(ic)::value>), dim3(grid), dim3(s.waves * kWave),
                           size_t(s.waves) * win_adjoint_lds<VT>(), st, descs, items, wrec, wrec_u, stride, nitems);
        return hipGetLastError();
    });
}

int batch_adjoint_win_occupancy(csrk_dtype store, Shape s, bool ind) {
    int blocks = 1;
    const hipError_t e = by_store_ind(store, ind, [&](auto vt, auto ic) -> hipError_t {
        using VT = decltype(vt);
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_batch_adjoint_win<VT, decltype(ic)::value>,
                                                            s.waves * kWave, size_t(s.waves) * win_adjoint_lds<VT>());
    });
    return (e != hipSuccess || blocks < 1) ? 1 : blocks;
}

}  // namespace dev
}  // namespace csrk
