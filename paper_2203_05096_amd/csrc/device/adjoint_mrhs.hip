// The one-pass adjoint for blocks of right-hand sides by the window walk: one
// matrix and batched launches.
#include "window_mrhs.hpp"

namespace csrk {
namespace dev {

namespace {

template <typename VT, int RL, int VX, bool EXACT, bool IND, bool UNI, bool GX, bool KEEP>
__global__ void __launch_bounds__(1024) k_adjoint_win_mrhs(WinArrays win, int32_t stride,
                                                           const int32_t *__restrict__ src,
                                                           const VT *__restrict__ vals,
                                                           const typename Store<VT>::X *__restrict__ x,
                                                           const typename Store<VT>::X *__restrict__ g,
                                                           typename Store<VT>::X *__restrict__ gx,
                                                           typename Store<VT>::A *__restrict__ gv, int64_t nnz,
                                                           int nrhs, XcdSplit split) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x / kWave);
    const int nw = blockDim.x / kWave;
    const int cap = UNI ? win.ucap : win.cap;
    unsigned char *lds = smem + size_t(wave) * win_mrhs_lds<VT>(cap, win_gv_apart<VT>(nrhs, RL * VX));
    const int32_t t = ssr_of_block(split, int32_t(blockIdx.x));
    if (t < 0) return;
    for (int32_t w = wave; w < stride; w += nw) {
        const int64_t slot = int64_t(t) * stride + w;
        const WinRec rec = win.rec[slot];
        if (rec.rows() == 0) break;
        win_adjoint_mrhs<VT, RL, VX, EXACT, IND, UNI, GX>(rec, UNI ? win.urec[slot] : rec, win.rend, win.xend,
                                                   UNI ? win.ucols : win.cols, src, vals, x, g, gx, gv, nnz, nrhs,
                                                   cap, std::bool_constant<KEEP>{}, lds, lane);
    }
}

// Items and XCD order as in k_batch_forward.  SYM: every pattern is symmetric
// (an instantiation without the union form's registers: 80 against 96 in FP32
// with 8 columns).
template <typename VT, int RL, int VX, bool EXACT, bool IND, bool SYM>
__global__ void __launch_bounds__(1024) k_batch_adjoint_win_mrhs(const MatDesc *__restrict__ descs,
                                                                 const int2 *__restrict__ items,
                                                                 const WinRec *__restrict__ wrec,
                                                                 const WinRec *__restrict__ wrec_u, int32_t stride,
                                                                 int32_t nitems, int nrhs, int cap) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x / kWave);
    const int nw = blockDim.x / kWave;
    unsigned char *lds = smem + size_t(wave) * win_mrhs_lds<VT>(cap, win_gv_apart<VT>(nrhs, RL * VX));
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
            if constexpr (!SYM) {
                if (d.uni) {
                    win_adjoint_mrhs<VT, RL, VX, EXACT, IND, true, true>(
                        rec, wrec_u[slot], rend, global_ptr(d.wxend), global_ptr(d.wucols), global_ptr(d.u_src),
                        global_ptr(static_cast<const VT *>(IND ? d.vals : d.u_vals)), x, g, gx, gv, d.nu, nrhs, cap,
                        std::false_type{}, lds, lane);
                    continue;
                }
            }
            win_adjoint_mrhs<VT, RL, VX, EXACT, IND, false, true>(rec, rec, rend, nullptr, global_ptr(d.wcols),
                                                           global_ptr(d.t_src),
                                                           global_ptr(static_cast<const VT *>(d.vals)), x, g, gx, gv,
                                                           d.nnz, nrhs, cap, std::false_type{}, lds, lane);
        }
    }
}

template <typename F>
hipError_t by_store_block_ind(csrk_dtype store, int nrhs, bool ind, F &&f) {
    return by_dtype(store, [&](auto vt) -> hipError_t {
        return by_block<typename Store<decltype(vt)>::X>(nrhs, [&](auto rc, auto vc) -> hipError_t {
            if (nrhs % decltype(vc)::value == 0)
                return ind ? f(vt, rc, vc, std::true_type{}, std::true_type{})
                           : f(vt, rc, vc, std::true_type{}, std::false_type{});
            return ind ? f(vt, rc, vc, std::false_type{}, std::true_type{})
                       : f(vt, rc, vc, std::false_type{}, std::false_type{});
        });
    });
}

}  // namespace

hipError_t adjoint_win_mrhs(const Arrays &a, csrk_dtype store, const void *vals, const void *x, const void *g, void *gx,
                            void *gv, int nrhs, Shape s, hipStream_t st) {
    // grad_vals alone does not read the values
    return by_store_block_ind(store, nrhs, gx && vals, [&](auto vt, auto rc, auto vc, auto xc, auto ic) -> hipError_t {
        using VT = decltype(vt);
        using X = typename Store<VT>::X;
        using A = typename Store<VT>::A;
        constexpr int RL = decltype(rc)::value, VX = decltype(vc)::value;
        constexpr bool EXACT = decltype(xc)::value, IND = decltype(ic)::value;
        auto go = [&](auto uc, auto gc, const int32_t *src, const void *v, int64_t entries) -> hipError_t {
            constexpr bool UNI = decltype(uc)::value, GX = decltype(gc)::value;
            const size_t lds = size_t(s.waves) *
                               win_mrhs_lds<VT>(UNI ? a.win.ucap : a.win.cap, win_gv_apart<VT>(nrhs, RL * VX));
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(a.split_adj.width * kXcds), dim3(s.waves * kWave), lds, st, a.win,
                                   a.srec_stride, src, static_cast<const VT *>(v), static_cast<const X *>(x),
                                   static_cast<const X *>(g), static_cast<X *>(gx), static_cast<A *>(gv), entries, nrhs,
                                   a.split_adj);
                return hipGetLastError();
            };
            if constexpr (GX && !IND)
                if (win_keep<VT>(a, nrhs, true))
                    return launch(k_adjoint_win_mrhs<VT, RL, VX, EXACT, IND, UNI, GX, true>);
            return launch(k_adjoint_win_mrhs<VT, RL, VX, EXACT, IND, UNI, GX, false>);
        };
        if (!gx) {
            if constexpr (!IND)
                return go(std::false_type{}, std::false_type{}, a.t_src, nullptr, a.nnz);
            else
                return hipErrorInvalidValue;  // never chosen
        }
        if (a.sym) return go(std::false_type{}, std::true_type{}, a.t_src, IND ? vals : a.vals_t, a.nnz);
        return go(std::true_type{}, std::true_type{}, a.u_src, IND ? vals : a.u_vals, a.nu);
    });
}

hipError_t batch_adjoint_win_mrhs(const MatDesc *descs, const int2 *items, const BatchWin &win, int32_t stride,
                                  int32_t nitems, csrk_dtype store, int nrhs, Shape s, int grid, bool ind,
                                  hipStream_t st) {
    return by_store_block_ind(store, nrhs, ind, [&](auto vt, auto rc, auto vc, auto xc, auto ic) -> hipError_t {
        using VT = decltype(vt);
        constexpr int RL = decltype(rc)::value, VX = decltype(vc)::value;
        constexpr bool EXACT = decltype(xc)::value, IND = decltype(ic)::value;
        const dim3 block(s.waves * kWave);
        const size_t lds = size_t(s.waves) * win_mrhs_lds<VT>(win.ucap, win_gv_apart<VT>(nrhs, RL * VX));
        if (win.sym)
            hipLaunchKernelGGL((k_batch_adjoint_win_mrhs<VT, RL, VX, EXACT, IND, true>), dim3(grid), block, lds, st, descs,
                               items, win.rec, win.urec, stride, nitems, nrhs, win.ucap);
        else
            hipLaunchKernelGGL((k_batch_adjoint_win_mrhs<VT, RL, VX, EXACT, IND, false>), dim3(grid), block, lds, st, descs,
                               items, win.rec, win.urec, stride, nitems, nrhs, win.ucap);
        return hipGetLastError();
    });
}

int batch_adjoint_win_mrhs_occupancy(csrk_dtype store, int nrhs, const BatchWin &win, Shape s, bool ind) {
    int blocks = 1;
    const hipError_t e = by_store_block_ind(store, nrhs, ind, [&](auto vt, auto rc, auto vc, auto xc, auto ic) -> hipError_t {
        using VT = decltype(vt);
        constexpr int RL = decltype(rc)::value, VX = decltype(vc)::value;
        constexpr bool EXACT = decltype(xc)::value, IND = decltype(ic)::value;
        const size_t lds = size_t(s.waves) * win_mrhs_lds<VT>(win.ucap, win_gv_apart<VT>(nrhs, RL * VX));
        if (win.sym)
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &blocks, k_batch_adjoint_win_mrhs<VT, RL, VX, EXACT, IND, true>, s.waves * kWave, lds);
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, k_batch_adjoint_win_mrhs<VT, RL, VX, EXACT, IND, false>, s.waves * kWave, lds);
    });
    return (e != hipSuccess || blocks < 1) ? 1 : blocks;
}

}  // namespace dev
}  // namespace csrk
