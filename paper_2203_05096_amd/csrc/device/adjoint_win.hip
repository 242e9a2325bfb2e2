// The one-pass adjoint by the window walk (single right-hand side, every
// super-row one window of 16-bit columns): one matrix and batched launches.
#include "window.hpp"

namespace csrk {
namespace dev {

namespace {

template <typename VT, int LL, bool IND, bool UNI, bool KEEP>
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
            win_adjoint<VT, LL, IND, true>(rec, win.urec[slot], win.rend, win.xend, win.ucols, src, vals, x, g, gx, gv,
                                       nnz, std::bool_constant<KEEP>{}, lds, lane);
        else
            win_adjoint<VT, LL, IND, false>(rec, rec, win.rend, nullptr, win.cols, src, vals, x, g, gx, gv, nnz,
                                        std::bool_constant<KEEP>{}, lds, lane);
    }
}

// Batched: items and XCD order as in k_batch_forward; LL as in
// k_batch_forward_win.  SYM: every pattern is symmetric; otherwise a matrix
// takes the union form where its own is not (its descriptor's uni).
template <typename VT, int LL, bool IND, bool SYM>
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
            auto go = [&](auto lc) {
                constexpr int L = decltype(lc)::value;
                if constexpr (!SYM) {
                    if (d.uni) {
                        win_adjoint<VT, L, IND, true>(rec, wrec_u[slot], rend, global_ptr(d.wxend),
                                                      global_ptr(d.wucols), global_ptr(d.u_src),
                                                      global_ptr(static_cast<const VT *>(IND ? d.vals : d.u_vals)), x,
                                                      g, gx, gv, d.nu, std::false_type{}, lds, lane);
                        return;
                    }
                }
                win_adjoint<VT, L, IND, false>(rec, rec, rend, nullptr, global_ptr(d.wcols), global_ptr(d.t_src),
                                               global_ptr(static_cast<const VT *>(d.vals)), x, g, gx, gv, d.nnz,
                                               std::false_type{}, lds, lane);
            };
            if constexpr (LL)
                go(std::integral_constant<int, LL>{});
            else
                by_win_lanes_dev(d.wlanes, go);
        }
    }
}

// Calls f(VT{}, integral_constant<LL>, bool_constant<IND>, bool_constant<SYM>).
template <typename F>
hipError_t by_adj_win(csrk_dtype store, int lanes, bool ind, bool sym, F &&f) {
    return by_batch_win(store, lanes, [&](auto vt, auto lc) -> hipError_t {
        if (ind)
            return sym ? f(vt, lc, std::true_type{}, std::true_type{}) : f(vt, lc, std::true_type{}, std::false_type{});
        return sym ? f(vt, lc, std::false_type{}, std::true_type{}) : f(vt, lc, std::false_type{}, std::false_type{});
    });
}

}  // namespace

hipError_t adjoint_win(const Arrays &a, csrk_dtype store, const void *vals, const void *x, const void *g, void *gx,
                       void *gv, Shape s, hipStream_t st) {
    if (a.ngroups == 0) return hipSuccess;
    return by_adj_win(store, a.win.lanes, vals != nullptr, a.sym, [&](auto vt, auto lc, auto ic, auto sc) -> hipError_t {
        using VT = decltype(vt);
        using X = typename Store<VT>::X;
        using A = typename Store<VT>::A;
        constexpr int LL = decltype(lc)::value;
        constexpr bool IND = decltype(ic)::value, SYM = decltype(sc)::value;
        if constexpr (LL == 0) {
            return hipErrorInvalidValue;  // batches only
        } else {
            auto go = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(a.split_adj.width * kXcds), dim3(s.waves * kWave),
                                   size_t(s.waves) * win_adjoint_lds<VT>(), st, a.win, a.srec_stride,
                                   SYM ? a.t_src : a.u_src,
                                   static_cast<const VT *>(IND ? vals : SYM ? a.vals_t : a.u_vals),
                                   static_cast<const X *>(x), static_cast<const X *>(g), static_cast<X *>(gx),
                                   static_cast<A *>(gv), SYM ? a.nnz : a.nu, a.split_adj);
                return hipGetLastError();
            };
            if constexpr (!IND)
                if (win_keep<VT>(a, 1, true)) return go(k_adjoint_win<VT, LL, IND, !SYM, true>);
            return go(k_adjoint_win<VT, LL, IND, !SYM, false>);
        }
    });
}

hipError_t batch_adjoint_win(const MatDesc *descs, const int2 *items, const BatchWin &win, int32_t stride,
                             int32_t nitems, csrk_dtype store, Shape s, int grid, bool ind, hipStream_t st) {
    return by_adj_win(store, win.lanes, ind, win.sym, [&](auto vt, auto lc, auto ic, auto sc) -> hipError_t {
        using VT = decltype(vt);
        hipLaunchKernelGGL((k_batch_adjoint_win<VT, decltype(lc)::value, decltype(ic)::value, decltype(sc)::value>),
                           dim3(grid), dim3(s.waves * kWave), size_t(s.waves) * win_adjoint_lds<VT>(), st, descs, items,
                           win.rec, win.urec, stride, nitems);
        return hipGetLastError();
    });
}

int batch_adjoint_win_occupancy(csrk_dtype store, const BatchWin &win, Shape s, bool ind) {
    int blocks = 1;
    const hipError_t e =
        by_adj_win(store, win.lanes, ind, win.sym, [&](auto vt, auto lc, auto ic, auto sc) -> hipError_t {
            using VT = decltype(vt);
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &blocks, k_batch_adjoint_win<VT, decltype(lc)::value, decltype(ic)::value, decltype(sc)::value>,
                s.waves * kWave, size_t(s.waves) * win_adjoint_lds<VT>());
        });
    return (e != hipSuccess || blocks < 1) ? 1 : blocks;
}

}  // namespace dev
}  // namespace csrk
