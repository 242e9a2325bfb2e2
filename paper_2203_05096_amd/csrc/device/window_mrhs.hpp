// Window walk for blocks of right-hand sides (row-major n x nrhs), in the
// layout of window.hpp: one super-row's values and 16-bit columns are staged in
// LDS; a row's columns are spread over RL lanes with VX consecutive columns
// each, and its entries over as many groups of RL lanes as the super-row's
// rows leave (win_groups), so that few long rows fill the wavefront too.
//
// Slices are VX columns wide for any nrhs >= VX and any alignment of the block
// (16 bytes; 8 for two or three FP32 columns): the last one is moved back so
// that it ends with the row, and its first columns repeat the slice before it
// (equal results, written twice; counted once in grad_vals).  gfx950 loads and
// stores 16 bytes from any 4-byte boundary.
//
// What bounds it: waiting for its chain of loads (record, stream, batches of
// gathers) at the wavefronts that its registers leave resident; the counters do not
// tell latency from bandwidth there.  One MI355X, three matrices used in turn, us,
// forward / adjoint, general walk -> window walk: 3D 7-point, 16 matrices of sides
// 16 to 72, 8 columns, FP32 56.3 / 96.6 -> 49.8 / 91.0; 3D 19-point 61x64x67, 8
// columns, FP32 21.5 / 43.1 -> 15.8 / 27.5; 2D 5-point 707x601, 5 columns, FP64 (one
// column per lane before, as rows end off 16 bytes) 22.1 / 47.3 -> 14.3 / 23.3.
#pragma once

#include "window.hpp"

namespace csrk {
namespace dev {

namespace {

// LDS bytes per wavefront for windows of at most `cap` entries (cap a multiple
// of 8, including the up to 7 entries before the window's first): values,
// columns, and grad_vals where they cannot take their values' place.
template <typename VT>
__host__ __device__ constexpr int win_mrhs_lds(int cap, bool gv_apart) {
    return cap * int(sizeof(VT) + sizeof(uint16_t) + (gv_apart ? sizeof(typename Store<VT>::A) : 0));
}

// grad_vals take the place of the values used for them when they have one
// size and a row's columns are walked in one go.
template <typename VT>
__host__ __device__ constexpr bool win_gv_apart(int nrhs, int cols_per_pass) {
    return sizeof(VT) != sizeof(typename Store<VT>::A) || nrhs > cols_per_pass;
}

// VX consecutive elements at any element boundary.
template <typename X, int VX>
struct Slice {
    typedef X V __attribute__((ext_vector_type(VX), aligned(sizeof(X))));
    V v;
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int e = 0; e < VX; ++e) v[e] = X(0);
    }
    // at base + byte offset `off` (32 bits: the window's rows lie within 65536 of its base)
    __device__ __forceinline__ void load(const X *__restrict__ base, uint32_t off) {
        v = *reinterpret_cast<const V *>(reinterpret_cast<const char *>(base) + off);
    }
    // past the caches: results are not read again by the launch (3D 7-point, 16 matrices, 8 FP32 columns: forward
    // 53.9 -> 49.9 us, adjoint 96.2 -> 94.7)
    __device__ __forceinline__ void store(X *__restrict__ p) const {
        __builtin_nontemporal_store(v, reinterpret_cast<V *>(p));
    }
};

// log2 of the groups of RL lanes per row: the largest power of two that still
// walks `nrows` rows at once (1 if they need more than one pass anyway), at
// most 8.
__device__ __forceinline__ int win_groups(int nrows, int RL) {
    int le = 0;
    while (le < 3 && ((nrows * RL) << (le + 1)) <= kWave) ++le;
    return le;
}

// The window's columns (and, with VALS, its values) into LDS.
template <typename VT, bool IND, bool UNI, bool VALS, bool K>
__device__ __forceinline__ void win_fetch(int32_t e0, int32_t nent, const uint16_t *__restrict__ cols,
                                          const int32_t *__restrict__ src, const VT *__restrict__ vals, int64_t nnz,
                                          std::bool_constant<K> keep, VT *sval, uint16_t *scol, int lane) {
    if constexpr (VALS) {
        WinStream<VT> w;
        win_load<VT, IND, UNI>(w, e0, nent, cols, src, vals, nnz, keep, lane);
        win_stage<VT>(w, e0, nent, sval, scol, lane);
    } else {
        const int32_t ea = e0 & ~(Store<VT>::V - 1);  // LDS index k - ea in both forms
        const int end = e0 - ea + nent;
        for (int at = lane * 8; at < end; at += kWave * 8)
#pragma unroll
            for (int h = 0; h < 8; h += Store<VT>::V)
                if (at + h < end)
                    *reinterpret_cast<typename WinStream<VT>::CC *>(scol + at + h) =
                        *reinterpret_cast<const typename WinStream<VT>::CC *>(cols + ea + at + h);
    }
}

// Entries gathered per batch and lane.  More of them save round trips to L2
// and cost the registers that keep wavefronts resident (us, forward / adjoint):
//   3D 7-point, 16 matrices, 8 columns, FP32   8 and 4: 53.6 / 96.6   4 and 3: 54.3 / 99.7   7 and 7: 51.1 / 115.5
//   3D 19-point 61x64x67, 8 columns, FP32      8 and 4: 18.7 / 29.5   4 and 3: 17.4 / 29.9   7 and 7: 17.5 / 37.6
//   2D 5-point 707x601, 5 columns, FP64        8 and 4: 16.3 / 27.8   4 and 3: 15.6 / 23.6   7 and 7: 15.1 / 30.0
constexpr int kMrhsBatchFwd = 4;
template <typename X>
constexpr int mrhs_batch_adj() {
    return sizeof(X) == 8 ? 3 : 4;
}

template <typename VT, int RL, int VX, bool K>
__device__ __forceinline__ void win_forward_mrhs(const WinRec &rec, const uint16_t *__restrict__ rend16,
                                                 const uint16_t *__restrict__ cols, const VT *__restrict__ vals,
                                                 const typename Store<VT>::X *__restrict__ x,
                                                 typename Store<VT>::X *__restrict__ y, int64_t nnz, int nrhs, int cap,
                                                 std::bool_constant<K> keep,
                                                 unsigned char *__restrict__ lds, int lane) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    constexpr int B = kMrhsBatchFwd;
    VT *sval = reinterpret_cast<VT *>(lds);
    uint16_t *scol = reinterpret_cast<uint16_t *>(lds + cap * sizeof(VT));
    const int nrows = rec.rows(), nent = rec.entries(), off = rec.e0 & (Store<VT>::V - 1);
    const int my_end = lane < nrows ? int(rend16[rec.r0 + lane]) : 0;
    win_fetch<VT, false, false, true>(rec.e0, nent, cols, nullptr, vals, nnz, keep, sval, scol, lane);
    wave_lds_sync();
    const int le = win_groups(nrows, RL), E = 1 << le;
    const int q = lane % RL, sub = (lane / RL) & (E - 1), rsub = (lane / RL) >> le, rows_per_pass = (kWave / RL) >> le;
    const X *xb = x + int64_t(rec.base) * nrhs;
    const uint32_t row_bytes = uint32_t(nrhs) * sizeof(X);
#pragma unroll 1
    for (int b = 0; b < nrows; b += rows_per_pass) {
        const int rr = b + rsub;
        const bool act = rr < nrows;
        const int rend = __shfl(my_end, act ? rr : 0), prev = __shfl(my_end, (act && rr > 0) ? rr - 1 : 0);
        const int kb = off + (rr > 0 ? prev : 0) + sub;
#pragma unroll 1
        for (int cb = 0; cb < nrhs; cb += RL * VX) {
            const bool cok = act && cb + q * VX < nrhs;
            const int col0 = min(cb + q * VX, nrhs - VX);
            const uint32_t col_bytes = uint32_t(cok ? col0 : 0) * sizeof(X);
            const int ke = cok ? off + rend : 0;
            A acc[VX];
#pragma unroll
            for (int e = 0; e < VX; ++e) acc[e] = A(0);
            for (int k = kb; __any(k < ke); k += B * E) {
                Slice<X, VX> xv[B];
                uint32_t at[B];
#pragma unroll
                for (int j = 0; j < B; ++j) at[j] = scol[k + j * E < ke ? k + j * E : off] * row_bytes + col_bytes;
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    xv[j].zero();
                    if (k + j * E < ke) xv[j].load(xb, at[j]);
                }
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    const bool ok = k + j * E < ke;
                    const A v = Store<VT>::widen(sval[ok ? k + j * E : off]), a = ok ? v : A(0);
#pragma unroll
                    for (int e = 0; e < VX; ++e) acc[e] += a * A(xv[j].v[e]);
                }
            }
            for (int o = RL; o < RL * E; o *= 2)
#pragma unroll
                for (int e = 0; e < VX; ++e) acc[e] += __shfl_xor(acc[e], o);
            if (cok && sub == 0) {
                Slice<X, VX> out;
#pragma unroll
                for (int e = 0; e < VX; ++e) out.v[e] = X(acc[e]);
                out.store(y + int64_t(rec.r0 + rr) * nrhs + col0);
            }
        }
    }
    wave_lds_sync();
}

// Both gradients of one super-row (GX), or grad_vals alone; UNI as in
// win_adjoint (with GX only).  EXACT: the slices do not overlap (nrhs % VX == 0).
template <typename VT, int RL, int VX, bool EXACT, bool IND, bool UNI, bool GX, bool K>
__device__ __forceinline__ void win_adjoint_mrhs(const WinRec &ra, const WinRec &ru,
                                                 const uint16_t *__restrict__ rend16,
                                                 const uint16_t *__restrict__ xend16,
                                                 const uint16_t *__restrict__ cols, const int32_t *__restrict__ src,
                                                 const VT *__restrict__ vals,
                                                 const typename Store<VT>::X *__restrict__ x,
                                                 const typename Store<VT>::X *__restrict__ g,
                                                 typename Store<VT>::X *__restrict__ gx,
                                                 typename Store<VT>::A *__restrict__ gv, int64_t nnz, int nrhs, int cap,
                                                 std::bool_constant<K> keep, unsigned char *__restrict__ lds, int lane) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    constexpr int V = Store<VT>::V;
    constexpr int B = mrhs_batch_adj<X>();
    const bool apart = win_gv_apart<VT>(nrhs, RL * VX);
    VT *sval = reinterpret_cast<VT *>(lds);
    uint16_t *scol = reinterpret_cast<uint16_t *>(lds + cap * sizeof(VT));
    A *sgv = reinterpret_cast<A *>(apart ? lds + cap * (sizeof(VT) + sizeof(uint16_t)) : lds);
    const int nrows = ra.rows(), nent = ra.entries(), off = ru.e0 & (V - 1);
    const int my_end = lane < nrows ? int(rend16[ra.r0 + lane]) : 0;
    const int my_xend = UNI && lane < nrows ? int(xend16[ra.r0 + lane]) : 0;
    win_fetch<VT, IND, UNI, GX>(ru.e0, ru.entries(), cols, src, vals, nnz, keep, sval, scol, lane);
    wave_lds_sync();
    const int le = win_groups(nrows, RL), E = 1 << le;
    const int q = lane % RL, sub = (lane / RL) & (E - 1), rsub = (lane / RL) >> le, rows_per_pass = (kWave / RL) >> le;
    const X *xb = x + int64_t(ru.base) * nrhs, *gb = g + int64_t(ru.base) * nrhs;
    const uint32_t row_bytes = uint32_t(nrhs) * sizeof(X);
#pragma unroll 1
    for (int b = 0; b < nrows; b += rows_per_pass) {
        const int rr = b + rsub;
        const bool act = rr < nrows;
        const int at = act ? rr : 0, before = (act && rr > 0) ? rr - 1 : 0;
        const int rend = __shfl(my_end, at), prev = __shfl(my_end, before);
        const int xend = UNI ? __shfl(my_xend, at) : 0, xprev = UNI ? __shfl(my_xend, before) : 0;
        const int kb = off + (rr > 0 ? prev : 0) + sub, ke = act ? off + rend : 0;
#pragma unroll 1
        for (int cb = 0; cb < nrhs; cb += RL * VX) {
            const bool cok = cb + q * VX < nrhs;
            const int col0 = min(cb + q * VX, nrhs - VX);
            const int twice = cb + q * VX - col0;  // leading columns that the slice before counts (if cok)
            const uint32_t col_bytes = uint32_t(cok ? col0 : 0) * sizeof(X);
            A gi[VX], acc[VX];
#pragma unroll
            for (int e = 0; e < VX; ++e) gi[e] = acc[e] = A(0);
            if (act && cok) {
                Slice<X, VX> t;
                t.load(g + int64_t(ra.r0 + rr) * nrhs, col_bytes);
#pragma unroll
                for (int e = 0; e < VX; ++e) gi[e] = EXACT || e >= twice ? A(t.v[e]) : A(0);
            }
            for (int k = kb; __any(k < ke); k += B * E) {
                Slice<X, VX> xv[B], gw[B];
                uint32_t at_col[B];
#pragma unroll
                for (int j = 0; j < B; ++j)
                    at_col[j] = scol[k + j * E < ke ? k + j * E : off] * row_bytes + col_bytes;
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    xv[j].zero();
                    gw[j].zero();
                    if (cok && k + j * E < ke) {
                        xv[j].load(xb, at_col[j]);
                        if constexpr (GX) gw[j].load(gb, at_col[j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    const bool ok = k + j * E < ke;
                    if constexpr (GX) {  // before grad_vals can take the value's place
                        const A v = Store<VT>::widen(sval[ok ? k + j * E : off]), a = ok ? v : A(0);
                        if (!UNI || has_mirror(a)) {
#pragma unroll
                            for (int e = 0; e < VX; ++e) acc[e] += a * A(gw[j].v[e]);
                        }
                    }
                    A p = 0;
#pragma unroll
                    for (int e = 0; e < VX; ++e) p += gi[e] * (EXACT || e >= twice ? A(xv[j].v[e]) : A(0));
                    p = row_sum<RL>(p);
                    if (q == 0 && ok) sgv[k + j * E] = cb == 0 ? p : sgv[k + j * E] + p;
                }
            }
            if constexpr (GX) {
                if constexpr (UNI) {
                    const int xe = act ? off + nent + xend : 0;
                    for (int k = off + nent + (rr > 0 ? xprev : 0) + sub; __any(k < xe); k += 2 * E) {
                        Slice<X, VX> gw[2];
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            gw[j].zero();
                            if (cok && k + j * E < xe) gw[j].load(gb, scol[k + j * E] * row_bytes + col_bytes);
                        }
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const A a = k + j * E < xe ? Store<VT>::widen(sval[k + j * E]) : A(0);
#pragma unroll
                            for (int e = 0; e < VX; ++e) acc[e] += a * A(gw[j].v[e]);
                        }
                    }
                }
                for (int o = RL; o < RL * E; o *= 2)
#pragma unroll
                    for (int e = 0; e < VX; ++e) acc[e] += __shfl_xor(acc[e], o);
                if (act && cok && sub == 0) {
                    Slice<X, VX> out;
#pragma unroll
                    for (int e = 0; e < VX; ++e) out.v[e] = X(acc[e]);
                    out.store(gx + int64_t(ra.r0 + rr) * nrhs + col0);
                }
            }
        }
    }
    wave_lds_sync();
    win_store_gv<A>(sgv, off, nent, gv + (ra.e0 & ~(V - 1)), lane);
    wave_lds_sync();
}

// ------------------------------------------------------------------ dispatch

// Calls f(integral_constant<RL>, integral_constant<VX>) for a block of nrhs
// columns (nrhs >= 2): slices of 16 bytes where a row holds one, RL the power
// of two of lanes that covers a row, at most 16 (wider blocks are walked in
// chunks of 16 slices).
template <typename X, typename F>
hipError_t by_block(int nrhs, F &&f) {
    constexpr int W = 16 / int(sizeof(X));
    auto lanes = [&](auto vc) -> hipError_t {
        constexpr int VX = decltype(vc)::value;
        const int slices = (nrhs + VX - 1) / VX;
        if (slices <= 1) return f(std::integral_constant<int, 1>{}, vc);
        if (slices <= 2) return f(std::integral_constant<int, 2>{}, vc);
        if constexpr (VX < W) {
            return hipErrorInvalidValue;  // narrow slices serve at most 3 columns
        } else {
            if (slices <= 4) return f(std::integral_constant<int, 4>{}, vc);
            if (slices <= 8) return f(std::integral_constant<int, 8>{}, vc);
            return f(std::integral_constant<int, 16>{}, vc);
        }
    };
    if constexpr (W > 2) {
        if (nrhs < W) return lanes(std::integral_constant<int, 2>{});
    }
    return lanes(std::integral_constant<int, W>{});
}

}  // namespace

}  // namespace dev
}  // namespace csrk
