// Row-lane window walk for regular matrices (one right-hand side): every
// super-row is one staging window of at most kWave rows and kWinEntries
// entries whose columns span at most 65536, so its columns are kept as 16-bit
// offsets from the super-row's first column and its row ends as 16-bit offsets
// from its first entry (WinArrays, built on the device at upload).
//
// A wavefront streams one super-row's values and column offsets with 16-byte
// (8-, 4-byte) loads straight from its record into LDS, as they are; then LL
// lanes per row walk the row's entries in LDS, gather x and sum in registers.
// LL is the matrix's (window_lanes), a template argument: one body that picks
// LL per super-row took 72 instead of 60 registers in the FP64 forward, 84
// instead of 70 in the adjoint, and with them a wavefront per SIMD.
//
// What bounds it, and why it is laid out so (one MI355X, three matrices used
// in turn, us before -> after):
//  - HBM: 2 bytes less per entry and per row.  3D 7-point 128^3 FP64 reads
//    184 MB instead of 217 MB.
//  - Gathers.  In entry order (the general walk) a gather instruction's lanes
//    lie V entries apart, so they touch up to 64 lines; here neighbouring
//    lanes hold neighbouring rows, whose e-th columns lie next to each other.
//    Forward with 16-bit columns, entry order -> row order: 3D 7-point 128^3
//    FP64 32.9 -> 28.4 us (32-bit columns, entry order: 47.4), 27-point
//    87x90x91 BF16 29.6 -> 20.5 (35.6), 27-point 75x80x77 FP32 22.5 -> 16.6
//    (25.5).
//  - The row sums need no second pass over LDS, and the adjoint no map from
//    entries to rows: a row's g stays in its lanes' registers.
// Measured and not kept: a resident grid that prefetches the next super-row
// into registers (3D 7-point 32.9 -> 35.3 us), lane-contiguous scalar loads of
// the stream (39.3 us), BF16 (value, column) pairs packed in one LDS word
// (20.5 -> 21.5 us).
#pragma once

#include "common.hpp"

namespace csrk {
namespace dev {

namespace {

// Gathers of one lane in flight at once.  8 hold a 7-point row or a quarter of
// a 27-point row (4 measured 2-10% slower on both); 4-byte vectors leave the
// registers for 12, which takes a 9-point row in one batch (forward, 2D 9-point
// 1201x999 FP32 18.3 -> 16.1 us; with 8-byte vectors 12 cost the 7-point forward
// 29.2 -> 32.5 us).
template <typename X>
constexpr int win_batch() {
    return sizeof(X) == 8 ? 8 : 12;
}

static_assert(kWinEntries <= kStageEntries - 8, "a window must fit the staging area from any 16-byte boundary");

template <typename VT>
struct WinStream {
    static constexpr int V = Store<VT>::V;
    static constexpr int U = kStageEntries / (kWave * V);
    typedef VT VV __attribute__((ext_vector_type(V)));
    typedef uint16_t CC __attribute__((ext_vector_type(V)));
    VV v[U];
    CC c[U];
};

// The window's values and column offsets, entries [e0, e0 + nent), in whole
// groups of V from the 16-byte boundary at or below e0.  `cols` is padded to a
// whole group; the values are the caller's or the handle's nnz elements, so
// the last group of the array is read one by one.  IND: value k is
// the caller's at src[k], src holding nnz elements too (UNI: the union's).  K: the
// values are read through the caches (win_keep), otherwise past them; a constant,
// since the compiler merges the two loads of a branch into one plain load.
template <typename VT, bool IND, bool UNI, bool K>
__device__ __forceinline__ void win_load(WinStream<VT> &w, int32_t e0, int32_t nent, const uint16_t *__restrict__ cols,
                                         const int32_t *__restrict__ src, const VT *__restrict__ vals, int64_t nnz,
                                         std::bool_constant<K>, int lane) {
    using W = WinStream<VT>;
    constexpr int V = W::V;
    typedef int32_t SV __attribute__((ext_vector_type(V)));
    const int32_t ea = e0 & ~(V - 1), ce = e0 + nent;
    SV sv[IND ? W::U : 1];
#pragma unroll
    for (int u = 0; u < W::U; ++u) {
        const int64_t pos = int64_t(ea) + (u * kWave + lane) * V;
        if (pos < ce) {
            w.c[u] = *reinterpret_cast<const typename W::CC *>(cols + pos);
            if (pos + V <= nnz) {
                if constexpr (IND) {
                    sv[u] = *reinterpret_cast<const SV *>(src + pos);
#pragma unroll
                    for (int e = 0; e < V; ++e) w.v[u][e] = fetch_at<VT, UNI>(vals, sv[u][e]);
                } else if constexpr (K) {
                    w.v[u] = *reinterpret_cast<const typename W::VV *>(vals + pos);
                } else {
                    w.v[u] = __builtin_nontemporal_load(reinterpret_cast<const typename W::VV *>(vals + pos));
                }
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const bool ok = pos + e < nnz;
                    if constexpr (IND) {
                        sv[u][e] = ok ? src[pos + e] : 0;
                        w.v[u][e] = ok ? fetch_at<VT, UNI>(vals, sv[u][e]) : VT(0);
                    } else {
                        w.v[u][e] = ok ? vals[pos + e] : VT(0);
                    }
                }
            }
        }
    }
    if constexpr (IND && UNI) {
#pragma unroll
        for (int u = 0; u < W::U; ++u)
            if (int64_t(ea) + (u * kWave + lane) * V < ce)
#pragma unroll
                for (int e = 0; e < V; ++e) w.v[u][e] = value_of<VT, UNI>(w.v[u][e], sv[u][e]);
    }
}

// Stages the stream in LDS: entry k of the array at index k - ea.  Groups
// past the window's end are not loaded and not staged.
template <typename VT>
__device__ __forceinline__ void win_stage(const WinStream<VT> &w, int32_t e0, int32_t nent, VT *__restrict__ sval,
                                          uint16_t *__restrict__ scol, int lane) {
    using W = WinStream<VT>;
    constexpr int V = W::V;
    const int end = (e0 & (V - 1)) + nent;
#pragma unroll
    for (int u = 0; u < W::U; ++u) {
        const int at = (u * kWave + lane) * V;
        if (at < end) {
            *reinterpret_cast<typename W::CC *>(scol + at) = w.c[u];
            *reinterpret_cast<typename W::VV *>(sval + at) = w.v[u];
        }
    }
}

// LDS bytes per wavefront of the forward walk: values and column offsets.
template <typename VT>
__host__ __device__ constexpr int win_forward_lds() {
    return kStageEntries * int(sizeof(VT) + sizeof(uint16_t));
}

// The product of one super-row with a vector given by its entries: ready() is
// called once the stream is requested, gather(c) returns x at column base + c,
// and one lane per row calls emit(row, sum), the row counted from r0.
template <typename VT, int LL, bool K, typename R, typename G, typename E>
__device__ __forceinline__ void win_product(const WinRec &rec, const uint16_t *__restrict__ rend16,
                                            const uint16_t *__restrict__ cols, const VT *__restrict__ vals, int64_t nnz,
                                            std::bool_constant<K> keep, unsigned char *__restrict__ lds, int lane,
                                            R &&ready, G &&gather, E &&emit) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    constexpr int V = Store<VT>::V;
    constexpr int B = win_batch<X>();
    VT *sval = reinterpret_cast<VT *>(lds);
    uint16_t *scol = reinterpret_cast<uint16_t *>(lds + kStageEntries * sizeof(VT));
    const int nrows = rec.rows(), nent = rec.entries(), off = rec.e0 & (V - 1);
    WinStream<VT> w;
    win_load<VT, false, false>(w, rec.e0, nent, cols, nullptr, vals, nnz, keep, lane);
    const int my_end = lane < nrows ? int(rend16[rec.r0 + lane]) : 0;
    ready();
    win_stage<VT>(w, rec.e0, nent, sval, scol, lane);
    wave_lds_sync();
    const int rr = lane / LL;
    const bool act = rr < nrows;
    const int rend = __shfl(my_end, act ? rr : 0);
    const int prev = __shfl(my_end, (act && rr > 0) ? rr - 1 : 0);
    int k = off + (rr > 0 ? prev : 0) + lane % LL;
    const int ke = act ? off + rend : 0;
    A acc = 0;
    while (__any(k < ke)) {
        X xv[B];
        A a[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const bool ok = k + j * LL < ke;
            const int kk = ok ? k + j * LL : off;
            const uint32_t c = scol[kk];
            a[j] = ok ? Store<VT>::widen(sval[kk]) : A(0);
            xv[j] = ok ? gather(c) : X(0);
        }
#pragma unroll
        for (int j = 0; j < B; ++j) acc += a[j] * A(xv[j]);
        k += B * LL;
    }
    acc = row_sum<LL>(acc);
    if (act && lane % LL == 0) emit(rr, acc);
    wave_lds_sync();
}

// y for the rows of one super-row.
template <typename VT, int LL, bool K>
__device__ __forceinline__ void win_forward(const WinRec &rec, const uint16_t *__restrict__ rend16,
                                            const uint16_t *__restrict__ cols, const VT *__restrict__ vals,
                                            const typename Store<VT>::X *__restrict__ x,
                                            typename Store<VT>::X *__restrict__ y, int64_t nnz,
                                            std::bool_constant<K> keep, unsigned char *__restrict__ lds, int lane) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    const X *xb = x + rec.base;
    win_product<VT, LL>(
        rec, rend16, cols, vals, nnz, keep, lds, lane, [] {}, [&](uint32_t c) { return xb[c]; },
        [&](int rr, A acc) { y[rec.r0 + rr] = X(acc); });
}

// ------------------------------------------------------------------ adjoint
//
// Both gradients in one pass, in the forward's layout: the lanes of row i
// gather x_j and g_j of its entries, add a_ji g_j to grad_x[i] in registers
// and leave grad_vals = g_i x_j in LDS (over the value just used where the two
// have one size), from where they go out as 16-byte stores; stored straight by
// the row lanes they cost the 3D 7-point matrix below half as much time again.
// Bound by HBM: per entry it reads 2 bytes of columns and a value and writes a
// grad_vals, near the rate of a plain copy (entry-order gathers, 32-bit columns and
// a map from entries to rows in LDS before; three matrices in turn, us before ->
// after): 3D 7-point 101x97x113 FP64 41.0 -> 34.3, 27-point 75x80x77 FP32 43.5 ->
// 31.7, BF16 43.2 -> 29.5, FP64 57.0 -> 46.9.

// LDS bytes per wavefront: values (overwritten by grad_vals of the same size),
// grad_vals where values are smaller, and column offsets.
template <typename VT>
__host__ __device__ constexpr int win_adjoint_lds() {
    using A = typename Store<VT>::A;
    return kStageEntries * int((sizeof(VT) == sizeof(A) ? 0 : sizeof(VT)) + sizeof(A) + sizeof(uint16_t));
}

// grad_vals of LDS entries [off, off + nent) to gv (the array position of LDS
// entry 0, 16-byte aligned).
template <typename A>
__device__ __forceinline__ void win_store_gv(const A *__restrict__ sgv, int off, int nent, A *__restrict__ gv,
                                             int lane) {
    constexpr int VA = 16 / int(sizeof(A));
    typedef A AV __attribute__((ext_vector_type(VA)));
#pragma unroll
    for (int u = 0; u < kStageEntries / (kWave * VA); ++u) {
        const int p = (u * kWave + lane) * VA;
        if (p >= off && p + VA <= off + nent) {
            *reinterpret_cast<AV *>(gv + p) = *reinterpret_cast<const AV *>(sgv + p);
        } else {
#pragma unroll
            for (int e = 0; e < VA; ++e)
                if (p + e >= off && p + e < off + nent) gv[p + e] = sgv[p + e];
        }
    }
}

// Both gradients of one super-row.  UNI false: symmetric pattern, `ru` == `ra`
// and values in A'^T order (vals) or the caller's through src (IND).  UNI true:
// the super-row's union range `ru` holds its A' entries (at a fixed offset, a
// multiple of 8, from their A' positions; no_mirror where A'^T has none) and then
// its rows' extras, whose ends are xend16; columns, values and src are the
// union's, `nnz` its entries.
template <typename VT, int LL, bool IND, bool UNI, bool K>
__device__ __forceinline__ void win_adjoint(const WinRec &ra, const WinRec &ru, const uint16_t *__restrict__ rend16,
                                            const uint16_t *__restrict__ xend16, const uint16_t *__restrict__ cols,
                                            const int32_t *__restrict__ src, const VT *__restrict__ vals,
                                            const typename Store<VT>::X *__restrict__ x,
                                            const typename Store<VT>::X *__restrict__ g,
                                            typename Store<VT>::X *__restrict__ gx,
                                            typename Store<VT>::A *__restrict__ gv, int64_t nnz,
                                            std::bool_constant<K> keep, unsigned char *__restrict__ lds, int lane) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    constexpr int V = Store<VT>::V;
    constexpr int B = win_batch<X>();
    constexpr bool OVER = sizeof(VT) == sizeof(A);
    A *sgv = reinterpret_cast<A *>(lds);
    VT *sval = reinterpret_cast<VT *>(lds + (OVER ? 0 : kStageEntries * sizeof(A)));
    uint16_t *scol = reinterpret_cast<uint16_t *>(lds + win_adjoint_lds<VT>() - kStageEntries * sizeof(uint16_t));
    const int nrows = ra.rows(), nent = ra.entries(), off = ru.e0 & (V - 1);
    WinStream<VT> w;
    win_load<VT, IND, UNI>(w, ru.e0, ru.entries(), cols, src, vals, nnz, keep, lane);
    const int my_end = lane < nrows ? int(rend16[ra.r0 + lane]) : 0;
    const int my_xend = UNI && lane < nrows ? int(xend16[ra.r0 + lane]) : 0;
    const A my_g = lane < nrows ? A(g[ra.r0 + lane]) : A(0);
    win_stage<VT>(w, ru.e0, ru.entries(), sval, scol, lane);
    wave_lds_sync();
    const X *xb = x + ru.base, *gb = g + ru.base;
    const int rr = lane / LL;
    const bool act = rr < nrows;
    const int at = act ? rr : 0, before = (act && rr > 0) ? rr - 1 : 0;
    const int rend = __shfl(my_end, at), prev = __shfl(my_end, before);
    const A gi = __shfl(my_g, at);
    int k = off + (rr > 0 ? prev : 0) + lane % LL;
    int ke = act ? off + rend : 0;
    A acc = 0;
    while (__any(k < ke)) {
        X xv[B], gw[B];
        uint32_t c[B];
#pragma unroll
        for (int j = 0; j < B; ++j) c[j] = scol[k + j * LL < ke ? k + j * LL : off];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            xv[j] = gw[j] = X(0);
            if (k + j * LL < ke) {
                xv[j] = xb[c[j]];
                gw[j] = gb[c[j]];
            }
        }
#pragma unroll
        for (int j = 0; j < B; ++j)
            if (k + j * LL < ke) {
                const A a = Store<VT>::widen(sval[k + j * LL]);
                if (!UNI || has_mirror(a)) acc += a * A(gw[j]);
                sgv[k + j * LL] = gi * A(xv[j]);
            }
        k += B * LL;
    }
    if constexpr (UNI) {
        constexpr int BX = 2;  // a dropped entry in ten leaves a row about one extra
        const int xend = __shfl(my_xend, at), xprev = __shfl(my_xend, before);
        k = off + nent + (rr > 0 ? xprev : 0) + lane % LL;
        ke = act ? off + nent + xend : 0;
        while (__any(k < ke)) {
            X gw[BX];
#pragma unroll
            for (int j = 0; j < BX; ++j) gw[j] = k + j * LL < ke ? gb[uint32_t(scol[k + j * LL])] : X(0);
#pragma unroll
            for (int j = 0; j < BX; ++j)
                if (k + j * LL < ke) acc += Store<VT>::widen(sval[k + j * LL]) * A(gw[j]);
            k += BX * LL;
        }
    }
    acc = row_sum<LL>(acc);
    if (act && lane % LL == 0) gx[ra.r0 + rr] = X(acc);
    wave_lds_sync();
    win_store_gv<A>(sgv, off, nent, gv + (ra.e0 & ~(V - 1)), lane);
    wave_lds_sync();
}

// ------------------------------------------------------------------ dispatch

// Calls f(integral_constant<int, LL>) for a matrix's lanes per row.
template <typename F>
hipError_t by_win_lanes(int lanes, F &&f) {
    static_assert(kWinMaxLanes == 16, "");
    switch (lanes) {
    case 1:
        return f(std::integral_constant<int, 1>{});
    case 2:
        return f(std::integral_constant<int, 2>{});
    case 4:
        return f(std::integral_constant<int, 4>{});
    case 8:
        return f(std::integral_constant<int, 8>{});
    case 16:
        return f(std::integral_constant<int, 16>{});
    }
    return hipErrorInvalidValue;
}

// The same inside a kernel (a batch whose matrices differ; uniform).
template <typename F>
__device__ __forceinline__ void by_win_lanes_dev(int lanes, F &&f) {
    if (lanes == 1)
        f(std::integral_constant<int, 1>{});
    else if (lanes == 2)
        f(std::integral_constant<int, 2>{});
    else if (lanes == 4)
        f(std::integral_constant<int, 4>{});
    else if (lanes == 8)
        f(std::integral_constant<int, 8>{});
    else
        f(std::integral_constant<int, 16>{});
}

// Calls f(VT{}, integral_constant<int, LL>) for a batch (LL = 0 where lanes is).
template <typename F>
hipError_t by_batch_win(csrk_dtype store, int lanes, F &&f) {
    return by_dtype(store, [&](auto vt) -> hipError_t {
        if (lanes == 0) return f(vt, std::integral_constant<int, 0>{});
        return by_win_lanes(lanes, [&](auto lc) { return f(vt, lc); });
    });
}

// Whether a launch over nrhs columns reads the values through the caches: its
// whole traffic (values, columns, vectors, grad_vals) is at most kWinKeepBytes, so
// that the next launch still finds it in the 256 MB Infinity Cache; more is read
// past them, which leaves the caches to the vectors.  Three matrices in turn, us,
// past / through: 82 MB, 3D 27-point 87x90x91 BF16 forward 22.0 / 20.1; 84 MB, 3D
// 7-point 80^3 FP64 adjoint 18.8 / 15.2; 73 MB, 3D 19-point 61x64x67, 8 FP32
// columns, forward and adjoint 44.8 / 40.4; 117 MB, 2D 9-point 1201x999 FP32
// adjoint 33.0 / 36.3; 184 MB, 3D 7-point 128^3 FP64 forward 29.2 / 36.5.
// Batched launches read past them at any size: 16 3D 7-point matrices, 8 FP32
// columns, 83 MB, forward 29.7 / 28.7, 118 MB, adjoint 56.2 / 54.8; one column, 205
// MB, FP64 forward 30.6 / 36.7, 330 MB, adjoint 60.7 / 64.7; the same below 80 MB.
constexpr int64_t kWinKeepBytes = 96 << 20;
template <typename VT>
bool win_keep(const Arrays &a, int nrhs, bool adjoint) {
    const int64_t entries = (adjoint && !a.sym ? a.nu : a.nnz) * int64_t(sizeof(VT) + sizeof(uint16_t));
    const int64_t grad = adjoint ? a.nnz * int64_t(sizeof(typename Store<VT>::A)) : 0;
    return entries + grad + (adjoint ? 3 : 2) * int64_t(a.n) * nrhs * int64_t(sizeof(typename Store<VT>::X)) <=
           kWinKeepBytes;
}

}  // namespace

}  // namespace dev
}  // namespace csrk
