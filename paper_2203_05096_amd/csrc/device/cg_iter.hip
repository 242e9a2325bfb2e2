// Conjugate-gradient iterations.  The scalars of an iteration are sums of one
// partial per workgroup; the kernels that need them add the partials themselves,
// every wavefront or workgroup in the same order, so all use the same bits and no
// launch is spent on a sum.  Launches that wait for each other cost 4 to 5 us
// each; with a launch per sum an iteration had five, 27 us of them on a 3D
// 7-point 64^3 matrix.
//   Two launches (small matrices with the window layout, CgIter::two):
//     k_cg_product: beta from the residual's partials; the product gathers
//       p = r + beta p_old entry by entry (both at the column), its rows write p
//       and x += alpha p_old, and each workgroup its part of p . q;
//     k_cg_residual: alpha from those parts; r -= alpha q and the parts of r . r.
//     p has two buffers, since rows read their neighbours' old p, and x lags by
//     one update (k_cg_last).
//   Three launches (any matrix): the product with its parts of p . q (spmv_dot),
//     k_cg_residual, and k_cg_update: beta, x += alpha p, p = r + beta p.
// The first saves a launch and the passes over p and r, the second the second
// gather of every entry; the line between them is at cg_two_launches.
//
// s: s[1] = p . q and s[2] = alpha of the last iteration, s[6 + (it & 1)] = r . r
// at the start of iteration it (written before k_cg_residual of that iteration,
// read by it and by what makes beta of the next).
#include "window.hpp"

namespace csrk {
namespace dev {

namespace {

constexpr int kBlock = 256;

// Threads per workgroup of the passes over the vectors.  Every workgroup reads the
// whole list of parts, so many rows take few, large ones: at 128^3 rows 1024 of 256
// threads read 134 MB of parts of p . q out of L2, 256 of 1024 a quarter of it (50
// iterations, us, FP64: 3363 -> 3046; 97x91x88 1671 -> 1583).  Fewer rows take small
// ones, which then reach more of the CUs (64^3 gives every CU one).
constexpr int kWideBlock = 1024;
constexpr int64_t kWideRows = 1 << 19;
int cg_block(int64_t n) { return n > kWideRows ? kWideBlock : kBlock; }

// part[first], part[first + step], ... below count, added in that order.  B are
// requested at a time, the last batch filled up with zeros: each batch waits once
// for L2.  50 iterations, us, eights with the rest one by one -> sixteens: 3D
// 7-point 97x91x88 FP64 1774 -> 1671, 128^3 3396 -> 3363.
template <int B>
__device__ __forceinline__ double part_sum(const double *__restrict__ part, int count, int first, int step) {
    double acc = 0;
    for (int i = first; i < count; i += B * step) {
        double v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = i + u * step < count ? part[i + u * step] : 0.0;
#pragma unroll
        for (int u = 0; u < B; ++u) acc += v[u];
    }
    return acc;
}

// part[0..count) added by one wavefront: lane l takes l, l + 64, ..., then the
// lanes in a fixed order; the same bits in every lane of every wavefront.
template <int B>
__device__ __forceinline__ double wave_total(const double *__restrict__ part, int count, int lane) {
    double acc = part_sum<B>(part, count, lane, kWave);
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    return acc;
}

// The matrix is read through the caches: 3 M entries, the most that come here, and
// the vectors stay in the Infinity Cache from one iteration to the next.
template <typename VT, int LL>
__global__ void __launch_bounds__(1024) k_cg_product(WinArrays win, int32_t stride, const VT *__restrict__ vals,
                                                     const double *__restrict__ r, const double *__restrict__ p_old,
                                                     double *__restrict__ p, double *__restrict__ x,
                                                     typename Store<VT>::X *__restrict__ q, int64_t nnz, XcdSplit split,
                                                     const double *__restrict__ rr_part, int rr_parts,
                                                     double *__restrict__ s, int it, double *__restrict__ pq_part) {
    using A = typename Store<VT>::A;
    using X = typename Store<VT>::X;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double wsum[1024 / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x / kWave);
    const int nw = blockDim.x / kWave;
    unsigned char *lds = smem + size_t(wave) * win_forward_lds<VT>();
    const int32_t t = ssr_of_block(split, int32_t(blockIdx.x));
    double dot = 0, alpha = 0, beta = 0;
    bool known = false;
    // iteration 0: p = r and x unchanged (the caller passes r as p_old)
    auto scalars = [&]() {
        if (known) return;
        known = true;
        const double rr = wave_total<4>(rr_part, rr_parts, lane);
        if (blockIdx.x == 0 && threadIdx.x == 0) s[6 + (it & 1)] = rr;
        if (it > 0) {
            alpha = s[2];
            beta = rr / s[6 + ((it + 1) & 1)];
        }
    };
    if (t >= 0) {
        for (int32_t w = wave; w < stride; w += nw) {
            const WinRec rec = win.rec[int64_t(t) * stride + w];
            if (rec.rows() == 0) break;
            const double *rb = r + rec.base, *pb = p_old + rec.base;
            const int rr = lane / LL;
            double pi = 0;
            win_product<VT, LL>(
                rec, win.rend, win.cols, vals, nnz, std::true_type{}, lds, lane,
                [&]() {
                    const bool own = rr < rec.rows() && lane % LL == 0;
                    const int64_t i = rec.r0 + rr;
                    const double ri = own ? r[i] : 0, po = own ? p_old[i] : 0, xi = own ? x[i] : 0;
                    scalars();
                    if (own) {
                        pi = __builtin_fma(beta, po, ri);
                        p[i] = pi;
                        x[i] = __builtin_fma(alpha, po, xi);
                    }
                },
                [&](uint32_t c) { return X(__builtin_fma(beta, pb[c], rb[c])); },
                [&](int, A acc) {
                    q[rec.r0 + rr] = X(acc);
                    dot += double(X(acc)) * pi;
                });
        }
    }
    if (blockIdx.x == 0 && wave == 0) scalars();  // s is written also where block 0 has no rows
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) dot += __shfl_xor(dot, off);
    if (lane == 0) wsum[wave] = dot;
    __syncthreads();
    if (threadIdx.x == 0) {
        double d = 0;
        for (int w = 0; w < nw; ++w) d += wsum[w];
        pq_part[blockIdx.x] = d;
    }
}

// r -= alpha q; rr_part[block] = its part of r . r.  The first elements are
// requested before alpha is summed.
template <typename TQ, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_cg_residual(double *__restrict__ r, const TQ *__restrict__ q, int64_t n,
                                                        const double *__restrict__ pq_part, int pq_parts,
                                                        double *__restrict__ s, int it, double *__restrict__ rr_part) {
    constexpr int W = 4;
    __shared__ double sh[2][BLOCK / kWave];
    const int64_t step = int64_t(gridDim.x) * BLOCK, first = int64_t(blockIdx.x) * BLOCK + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    double rv[W], qv[W];
    auto load = [&](int64_t i) {
#pragma unroll
        for (int u = 0; u < W; ++u) {
            const bool in = i + u * step < n;
            rv[u] = in ? r[i + u * step] : 0.0;
            qv[u] = in ? double(q[i + u * step]) : 0.0;
        }
    };
    load(first);
    const double rr = s[6 + (it & 1)];
    double pq = part_sum<16>(pq_part, pq_parts, threadIdx.x, BLOCK);
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) pq += __shfl_xor(pq, off);
    if (lane == 0) sh[0][wave] = pq;
    __syncthreads();
    pq = 0;
    for (int w = 0; w < BLOCK / kWave; ++w) pq += sh[0][w];
    const double alpha = rr / pq;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        s[1] = pq;
        s[2] = alpha;
    }
    double acc = 0;
    for (int64_t i = first; i < n; i += W * step) {
        if (i != first) load(i);
#pragma unroll
        for (int u = 0; u < W; ++u) {
            const double v = __builtin_fma(-alpha, qv[u], rv[u]);
            if (i + u * step < n) {
                r[i + u * step] = v;
                acc += v * v;
            }
        }
    }
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) sh[1][wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0;
        for (int w = 0; w < BLOCK / kWave; ++w) t += sh[1][w];
        rr_part[blockIdx.x] = t;
    }
}

// x += alpha p, the update that k_cg_product leaves to the next iteration.
__global__ void __launch_bounds__(kBlock) k_cg_last(double *__restrict__ x, const double *__restrict__ p,
                                                    const double *__restrict__ s, int64_t n) {
    const double alpha = s[2];
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock)
        x[i] = __builtin_fma(alpha, p[i], x[i]);
}

// Three launches: beta = r . r / its value before, x += alpha p, p = r + beta p,
// and p_lo = p in the product's vector type when that is not FP64.
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_cg_update(double *__restrict__ x, double *__restrict__ p,
                                                      float *__restrict__ p_lo, const double *__restrict__ r, int64_t n,
                                                      const double *__restrict__ rr_part, int rr_parts,
                                                      double *__restrict__ s, int it) {
    constexpr int W = 4;
    const int64_t step = int64_t(gridDim.x) * BLOCK, first = int64_t(blockIdx.x) * BLOCK + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    double xv[W], pv[W], rv[W];
    auto load = [&](int64_t i) {
#pragma unroll
        for (int u = 0; u < W; ++u) {
            const bool in = i + u * step < n;
            xv[u] = in ? x[i + u * step] : 0.0;
            pv[u] = in ? p[i + u * step] : 0.0;
            rv[u] = in ? r[i + u * step] : 0.0;
        }
    };
    load(first);
    const double rr = wave_total<16>(rr_part, rr_parts, lane);
    const double alpha = s[2], beta = rr / s[6 + (it & 1)];
    if (blockIdx.x == 0 && threadIdx.x == 0) s[6 + ((it + 1) & 1)] = rr;
    for (int64_t i = first; i < n; i += W * step) {
        if (i != first) load(i);
#pragma unroll
        for (int u = 0; u < W; ++u) {
            const int64_t at = i + u * step;
            if (at >= n) break;
            x[at] = __builtin_fma(alpha, pv[u], xv[u]);
            const double pn = __builtin_fma(beta, pv[u], rv[u]);
            p[at] = pn;
            if (p_lo) p_lo[at] = float(pn);
        }
    }
}

}  // namespace

int cg_iter_grid(int64_t n) {
    const int64_t per = 4 * cg_block(n), g = (n + per - 1) / per;  // one batch of loads per thread
    const int64_t most = int64_t(kCgGrid) * kBlock / cg_block(n);
    return int(g < 1 ? 1 : (g > most ? most : g));
}

namespace {

// s[6] = s[0]: r . r before iteration 0, for three launches.
__global__ void k_cg_first(double *s) { s[6] = s[0]; }

hipError_t product_two(const Arrays &a, csrk_dtype store, const void *vals, const CgIter &w, int it, Shape s,
                       hipStream_t st) {
    return by_dtype(store, [&](auto vt) -> hipError_t {
        using VT = decltype(vt);
        using X = typename Store<VT>::X;
        return by_win_lanes(a.win.lanes, [&](auto lc) -> hipError_t {
            hipLaunchKernelGGL((k_cg_product<VT, decltype(lc)::value>), dim3(spmv_grid(a)), dim3(s.waves * kWave),
                               size_t(s.waves) * win_forward_lds<VT>(), st, a.win, a.srec_stride,
                               static_cast<const VT *>(vals), static_cast<const double *>(w.r),
                               static_cast<const double *>(it == 0 ? w.r : w.p[(it + 1) & 1]), w.p[it & 1], w.x,
                               static_cast<X *>(w.q), a.nnz, a.split_fwd, static_cast<const double *>(w.rr_part),
                               it == 0 ? w.rr_parts0 : cg_iter_grid(a.n), w.s, it, w.pq_part);
            return hipGetLastError();
        });
    });
}

}  // namespace

hipError_t cg_iteration(const Arrays &a, csrk_dtype store, const void *vals, const CgIter &w, int it, Shape s,
                        hipStream_t st) {
    const int parts = spmv_grid(a);
    const dim3 grid(cg_iter_grid(a.n));
    if (!w.two && it == 0) hipLaunchKernelGGL(k_cg_first, dim3(1), dim3(1), 0, st, w.s);
    const void *in = store == CSRK_F64 ? static_cast<const void *>(w.p[0]) : static_cast<const void *>(w.p_lo);
    const hipError_t e = w.two ? product_two(a, store, vals, w, it, s, st)
                               : spmv_dot(a, store, vals, in, w.q, w.p[0], w.pq_part, s, st);
    if (e != hipSuccess) return e;
    auto passes = [&](auto bc) {
        constexpr int BLOCK = decltype(bc)::value;
        if (store == CSRK_F64)
            hipLaunchKernelGGL((k_cg_residual<double, BLOCK>), grid, dim3(BLOCK), 0, st, w.r,
                               static_cast<const double *>(w.q), int64_t(a.n), w.pq_part, parts, w.s, it, w.rr_part);
        else
            hipLaunchKernelGGL((k_cg_residual<float, BLOCK>), grid, dim3(BLOCK), 0, st, w.r,
                               static_cast<const float *>(w.q), int64_t(a.n), w.pq_part, parts, w.s, it, w.rr_part);
        if (!w.two)
            hipLaunchKernelGGL((k_cg_update<BLOCK>), grid, dim3(BLOCK), 0, st, w.x, w.p[0], w.p_lo, w.r, int64_t(a.n),
                               w.rr_part, int(grid.x), w.s, it);
    };
    if (cg_block(a.n) == kBlock)
        passes(std::integral_constant<int, kBlock>{});
    else
        passes(std::integral_constant<int, kWideBlock>{});
    return hipGetLastError();
}

hipError_t cg_last(const CgIter &w, int iterations, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_cg_last, dim3(cg_iter_grid(n)), dim3(kBlock), 0, st, w.x, w.p[(iterations + 1) & 1], w.s, n);
    return hipGetLastError();
}

}  // namespace dev
}  // namespace csrk
