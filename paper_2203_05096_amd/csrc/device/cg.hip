// Conjugate gradients on top of the CSR-k product (the paper names CG for
// PDE systems as the application its format is meant for: Section 1 and the
// conclusions).  The matrix product runs in the handle's storage precision;
// the CG vectors x, r, p and every reduction are FP64, so the residual that
// decides convergence is accumulated in FP64 whatever the matrix storage.
//
// This file holds the start of a solve (residual, norms, p = r); the iterations
// are in cg_iter.hip.  Reductions are deterministic: a fixed grid writes one FP64
// partial sum per workgroup (each summed in a fixed order), and the partials are
// added in a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch.hpp"

namespace csrk {
namespace dev {

namespace {

constexpr int kBlock = 256;
constexpr int kWaveSize = 64;

// Sum of v over the workgroup (kBlock threads) in a fixed order; valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *sh) {
#pragma unroll
    for (int off = kWaveSize / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    const int wave = threadIdx.x / kWaveSize;
    if ((threadIdx.x % kWaveSize) == 0) sh[wave] = v;
    __syncthreads();
    double t = 0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kBlock / kWaveSize; ++w) t += sh[w];
    __syncthreads();
    return t;
}

// part[block] = sum over this block's grid-stride share of a[i] * b[i].
template <typename TB>
__global__ void __launch_bounds__(kBlock) k_dot_partial(const double *__restrict__ a, const TB *__restrict__ b,
                                                        int64_t n, double *__restrict__ part) {
    __shared__ double sh[kBlock / kWaveSize];
    double acc = 0;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock)
        acc += a[i] * double(b[i]);
    const double t = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

constexpr int kFinishBlock = 1024;

// s[slot] = sum of part[0..count) (one workgroup), and also = (s[slot], s[1]) to
// `out` when given.  Thread t adds part[t], part[t + 1024], ... in that order
// (coalesced; the loads of a thread are independent, so they are issued
// together), then the threads' sums are combined in a fixed order.
__global__ void __launch_bounds__(kFinishBlock) k_finish(const double *__restrict__ part, int count,
                                                         double *__restrict__ to, const double *__restrict__ s,
                                                         double *__restrict__ out) {
    __shared__ double sh[kFinishBlock / kWaveSize];
    double acc = 0;
#pragma unroll 8
    for (int i = threadIdx.x; i < count; i += kFinishBlock) acc += part[i];
#pragma unroll
    for (int off = kWaveSize / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x % kWaveSize) == 0) sh[threadIdx.x / kWaveSize] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0;
        for (int w = 0; w < kFinishBlock / kWaveSize; ++w) t += sh[w];
        if (to) *to = t;
        if (out) {
            out[0] = t;
            out[1] = s[1];
        }
    }
}

// p = r; p_lo = p rounded to the product's vector type when that is not FP64.
__global__ void __launch_bounds__(kBlock) k_set_p(const double *__restrict__ r, double *__restrict__ p,
                                                  float *__restrict__ p_lo, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
        p[i] = r[i];
        if (p_lo) p_lo[i] = float(r[i]);
    }
}

// r = b - q (q = A x0), part = partial sums of r . r.
template <typename TQ>
__global__ void __launch_bounds__(kBlock) k_residual(const double *__restrict__ b, const TQ *__restrict__ q,
                                                     double *__restrict__ r, int64_t n, double *__restrict__ part) {
    __shared__ double sh[kBlock / kWaveSize];
    double acc = 0;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
        const double ri = b[i] - double(q[i]);
        r[i] = ri;
        acc += ri * ri;
    }
    const double t = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ void __launch_bounds__(kBlock) k_round_f32(const double *__restrict__ v, float *__restrict__ out,
                                                      int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock)
        out[i] = float(v[i]);
}

}  // namespace

int cg_grid(int64_t n) {
    const int64_t g = (n + kBlock - 1) / kBlock;
    return int(g < 1 ? 1 : (g > kCgGrid ? kCgGrid : g));
}

hipError_t cg_residual(const double *b, const void *q, bool q_f32, double *r, int64_t n, double *part, double *s,
                       hipStream_t st) {
    const int grid = cg_grid(n);
    if (q_f32)
        hipLaunchKernelGGL((k_residual<float>), dim3(grid), dim3(kBlock), 0, st, b, static_cast<const float *>(q),
                           r, n, part);
    else
        hipLaunchKernelGGL((k_residual<double>), dim3(grid), dim3(kBlock), 0, st, b, static_cast<const double *>(q),
                           r, n, part);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kFinishBlock), 0, st, part, grid, s, s, nullptr);
    return hipGetLastError();
}

hipError_t cg_norm2(const double *b, int64_t n, double *part, double *s, hipStream_t st) {
    const int grid = cg_grid(n);
    hipLaunchKernelGGL((k_dot_partial<double>), dim3(grid), dim3(kBlock), 0, st, b, b, n, part);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kFinishBlock), 0, st, part, grid, s + 5, s, nullptr);
    return hipGetLastError();
}

hipError_t cg_set_p(const double *r, double *p, float *p_lo, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_set_p, dim3(cg_grid(n)), dim3(kBlock), 0, st, r, p, p_lo, n);
    return hipGetLastError();
}

hipError_t cg_report(const double *part, int count, const double *s, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kFinishBlock), 0, st, part, count, nullptr, s, out);
    return hipGetLastError();
}

hipError_t cg_round(const double *v, float *out, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_round_f32, dim3(cg_grid(n)), dim3(kBlock), 0, st, v, out, n);
    return hipGetLastError();
}

}  // namespace dev
}  // namespace csrk
