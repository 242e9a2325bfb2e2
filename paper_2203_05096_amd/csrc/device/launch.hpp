// Launchers of the gfx950 kernels (device/forward.hip, adjoint.hip, batch.hip,
// util.hip, cg.hip).  C++ linkage, used only by the C ABI layer.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../../include/csrk.h"

namespace csrk {
namespace dev {

// Rows with more nonzeros than this are computed by a workgroup of their own
// (split over its wavefronts) instead of by their super-row's wavefront; the
// handle lists them at upload.
constexpr int32_t kLongRow = CSRK_LONG_ROW;

// A nonsymmetric pattern gets a union-pattern index (one-pass adjoint) when
// every super-row has at most kUnionRows rows and at most kUnionWindow union
// entries: one wavefront's staging window (512 entries) less one load step of
// the widest entry group (8), as the window walk requires.
constexpr int32_t kUnionRows = 64;
constexpr int32_t kUnionWindow = 512 - 8;

// Workgroups are dispatched to the 8 XCDs (each with its own L2) round-robin
// by block index.  SSR block b (counted after the long-row blocks, a multiple
// of 8 of them) runs super-super-row b[b % 8] + b / 8 of XCD b % 8's
// contiguous range [b[x], b[x+1]); blocks past the end of their range exit at
// once.  The ranges are cut so that each XCD gets about the same work.
constexpr int kXcds = 8;
struct XcdSplit {
    int32_t b[kXcds + 1] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    int32_t width = 0;  // largest range: the grid is width * kXcds blocks
};

// Bounds of one super-row: rows [r0, r1) and their entries [e0, e1).  The
// handle keeps one record per (super-super-row, slot), slot w < stride holding
// the SSR's w-th super-row (empty records, r0 == r1, pad short SSRs), so a
// workgroup finds its super-rows' rows and entries with one load instead of
// the chain ssr_ptr -> sr_ptr -> row_ptr.
struct __attribute__((aligned(16))) SrRec {
    int32_t r0, r1, e0, e1;
};

// Row-lane window walk (device/window.hpp): the matrices whose super-rows all
// have at most kWave (64) rows, at most kWinEntries entries (a staging window
// of 512 less one load step of the widest group) and columns within 65536 of
// each other.  A row is walked by 1 to kWinMaxLanes lanes (WinArrays::lanes) in
// batches of 8 entries per lane; a matrix with a row longer than
// kWinMaxBatches batches keeps the general walk, which sums such rows by more
// lanes.
constexpr int32_t kWinRows = 64;
constexpr int32_t kWinEntries = 512 - 8;
constexpr int32_t kWinSpan = 65536;
constexpr int32_t kWinMaxBatches = 4;
constexpr int32_t kWinMaxLanes = 16;

// One super-row of the window walk: rows [r0, r0 + rows()), entries
// [e0, e0 + entries()), columns base + cols16[k].  Slots as in SrRec (rows()
// == 0: empty).
struct __attribute__((aligned(16))) WinRec {
    int32_t r0, e0;
    uint32_t count;  // rows | entries << 16
    int32_t base;
    __host__ __device__ int rows() const { return int(count & 0xffffu); }
    __host__ __device__ int entries() const { return int(count >> 16); }
};

// A' for the window walk; rec == nullptr when the matrix does not qualify.
struct WinArrays {
    const WinRec *rec = nullptr;       // per (SSR, slot), like Arrays::srec
    const uint16_t *cols = nullptr;    // nnz offsets from the super-row's base, padded to a whole load
    const uint16_t *rend = nullptr;    // n row ends, from the super-row's first entry
    // the union pattern's, for the adjoint of a nonsymmetric pattern (nullptr: general walk)
    const WinRec *urec = nullptr;      // r0, first U entry, rows, U entries, base
    const uint16_t *ucols = nullptr;   // nu offsets, padded to a whole load
    const uint16_t *xend = nullptr;    // n ends of the rows' extras, from the super-row's first extra
    // LDS entries that hold any window from the 16-byte boundary before it (multiples of 8)
    int32_t cap = 0, ucap = 0;
    int32_t lanes = 1;  // lanes per row, one right-hand side (a power of two)
};

// Row bytes that a block of right-hand sides may have for the window walk: the
// byte offset of a gathered row from the window's first column is 32-bit.
constexpr int64_t kWinBlockBytes = 65536;

// Device arrays of one CSR-k matrix.
struct Arrays {
    int32_t n = 0;
    int64_t nnz = 0;
    int32_t ngroups = 0;  // groups of windows, one workgroup each (the super-super-rows where none is cut)
    const int32_t *row_ptr = nullptr;
    const int32_t *col_idx = nullptr;
    const int32_t *perm = nullptr;
    // A'^T: row j lists column j of A' by increasing row (t_col) with each
    // entry's position in A' (t_src).  For a symmetric pattern t_row_ptr and
    // t_col are row_ptr and col_idx.
    const int32_t *t_row_ptr = nullptr;
    const int32_t *t_col = nullptr;
    const int32_t *t_src = nullptr;
    const void *vals_t = nullptr;  // the handle's values in A'^T order (aligned with t_col)
    bool sym = false;              // pattern of A' is symmetric: A'^T has the pattern of A'
    // Rows of A' (long_rows) and of A'^T (t_long_rows) longer than kLongRow,
    // ascending; for a symmetric pattern the two lists are the same.
    const int32_t *long_rows = nullptr;
    int32_t nlong = 0;
    const int32_t *t_long_rows = nullptr;
    int32_t t_nlong = 0;
    XcdSplit split_fwd;  // by the forward's work (rows of A')
    XcdSplit split_adj;  // by the adjoint's work (rows of A' and of A'^T)
    int32_t max_row = 0;  // longest row of A' or of A'^T (nonzeros)
    const SrRec *srec = nullptr;    // ngroups * srec_stride window records
    const SrRec *srec_t = nullptr;  // the same rows of A'^T (entries of t_row_ptr); == srec if symmetric
    int32_t srec_stride = 0;        // most windows in one group
    // Union pattern of a nonsymmetric A' (host union_index): per super-row its
    // A' entries, then its rows' extras (entries of A'^T missing from A'),
    // each U entry (i, j) carrying a'_ji.  Present (srec_u != nullptr) only
    // when every super-row fits one staging window; the single-right-hand-side
    // adjoint then takes both gradients in one pass over it.
    const int32_t *u_col = nullptr;
    const int32_t *u_src = nullptr;  // position of a'_ji in A', -1 where A' has no (j, i)
    const void *u_vals = nullptr;    // the handle's values a'_ji in U order (a marker where u_src is -1)
    const int32_t *erow_ptr = nullptr;  // extras of the rows before row i
    const SrRec *srec_u = nullptr;      // per (SSR, slot): rows [r0, r1), U entries [e0, e1)
    int64_t nu = 0;                     // U entries (with padding)
    WinArrays win;  // 16-bit form of A' for the window walk
};

// Whether windows of few rows get more lanes per row (window_row_sums): only
// for matrices with rows far longer than L lanes per row is meant for, so that
// regular matrices run the plain reduction.
inline bool adapt_windows(const Arrays &a, int L) { return a.max_row > 16 * L; }

// Per-matrix record of a batched launch (device-resident table).
struct MatDesc {
    const int32_t *row_ptr;
    const int32_t *col_idx;
    const int32_t *t_row_ptr;
    const int32_t *t_col;
    const int32_t *t_src;
    const void *vals;
    const void *x;
    void *y;
    const void *g;
    void *gx;
    void *gv;
    int64_t nnz;
    int32_t n;
    int32_t wlanes;
    int32_t sym;
    int32_t uni;  // the matrix has a union-pattern index (Arrays::u_col ...): the adjoint takes one pass
    const int32_t *u_col;
    const int32_t *u_src;
    const int32_t *erow_ptr;
    const void *u_vals;
    int64_t nu;
    const uint16_t *wcols;  // WinArrays of A' (batches whose matrices all have them)
    const uint16_t *wrend;
    const uint16_t *wucols;  // their union's, where the pattern is nonsymmetric
    const uint16_t *wxend;
};

// Kernel-shape knobs: lanes per row in the reduction, wavefronts per workgroup.
struct Shape {
    int lanes_per_row = 1;
    int waves = 4;
};

// y = A'x (one right-hand side) and part[w] = the partial sum of y_i pdot_i
// over workgroup w's rows, for w < spmv_grid(a) (CG's p . Ap; FP64).
int spmv_grid(const Arrays &a);
hipError_t spmv_dot(const Arrays &a, csrk_dtype store, const void *vals, const void *x, void *y, const double *pdot,
                    double *part, Shape s, hipStream_t st);

hipError_t spmv(const Arrays &a, csrk_dtype store, const void *vals, const void *x, void *y, int nrhs, Shape s,
                hipStream_t st);
hipError_t spmv_plain(const Arrays &a, csrk_dtype store, const void *vals, const void *x, void *y, int nrhs,
                      Shape s, hipStream_t st);
hipError_t adjoint(const Arrays &a, csrk_dtype store, const void *vals, const void *x, const void *g, void *gx,
                   void *gv, int nrhs, Shape s, hipStream_t st);
// adjoint with both outputs and one right-hand side by the window walk: a.win.rec
// set and, for a nonsymmetric pattern, a.win.urec.
hipError_t adjoint_win(const Arrays &a, csrk_dtype store, const void *vals, const void *x, const void *g, void *gx,
                       void *gv, Shape s, hipStream_t st);
// The same for blocks of right-hand sides (nrhs >= 2, rows of at most
// kWinBlockBytes): the product, and the adjoint with both outputs or (gx ==
// nullptr) grad_vals alone.
hipError_t spmv_win_mrhs(const Arrays &a, csrk_dtype store, const void *vals, const void *x, void *y, int nrhs,
                         Shape s, hipStream_t st);
hipError_t adjoint_win_mrhs(const Arrays &a, csrk_dtype store, const void *vals, const void *x, const void *g, void *gx,
                            void *gv, int nrhs, Shape s, hipStream_t st);
// vals_t[p] = vals[t_src[p]]: the values in A'^T order.
hipError_t transpose_values(const Arrays &a, csrk_dtype store, const void *vals, void *vals_t, hipStream_t st);
// u_vals[p] = vals[u_src[p]] for p < nu, marked as without a mirror where u_src[p] < 0.
hipError_t union_values(const int32_t *u_src, int64_t nu, csrk_dtype store, const void *vals, void *u_vals,
                        hipStream_t st);
// Fills a window layout from `count` super-row records: each slot's WinRec, its
// entries' 16-bit column offsets and its rows' 16-bit ends (rp[r + 1] - rp[r0]).
// *wide (one int32, cleared by the caller) becomes nonzero when some super-row's
// columns span more than kWinSpan.  `cols` must be able to hold every entry.
hipError_t window_layout(const SrRec *srec, int64_t count, const int32_t *col_idx, const int32_t *rp, WinRec *rec,
                         uint16_t *cols, uint16_t *rend, int32_t *wide, hipStream_t st);
hipError_t permute(const Arrays &a, int dir, const void *in, void *out, int nrhs, int elem_bytes, hipStream_t st);
hipError_t convert_values(const double *src, void *dst, int64_t count, csrk_dtype store, hipStream_t st);

// Batched launches: one grid over `nitems` (matrix, super-super-row) items.
// `vec`: every right-hand-side block pointer is 16-byte aligned.
// `brec`: per item, `stride` super-row records (SrRec) of its SSR.
// `win`: the same slots' window records when every matrix has the window
// layout (rec == nullptr otherwise).
struct BatchWin {
    const WinRec *rec = nullptr;   // of A'
    const WinRec *urec = nullptr;  // of what the adjoint streams: the union where A' is nonsymmetric
    int32_t cap = 0, ucap = 0;     // WinArrays::cap over all matrices, and over what the adjoint streams
    int32_t lanes = 0;             // WinArrays::lanes of every matrix, 0 when they differ
    bool sym = true;               // every pattern is symmetric
};
hipError_t batch_forward(const MatDesc *descs, const int2 *items, const SrRec *brec, const BatchWin &win,
                         int32_t stride, int32_t nitems, csrk_dtype store, int nrhs, Shape s, int grid, bool vec, hipStream_t st);
// `ind`: the descriptors' vals are caller values in CSR-k order (reached
// through t_src); otherwise they are the handles' transposed copies.
// `all_sym`: every matrix of the batch has a symmetric pattern; `both`: both
// gradients are wanted (then a multi-right-hand-side launch with FP32
// accumulation runs the fused-only kernel).
// `brec_u`: per item, the same slots' union-pattern records (for matrices
// with uni set; other slots repeat brec).
// `win`: as for batch_forward, rec and urec set when both outputs of every
// matrix are wanted.
hipError_t batch_adjoint(const MatDesc *descs, const int2 *items, const SrRec *brec, const SrRec *brec_u,
                         const BatchWin &win, int32_t stride, int32_t nitems, csrk_dtype store, int nrhs, Shape s, int grid, bool ind,
                         bool vec, bool all_sym, bool both, hipStream_t st);

// batch_adjoint's window walk (one right-hand side, both outputs), and the
// workgroups per CU it can keep resident.
hipError_t batch_adjoint_win(const MatDesc *descs, const int2 *items, const BatchWin &win, int32_t stride,
                             int32_t nitems, csrk_dtype store, Shape s, int grid, bool ind, hipStream_t st);
int batch_adjoint_win_occupancy(csrk_dtype store, const BatchWin &win, Shape s, bool ind);
// The window walks for blocks of right-hand sides, and their occupancies.
hipError_t batch_forward_win_mrhs(const MatDesc *descs, const int2 *items, const BatchWin &win, int32_t stride,
                                  int32_t nitems, csrk_dtype store, int nrhs, Shape s, int grid, hipStream_t st);
int batch_forward_win_mrhs_occupancy(csrk_dtype store, int nrhs, const BatchWin &win, Shape s);
hipError_t batch_adjoint_win_mrhs(const MatDesc *descs, const int2 *items, const BatchWin &win, int32_t stride,
                                  int32_t nitems, csrk_dtype store, int nrhs, Shape s, int grid, bool ind,
                                  hipStream_t st);
int batch_adjoint_win_mrhs_occupancy(csrk_dtype store, int nrhs, const BatchWin &win, Shape s, bool ind);

// Workgroups per CU the batched kernels can keep resident (for sizing the grid).
int batch_occupancy(csrk_dtype store, int nrhs, Shape s, bool adjoint, bool ind, bool vec, bool all_sym,
                    bool both, const BatchWin &win);

// Bandwidth probes (device/util.hip): a streaming read of `bytes` (a multiple of
// 16, 16-byte aligned) writing one word per workgroup to part[0 .. probe_grid()),
// and a copy of `bytes` from src to dst.
int probe_grid();
hipError_t probe_read(const void *buf, int64_t bytes, double *part, hipStream_t st);
hipError_t probe_copy(const void *src, void *dst, int64_t bytes, hipStream_t st);

// Conjugate-gradient vector kernels (device/cg.hip).  FP64 vectors; q (the
// product's output) is FP32 when q_f32.  part holds kCgGrid partial sums; s the
// scalars rr and bb at s[0] and s[5].
constexpr int kCgGrid = 1024;
int cg_grid(int64_t n);
// r = b - q, s[0] = r . r
hipError_t cg_residual(const double *b, const void *q, bool q_f32, double *r, int64_t n, double *part, double *s,
                       hipStream_t st);
// s[5] = b . b
hipError_t cg_norm2(const double *b, int64_t n, double *part, double *s, hipStream_t st);
// p = r; p_lo = float(p) when p_lo != NULL
hipError_t cg_set_p(const double *r, double *p, float *p_lo, int64_t n, hipStream_t st);
// out = float(v)
hipError_t cg_round(const double *v, float *out, int64_t n, hipStream_t st);

// CG iterations without launches for their sums (device/cg_iter.hip).  x, r and
// p hold n doubles, q the product's vector type, p_lo n floats (FP32/BF16
// storage, three launches), pq_part spmv_grid(a) and rr_part kCgGrid partial
// sums (rr_parts0 of them before iteration 0), s 8 scalars.  s[1] is p . q of the
// last iteration; r . r after it is rr_part's sum.
struct CgIter {
    bool two = false;  // two launches an iteration: a.win.rec set, p has two buffers
    double *x = nullptr, *r = nullptr, *p[2] = {nullptr, nullptr};
    float *p_lo = nullptr;
    void *q = nullptr;
    double *pq_part = nullptr, *rr_part = nullptr, *s = nullptr;
    int rr_parts0 = 0;
};
int cg_iter_grid(int64_t n);  // partial sums of r . r after an iteration
hipError_t cg_iteration(const Arrays &a, csrk_dtype store, const void *vals, const CgIter &w, int it, Shape s,
                        hipStream_t st);
// x += alpha p after `iterations` >= 1 iterations of two launches
hipError_t cg_last(const CgIter &w, int iterations, int64_t n, hipStream_t st);
// out[0] = sum of part[0..count), out[1] = s[1] (out: mapped host memory)
hipError_t cg_report(const double *part, int count, const double *s, double *out, hipStream_t st);

}  // namespace dev
}  // namespace csrk
