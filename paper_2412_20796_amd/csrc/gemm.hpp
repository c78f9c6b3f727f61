// GEMMs with gathered operands and fused epilogues, and split-K weight
// gradients (gfx950).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

namespace chg {

// ---------------------------------------------------------------------------
// Weights as the B operand of the matrix products.
//
// An fp32 number is the sum of three bf16 numbers, x = h + m + l, each the
// rounded remainder of the ones before it (8 significand bits each: |m| <=
// 2^-8 |x|, |l| <= 2^-17 |x|). The products run on the bf16 matrix cores as
// the six terms hh + hm + mh + hl + lh + mm; the terms left out are at most
// 2^-24 of |x y| (2^-27.5 rms; the rounding of one fp32 product is at most
// 2^-24, 2^-25.6 rms). Six bf16 passes take 6/16 of the fp32 matrix cores'
// time.
// These matrix cores cut the bits of a small addend that fall below the sum
// towards minus infinity, half a last place on average: nothing in one
// element, but the same sign in every element, so that a gradient summed over
// 50,000 rows was off by 2e-6 of its size where fp32 products gave 7e-7.
// Odd rows are therefore multiplied with -1 and their results turned back,
// which gives their errors the other sign.
// The six terms of a step share an accumulator; a sum of one step (at most 16
// deep) keeps hh apart from the small terms, whose cut is then 2^-8 as large,
// and adds the two at the end. Error of 262,144 sums of k products of random
// numbers against 64 bits, rms relative to the rms sum:
//   k                       1        2        16       31       64       512
//   fp32 matrix cores       2.5e-8   2.9e-8   7.4e-8   1.0e-7   1.5e-7   4.0e-7
//   one accumulator         3.3e-8   3.3e-8   3.3e-8   7.0e-8   1.1e-7   3.4e-7
//   small terms apart       2.6e-8   2.6e-8   3.2e-8   3.9e-8   4.7e-8   1.2e-7
// (Apart in every step, the registers cost k_gemm_p 5 to 15 % and k_gemm_k
// its second block a compute unit.)
// A part of an infinite x, or of a finite one above the largest bf16 number
// (3.39e38), is not finite. A wavefront looks at its tile when it is done and
// forms one with a value that is not finite again with fp32 products, so that
// the range and the infinities are those of fp32. (Of operands below 2^-110
// the bits under 2^-126 are lost.)
//
// The weights are split once a pass: a matrix is packed, as B (k, n) =
// W[k][n] and, for backward passes, as W[n][k], into tiles of 16 k x 32
// columns in fragment order, three planes (h, m, l) of 64 lanes x 8 values
// (lane l: column l % 32, k = 8 (l / 32) ..), so that a wavefront reads a
// plane as one contiguous kilobyte. k and columns past the matrix are zero.
// ---------------------------------------------------------------------------
constexpr int kPackTile = 3 * 64;  // 16-byte pieces of a tile
struct PackMat {
  int64_t off;      // first value of the matrix in the aligned weight copy
  int64_t src;      // and in the public layout
  int rows, cols;
  int64_t n0, t0;   // first tile of W[k][n] and of W[n][k]
};
struct PackTable {
  std::vector<PackMat> m;  // in order of `off`
  int64_t n_tiles = 0, t_tiles = 0;  // t tiles follow the n tiles
  void add(int64_t off, int64_t src, int rows, int cols);
  void finish();
};
// Packs every matrix (with_t: also the transposes) of the weights `src`
// (public layout) into `out`.
int pack_weights(const PackTable& t, const float* src, uint4* out, bool with_t, hipStream_t st);

// One K-segment of an NN product: rows of A (gathered by the problem's
// a_rows) times B. B element (k, n) = trans ? B[n*ldb + k] : B[k*ldb + n],
// B a block of a packed weight matrix whose first column (trans: row) is a
// multiple of 32 and first row (trans: column) a multiple of 16.
struct GemmSeg {
  const float* A;
  int lda;
  int a_col;  // first column of A used by this segment
  int K;
  const float* B;
  int ldb;
  int trans;
  // set by gemm_resolve
  const uint4* Bp;  // packed tile of column 0, k 0
  int bnt;          // tiles from one 32-column group to the next
  int ks0;          // 16-deep steps of the segments before
};

enum GemmAct { ACT_NONE = 0, ACT_SILU_OUT = 1, ACT_DSILU_MUL = 2 };

// C[c_rows(r), c] (+)= sum_seg A[a_rows(r), a_col + k] B(k, c) + bias[c]
//                      + res[res_rows(r), c]
// ACT_SILU_OUT: also C2[r, c] = silu(value) (C may then be null: not stored).
// ACT_DSILU_MUL: value *= silu'(mul[r, c]) before bias/adds (backward of an
//                activation; use without bias/adds/res).
struct GemmProblem {
  int M, N;
  const int* a_rows;
  int nseg;
  GemmSeg seg[4];
  const float* bias;
  const float* res;
  int res_ld;
  const int* res_rows;
  float* C;
  int ldc;
  const int* c_rows;
  int accumulate;
  int act;
  float* C2;
  int ldc2;
  const float* mul;
  int mul_ld;
  int nks;  // 16-deep steps (set by gemm_resolve)
};

constexpr int kMaxGemmProblems = 6;
struct GemmBatch {
  int n;
  GemmProblem p[kMaxGemmProblems];
};

// The packed tiles of a problem's weights: `P` is the aligned weight copy that
// its B pointers point into.
int gemm_resolve(GemmProblem& p, const PackTable& t, const float* P, const uint4* packed);
int gemm_launch(const GemmBatch& b, hipStream_t st, const char* tag);

// dW[m, n] (+)= sum_r X[x_rows(r), x_col + m] * Y[y_rows(r), y_col + n]
// over r in [0, R); X == nullptr means a single column of ones (M = 1, the
// bias gradient). Deterministic: per-chunk partials, then an ordered fp64 sum.
struct TnProblem {
  int R, M, N;
  const float* X;
  int ldx, x_col;
  const int* x_rows;
  const float* Y;
  int ldy, y_col;
  const int* y_rows;
  float* out;  // out[m * ld_out + n] += result
  int ld_out;
  // optional column split: columns [q*owidth, (q+1)*owidth) go to outs[q]
  // (outs[0] unused: out), owidth = 0 means a single output
  int owidth;
  float* outs[4];
};

constexpr int kMaxTnProblems = 16;
struct TnBatch {
  int n;
  TnProblem p[kMaxTnProblems];
};

// part: scratch of part_cap floats.
int tn_launch(const TnBatch& b, float* part, int64_t part_cap, hipStream_t st, const char* tag);

struct ReduceJob {
  const float* part;
  int nchunks;
  int64_t stride;
  int count;
  float* out;
};
constexpr int kMaxReduceJobs = 20;
struct ReduceJobs {
  int n;
  ReduceJob j[kMaxReduceJobs];
};
// Up to kMaxReduceJobs independent reductions in two launches (32 ordered
// group sums, then their ordered sum); scratch: n * 32 * 1024 doubles.
int reduce_rows_multi(const ReduceJobs& J, double* scratch, hipStream_t st);

// out[k] += sum_c part[c*stride + k] (k < count), in a fixed order, in fp64.
// scratch: 32 * count doubles.
int reduce_rows_launch(const float* part, int nchunks, int64_t stride, int count, float* out, double* scratch,
                       hipStream_t st);

}  // namespace chg
