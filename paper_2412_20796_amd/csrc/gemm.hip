// Matrix products of the per-atom, per-edge and per-angle linear layers.
//
// k_gemm_p: products with a weight block, at most 128 deep, over many rows;
// k_gemm_k: the same over few rows or deeper, k split over wavefronts. Both
// multiply split operands on the bf16 matrix cores (see gemm.hpp). k_tn:
// split-K weight-gradient products X^T Y. Operand rows may be gathered
// through an index array (edge -> source atom, bond -> edge, angle -> bond),
// so the concatenated GatedMLP inputs of Eq. (4)-(6) never exist in memory:
// the products of their blocks are summed in the epilogue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "common.hpp"
#include "gemm.hpp"
#include "split.hpp"

namespace chg {

namespace {

__device__ __forceinline__ float sigm(float x) { return 1.0f / (1.0f + __expf(-x)); }

typedef float v16f __attribute__((ext_vector_type(16)));

// Epilogue of one row and 4 consecutive columns: activation, bias,
// residual, optional accumulation, 16-byte stores when aligned.
__device__ __forceinline__ bool gemm_cvec(const GemmProblem& P) {
  return (P.ldc & 3) == 0 && ((uintptr_t)P.C & 15) == 0 &&
         (!P.res || ((P.res_ld & 3) == 0 && ((uintptr_t)P.res & 15) == 0)) &&
         (P.act != ACT_DSILU_MUL || ((P.mul_ld & 3) == 0 && ((uintptr_t)P.mul & 15) == 0)) &&
         (P.act != ACT_SILU_OUT || ((P.ldc2 & 3) == 0 && ((uintptr_t)P.C2 & 15) == 0));
}

__device__ __forceinline__ void gemm_store4(const GemmProblem& P, int row, int col, float4 sv, bool cvec) {
  if (row >= P.M || col >= P.N) return;
  float v[4] = {sv.x, sv.y, sv.z, sv.w};
  const int64_t rr = P.res ? (P.res_rows ? P.res_rows[row] : row) * (int64_t)P.res_ld : 0;
  const int64_t cr = (P.c_rows ? P.c_rows[row] : row) * (int64_t)P.ldc;
  if (cvec && col + 3 < P.N) {
    if (P.act == ACT_DSILU_MUL) {
      const float4 x4 = *reinterpret_cast<const float4*>(P.mul + (int64_t)row * P.mul_ld + col);
      const float xs[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float sg = sigm(xs[u]);
        v[u] *= sg * (1.0f + xs[u] * (1.0f - sg));
      }
    }
    if (P.bias)
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += P.bias[col + u];
    if (P.res) {
      const float4 r4 = *reinterpret_cast<const float4*>(P.res + rr + col);
      v[0] += r4.x; v[1] += r4.y; v[2] += r4.z; v[3] += r4.w;
    }
    float4* dst = reinterpret_cast<float4*>(P.C + cr + col);
    if (P.accumulate) {
      const float4 o = *dst;
      v[0] += o.x; v[1] += o.y; v[2] += o.z; v[3] += o.w;
    }
    if (P.C) *dst = make_float4(v[0], v[1], v[2], v[3]);
    if (P.act == ACT_SILU_OUT)
      *reinterpret_cast<float4*>(P.C2 + (int64_t)row * P.ldc2 + col) =
          make_float4(v[0] * sigm(v[0]), v[1] * sigm(v[1]), v[2] * sigm(v[2]), v[3] * sigm(v[3]));
    return;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int cc = col + u;
    if (cc >= P.N) break;
    float x = v[u];
    if (P.act == ACT_DSILU_MUL) {
      const float m = P.mul[(int64_t)row * P.mul_ld + cc];
      const float sg = sigm(m);
      x *= sg * (1.0f + m * (1.0f - sg));
    }
    if (P.bias) x += P.bias[cc];
    if (P.res) x += P.res[rr + cc];
    float* dst = P.C + cr + cc;
    if (P.accumulate) x += *dst;
    if (P.C) *dst = x;
    if (P.act == ACT_SILU_OUT) P.C2[(int64_t)row * P.ldc2 + cc] = x * sigm(x);
  }
}

// segment of a 16-deep step (uniform over the wavefront)
__device__ __forceinline__ int seg_of(const GemmProblem& P, int ks) {
  int s = 0;
  while (s + 1 < P.nseg && ks >= P.seg[s + 1].ks0) ++s;
  return s;
}

// The sign that odd rows are multiplied with (see gemm.hpp): `flip_odd` for a
// lane that holds row lane % 32 of A, `unflip` for a 32 x 32 accumulator,
// whose value j belongs to row 8 (j / 4) + 4 (lane / 32) + j % 4.
__device__ __forceinline__ void flip_odd(float (&v)[8], int lane) {
  const unsigned s = (unsigned)lane << 31;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(__float_as_uint(v[e]) ^ s);
}
__device__ __forceinline__ void unflip(v16f& acc) {
#pragma unroll
  for (int j = 1; j < 16; j += 2) acc[j] = -acc[j];
}

// acc += x y over 16 k; `only`: the one step of its sum, with the small terms
// in an accumulator of their own (see gemm.hpp)
__device__ __forceinline__ void mul_step(const Split8& x, const Split8& y, bool only, v16f& acc) {
  if (!only) {
    mfma_split(x, y, acc, acc);
    return;
  }
  v16f lo;
#pragma unroll
  for (int j = 0; j < 16; ++j) lo[j] = 0.f;
  mfma_split(x, y, acc, lo);
  acc += lo;
}

// this lane's eight A values of a step (its row, k = 16 step + 8 (lane / 32) ..)
__device__ __forceinline__ void load_a(const GemmProblem& P, int ks, int64_t arow, int h, float (&v)[8]) {
  const GemmSeg& S = P.seg[seg_of(P, ks)];
  const int k0 = (ks - S.ks0) * 16, k = k0 + 8 * h;
  const float* p = S.A + arow * S.lda + S.a_col + k;
  if (k0 + 16 <= S.K) {  // uniform
    const f4u a = *reinterpret_cast<const f4u*>(p), b = *reinterpret_cast<const f4u*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = k + e < S.K ? p[e] : 0.f;
  }
}

// 0 x over an accumulator's values, added to s: 0, or NaN where one is not
// finite. An operand's value with a part that is not finite leaves its whole
// row (left) or column (right) of the sums of products so, as part times 0 is
// not finite either: a look at one accumulator and one value of its neighbour
// finds both. The neighbour's other values may be infinite on their own, where
// a product of leading parts overflows (rounded up, by 2^-8 at most).
__device__ __forceinline__ float zero_of(const v16f& x, float s) {
  float t = 0.f;
#pragma unroll
  for (int j = 0; j < 16; j += 2) {
    s = fmaf(x[j], 0.f, s);
    t = fmaf(x[j + 1], 0.f, t);
  }
  return s + t;
}
__device__ __forceinline__ float zero_of_next(const v16f& x, float s) {
  float m = 0.f;
#pragma unroll
  for (int j = 0; j < 16; j += 2) m = fmaxf(fmaxf(fabsf(x[j]), fabsf(x[j + 1])), m);
  return fmaf(x[0], 0.f, fmaf(m, 0.f, s));
}
__device__ __forceinline__ bool any_nan(float s) { return __ballot(s != 0.f) != 0; }

// A wavefront's tile over the steps [lo, hi) with fp32 products, for a tile
// whose split products are not all finite (see gemm.hpp).
__device__ __forceinline__ void gemm_tile_fp32(const GemmProblem& P, int lo, int hi, int64_t arow, int c0, bool two,
                                               int lane, v16f (&acc)[2]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[t][j] = 0.f;
#pragma unroll 1
  for (int ks = lo; ks < hi; ++ks) {
    float a[8];
    load_a(P, ks, arow, lane >> 5, a);
    const GemmSeg& S = P.seg[seg_of(P, ks)];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t == 1 && !two) break;
      float b[8];
      unsplit8(packed8(S.Bp + ((int64_t)(c0 / 32 + t) * S.bnt + ks - S.ks0) * kPackTile + lane), b);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc[t], 0, 0, 0);
    }
  }
}

// the value that lane lr + 4 h holds, for both halves h of a wavefront (all
// lanes active, so that the lanes read from hold it)
__device__ __forceinline__ int row_lane(int v, int lr, int h) {
  const int a = __builtin_amdgcn_readlane(v, lr), b = __builtin_amdgcn_readlane(v, lr + 4);
  return h ? b : a;
}

// The 32 x 32 accumulator tiles of a wavefront (32 rows at r0, NT tiles at
// column c0) to C: lane (c, h) holds column c of rows 8 (j / 4) + 4 h + j % 4,
// so a store instruction writes whole 128-byte pieces of two rows (with the
// operands swapped, a lane has 16 bytes of one row: 32-byte pieces of 32
// rows, 88 -> 116 us for the embeddings of 4,096 atoms).
// A tile's 16 values a lane of the residual, the factor and the old C are all
// loaded before the first of its stores, which they could not pass otherwise.
template <int NT>
__device__ __forceinline__ void gemm_put(const GemmProblem& P, int r0, int c0, const v16f (&acc)[NT],
                                         const float (&bias)[2], int lane) {
  const int c = lane & 31, h = lane >> 5;
  const bool full = r0 + 32 <= P.M && c0 + 32 * NT <= P.N;  // uniform
  const bool plain = full && !P.res_rows && !P.c_rows;
  const int mine = min(r0 + c, P.M - 1);
  const int rr = P.res_rows ? P.res_rows[mine] : mine, cr = P.c_rows ? P.c_rows[mine] : mine;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int col = c0 + 32 * t + c;
    float x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = acc[t][j];
    if (plain) {
      // rows at a fixed distance: one offset a lane, the rest uniform
      if (P.act == ACT_DSILU_MUL) {
        const float* q = P.mul + (int64_t)r0 * P.mul_ld + (4 * h * P.mul_ld + col);
        float m[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) m[j] = q[(8 * (j >> 2) + (j & 3)) * P.mul_ld];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const float sg = sigm(m[j]);
          x[j] *= sg * (1.0f + m[j] * (1.0f - sg));
        }
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] += bias[t];
      if (P.res) {
        const float* q = P.res + (int64_t)r0 * P.res_ld + (4 * h * P.res_ld + col);
        float m[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) m[j] = q[(8 * (j >> 2) + (j & 3)) * P.res_ld];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] += m[j];
      }
      float* d = P.C + (int64_t)r0 * P.ldc + (4 * h * P.ldc + col);
      if (P.accumulate) {
        float m[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) m[j] = d[(8 * (j >> 2) + (j & 3)) * P.ldc];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] += m[j];
      }
      if (P.C)
#pragma unroll
        for (int j = 0; j < 16; ++j) d[(8 * (j >> 2) + (j & 3)) * P.ldc] = x[j];
      if (P.act == ACT_SILU_OUT) {
        float* d2 = P.C2 + (int64_t)r0 * P.ldc2 + (4 * h * P.ldc2 + col);
#pragma unroll
        for (int j = 0; j < 16; ++j) d2[(8 * (j >> 2) + (j & 3)) * P.ldc2] = x[j] * sigm(x[j]);
      }
      continue;
    }
    // gathered or scattered rows, and the edges of C: rows and columns past
    // the end are clamped and not stored
    const bool in = col < P.N;
    const int cl = min(col, P.N - 1);
    auto row = [&](int j) { return r0 + 8 * (j >> 2) + 4 * h + (j & 3); };
    auto row_at = [&](const int* rows, int v, int j) {
      return rows ? row_lane(v, 8 * (j >> 2) + (j & 3), h) : min(row(j), P.M - 1);
    };
    if (P.act == ACT_DSILU_MUL) {
      float m[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) m[j] = P.mul[(int64_t)min(row(j), P.M - 1) * P.mul_ld + cl];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float sg = sigm(m[j]);
        x[j] *= sg * (1.0f + m[j] * (1.0f - sg));
      }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] += bias[t];
    if (P.res) {
      float m[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) m[j] = P.res[(int64_t)row_at(P.res_rows, rr, j) * P.res_ld + cl];
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] += m[j];
    }
    if (P.accumulate) {
      float m[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) m[j] = P.C[(int64_t)row_at(P.c_rows, cr, j) * P.ldc + cl];
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] += m[j];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int64_t at = row_at(P.c_rows, cr, j);
      if (!in || row(j) >= P.M) continue;
      if (P.C) P.C[at * P.ldc + col] = x[j];
      if (P.act == ACT_SILU_OUT) P.C2[(int64_t)row(j) * P.ldc2 + col] = x[j] * sigm(x[j]);
    }
  }
}

// Products over many rows. A block takes 64 columns and keeps their packed
// weights, KS steps of 16 k, in LDS; its four wavefronts walk 32-row tiles: a
// step's eight A values a lane are split and multiplied, and the same
// registers take the values of that step of the next tile (DEEP: of the next
// KS steps), so they are in flight meanwhile. Problems at most 16 KS deep load
// the weights once and run without a further barrier; deeper ones (DEEP) take
// them KS steps at a time through two LDS buffers, the next steps loaded
// straight into LDS while these are multiplied, one barrier a chunk.
// Bound by the latency of the rows of A and of the stores: the two wavefronts
// a SIMD that are there on average wait for memory half of their time (0.47 to
// 0.60 of it by the counters), while the matrix cores are 6 % (k = 64) to 17 %
// (k = 256) busy, the vector unit issues in 17 to 30 % of the cycles and 1.8
// to 2.4 TB/s move. Against the fp32 matrix cores with both operands staged
// through LDS, kernel time: a layer's bond projections of 4,096 atoms (36,300
// x 512 x 64) 52 -> 40 us, its embeddings 115 -> 84 us; wide128's launches of
// k = 128 92-170 -> 89 us; the Eq. 10 block's input gradients (k = 256) of 64
// cells 145 -> 119 us. Blocks: three a compute unit (four for KS = 1, 2);
// with registers for four at KS = 4 the epilogue spilled (37 -> 66 us).
struct GemmPArgs {
  GemmBatch b;
  int block0[kMaxGemmProblems + 1];  // first block of each problem (multiples of 8)
};
template <int KS, bool DEEP>
__global__ void __launch_bounds__(256, KS <= 2 ? 4 : 3) k_gemm_p(GemmPArgs args) {
  int pi = 0;
  while (pi + 1 < args.b.n && (int)blockIdx.x >= args.block0[pi + 1]) ++pi;
  const GemmProblem& P = args.b.p[pi];
  // Workgroups are dealt to the 8 XCDs in turn: the column groups of one row
  // worker sit 8 apart, on one XCD, and its A rows are fetched into one L2.
  const int ncol = (P.N + 63) / 64, nb = args.block0[pi + 1] - args.block0[pi], workers = nb / ncol;
  int bx, by;
  {
    const int p = (int)blockIdx.x - args.block0[pi], j = p >> 3;
    by = j % ncol;
    bx = 8 * (j / ncol) + (p & 7);
  }
  const int c0 = by * 64, ntiles = (P.M + 31) / 32;
  if (bx * 4 >= ntiles) return;  // uniform over the block
  constexpr int kPanel = 2 * KS * kPackTile;
  __shared__ uint4 Bs[(DEEP ? 2 : 1) * kPanel];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nks = P.nks;
  const bool two = c0 + 32 < P.N;  // uniform
  auto load_b = [&](int k0) {
    const int n = min(KS, nks - k0);
    for (int u = tid; u < (two ? 2 : 1) * n * kPackTile; u += 256) {
      const int t = u / (n * kPackTile), ks = (u / kPackTile) % n, o = u % kPackTile;
      const GemmSeg& S = P.seg[seg_of(P, k0 + ks)];
      Bs[(t * KS + ks) * kPackTile + o] = S.Bp[((int64_t)(c0 / 32 + t) * S.bnt + k0 + ks - S.ks0) * kPackTile + o];
    }
  };
  const int step = workers * 4;
  int tile = bx * 4 + wave;
  auto row_of = [&](int t) -> int64_t {
    const int r = min(t * 32 + (lane & 31), P.M - 1);
    return P.a_rows ? P.a_rows[r] : r;
  };
  // A steps in flight: more registers for the eight of KS = 8 would spill
  constexpr int RA = KS < 4 ? KS : 4;
  float a[RA][8];
  int64_t ar = row_of(tile);
#pragma unroll
  for (int ks = 0; ks < RA; ++ks)
    if (ks < nks) load_a(P, ks, ar, h, a[ks]);
  int buf = 0;
  load_b(0);
  __syncthreads();
  if (!DEEP && tile >= ntiles) return;
  float bias[2] = {0.f, 0.f};
  if (P.bias)
#pragma unroll
    for (int t = 0; t < 2; ++t) bias[t] = P.bias[min(c0 + 32 * t + (lane & 31), P.N - 1)];
  auto put = [&](v16f (&acc)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) unflip(acc[t]);
    if (any_nan(zero_of(acc[0], zero_of_next(acc[1], 0.f)))) gemm_tile_fp32(P, 0, nks, row_of(tile), c0, two, lane, acc);
    if (two) {
      gemm_put<2>(P, tile * 32, c0, acc, bias, lane);
    } else {
      const v16f one[1] = {acc[0]};
      gemm_put<1>(P, tile * 32, c0, one, bias, lane);
    }
  };
  // DEEP: the panel of steps k0 .. k0 + KS - 1 straight into LDS, a kilobyte
  // (a plane of a tile) a wavefront at a time; steps and columns past the end
  // are clamped and not used
  auto fetch_b = [&](int k0, int to) {
#pragma unroll
    for (int q = 0; q < 2 * KS * 3 / 4; ++q) {
      const int pc = wave + 4 * q, t = two ? pc / (KS * 3) : 0;
      const int ks = min(k0 + (pc / 3) % KS, nks - 1);
      const GemmSeg& S = P.seg[seg_of(P, ks)];
      const uint4* src = S.Bp + ((int64_t)(c0 / 32 + t) * S.bnt + ks - S.ks0) * kPackTile + 64 * (pc % 3) + lane;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) unsigned*)src,
                                       (__attribute__((address_space(3))) unsigned*)(Bs + to * kPanel + 64 * pc), 16, 0, 0);
    }
  };
  auto mul = [&](const uint4* B, int ks, const Split8& x, v16f (&acc)[2]) {
    const uint4* b0 = B + ks * kPackTile + lane;
    mul_step(x, packed8(b0), KS == 1, acc[0]);
    if (two) mul_step(x, packed8(b0 + KS * kPackTile), KS == 1, acc[1]);
  };
  // (DEEP: every wavefront runs the block's rounds; a tile past the end is
  // clamped rows, not stored)
  for (int base = bx * 4; base < ntiles; base += step, tile += step) {
    if (!DEEP && tile >= ntiles) break;
    const bool more = (DEEP ? base : tile) + step < ntiles;
    v16f acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[t][j] = 0.f;
    if constexpr (!DEEP) {
      const int64_t arn = more ? row_of(tile + step) : ar;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks >= nks) break;
        flip_odd(a[ks % RA], lane);
        const Split8 x = split8(a[ks % RA]);
        // the next step that takes these registers, of this tile or the next
        if (KS > RA && ks + RA < nks) load_a(P, ks + RA, ar, h, a[ks % RA]);
        else load_a(P, ks % RA, arn, h, a[ks % RA]);
        mul(Bs, ks, x, acc);
      }
      ar = arn;
      put(acc);
    } else {
      for (int k0 = 0; k0 < nks; k0 += KS) {
        const bool last = k0 + KS >= nks;
        const uint4* B = Bs + buf * kPanel;
        if (!last || more) fetch_b(last ? 0 : k0 + KS, buf ^ 1);
        const int64_t arn = last && more ? row_of(tile + step) : ar;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          if (k0 + ks >= nks) break;
          flip_odd(a[ks], lane);
          const Split8 x = split8(a[ks]);
          const int nx = last ? ks : k0 + KS + ks;
          if (nx < nks) load_a(P, nx, arn, h, a[ks]);
          mul(B, ks, x, acc);
        }
        // steps of the next tile whose registers this short chunk did not use
        if (last && more)
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            if (k0 + ks >= nks && ks < nks) load_a(P, ks, arn, h, a[ks]);
        if (last) ar = arn;
        // (the other buffer was last read before the barrier before this one)
        buf ^= 1;
        __builtin_amdgcn_s_waitcnt(0);  // the panel is in LDS
        __syncthreads();
      }
      if (tile < ntiles) put(acc);
    }
  }
}

// Products over few rows: each wavefront owns a 32 x 64 tile of C and streams
// both operands from global memory (the packed weights
// as contiguous kilobytes), one step in flight ahead of the matrix cores. The
// WK wavefronts of a tile take contiguous runs of its steps and their partial
// tiles are added in wave order in LDS before the epilogue.
constexpr int kGwWaves = 8;
constexpr int kGwLd = 64 + 4;

template <int WK>
__global__ void __launch_bounds__(512, 2) k_gemm_k(GemmBatch batch) {
  __shared__ __attribute__((aligned(16))) float slot[WK > 1 ? kGwWaves * 32 * kGwLd : 4];
  const GemmProblem& P = batch.p[blockIdx.z];
  constexpr int TPB = kGwWaves / WK;  // row tiles per block
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tl = wave / WK, kp = wave % WK;
  const int r0 = (blockIdx.x * TPB + tl) * 32, n0 = blockIdx.y * 64;
  if ((int)blockIdx.x * TPB * 32 >= P.M || n0 >= P.N) return;  // uniform over the block
  const int lo = kp * P.nks / WK, hi = (kp + 1) * P.nks / WK;
  const int arow_i = min(r0 + c, P.M - 1);
  const int64_t arow = P.a_rows ? P.a_rows[arow_i] : arow_i;
  const bool two = n0 + 32 < P.N;  // uniform
  v16f acc[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[u][j] = 0.f;
  float a[2][8];
  uint4 b[2][2][3];
  auto fetch = [&](int ks, int q) {
    load_a(P, ks, arow, h, a[q]);
    const GemmSeg& S = P.seg[seg_of(P, ks)];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t == 1 && !two) break;
      const uint4* src = S.Bp + ((int64_t)(n0 / 32 + t) * S.bnt + ks - S.ks0) * kPackTile + lane;
#pragma unroll
      for (int pl = 0; pl < 3; ++pl) b[q][t][pl] = src[64 * pl];
    }
  };
  auto compute = [&](int q, bool only = false) {
    flip_odd(a[q], lane);
    const Split8 x = split8(a[q]);
    mul_step(x, as_split8(b[q][0]), only, acc[0]);
    if (two) mul_step(x, as_split8(b[q][1]), only, acc[1]);
  };
  if (r0 < P.M && hi - lo == 1) {
    // apart from the loop, whose second set of operands it does not need
    fetch(lo, 0);
    compute(0, true);
  } else if (r0 < P.M) {
    if (lo < hi) fetch(lo, 0);
    for (int ks = lo; ks < hi; ks += 2) {
      if (ks + 1 < hi) fetch(ks + 1, 1);
      compute(0);
      if (ks + 2 < hi) fetch(ks + 2, 0);
      if (ks + 1 < hi) compute(1);
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) unflip(acc[u]);
  if (any_nan(zero_of(acc[0], zero_of_next(acc[1], 0.f)))) gemm_tile_fp32(P, lo, hi, arow, n0, two, lane, acc);
  if constexpr (WK == 1) {
    if (r0 >= P.M) return;
    float bias[2] = {0.f, 0.f};
    if (P.bias)
#pragma unroll
      for (int t = 0; t < 2; ++t) bias[t] = P.bias[min(n0 + 32 * t + c, P.N - 1)];
    if (two) {
      gemm_put<2>(P, r0, n0, acc, bias, lane);
    } else {
      const v16f one[1] = {acc[0]};
      gemm_put<1>(P, r0, n0, one, bias, lane);
    }
    return;
  }
  // partial tiles -> LDS
  float* my = slot + wave * 32 * kGwLd;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int j = 0; j < 16; ++j) my[(8 * (j >> 2) + 4 * h + (j & 3)) * kGwLd + 32 * u + c] = acc[u][j];
  __syncthreads();
  // wave-ordered sum of each tile's WK partials, epilogue with row-contiguous
  // 4-column pieces: 32 rows x 16 pieces per tile
  const bool cvec = gemm_cvec(P);
  for (int q = tid; q < TPB * 32 * 16; q += 512) {
    const int t = q / (32 * 16), rr = (q / 16) % 32, cl = 4 * (q % 16);
    const float* base = slot + (t * WK) * 32 * kGwLd + rr * kGwLd + cl;
    float4 sum = *reinterpret_cast<const float4*>(base);
#pragma unroll
    for (int p = 1; p < WK; ++p) {
      const float4 v = *reinterpret_cast<const float4*>(base + p * 32 * kGwLd);
      sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    gemm_store4(P, (blockIdx.x * TPB + t) * 32 + rr, n0 + cl, sum, cvec);
  }
}

// Packing of the weights: a wavefront a tile.
constexpr int kPackMats = 96;
struct PackArgs {
  int n;
  int64_t tiles;
  struct { int src, rows, cols, tile0; } m[kPackMats];  // tile0: within the launch, ascending
};
template <bool T>
__global__ void __launch_bounds__(256) k_pack_split(PackArgs A, const float* __restrict__ src, uint4* __restrict__ out) {
  const int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tile >= A.tiles) return;
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = A.n;  // matrix with tile0 <= tile
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (A.m[mid].tile0 <= tile) lo = mid;
    else hi = mid;
  }
  const auto& M = A.m[lo];
  const int K = T ? M.cols : M.rows, N = T ? M.rows : M.cols;
  const int nks = (K + 15) / 16, l = (int)(tile - M.tile0);
  const int n = (l / nks) * 32 + (lane & 31), k0 = (l % nks) * 16 + 8 * (lane >> 5);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = k0 + e;
    v[e] = n < N && k < K ? src[M.src + (T ? (int64_t)n * M.cols + k : (int64_t)k * M.cols + n)] : 0.f;
  }
  const Split8 x = split8_all(v);
  uint4* o = out + tile * kPackTile + lane;
  o[0] = __builtin_bit_cast(uint4, x.h);
  o[64] = __builtin_bit_cast(uint4, x.m);
  o[128] = __builtin_bit_cast(uint4, x.l);
}

struct TnPlan {
  TnProblem p;
  int vx, vy;            // fragment widths: a wave tile is 32 vx x 32 vy
  int tiles_m, tiles_n;  // wave tiles per chunk (tiles_m = 0: column sums only)
  int rpc;               // rows per chunk (a multiple of 64: four wave ranges of 16-row groups)
  int nchunks;
  int block0;            // first block of this problem in the launch
  int has_bias;          // partials carry one more row: the column sums of Y
  float* bout;           // destination of the column sums (split like out)
  int bowidth;
  float* bouts[4];
  int64_t off;  // partial offset; a chunk's partial is (M + has_bias) x N
};
struct TnLaunch {
  int n;
  TnPlan q[kMaxTnProblems];
};

// Split-K X^T Y without LDS tiles: each wavefront streams its own row range
// and loads its fragments straight from global memory, 16 rows a step: lane
// half h supplies rows 8 h .. 8 h + 7; lane c = lane % 32 holds columns
// vx c + v (v < vx) of the X rows and vy c + u of the Y rows, so wave tile v
// of X and u of Y are column-interleaved and the loads are 4- or 8-byte
// vectors. Both
// operands are split into three bf16 parts and multiplied on the bf16 matrix
// cores (see gemm.hpp; odd wavefronts multiply -X, so that the one-sided
// rounding cancels in the block's sum; a range's last step, of fewer than 16
// rows, which may be its only one, keeps the small terms apart: in every step
// that took 242 registers for 181, no block of the kernels this one overlaps
// with fitted beside it, and its launches went from 266 to 362 us a step on 40
// crystals of 1,076 atoms). The next steps' rows are loaded while a step is
// multiplied. The four wavefronts of a block take consecutive
// quarters of the block's rows; their tiles are added in wave order in LDS.
// A problem with a bias row also sums the Y columns (the bias gradient of a
// layer whose weight gradient is X^T Y).
// Bound by the vector instructions that split the operands (about 230 a step
// against 24 matrix instructions of 32 cycles) and, beside the gate kernels,
// by the compute units those leave. Against the fp32 matrix cores (64 x 128
// wave tiles on large launches): wide128 step 21.9 -> 19.8 ms, 64 tail cells
// with the Eq. 10 block 4.13 -> 3.87 ms, conservative training 6.87 -> 6.58.
// ROLE only names the instantiation (1: interaction-block weight gradients).
// reduction buffer: two wave tiles and four wavefronts' column sums
constexpr int kTnRedFloats = 2 * 64 * 64 + 4 * 64;
constexpr int kTnBuffers = 2;
constexpr int kTnSlots = 2 * 256;  // resident blocks
// Rows per split-K chunk at most: the eight output tiles of a chunk stream
// the same rows on one XCD, and a chunk of 2048 rows of 384 floats (3 MB)
// stays in that XCD's 4 MB L2 while they do (4480-row chunks measured 1.30
// ms per wide128 layer launch against 1.01 ms).
constexpr int kTnMaxChunkRows = 2048;
// rows of one wavefront's range (a quarter of a chunk): the size of its
// LDS row-index tables
constexpr int kTnWaveRows = kTnMaxChunkRows / 4;
// RIDX: the problem gathers X or Y rows through an index array. The wave
// first copies its range's row indices to LDS (ridx: [2][kTnWaveRows], in the
// reduction buffer, which the block takes over once every wave is past its
// rows), so the fragment loads depend on no other global load and the loads
// of the steps ahead stay in flight.
template <int VX, int VY, bool XFULL, bool YFULL, bool HASX, bool RIDX>
__device__ __forceinline__ void tn_wave(const TnPlan& Q, int chunk, int m0, int n0, bool colsum, float* red,
                                        int* ridx, float* __restrict__ part) {
  // (the plan's fields by value: through a reference the whole argument block
  // went to scratch memory)
  const float *const PX = Q.p.X + (HASX ? Q.p.x_col : 0), *const PY = Q.p.Y + Q.p.y_col;
  const int *const x_rows = Q.p.x_rows, *const y_rows = Q.p.y_rows;
  const int ldx = Q.p.ldx, ldy = Q.p.ldy, PM = Q.p.M, PN = Q.p.N, PR = Q.p.R;
  const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: scalar row range
  const int wr = Q.rpc / 4;
  const int rlo = chunk * Q.rpc + wave * wr;
  const int rhi = min(PR, rlo + wr);
  const int xm = m0 + VX * c, yn = n0 + VY * c;
  v16f acc[VX][VY];
#pragma unroll
  for (int v = 0; v < VX; ++v)
#pragma unroll
    for (int u = 0; u < VY; ++u)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[v][u][j] = 0.f;
  float ysum[VY];
#pragma unroll
  for (int u = 0; u < VY; ++u) ysum[u] = 0.f;
  // register buffers: NB - 1 steps in flight ahead of the matrix cores
  constexpr int NB = kTnBuffers;
  float xf[NB][8][VX], yf[NB][8][VY];
  // Branch-free loads: rows and columns are clamped into the matrix. Columns
  // past M or N only reach outputs that are not stored; rows past the wave's
  // range are zeroed in the range's last step.
  if (RIDX) {
    for (int r = rlo + lane; r < rhi; r += 64) {
      ridx[r - rlo] = x_rows ? x_rows[r] : r;
      ridx[kTnWaveRows + r - rlo] = y_rows ? y_rows[r] : r;
    }
  }
  auto load_x = [&](const float* xp, int i, int b, int col) {
    if (XFULL) {
      const float2 t = *reinterpret_cast<const float2*>(xp + col);
      xf[b][i][0] = t.x;
      xf[b][i][VX - 1] = t.y;
    } else {
#pragma unroll
      for (int v = 0; v < VX; ++v) xf[b][i][v] = xp[col - xm + min(xm + v, PM - 1)];
    }
  };
  auto load_y = [&](const float* yp, int i, int b, int col) {
    if (YFULL) {
      const float2 t = *reinterpret_cast<const float2*>(yp + col);
      yf[b][i][0] = t.x;
      yf[b][i][VY - 1] = t.y;
    } else {
#pragma unroll
      for (int u = 0; u < VY; ++u) yf[b][i][u] = yp[col - yn + min(yn + u, PN - 1)];
    }
  };
  // a lane's offset from the first row of a step (rows in order): the row's
  // own address is uniform, so a load needs no address arithmetic
  const int xo = 8 * h * ldx + xm, yo = 8 * h * ldy + yn;
  // the 16 rows from g, all inside the range (in order: g is uniform)
  auto fetch = [&](int g, int b) {
    if constexpr (!RIDX) {
      const float* xb = HASX ? PX + (int64_t)g * ldx : nullptr;
      const float* yb = PY + (int64_t)g * ldy;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (HASX) load_x(xb + (int64_t)i * ldx, i, b, xo);
        load_y(yb + (int64_t)i * ldy, i, b, yo);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int at = g - rlo + 8 * h + i;
        if (HASX) load_x(PX + (int64_t)ridx[at] * ldx, i, b, xm);
        load_y(PY + (int64_t)ridx[kTnWaveRows + at] * ldy, i, b, yn);
      }
    }
  };
  const unsigned flip = (unsigned)(wave & 1) << 31;
  // (last: the range's last step, of fewer than 16 rows)
  auto compute = [&](int b, bool last) {
    if (colsum) {
#pragma unroll
      for (int u = 0; u < VY; ++u)
        ysum[u] += ((yf[b][0][u] + yf[b][1][u]) + (yf[b][2][u] + yf[b][3][u])) +
                   ((yf[b][4][u] + yf[b][5][u]) + (yf[b][6][u] + yf[b][7][u]));
    }
    if (HASX) {
      Split8 xs[VX];
#pragma unroll
      for (int v = 0; v < VX; ++v) {
        float t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = __uint_as_float(__float_as_uint(xf[b][i][v]) ^ flip);
        xs[v] = split8(t);
      }
#pragma unroll
      for (int u = 0; u < VY; ++u) {
        float t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = yf[b][i][u];
        const Split8 y = split8(t);
#pragma unroll
        for (int v = 0; v < VX; ++v) mul_step(xs[v], y, last, acc[v][u]);
      }
    }
  };
  // the rows left after the range's whole steps: clamped into the range, those
  // past it zeroed (the clamped X row as well, so that a value that is not
  // finite does not reach the sum)
  const int nf = rhi > rlo ? (rhi - rlo) / 16 : 0;
  auto fetch_rest = [&]() {
    const int g = rlo + 16 * nf;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = min(g + 8 * h + i, rhi - 1), at = r - rlo;
      const bool in = g + 8 * h + i < rhi;
      if (HASX) {
        load_x(PX + (int64_t)(RIDX ? ridx[at] : r) * ldx, i, 0, xm);
#pragma unroll
        for (int v = 0; v < VX; ++v) xf[0][i][v] = in ? xf[0][i][v] : 0.f;
      }
      load_y(PY + (int64_t)(RIDX ? ridx[kTnWaveRows + at] : r) * ldy, i, 0, yn);
#pragma unroll
      for (int u = 0; u < VY; ++u) yf[0][i][u] = in ? yf[0][i][u] : 0.f;
    }
  };
  const bool rest = rlo + 16 * nf < rhi;
  // the whole steps, through a ring of NB register buffers with constant
  // indices (a step past the last loads the last one again)
  if (nf > 0) {
    auto step = [&](int s) { return rlo + 16 * min(s, nf - 1); };
#pragma unroll
    for (int b = 0; b < NB - 1; ++b) fetch(step(b), b);
    for (int s = 0; s < nf; s += NB) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        fetch(step(s + b + NB - 1), (b + NB - 1) % NB);
        if (s + b < nf) compute(b, false);
      }
    }
  }
  if (rest) {
    fetch_rest();
    compute(0, true);
  }
  if (HASX) {
    float z = 0.f;
#pragma unroll
    for (int v = 0; v < VX; ++v) {
      z = zero_of(acc[v][0], z);
      if (VY > 1) z = zero_of_next(acc[v][VY - 1], z);
    }
    if (any_nan(z)) {  // with fp32 products (see gemm.hpp)
#pragma unroll
      for (int v = 0; v < VX; ++v)
#pragma unroll
        for (int u = 0; u < VY; ++u)
#pragma unroll
          for (int j = 0; j < 16; ++j) acc[v][u][j] = 0.f;
#pragma unroll 1
      for (int s = 0; s < nf + (rest ? 1 : 0); ++s) {
        if (s < nf) fetch(rlo + 16 * s, 0);
        else fetch_rest();
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int v = 0; v < VX; ++v)
#pragma unroll
            for (int u = 0; u < VY; ++u)
              acc[v][u] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(__float_as_uint(xf[0][i][v]) ^ flip),
                                                               yf[0][i][u], acc[v][u], 0, 0, 0);
      }
    }
  }
  // the row-index tables share this LDS: every wavefront is past its rows
  if (RIDX) __syncthreads();
  constexpr int TILE = VX * VY * 16 * 64, CS = 32 * VY;  // a wave tile; a wavefront's column sums
  // column sums: the two lane halves hold different rows of the same column
  if (colsum) {
#pragma unroll
    for (int u = 0; u < VY; ++u) ysum[u] += __shfl_xor(ysum[u], 32);
    if (h == 0) {
#pragma unroll
      for (int u = 0; u < VY; ++u) red[2 * TILE + wave * CS + u * 32 + c] = ysum[u];
    }
  }
  // wave tiles added in the order (w0 + w1) + (w2 + w3)
  auto put = [&](float* dst) {
#pragma unroll
    for (int v = 0; v < VX; ++v)
#pragma unroll
      for (int u = 0; u < VY; ++u)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          dst[((v * VY + u) * 16 + j) * 64 + lane] = __uint_as_float(__float_as_uint(acc[v][u][j]) ^ flip);
  };
  auto add = [&](const float* src) {
#pragma unroll
    for (int v = 0; v < VX; ++v)
#pragma unroll
      for (int u = 0; u < VY; ++u)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[v][u][j] += src[((v * VY + u) * 16 + j) * 64 + lane];
  };
  if (wave == 1) put(red);
  if (wave == 3) put(red + TILE);
  __syncthreads();
  if (wave == 0) add(red);
  if (wave == 2) add(red + TILE);
  __syncthreads();
  if (wave == 2) put(red);
  __syncthreads();
  if (wave != 0) return;
  add(red);
  const int rows_out = PM + Q.has_bias;
  float* out = part + Q.off + (int64_t)chunk * rows_out * PN;
  if (HASX) {
#pragma unroll
    for (int v = 0; v < VX; ++v)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int m = m0 + VX * (8 * (j >> 2) + 4 * h + (j & 3)) + v;
        if (m >= PM) continue;
#pragma unroll
        for (int u = 0; u < VY; ++u) {
          const int n = yn + u;
          if (n < PN) out[(int64_t)m * PN + n] = acc[v][u][j];
        }
      }
  }
  if (colsum && h == 0) {
    const float* ys = red + 2 * TILE;
#pragma unroll
    for (int u = 0; u < VY; ++u) {
      const int k = u * 32 + c;
      const float s = (ys[k] + ys[CS + k]) + (ys[2 * CS + k] + ys[3 * CS + k]);
      const int n = yn + u;
      if (n < PN) out[(int64_t)PM * PN + n] = s;
    }
  }
}

template <bool RIDX>
__device__ __forceinline__ void tn_dispatch(const TnPlan& Q, int chunk, int m0, int n0, bool colsum, bool xf, bool yf,
                                            float* red, int* ridx, float* __restrict__ part) {
  if (Q.tiles_m == 0) {
    // column sums only
    if (yf) tn_wave<1, 2, false, true, false, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
    else if (Q.vy == 2) tn_wave<1, 2, false, false, false, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
    else tn_wave<1, 1, false, false, false, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
  } else if (Q.vx == 2 && Q.vy == 2) {
    if (xf && yf) tn_wave<2, 2, true, true, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
    else if (xf) tn_wave<2, 2, true, false, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
    else if (yf) tn_wave<2, 2, false, true, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
    else tn_wave<2, 2, false, false, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
  } else if (Q.vx == 2) {
    if (xf) tn_wave<2, 1, true, false, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
    else tn_wave<2, 1, false, false, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
  } else if (Q.vy == 2) {
    if (yf) tn_wave<1, 2, false, true, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
    else tn_wave<1, 2, false, false, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
  } else {
    tn_wave<1, 1, false, false, true, RIDX>(Q, chunk, m0, n0, colsum, red, ridx, part);
  }
}

template <int ROLE>
__global__ void __launch_bounds__(256, 2) k_tn(TnLaunch L, float* __restrict__ part) {
  __shared__ float red[kTnRedFloats];
  static_assert(4 * 2 * kTnWaveRows <= kTnRedFloats, "row-index tables fit in the reduction buffer");
  const int bid = (int)blockIdx.x;
  int k = 0;
  while (k + 1 < L.n && bid >= L.q[k + 1].block0) ++k;
  const TnPlan& Q = L.q[k];
  const int lb = bid - Q.block0;
  const int tiles = max(Q.tiles_m, 1) * Q.tiles_n;
  // The tiles of a row chunk sit 8 block indices apart, so that they run on
  // one XCD (blocks are dealt to the 8 XCDs in turn) and share its L2 for the
  // chunk's rows; chunks after the last full group of 8 keep consecutive tiles.
  const int grouped = (Q.nchunks / 8) * 8 * tiles;
  int chunk, tile;
  if (lb < grouped) {
    const int g = lb / (8 * tiles), rem = lb % (8 * tiles);
    tile = rem / 8;
    chunk = g * 8 + rem % 8;
  } else {
    chunk = (Q.nchunks / 8) * 8 + (lb - grouped) / tiles;
    tile = (lb - grouped) % tiles;
  }
  const int tm = tile / Q.tiles_n, tn = tile % Q.tiles_n;
  const int m0 = tm * 32 * Q.vx, n0 = tn * 32 * Q.vy;
  const bool colsum = Q.has_bias && tm == 0;
  // 8-byte fragment loads where the wave tile lies inside the matrix and
  // the rows are 8-byte aligned
  const TnProblem& P = Q.p;
  const bool xf = Q.vx == 2 && P.X && ((P.ldx | P.x_col) & 1) == 0 && ((uintptr_t)P.X & 7) == 0 && m0 + 64 <= P.M;
  const bool yf = Q.vy == 2 && ((P.ldy | P.y_col) & 1) == 0 && ((uintptr_t)P.Y & 7) == 0 && n0 + 64 <= P.N;
  int* ridx = reinterpret_cast<int*>(red) + (threadIdx.x >> 6) * 2 * kTnWaveRows;
  if (P.x_rows || P.y_rows) tn_dispatch<true>(Q, chunk, m0, n0, colsum, xf, yf, red, ridx, part);
  else tn_dispatch<false>(Q, chunk, m0, n0, colsum, xf, yf, red, ridx, part);
}

// Ordered column sums of chunk partials: 16 wavefronts per block, wave w
// sums chunks w, w+16, ... (fp64), then the 16 partial sums are added in
// wave order. The result is independent of scheduling.
__device__ __forceinline__ double sum_chunks(const float* __restrict__ src, int nchunks, int64_t stride, int w) {
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  int c = w;
  for (; c + 48 < nchunks; c += 64) {
    s0 += (double)src[(int64_t)c * stride];
    s1 += (double)src[(int64_t)(c + 16) * stride];
    s2 += (double)src[(int64_t)(c + 32) * stride];
    s3 += (double)src[(int64_t)(c + 48) * stride];
  }
  for (; c < nchunks; c += 16) s0 += (double)src[(int64_t)c * stride];
  return (s0 + s1) + (s2 + s3);
}

__global__ void __launch_bounds__(1024) k_tn_reduce(TnLaunch L, const float* __restrict__ part) {
  __shared__ double red[16][64];
  const TnPlan& Q = L.q[blockIdx.y];
  const TnProblem& P = Q.p;
  const int64_t mn = (int64_t)(P.M + Q.has_bias) * P.N;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t k = (int64_t)blockIdx.x * 64 + lane;
  if ((int64_t)blockIdx.x * 64 >= mn) return;
  red[w][lane] = k < mn ? sum_chunks(part + Q.off + k, Q.nchunks, mn, w) : 0.0;
  __syncthreads();
  if (w == 0 && k < mn) {
    double s = 0.0;
    for (int q = 0; q < 16; ++q) s += red[q][lane];
    const int m = (int)(k / P.N), n = (int)(k % P.N);
    float* o;
    if (m < P.M) {
      const int q = P.owidth > 0 ? n / P.owidth : 0;
      const int nn = P.owidth > 0 ? n - q * P.owidth : n;
      o = (q == 0 ? P.out : P.outs[q]) + (int64_t)m * P.ld_out + nn;
    } else {
      const int q = Q.bowidth > 0 ? n / Q.bowidth : 0;
      const int nn = Q.bowidth > 0 ? n - q * Q.bowidth : n;
      o = (q == 0 ? Q.bout : Q.bouts[q]) + nn;
    }
    *o = (float)((double)*o + s);
  }
}

// Ordered reduction of chunk partials, two launches. Level 1: block
// (x, g, job) sums the chunks of group g for 64 columns (4 wavefronts, fixed
// order, fp64) into part2[job][g]. Level 2: block (x, job) adds the groups in
// order (4 wavefronts x 8 groups, then the 4 wave sums in order).
__global__ void __launch_bounds__(256) k_reduce_rows1(ReduceJobs J, int groups_max, double* __restrict__ part2_all) {
  __shared__ double red[4][64];
  const ReduceJob& R = J.j[blockIdx.z];
  const int count = R.count, nchunks = R.nchunks;
  const int groups = max(1, min(groups_max, nchunks));
  const int per = (nchunks + groups - 1) / groups;
  if ((int)blockIdx.y >= groups || (int)blockIdx.x * 64 >= count) return;
  double* part2 = part2_all + (int64_t)blockIdx.z * groups_max * 8 * 128;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = blockIdx.x * 64 + lane, g = blockIdx.y;
  const int c0 = g * per, c1 = min(nchunks, c0 + per);
  double s = 0.0;
  if (k < count)
    for (int c = c0 + w; c < c1; c += 4) s += (double)R.part[(int64_t)c * R.stride + k];
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && k < count) part2[(int64_t)g * count + k] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

__global__ void __launch_bounds__(256) k_reduce_rows2(ReduceJobs J, int groups_max, const double* __restrict__ part2_all) {
  __shared__ double red[4][64];
  const ReduceJob& R = J.j[blockIdx.y];
  const int count = R.count;
  const int groups = max(1, min(groups_max, R.nchunks));
  if ((int)blockIdx.x * 64 >= count) return;
  const double* part2 = part2_all + (int64_t)blockIdx.y * groups_max * 8 * 128;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = blockIdx.x * 64 + lane;
  double v[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int q = w + 4 * u;
    v[u] = (k < count && q < groups) ? part2[(int64_t)q * count + k] : 0.0;
  }
  double t = 0.0;
#pragma unroll
  for (int u = 0; u < 8; ++u) t += v[u];
  red[w][lane] = t;
  __syncthreads();
  if (w == 0 && k < count) R.out[k] = (float)((double)R.out[k] + (((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane]));
}


}  // namespace

void PackTable::add(int64_t off, int64_t src, int rows, int cols) {
  PackMat q{off, src, rows, cols, n_tiles, t_tiles};
  n_tiles += cdiv(cols, 32) * cdiv(rows, 16);
  t_tiles += cdiv(rows, 32) * cdiv(cols, 16);
  m.push_back(q);
}
void PackTable::finish() {
  std::sort(m.begin(), m.end(), [](const PackMat& a, const PackMat& b) { return a.off < b.off; });
}

int pack_weights(const PackTable& t, const float* src, uint4* out, bool with_t, hipStream_t st) {
  if ((int)t.m.size() > kPackMats) return fail(CHGNET_EINVAL, "pack: too many weight matrices");
  for (int tr = 0; tr <= (with_t ? 1 : 0); ++tr) {
    PackArgs A{};
    A.tiles = tr ? t.t_tiles : t.n_tiles;
    std::vector<const PackMat*> by(t.m.size());
    for (size_t i = 0; i < t.m.size(); ++i) by[i] = &t.m[i];
    std::sort(by.begin(), by.end(), [&](const PackMat* a, const PackMat* b) { return tr ? a->t0 < b->t0 : a->n0 < b->n0; });
    for (const PackMat* q : by) A.m[A.n++] = {(int)q->src, q->rows, q->cols, (int)(tr ? q->t0 : q->n0)};
    const unsigned blocks = (unsigned)cdiv(A.tiles, 4);
    if (tr) KLAUNCH(st, "k_pack_params", k_pack_split<true><<<blocks, 256, 0, st>>>(A, src, out + t.n_tiles * kPackTile));
    else KLAUNCH(st, "k_pack_params", k_pack_split<false><<<blocks, 256, 0, st>>>(A, src, out));
  }
  return CHGNET_OK;
}

int gemm_resolve(GemmProblem& p, const PackTable& t, const float* P, const uint4* packed) {
  p.nks = 0;
  for (int s = 0; s < p.nseg; ++s) {
    GemmSeg& S = p.seg[s];
    const int64_t off = S.B - P;
    auto it = std::upper_bound(t.m.begin(), t.m.end(), off, [](int64_t o, const PackMat& q) { return o < q.off; });
    if (it == t.m.begin()) return fail(CHGNET_EINVAL, "gemm: weights not packed");
    const PackMat& q = *--it;
    const int64_t at = off - q.off, r = at / q.cols, c = at % q.cols;
    // the block's first k and first column in the packed orientation
    const int64_t k0 = S.trans ? c : r, n0 = S.trans ? r : c;
    const int64_t ks = cdiv(S.trans ? q.cols : q.rows, 16);
    const int64_t kmax = S.trans ? q.cols : q.rows, nmax = S.trans ? q.rows : q.cols;
    if (S.ldb != q.cols || at >= (int64_t)q.rows * q.cols || k0 % 16 || n0 % 32 || k0 + S.K > kmax || n0 + p.N > nmax ||
        (S.K % 16 && k0 + S.K != kmax))
      return fail(CHGNET_EINVAL, "gemm: weight block not aligned to the packed tiles");
    S.bnt = (int)ks;
    S.Bp = packed + ((S.trans ? t.n_tiles + q.t0 : q.n0) + (n0 / 32) * ks + k0 / 16) * kPackTile;
    S.ks0 = p.nks;
    p.nks += (int)cdiv(S.K, 16);
  }
  return CHGNET_OK;
}

int gemm_launch(const GemmBatch& b, hipStream_t st, const char* tag) {
  // Launches with enough 32 x 64 tiles for two wavefronts on every SIMD keep
  // their weights in LDS (k_gemm_p); those with fewer stream them (k_gemm_k),
  // k split over up to eight wavefronts so that the launch has about 2,048 of
  // them. (A product of 14 x 512 x 64 takes 5.4 us so, against 8.7 us with fp32
  // matrix cores and weights read across their rows; ten thousand rows 512
  // deep 14.8 against 28 us.)
  GemmBatch q{};
  int64_t tiles = 0, maxM = 0, maxN = 0;
  int maxks = 0;
  for (int i = 0; i < b.n; ++i) {
    const GemmProblem& p = b.p[i];
    if (p.M <= 0 || p.N <= 0) continue;
    q.p[q.n++] = p;
    tiles += cdiv(p.M, 32) * cdiv(p.N, 64);
    maxM = std::max<int64_t>(maxM, p.M);
    maxN = std::max<int64_t>(maxN, p.N);
    maxks = std::max(maxks, p.nks);
  }
  if (q.n == 0) return CHGNET_OK;
  const unsigned gy = (unsigned)cdiv(maxN, 64);
  if (tiles >= 2048) {
    // sums of one step have an instantiation of their own (see mul_step)
    const int ones = (int)std::count_if(q.p, q.p + q.n, [](const GemmProblem& p) { return p.nks == 1; });
    if (ones > 0 && ones < q.n) {
      GemmBatch part[2] = {};
      for (int i = 0; i < q.n; ++i) {
        GemmBatch& to = part[q.p[i].nks == 1];
        to.p[to.n++] = q.p[i];
      }
      CHG_TRY(gemm_launch(part[0], st, tag));
      return gemm_launch(part[1], st, tag);
    }
    // one resident round of blocks (four or three a compute unit), dealt to
    // the problems by their steps, row workers in multiples of 8 (one per XCD)
    const bool deep = maxks > 8;
    const int64_t slots = (maxks <= 2 ? 4 : 3) * 256;
    int64_t work = 0;
    for (int i = 0; i < q.n; ++i) work += cdiv(q.p[i].M, 32) * cdiv(q.p[i].N, 64) * (q.p[i].nks + 2);
    GemmPArgs A{};
    A.b = q;
    for (int i = 0; i < q.n; ++i) {
      const GemmProblem& p = q.p[i];
      const int64_t ncol = cdiv(p.N, 64), mine = cdiv(p.M, 32) * ncol * (p.nks + 2);
      const int64_t workers = std::min(cdiv(p.M, 128), std::max<int64_t>(1, slots * mine / (work * ncol)));
      A.block0[i + 1] = A.block0[i] + (int)(cdiv(workers, 8) * 8 * ncol);
    }
    const unsigned grid = (unsigned)A.block0[q.n];
    if (maxks == 1) KLAUNCH(st, tag, k_gemm_p<1, false><<<grid, 256, 0, st>>>(A));
    else if (maxks == 2) KLAUNCH(st, tag, k_gemm_p<2, false><<<grid, 256, 0, st>>>(A));
    else if (maxks <= 4) KLAUNCH(st, tag, k_gemm_p<4, false><<<grid, 256, 0, st>>>(A));
    else if (!deep) KLAUNCH(st, tag, k_gemm_p<8, false><<<grid, 256, 0, st>>>(A));
    else KLAUNCH(st, tag, k_gemm_p<4, true><<<grid, 256, 0, st>>>(A));
    return CHGNET_OK;
  }
  int wk = 1;
  while (wk < kGwWaves && tiles * wk < 2048 && 2 * wk <= maxks) wk *= 2;
  const dim3 grid((unsigned)cdiv(maxM, 32 * (kGwWaves / wk)), gy, q.n);
  if (wk == 1) KLAUNCH(st, tag, k_gemm_k<1><<<grid, 512, 0, st>>>(q));
  else if (wk == 2) KLAUNCH(st, tag, k_gemm_k<2><<<grid, 512, 0, st>>>(q));
  else if (wk == 4) KLAUNCH(st, tag, k_gemm_k<4><<<grid, 512, 0, st>>>(q));
  else KLAUNCH(st, tag, k_gemm_k<8><<<grid, 512, 0, st>>>(q));
  return CHGNET_OK;
}


int tn_launch(const TnBatch& b, float* part, int64_t part_cap, hipStream_t st, const char* tag) {
  if (b.n == 0) return CHGNET_OK;
  // A bias problem (X = ones, M = 1) becomes the column-sum row of a weight
  // problem over the same Y rows and columns, so Y is streamed once.
  TnLaunch L{};
  for (int i = 0; i < b.n; ++i) {
    const TnProblem& p = b.p[i];
    if (p.X == nullptr) continue;
    if (p.M <= 0 || p.N <= 0) return fail(CHGNET_EINVAL, "tn: empty output");
    TnPlan& q = L.q[L.n++];
    q = TnPlan{};
    q.p = p;
  }
  for (int i = 0; i < b.n; ++i) {
    const TnProblem& p = b.p[i];
    if (p.X != nullptr) continue;
    if (p.M != 1 || p.N <= 0) return fail(CHGNET_EINVAL, "tn: a problem without X must have one output row");
    TnPlan* host = nullptr;
    for (int j = 0; j < L.n && !host; ++j) {
      const TnProblem& w = L.q[j].p;
      if (!L.q[j].has_bias && w.X && w.R == p.R && w.N == p.N && w.Y == p.Y && w.ldy == p.ldy && w.y_col == p.y_col &&
          w.y_rows == p.y_rows)
        host = &L.q[j];
    }
    if (!host) {
      host = &L.q[L.n++];
      *host = TnPlan{};
      host->p = p;
      host->p.M = 0;
    }
    host->has_bias = 1;
    host->bout = p.out;
    host->bowidth = p.owidth;
    for (int q = 1; q < 4; ++q) host->bouts[q] = p.outs[q];
  }
  int64_t units = 0;
  for (int i = 0; i < L.n; ++i) {
    TnPlan& q = L.q[i];
    q.vx = q.p.M <= 32 ? 1 : 2;
    q.vy = q.p.N <= 32 ? 1 : 2;
    q.tiles_m = q.p.X ? (int)cdiv(q.p.M, 32 * q.vx) : 0;
    q.tiles_n = (int)cdiv(q.p.N, 32 * q.vy);
    units += cdiv(std::max(q.p.R, 0), 64) * std::max(q.tiles_m, 1) * q.tiles_n;
  }
  // about one block per resident slot (two 4-wave blocks per compute
  // unit): fewer, longer blocks measured faster than several rounds
  const int64_t per = std::max<int64_t>(1, cdiv(units, kTnSlots));
  const int rpc = (int)std::min<int64_t>(64 * per, kTnMaxChunkRows);
  int64_t off = 0, blocks = 0, maxmn = 0;
  for (int i = 0; i < L.n; ++i) {
    TnPlan& q = L.q[i];
    q.rpc = rpc;
    q.nchunks = q.p.R > 0 ? (int)cdiv(q.p.R, rpc) : 0;
    q.block0 = (int)blocks;
    q.off = off;
    const int64_t mn = (int64_t)(q.p.M + q.has_bias) * q.p.N;
    off += (int64_t)q.nchunks * mn;
    blocks += (int64_t)q.nchunks * std::max(q.tiles_m, 1) * q.tiles_n;
    maxmn = std::max(maxmn, mn);
  }
  if (off > part_cap) return fail(CHGNET_EWORKSPACE, "split-K partial buffer too small");
  if (blocks > 0x7fffffff) return fail(CHGNET_EINVAL, "tn: too many blocks");
  if (blocks > 0) {
    if (std::string(tag) == "tn_in") KLAUNCH(st, tag, k_tn<1><<<(unsigned)blocks, 256, 0, st>>>(L, part));
    else KLAUNCH(st, tag, k_tn<0><<<(unsigned)blocks, 256, 0, st>>>(L, part));
    KLAUNCH(st, "k_tn_reduce", k_tn_reduce<<<dim3((unsigned)cdiv(maxmn, 64), L.n), 1024, 0, st>>>(L, part));
  }
  return CHGNET_OK;
}

int reduce_rows_multi(const ReduceJobs& J, double* scratch, hipStream_t st) {
  if (J.n == 0) return CHGNET_OK;
  int maxc = 0, maxg = 1;
  for (int i = 0; i < J.n; ++i) {
    if (J.j[i].count > 8 * 128) return fail(CHGNET_EINVAL, "reduce: count too large");
    maxc = std::max(maxc, J.j[i].count);
    maxg = std::max(maxg, std::min(32, J.j[i].nchunks));
  }
  if (maxc == 0) return CHGNET_OK;
  KLAUNCH(st, "k_reduce_rows1", k_reduce_rows1<<<dim3((unsigned)cdiv(maxc, 64), maxg, J.n), 256, 0, st>>>(J, 32, scratch));
  KLAUNCH(st, "k_reduce_rows2", k_reduce_rows2<<<dim3((unsigned)cdiv(maxc, 64), J.n), 256, 0, st>>>(J, 32, scratch));
  return CHGNET_OK;
}

int reduce_rows_launch(const float* part, int nchunks, int64_t stride, int count, float* out, double* scratch,
                       hipStream_t st) {
  ReduceJobs J{};
  J.n = 1;
  J.j[0] = ReduceJob{part, nchunks, stride, count, out};
  return reduce_rows_multi(J, scratch, st);
}

}  // namespace chg
