// Periodic atom graph, bond graph and angle list on gfx950 (Sec. II-B (1)).
//
// Cell-list search: each crystal's cell is cut into n_a slabs per lattice
// axis, each at least r + margin thick (so the neighbours of an atom lie in
// the slabs within K_a = floor((r + margin) n_a / h_a) + 1 of its own, with
// periodic images handled by "virtual" slab indices), atoms are binned by
// their wrapped fractional coordinates into bin-ordered records, and one or
// four wavefronts per atom test all candidates with the exact fp32 inclusion
// expression. The accepted (j, n) keys of an atom are then put in LDS into
// the canonical (j, n1, n2, n3) order, so the output does not depend on the
// order in which atoms landed in their bins. One host wait reads the sizes
// E, B, A back.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <climits>
#include <cmath>
#include <cstring>
#include <mutex>

#include "common.hpp"

namespace chg {

namespace {

constexpr double kMargin = 0.05;      // Angstrom added to the cutoff for binning
constexpr int kMaxK = 64;             // max slab reach per axis
constexpr int kMaxWrap = 200;         // max |cell index| of an input position
constexpr float kMaxCoord = 1.0e4f;   // max |Cartesian coordinate|
constexpr int kMaxEdgesPerAtom = 8192;
constexpr int kImgBias = 512;         // image components stored as n + 512 in 10 bits

enum ErrBits { ERR_Z = 1, ERR_DET = 2, ERR_THIN = 4, ERR_FAR = 8, ERR_PTR = 32 };

struct StructInfo {
  double Linv[9];
  float L[9];
  int nb[3];
  int K[3];
  int bin_base;
  int pad;
};

struct GraphInfo {
  long long n_edges, n_bonds, n_angles;
  int max_count;
  int err;
  unsigned int max_disp2;  // MD neighbour-list reuse: largest squared displacement (fp32 bits)
  int pad;
};

// ---------------------------------------------------------------------------
// The exact fp32 cutoff expression: one rounding per operation, no FMA,
// evaluated in the canonical orientation of the pair {(i, j, n), (j, i, -n)}
// (i < j, or i = j with n lexicographically positive). (r_j + s) - r_i and
// (r_i - s) - r_j round differently, so without a fixed orientation an edge
// near the cutoff could pass while its reverse fails; with it both directions
// get the same D2 and every edge has its reverse.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float pair_d2(int i, int j, const float* ri, const float* rj, int n1, int n2, int n3,
                                         const float* L) {
#pragma clang fp contract(off)
  const bool canon = i < j || (i == j && (n1 > 0 || (n1 == 0 && (n2 > 0 || (n2 == 0 && n3 > 0)))));
  const float sg = canon ? 1.0f : -1.0f;  // exact: m = sg * n
  const float f1 = sg * (float)n1, f2 = sg * (float)n2, f3 = sg * (float)n3;
  const float sx = (f1 * L[0] + f2 * L[3]) + f3 * L[6];
  const float sy = (f1 * L[1] + f2 * L[4]) + f3 * L[7];
  const float sz = (f1 * L[2] + f2 * L[5]) + f3 * L[8];
  const float px = canon ? ri[0] : rj[0], py = canon ? ri[1] : rj[1], pz = canon ? ri[2] : rj[2];
  const float qx = canon ? rj[0] : ri[0], qy = canon ? rj[1] : ri[1], qz = canon ? rj[2] : ri[2];
  const float dx = (qx + sx) - px;
  const float dy = (qy + sy) - py;
  const float dz = (qz + sz) - pz;
  return (dx * dx + dy * dy) + dz * dz;
}

__device__ __forceinline__ int floor_mod(int v, int n) {
  int r = v % n;
  return r < 0 ? r + n : r;
}

__device__ __forceinline__ int find_struct(const int* atom_ptr, int S, int i) {
  int lo = 0, hi = S - 1;  // last s with atom_ptr[s] <= i
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (atom_ptr[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Per-structure setup: inverse lattice, slab counts and reach. One block.
// Inverse lattice, slab counts and reach of structure s (flags bad input).
__device__ StructInfo struct_info(int s, const int* __restrict__ atom_ptr, const float* __restrict__ lattice, float r,
                                  GraphInfo* ginfo) {
  StructInfo si{};
  double L[9];
  for (int k = 0; k < 9; ++k) {
    si.L[k] = lattice[s * 9 + k];
    L[k] = (double)si.L[k];
  }
  // rows a0, a1, a2; cofactor rows give the reciprocal basis
  double c0[3] = {L[4] * L[8] - L[5] * L[7], L[5] * L[6] - L[3] * L[8], L[3] * L[7] - L[4] * L[6]};
  double c1[3] = {L[7] * L[2] - L[8] * L[1], L[8] * L[0] - L[6] * L[2], L[6] * L[1] - L[7] * L[0]};
  double c2[3] = {L[1] * L[5] - L[2] * L[4], L[2] * L[3] - L[0] * L[5], L[0] * L[4] - L[1] * L[3]};
  double det = L[0] * c0[0] + L[1] * c0[1] + L[2] * c0[2];
  int n_s = atom_ptr[s + 1] - atom_ptr[s];
  if (!(fabs(det) >= 1e-6) || n_s < 0) {
    atomicOr(&ginfo->err, n_s < 0 ? ERR_PTR : ERR_DET);
    for (int k = 0; k < 9; ++k) si.Linv[k] = 0.0;
    si.nb[0] = si.nb[1] = si.nb[2] = 1;
    si.K[0] = si.K[1] = si.K[2] = 0;
    return si;
  }
  // frac = cart @ Linv, Linv = L^{-1}; column a of Linv = c_a / det
  for (int row = 0; row < 3; ++row) {
    si.Linv[row * 3 + 0] = c0[row] / det;
    si.Linv[row * 3 + 1] = c1[row] / det;
    si.Linv[row * 3 + 2] = c2[row] / det;
  }
  double vol = fabs(det);
  double h[3];
  const double* cs[3] = {c0, c1, c2};
  for (int a = 0; a < 3; ++a) h[a] = vol / sqrt(cs[a][0] * cs[a][0] + cs[a][1] * cs[a][1] + cs[a][2] * cs[a][2]);
  const double rr = (double)r + kMargin;
  long long nb[3];
  // slabs half a cutoff thick where the cell is at least one cutoff wide: the
  // 5 x 5 x 5 slabs around an atom then hold 0.58 times the candidates of
  // 3 x 3 x 3 slabs of a whole cutoff; in thinner cells, where every image is
  // searched anyway, more slabs would only make the runs shorter
  for (int a = 0; a < 3; ++a) {
    double q = h[a] >= rr ? floor(2.0 * h[a] / rr) : 1.0;
    nb[a] = q < 1.0 ? 1 : (q > 1024.0 ? 1024 : (long long)q);
  }
  long long cap = n_s > 1 ? n_s : 1;
  while (nb[0] * nb[1] * nb[2] > cap) {
    int a = 0;
    if (nb[1] > nb[a]) a = 1;
    if (nb[2] > nb[a]) a = 2;
    nb[a] -= 1;
  }
  bool thin = false;
  for (int a = 0; a < 3; ++a) {
    si.nb[a] = (int)nb[a];
    double kk = floor(rr * (double)nb[a] / h[a]) + 1.0;
    if (kk > kMaxK) { thin = true; kk = 0; }
    si.K[a] = (int)kk;
  }
  if (thin) atomicOr(&ginfo->err, ERR_THIN);
  si.bin_base = 0;
  return si;
}

// More bins than atoms and crystals can only come from a decreasing atom_ptr
// (refused afterwards): every crystal then takes bin 0, so that no bin index
// leaves the scratch arrays. Whole block; returns the number of bins.
__device__ int bins_checked(int nbins, int N, int S, StructInfo* info, GraphInfo* ginfo) {
  if (nbins <= N + S) return nbins;
  if (threadIdx.x == 0) atomicOr(&ginfo->err, ERR_PTR);
  for (int s = threadIdx.x; s < S; s += blockDim.x)
    for (int a = 0; a < 3; ++a) {
      info[s].nb[a] = 1;
      info[s].K[a] = 0;
      info[s].bin_base = 0;
    }
  return 1;
}

__global__ void __launch_bounds__(1024) k_struct_setup(int N, int S, const int* __restrict__ atom_ptr,
                                                       const float* __restrict__ lattice, float r,
                                                       StructInfo* info, int* __restrict__ total_bins,
                                                       GraphInfo* ginfo) {
  __shared__ int scan[1024];
  int carry = 0;  // bins of the structures of earlier rounds
  for (int s0 = 0; s0 < S; s0 += 1024) {
    const int s = s0 + (int)threadIdx.x;
    int bins = 0;
    if (s < S) {
      const StructInfo si = struct_info(s, atom_ptr, lattice, r, ginfo);
      info[s] = si;
      bins = si.nb[0] * si.nb[1] * si.nb[2];
    }
    // exclusive scan of the bin counts over the round (Hillis-Steele in LDS)
    scan[threadIdx.x] = bins;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const int y = threadIdx.x >= (unsigned)off ? scan[threadIdx.x - off] : 0;
      __syncthreads();
      scan[threadIdx.x] += y;
      __syncthreads();
    }
    if (s < S) info[s].bin_base = carry + scan[threadIdx.x] - bins;
    carry += scan[1023];
    __syncthreads();
  }
  __threadfence_block();
  __syncthreads();
  carry = bins_checked(carry, N, S, info, ginfo);
  if (threadIdx.x == 0) *total_bins = carry;
}

// An atom's structure, bin, cell (10 bits an axis: at most 1024 slabs) and
// wrap (floor of the fractional coordinate, |w| <= kMaxWrap, 10 bits an axis
// with a bias of 512).
struct AtomMeta {
  int s, bin, cell, wrap;
};
constexpr int kWrapBias = 512;
__device__ __forceinline__ int pack3(int a, int b, int c) { return a | (b << 10) | (c << 20); }
__device__ __forceinline__ void unpack3(int p, int bias, int (&v)[3]) {
  v[0] = (p & 1023) - bias;
  v[1] = ((p >> 10) & 1023) - bias;
  v[2] = ((p >> 20) & 1023) - bias;
}

__device__ __forceinline__ AtomMeta atom_meta(int i, int s, const float* __restrict__ pos, const int* __restrict__ Z,
                                              const StructInfo* __restrict__ info, GraphInfo* ginfo) {
  const int z = Z[i];
  int err = z < 1 || z > 94 ? ERR_Z : 0;
  const StructInfo& si = info[s];
  const float p[3] = {pos[i * 3 + 0], pos[i * 3 + 1], pos[i * 3 + 2]};
  int c[3], w[3];
  for (int a = 0; a < 3; ++a) {
    if (!(fabsf(p[a]) <= kMaxCoord)) err |= ERR_FAR;
    double f = (double)p[0] * si.Linv[0 * 3 + a] + (double)p[1] * si.Linv[1 * 3 + a] + (double)p[2] * si.Linv[2 * 3 + a];
    double fl = floor(f);
    if (!(fabs(fl) <= kMaxWrap)) { err |= ERR_FAR; f = fl = 0.0; }
    double fr = f - fl;
    int ca = (int)floor(fr * si.nb[a]);
    ca = ca < 0 ? 0 : (ca >= si.nb[a] ? si.nb[a] - 1 : ca);
    c[a] = ca;
    w[a] = (int)fl;
  }
  if (err) atomicOr(&ginfo->err, err);
  return AtomMeta{s, si.bin_base + (c[0] * si.nb[1] + c[1]) * si.nb[2] + c[2], pack3(c[0], c[1], c[2]),
                  pack3(w[0] + kWrapBias, w[1] + kWrapBias, w[2] + kWrapBias)};
}

__global__ void k_atom_bin(int N, int S, const int* __restrict__ atom_ptr, const float* __restrict__ pos,
                           const int* __restrict__ Z, const StructInfo* __restrict__ info, AtomMeta* __restrict__ meta,
                           int* __restrict__ bin_count, GraphInfo* ginfo) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const AtomMeta m = atom_meta(i, find_struct(atom_ptr, S, i), pos, Z, info, ginfo);
  meta[i] = m;
  atomicAdd(&bin_count[m.bin], 1);
}

// Scans in a fixed order: a wavefront's inclusive scan by lane shuffles,
// and a block's exclusive scan from its wavefronts' totals (sh: 17 slots of
// shared memory; every thread of the block takes part).
template <class T>
__device__ __forceinline__ T wave_incl_scan(T v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  return v;
}
template <class T>
__device__ __forceinline__ T block_excl_scan(T v, T* sh, T& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (int)(blockDim.x + 63) >> 6;
  const T inc = wave_incl_scan(v, lane);
  if (lane == 63) sh[w] = inc;
  __syncthreads();
  if (w == 0) {
    const T t = lane < nw ? sh[lane] : T(0);
    const T ti = wave_incl_scan(t, lane);
    if (lane < nw) sh[lane] = ti - t;
    if (lane == nw - 1) sh[16] = ti;
  }
  __syncthreads();
  const T r = sh[w] + inc - v;
  total = sh[16];
  __syncthreads();
  return r;
}

// Exclusive scan of n ints with one 1024-thread block (any n), 8 consecutive
// values a thread per pass. out[n] = total.
constexpr int kScanPer = 8;
__global__ void __launch_bounds__(1024) k_scan_single(int n, const int* __restrict__ in, int* __restrict__ out) {
  __shared__ int sh[17];
  int carry = 0;
  for (int base = 0; base < n; base += (int)blockDim.x * kScanPer) {
    const int i0 = base + (int)threadIdx.x * kScanPer;
    int v[kScanPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      v[q] = i0 + q < n ? in[i0 + q] : 0;
      sum += v[q];
    }
    int total;
    int run = carry + block_excl_scan(sum, sh, total);
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      if (i0 + q < n) out[i0 + q] = run;
      run += v[q];
    }
    carry += total;
  }
  if (threadIdx.x == 0) out[n] = carry;
}

// Bin-ordered record of an atom: position and index, and its wrap.
__device__ __forceinline__ void put_record(int slot, int i, int wrap, const float* __restrict__ pos,
                                           float4* __restrict__ bin_xyzj, int* __restrict__ bin_wrap) {
  bin_xyzj[slot] = make_float4(pos[i * 3 + 0], pos[i * 3 + 1], pos[i * 3 + 2], __int_as_float(i));
  bin_wrap[slot] = wrap;
}

__global__ void k_bin_fill(int N, const AtomMeta* __restrict__ meta, const int* __restrict__ bin_start,
                           int* __restrict__ bin_cursor, const float* __restrict__ pos, float4* __restrict__ bin_xyzj,
                           int* __restrict__ bin_wrap) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const AtomMeta m = meta[i];
  const int slot = atomicAdd(&bin_cursor[m.bin], 1);
  put_record(bin_start[m.bin] + slot, i, m.wrap, pos, bin_xyzj, bin_wrap);
}

// The whole binning (structure setup, bin counts, their scan, the records) in
// one block, with the counters in LDS, for batches whose bins fit there: each
// step is latency-bound at these sizes, and the five launches it takes the
// place of (each a few microseconds at least, kept below for larger batches)
// summed to 46 us on 128 crystals of 5,541 atoms, now 20 us, and to 29 us on
// one crystal of 4,096, now 15 us (kernel time under the profiler).
constexpr int kBinMax = 16384;      // bins (at most N + S)
constexpr int kBinAtomsPer = 8;     // atoms a thread at most
constexpr int kBinStructs = 2048;   // crystals whose offsets are searched in LDS
__global__ void __launch_bounds__(1024) k_bin(int N, int S, const int* __restrict__ atom_ptr,
                                              const float* __restrict__ pos, const int* __restrict__ Z,
                                              const float* __restrict__ lattice, float r, StructInfo* info,
                                              AtomMeta* __restrict__ meta, int* __restrict__ bin_start,
                                              float4* __restrict__ bin_xyzj, int* __restrict__ bin_wrap,
                                              GraphInfo* ginfo) {
  __shared__ int cnt[kBinMax];
  __shared__ int ptr_lds[kBinStructs + 1];
  __shared__ int sh[17];
  const int tid = threadIdx.x;
  if (S <= kBinStructs)
    for (int s = tid; s <= S; s += 1024) ptr_lds[s] = atom_ptr[s];
  if (tid == 0) *ginfo = GraphInfo{};
  __threadfence_block();
  __syncthreads();
  int nbins = 0;
  for (int s0 = 0; s0 < S; s0 += 1024) {
    const int s = s0 + tid;
    int bins = 0;
    StructInfo si{};
    if (s < S) {
      si = struct_info(s, atom_ptr, lattice, r, ginfo);
      bins = si.nb[0] * si.nb[1] * si.nb[2];
    }
    int total;
    const int base = nbins + block_excl_scan(bins, sh, total);
    if (s < S) {
      si.bin_base = base;
      info[s] = si;
    }
    nbins += total;
  }
  __threadfence_block();
  __syncthreads();
  nbins = bins_checked(nbins, N, S, info, ginfo);
  for (int b = tid; b < nbins; b += 1024) cnt[b] = 0;
  __threadfence_block();
  __syncthreads();
  int bin[kBinAtomsPer], slot[kBinAtomsPer], wrap[kBinAtomsPer];
#pragma unroll
  for (int q = 0; q < kBinAtomsPer; ++q) {
    const int i = tid + 1024 * q;
    bin[q] = -1;
    if (i < N) {
      const int st = S <= kBinStructs ? find_struct(ptr_lds, S, i) : find_struct(atom_ptr, S, i);
      const AtomMeta m = atom_meta(i, st, pos, Z, info, ginfo);
      meta[i] = m;
      bin[q] = m.bin;
      wrap[q] = m.wrap;
      slot[q] = atomicAdd(&cnt[m.bin], 1);
    }
  }
  __syncthreads();
  // exclusive scan of the counts, in place
  int carry = 0;
  for (int base = 0; base < nbins; base += 1024 * kScanPer) {
    const int i0 = base + tid * kScanPer;
    int v[kScanPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      v[q] = i0 + q < nbins ? cnt[i0 + q] : 0;
      sum += v[q];
    }
    int total;
    int run = carry + block_excl_scan(sum, sh, total);
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      if (i0 + q < nbins) {
        cnt[i0 + q] = run;
        bin_start[i0 + q] = run;
      }
      run += v[q];
    }
    carry += total;
  }
  if (tid == 0) bin_start[nbins] = carry;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kBinAtomsPer; ++q)
    if (bin[q] >= 0) put_record(cnt[bin[q]] + slot[q], tid + 1024 * q, wrap[q], pos, bin_xyzj, bin_wrap);
}

struct SearchArgs {
  int N;
  float rc2_atom, rc2_bond;
  const float* pos;
  const StructInfo* info;
  const AtomMeta* meta;
  const int* bin_start;
  const float4* bin_xyzj;
  const int* bin_wrap;
};

// Calls f(j, n1, n2, n3, d2, pass) on the lane that holds candidate (j, n) of
// atom i, once per 64 candidates of the calling wavefront (pass: it is within
// the atom cutoff; lanes past the end call with pass = false). The candidates
// are the atoms of the (2K+1)^3 virtual slabs around the atom's own. Bins of
// one (slab 0, slab 1) pair that lie in one image along axis 2 are contiguous
// in the bin order, so they form one run of records; a lane sizes one run, a
// wavefront scans 64 of them, and the flattened candidates are dealt 64 at a
// time: each run's lane sends its number to the lane that holds the run's
// first candidate, and a lane's run is the nearest such mark at or below it.
// Bound by the latency of its chain of loads: one 16-byte record a candidate
// (in place of three dependent loads through the atom's index) and two groups
// in flight (counting 4,096 atoms: 45 us with a block an atom, 22 us with a
// group at a time, 13 us so, with the finer slabs of struct_info).
// The W wavefronts of an atom take every W-th group of 64. No block barrier.
template <int W, class F>
__device__ __forceinline__ void wave_search(const SearchArgs& A, int i, int w, F&& f) {
  const int lane = threadIdx.x & 63;
  const AtomMeta me = A.meta[i];
  const StructInfo& si = A.info[me.s];
  float L[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) L[k] = si.L[k];
  const float ri[3] = {A.pos[i * 3 + 0], A.pos[i * 3 + 1], A.pos[i * 3 + 2]};
  int ci[3], wi[3];
  unpack3(me.cell, 0, ci);
  unpack3(me.wrap, kWrapBias, wi);
  const int nb0 = si.nb[0], nb1 = si.nb[1], nb2 = si.nb[2], K0 = si.K[0], K1 = si.K[1], K2 = si.K[2];
  const int w1 = 2 * K1 + 1;
  const int zlo = ci[2] - K2, zhi = ci[2] + K2;
  const int m2lo = (zlo - floor_mod(zlo, nb2)) / nb2, m2hi = (zhi - floor_mod(zhi, nb2)) / nb2;
  const int nz = m2hi - m2lo + 1;
  const int nruns = (2 * K0 + 1) * w1 * nz;
  for (int v0 = 0; v0 < nruns; v0 += 64) {
    const int v = v0 + lane;
    int cnt = 0, lo = 0, mp = 0;
    if (v < nruns) {
      const int pl = v / nz, m2 = m2lo + v % nz;
      const int x0 = ci[0] + pl / w1 - K0, b0 = floor_mod(x0, nb0);
      const int x1 = ci[1] + pl % w1 - K1, b1 = floor_mod(x1, nb1);
      const int base = si.bin_base + (b0 * nb1 + b1) * nb2;
      lo = A.bin_start[base + max(zlo - m2 * nb2, 0)];
      cnt = A.bin_start[base + min(zhi - m2 * nb2, nb2 - 1) + 1] - lo;
      // |m| is at most K / nb + 1 <= 65 along an axis
      mp = pack3((x0 - b0) / nb0 + kWrapBias, (x1 - b1) / nb1 + kWrapBias, m2 + kWrapBias);
    }
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(incl, off, 64);
      if (lane >= off) incl += y;
    }
    const int total = __shfl(incl, 63, 64), pre = incl - cnt;
    // two groups of 64 at a time, so that their loads overlap
    for (int c0 = 64 * w; c0 < total; c0 += 128 * W) {
      int idx[2], mq[2], wr[2];
      float4 q[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int cu = c0 + 64 * W * u;
        // run that holds candidate cu: the last non-empty one starting at or below it
        const unsigned long long below = __ballot(cnt > 0 && pre <= cu);
        int run = 63 - __clzll((long long)below);
        const bool marked = cnt > 0 && pre > cu && pre < cu + 64;
        // sent to lane pre - cu; a lane that nothing is sent to reads 0 (every
        // lane without a mark sends 0 to lane 0, whose run is `run` anyway)
        const int rec = __builtin_amdgcn_ds_permute(marked ? 4 * (pre - cu) : 0, marked ? lane + 1 : 0);
        const unsigned long long marks =
            __ballot(rec != 0 && lane > 0) & (lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1ull);
        const int other = __shfl(rec, marks ? 63 - __clzll((long long)marks) : 0, 64) - 1;
        if (marks) run = other;
        const int off = __shfl(lo - pre, run, 64);
        mq[u] = __shfl(mp, run, 64);
        // clamped, so that both groups' loads are issued at once
        idx[u] = off + cu + lane;
        if (cu + lane >= total) idx[u] = -1;
        const int at = max(idx[u], 0);
        q[u] = A.bin_xyzj[at];
        wr[u] = A.bin_wrap[at];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (c0 + 64 * W * u >= total) break;  // uniform over the wavefront
        int wj[3], n[3];
        unpack3(wr[u], kWrapBias, wj);
        unpack3(mq[u], kWrapBias, n);
        const int j = __float_as_int(q[u].w);
#pragma unroll
        for (int k = 0; k < 3; ++k) n[k] += wi[k] - wj[k];
        const float rj[3] = {q[u].x, q[u].y, q[u].z};
        const float dd = pair_d2(i, j, ri, rj, n[0], n[1], n[2], L);
        const bool pass = idx[u] >= 0 && dd < A.rc2_atom && !(j == i && n[0] == 0 && n[1] == 0 && n[2] == 0);
        f(j, n[0], n[1], n[2], dd, pass);
      }
    }
  }
}

constexpr int kSearchThreads = 256;

// Edges and bonds of each atom: W wavefronts an atom (four where few atoms
// would leave the chip idle), 4 / W atoms a block.
template <int W>
__global__ void __launch_bounds__(kSearchThreads) k_count(SearchArgs A, int* __restrict__ edge_count,
                                                          int* __restrict__ bond_count) {
  __shared__ int part[4][2];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blockIdx.x * (4 / W) + wave / W;
  int ne = 0, nb = 0;  // of the wavefront
  if (i < A.N)
    wave_search<W>(A, i, wave % W, [&](int, int, int, int, float dd, bool pass) {
      ne += __popcll(__ballot(pass));
      nb += __popcll(__ballot(pass && dd < A.rc2_bond));
    });
  if (W > 1) {
    if ((threadIdx.x & 63) == 0) {
      part[wave][0] = ne;
      part[wave][1] = nb;
    }
    __syncthreads();
    if (wave % W != 0) return;
    for (int q = 1; q < W; ++q) {
      ne += part[wave + q][0];
      nb += part[wave + q][1];
    }
  }
  if (i < A.N && (threadIdx.x & 63) == 0) {
    edge_count[i] = ne;
    bond_count[i] = nb;
  }
}

// Exclusive scans of edge counts, bond counts and k(k-1); totals, the largest
// edge count and (MD) the largest of the N squared displacements in `disp2`
// into ginfo and, if given, its host copy. One block; an atom has fewer than
// 2^18 edges and bonds here or the whole build is refused, so the 8,192 atoms
// of a pass sum to less than 2^31 and one 64-bit scan holds both counts.
__global__ void __launch_bounds__(1024) k_scan_counts(int N, const int* __restrict__ edge_count,
                                                     const int* __restrict__ bond_count, int* __restrict__ edge_ptr,
                                                     int* __restrict__ bond_ptr, long long* __restrict__ angle_base,
                                                     const float* __restrict__ disp2, GraphInfo* ginfo,
                                                     GraphInfo* host) {
  __shared__ unsigned long long sh_eb[17], sh_a[17];
  __shared__ int mx[16];
  __shared__ float md[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  long long ce = 0, cb = 0, ca = 0;
  int my_max = 0;
  float my_d2 = 0.f;
  for (int base = 0; base < N; base += 1024 * kScanPer) {
    const int i0 = base + (int)threadIdx.x * kScanPer;
    int ve[kScanPer], vb[kScanPer];
    unsigned long long seb = 0, sa = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      const bool in = i0 + q < N;
      // (a count past the limit is refused below through max_count)
      ve[q] = in ? min(edge_count[i0 + q], 1 << 18) : 0;
      vb[q] = in ? min(bond_count[i0 + q], 1 << 18) : 0;
      if (disp2 && in) my_d2 = fmaxf(my_d2, disp2[i0 + q]);
      seb += ((unsigned long long)vb[q] << 32) | (unsigned)ve[q];
      sa += (unsigned long long)vb[q] * (vb[q] - 1);
      my_max = max(my_max, ve[q]);
    }
    // block scan of both, two barriers
    const unsigned long long ieb = wave_incl_scan(seb, lane), ia = wave_incl_scan(sa, lane);
    if (lane == 63) {
      sh_eb[w] = ieb;
      sh_a[w] = ia;
    }
    __syncthreads();
    if (w == 0) {
      const unsigned long long t = lane < 16 ? sh_eb[lane] : 0, u = lane < 16 ? sh_a[lane] : 0;
      const unsigned long long ti = wave_incl_scan(t, lane), ui = wave_incl_scan(u, lane);
      if (lane < 16) {
        sh_eb[lane] = ti - t;
        sh_a[lane] = ui - u;
      }
      if (lane == 15) {
        sh_eb[16] = ti;
        sh_a[16] = ui;
      }
    }
    __syncthreads();
    const unsigned long long xeb = sh_eb[w] + ieb - seb, teb = sh_eb[16], ta = sh_a[16];
    long long e0 = ce + (long long)(xeb & 0xffffffffu), b0 = cb + (long long)(xeb >> 32);
    long long a0 = ca + (long long)(sh_a[w] + ia - sa);
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      if (i0 + q < N) {
        edge_ptr[i0 + q] = (int)(e0 < INT_MAX ? e0 : INT_MAX);
        bond_ptr[i0 + q] = (int)(b0 < INT_MAX ? b0 : INT_MAX);
        angle_base[i0 + q] = a0;
      }
      e0 += ve[q];
      b0 += vb[q];
      a0 += (long long)vb[q] * (vb[q] - 1);
    }
    ce += (long long)(teb & 0xffffffffu);
    cb += (long long)(teb >> 32);
    ca += (long long)ta;
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) {
    my_max = max(my_max, __shfl_xor(my_max, off, 64));
    my_d2 = fmaxf(my_d2, __shfl_xor(my_d2, off, 64));
  }
  if (lane == 0) {
    mx[w] = my_max;
    md[w] = my_d2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < 16; ++q) {
      my_max = max(my_max, mx[q]);
      my_d2 = fmaxf(my_d2, md[q]);
    }
    edge_ptr[N] = (int)(ce < INT_MAX ? ce : INT_MAX);
    bond_ptr[N] = (int)(cb < INT_MAX ? cb : INT_MAX);
    angle_base[N] = ca;
    GraphInfo r{};
    r.n_edges = ce;
    r.n_bonds = cb;
    r.n_angles = ca;
    r.max_count = my_max;
    r.err = disp2 ? 0 : ginfo->err;
    r.max_disp2 = __float_as_uint(my_d2);  // non-negative floats order as their bits
    *ginfo = r;
    if (host) *host = r;
  }
}

__device__ __forceinline__ unsigned long long make_key(int j, int n1, int n2, int n3, bool bond) {
  return ((unsigned long long)(unsigned)j << 31) | ((unsigned long long)(n1 + kImgBias) << 21) |
         ((unsigned long long)(n2 + kImgBias) << 11) | ((unsigned long long)(n3 + kImgBias) << 1) |
         (bond ? 1ull : 0ull);
}

// The canonical place of a key among the `count` keys of its atom, and the
// bonds before it (keys are distinct; the bond flag is a key's lowest bit).
__device__ __forceinline__ void write_edge(unsigned long long key, int rank, int brank, int e0, int b0,
                                           int* __restrict__ edge_dst, int* __restrict__ edge_img,
                                           int* __restrict__ bond_edge) {
  const int e = e0 + rank;
  edge_dst[e] = (int)(key >> 31);
  edge_img[e * 3 + 0] = (int)((key >> 21) & 1023) - kImgBias;
  edge_img[e * 3 + 1] = (int)((key >> 11) & 1023) - kImgBias;
  edge_img[e * 3 + 2] = (int)((key >> 1) & 1023) - kImgBias;
  if (key & 1ull) bond_edge[b0 + brank] = e;
}

// Gathers the accepted keys of an atom into LDS (in any order) and writes the
// edges in canonical order and the atom's bond list. A key's place is the
// number of smaller keys, counted against every key (broadcast LDS reads, no
// barrier between steps): about 80-100 keys an atom, where the bitonic
// network in its place ran 28 block barriers. With the search by wavefronts
// the launch went from 61 to 23 us on one crystal of 4,096 atoms. Past
// kRankMax keys the network's n log^2 n work is the smaller one and it is
// kept.
// W = 1: four atoms a block, at most kWaveKeys keys each. W = 4: a block an
// atom, `sort_size` (a power of two) keys in dynamic LDS.
constexpr int kWaveKeys = 256, kRankMax = 1024;
template <int W>
__global__ void __launch_bounds__(kSearchThreads) k_fill(SearchArgs A, int sort_size, const int* __restrict__ edge_ptr,
                                                         const int* __restrict__ bond_ptr, int* __restrict__ edge_dst,
                                                         int* __restrict__ edge_img, int* __restrict__ bond_edge) {
  extern __shared__ __attribute__((aligned(16))) unsigned long long keys_all[];
  __shared__ int nkeys, wsum[4];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const unsigned long long below = (1ull << lane) - 1ull;
  if constexpr (W == 1) {
    const int i = blockIdx.x * 4 + wave;
    if (i >= A.N) return;
    unsigned long long* keys = keys_all + wave * kWaveKeys;
    const int e0 = edge_ptr[i], b0 = bond_ptr[i];
    int n = 0;
    wave_search<1>(A, i, 0, [&](int j, int n1, int n2, int n3, float dd, bool pass) {
      const unsigned long long m = __ballot(pass);
      const int slot = n + __popcll(m & below);
      if (pass && slot < kWaveKeys) keys[slot] = make_key(j, n1, n2, n3, dd < A.rc2_bond);
      n += __popcll(m);
    });
    n = min(n, kWaveKeys);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // two keys a lane at a time
    for (int k0 = 0; k0 < n; k0 += 128) {
      unsigned long long mine[2];
      int rank[2] = {0, 0}, brank[2] = {0, 0};
#pragma unroll
      for (int q = 0; q < 2; ++q) mine[q] = k0 + 64 * q + lane < n ? keys[k0 + 64 * q + lane] : 0ull;
#pragma unroll 4
      for (int u = 0; u < n; ++u) {
        const unsigned long long k = keys[u];
        const int bond = (int)(k & 1ull);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const bool lt = k < mine[q];
          rank[q] += lt ? 1 : 0;
          brank[q] += lt ? bond : 0;
        }
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (k0 + 64 * q + lane < n) write_edge(mine[q], rank[q], brank[q], e0, b0, edge_dst, edge_img, bond_edge);
    }
    return;
  }
  unsigned long long* keys = keys_all;
  const int i = blockIdx.x;
  const int e0 = edge_ptr[i], b0 = bond_ptr[i];
  if (t == 0) nkeys = 0;
  __syncthreads();
  wave_search<4>(A, i, wave, [&](int j, int n1, int n2, int n3, float dd, bool pass) {
    const unsigned long long m = __ballot(pass);
    if (m == 0) return;
    int base = 0;
    if (lane == 0) base = atomicAdd(&nkeys, __popcll(m));
    base = __builtin_amdgcn_readfirstlane(base);
    const int slot = base + __popcll(m & below);
    if (pass && slot < sort_size) keys[slot] = make_key(j, n1, n2, n3, dd < A.rc2_bond);
  });
  __syncthreads();
  const int count = min(nkeys, sort_size);
  if (count <= kRankMax) {
    for (int k = t; k < count; k += kSearchThreads) {
      const unsigned long long mine = keys[k];
      int rank = 0, brank = 0;
#pragma unroll 4
      for (int u = 0; u < count; ++u) {
        const unsigned long long x = keys[u];
        const bool lt = x < mine;
        rank += lt ? 1 : 0;
        brank += lt ? (int)(x & 1ull) : 0;
      }
      write_edge(mine, rank, brank, e0, b0, edge_dst, edge_img, bond_edge);
    }
    return;
  }
  for (int k = count + t; k < sort_size; k += kSearchThreads) keys[k] = ~0ull;
  __syncthreads();
  // bitonic sort of sort_size (power of two) keys
  for (int size = 2; size <= sort_size; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int u = t; u < sort_size / 2; u += kSearchThreads) {
        const int lo = 2 * u - (u & (stride - 1));
        const int hi = lo + stride;
        const bool up = (lo & size) == 0;
        const unsigned long long a = keys[lo], b = keys[hi];
        if ((a > b) == up) { keys[lo] = b; keys[hi] = a; }
      }
      __syncthreads();
    }
  }
  int nb = 0;  // bonds written before this round of kSearchThreads keys
  for (int base = 0; base < count; base += kSearchThreads) {
    const int k = base + t;
    const unsigned long long key = k < count ? keys[k] : 0ull;
    const unsigned long long m = __ballot(k < count && (key & 1ull));
    if (lane == 0) wsum[wave] = __popcll(m);
    __syncthreads();
    int before = nb;
    for (int q = 0; q < wave; ++q) before += wsum[q];
    if (k < count) write_edge(key, k, before + __popcll(m & below), e0, b0, edge_dst, edge_img, bond_edge);
    for (int q = 0; q < kSearchThreads / 64; ++q) nb += wsum[q];
    __syncthreads();
  }
}

// Reverse map: binary search of (i, -n) in the sorted edge list of j. The
// search always succeeds: D2 is the same number in both directions (see
// pair_d2), and the cell list of j holds i at -n whenever that of i holds j
// at n (both cover every pair closer than r + kMargin, while D2 < r^2 implies
// a separation within fp32 rounding of r). Only the canonical direction of a
// pair searches and writes both entries; a probe loads the image only where
// the destination already equals i (few of a list's entries do).
__device__ __forceinline__ void rev_atoms(int blk, int N, const int* __restrict__ edge_ptr, const int* __restrict__ edge_dst,
                                          const int* __restrict__ edge_img, int* __restrict__ edge_rev) {
  const int i = blk * 4 + (threadIdx.x >> 6);
  if (i >= N) return;
  const int lane = threadIdx.x & 63;
  const int e1 = edge_ptr[i + 1];
  // two edges a lane at once: their chains of probes overlap
  for (int ea = edge_ptr[i] + lane; ea < e1; ea += 128) {
    int t[2][3], lo[2], hi[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = min(ea + 64 * u, e1 - 1);
      const int j = edge_dst[e];
#pragma unroll
      for (int k = 0; k < 3; ++k) t[u][k] = -edge_img[e * 3 + k];
      // n lexicographically negative on an atom's own image: not canonical
      const bool neg = t[u][0] > 0 || (t[u][0] == 0 && (t[u][1] > 0 || (t[u][1] == 0 && t[u][2] > 0)));
      const bool go = ea + 64 * u < e1 && (j > i || (j == i && !neg));
      lo[u] = edge_ptr[j];
      hi[u] = go ? edge_ptr[j + 1] - 1 : -1;
    }
    while (lo[0] < hi[0] || lo[1] < hi[1]) {  // first entry not below (i, -n)
      int mid[2], k0[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        mid[u] = lo[u] < hi[u] ? (lo[u] + hi[u]) >> 1 : 0;
        k0[u] = edge_dst[mid[u]];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (lo[u] >= hi[u]) continue;
        bool less = k0[u] < i;
        if (k0[u] == i) {
          const int k1 = edge_img[mid[u] * 3 + 0], k2 = edge_img[mid[u] * 3 + 1], k3 = edge_img[mid[u] * 3 + 2];
          less = k1 != t[u][0] ? k1 < t[u][0] : (k2 != t[u][1] ? k2 < t[u][1] : k3 < t[u][2]);
        }
        if (less) lo[u] = mid[u] + 1; else hi[u] = mid[u];
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (hi[u] >= 0) {
        edge_rev[ea + 64 * u] = lo[u];
        edge_rev[lo[u]] = ea + 64 * u;
      }
  }
}

// Angle list of atom i (one wavefront per atom): angle_ptr of its bonds and,
// if requested, the second bond of each of its k(k-1) angles.
__device__ __forceinline__ void angle_atoms(int blk, int N, const int* __restrict__ bond_ptr,
                                            const long long* __restrict__ angle_base, int* __restrict__ angle_ptr,
                                            int* __restrict__ angle_b2) {
  const int i = blk * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= N) return;
  const int b0 = bond_ptr[i], k = bond_ptr[i + 1] - b0;
  const long long a0 = angle_base[i];
  for (int p = lane; p < k; p += 64) angle_ptr[b0 + p] = (int)(a0 + (long long)p * (k - 1));
  if (i == N - 1 && lane == 0) angle_ptr[bond_ptr[N]] = (int)angle_base[N];
  if (angle_b2 && k > 1) {
    const int na = k * (k - 1);
    for (int x = lane; x < na; x += 64) {
      const int p = x / (k - 1), qq = x - p * (k - 1);
      angle_b2[a0 + x] = b0 + (qq < p ? qq : qq + 1);
    }
  }
}

// Reverse-edge map and angle lists in one launch: blocks [0, nb) take the
// reverse edges of atoms 4 b .. 4 b + 3, blocks [nb, 2 nb) their angle lists.
__global__ void __launch_bounds__(256) k_rev_angles(int N, const int* __restrict__ edge_ptr,
                                                    const int* __restrict__ edge_dst, const int* __restrict__ edge_img,
                                                    int* __restrict__ edge_rev, const int* __restrict__ bond_ptr,
                                                    const long long* __restrict__ angle_base, int* __restrict__ angle_ptr,
                                                    int* __restrict__ angle_b2) {
  const int nb = (N + 3) / 4;
  if ((int)blockIdx.x < nb) rev_atoms(blockIdx.x, N, edge_ptr, edge_dst, edge_img, edge_rev);
  else angle_atoms(blockIdx.x - nb, N, bond_ptr, angle_base, angle_ptr, angle_b2);
}

// Clears the graph info record and the bin counters (n each).
__global__ void k_zero_scratch(GraphInfo* __restrict__ ginfo, int* __restrict__ bin_count, int* __restrict__ bin_cursor,
                               int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *ginfo = GraphInfo{};
  if (i < n) {
    bin_count[i] = 0;
    bin_cursor[i] = 0;
  }
}

struct GraphScratch {
  StructInfo* info;
  GraphInfo* ginfo;
  int* total_bins;
  AtomMeta* meta;
  float4* bin_xyzj;
  int* bin_wrap;
  int *bin_count, *bin_start, *bin_cursor;
  int *edge_count, *bond_count;
  long long* angle_base;
};

void carve(Arena& ar, int64_t N, int64_t S, GraphScratch& g) {
  const int64_t nbins = N + S + 1;
  g.info = ar.take<StructInfo>(S);
  g.ginfo = ar.take<GraphInfo>(1);
  g.total_bins = ar.take<int>(1);
  g.meta = ar.take<AtomMeta>(N);
  g.bin_xyzj = ar.take<float4>(N);
  g.bin_wrap = ar.take<int>(N);
  g.bin_count = ar.take<int>(nbins + 1);
  g.bin_start = ar.take<int>(nbins + 1);
  g.bin_cursor = ar.take<int>(nbins + 1);
  g.edge_count = ar.take<int>(N);
  g.bond_count = ar.take<int>(N);
  g.angle_base = ar.take<long long>(N + 1);
}

// The calling thread's pinned record for the sizes (allocated on its first
// use): the scan kernel writes it directly, with no copy after it, on every
// device that the thread builds graphs on.
int pinned_info(GraphInfo*& out) {
  thread_local GraphInfo* pinned = nullptr;
  if (!pinned)
    CHG_HIP(hipHostMalloc(reinterpret_cast<void**>(&pinned), sizeof(GraphInfo),
                          hipHostMallocPortable | hipHostMallocMapped));
  out = pinned;
  return CHGNET_OK;
}

// From this many atoms on, one wavefront an atom gives every SIMD of the chip
// (1,024) one in the search kernels, and sizing the runs once an atom is
// cheaper than four times; below it four share an atom, each taking every
// fourth group of candidates (one 8-atom cell, 1,000 candidates an atom:
// counting 9.0 -> 6.4 us, against one block of 256 threads in lock step).
constexpr int kSearchWideAtoms = 1024;

}  // namespace

size_t graph_scratch_bytes(int64_t N, int64_t S) {
  Arena ar;
  GraphScratch g;
  carve(ar, N, S, g);
  return align_up(ar.used, 256);
}

int validate_batch(const chgnet_batch* b) {
  if (!b || b->n_struct < 1 || b->n_atoms < 1 || !b->atom_ptr || !b->pos || !b->lattice || !b->Z)
    return fail(CHGNET_EINVAL, "batch: need n_struct >= 1, n_atoms >= 1 and non-null arrays");
  return CHGNET_OK;
}

namespace {

// Graph build on a scratch region of ws_bytes at ws. With pinned_readback the
// sizes come back through a small pinned host buffer of the calling thread
// (allocated on its first use); otherwise through a pageable host variable.
int build_graph_impl(const chgnet_hparams* hp, const chgnet_batch* batch, chgnet_graph* graph, void* ws,
                     size_t ws_bytes, hipStream_t st, bool pinned_readback, bool candidates = false) {
  CHG_TRY(validate_hparams(hp));
  CHG_TRY(validate_batch(batch));
  if (!graph || !graph->edge_ptr || !graph->bond_ptr) return fail(CHGNET_EINVAL, "graph: edge_ptr and bond_ptr are required");
  const int N = batch->n_atoms, S = batch->n_struct;
  Arena ar{static_cast<char*>(ws), ws_bytes, 0};
  GraphScratch g;
  carve(ar, N, S, g);
  if (!ws || !ar.ok()) return fail(CHGNET_EWORKSPACE, "workspace too small for the graph build");
  const int64_t nbins_cap = (int64_t)N + S + 1;

  if (N <= 1024 * kBinAtomsPer && (int64_t)N + S <= kBinMax) {
    KLAUNCH(st, "k_bin", k_bin<<<1, 1024, 0, st>>>(N, S, batch->atom_ptr, batch->pos, batch->Z, batch->lattice, hp->r_atom,
                                                   g.info, g.meta, g.bin_start, g.bin_xyzj, g.bin_wrap, g.ginfo));
  } else {
    const int n = (int)(nbins_cap + 1);
    KLAUNCH(st, "k_zero_scratch", k_zero_scratch<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(g.ginfo, g.bin_count, g.bin_cursor, n));
    KLAUNCH(st, "k_struct_setup", k_struct_setup<<<1, 1024, 0, st>>>(N, S, batch->atom_ptr, batch->lattice, hp->r_atom, g.info, g.total_bins, g.ginfo));
    KLAUNCH(st, "k_atom_bin", k_atom_bin<<<cdiv(N, 256), 256, 0, st>>>(N, S, batch->atom_ptr, batch->pos, batch->Z, g.info, g.meta,
                                             g.bin_count, g.ginfo));
    // total bins <= N + S (each crystal has at most max(1, n_s) bins)
    KLAUNCH(st, "k_scan_single", k_scan_single<<<1, 1024, 0, st>>>((int)nbins_cap, g.bin_count, g.bin_start));
    KLAUNCH(st, "k_bin_fill", k_bin_fill<<<cdiv(N, 256), 256, 0, st>>>(N, g.meta, g.bin_start, g.bin_cursor, batch->pos, g.bin_xyzj, g.bin_wrap));
  }

  SearchArgs A;
  A.N = N;
  A.rc2_atom = hp->r_atom * hp->r_atom;
  A.rc2_bond = candidates ? -1.0f : hp->r_bond * hp->r_bond;  // a candidate list has no bonds
  A.pos = batch->pos;
  A.info = g.info;
  A.meta = g.meta;
  A.bin_start = g.bin_start;
  A.bin_xyzj = g.bin_xyzj;
  A.bin_wrap = g.bin_wrap;
  const bool wide = N >= kSearchWideAtoms;
  if (wide) KLAUNCH(st, "k_count", k_count<1><<<(unsigned)cdiv(N, 4), kSearchThreads, 0, st>>>(A, g.edge_count, g.bond_count));
  else KLAUNCH(st, "k_count", k_count<4><<<N, kSearchThreads, 0, st>>>(A, g.edge_count, g.bond_count));
  GraphInfo* pinned = nullptr;
  if (pinned_readback) CHG_TRY(pinned_info(pinned));
  KLAUNCH(st, "k_scan_counts", k_scan_counts<<<1, 1024, 0, st>>>(N, g.edge_count, g.bond_count, graph->edge_ptr, graph->bond_ptr, g.angle_base,
                                    nullptr, g.ginfo, pinned));
  GraphInfo hinfo;
  if (pinned) {
    CHG_HIP(hipStreamSynchronize(st));
    hinfo = *pinned;
  } else {
    CHG_HIP(hipMemcpyAsync(&hinfo, g.ginfo, sizeof(GraphInfo), hipMemcpyDeviceToHost, st));
    CHG_HIP(hipStreamSynchronize(st));
  }
  if (hinfo.err) {
    std::string m = "build_graph: invalid input:";
    if (hinfo.err & ERR_Z) m += " Z outside 1..94;";
    if (hinfo.err & ERR_DET) m += " |det L| < 1e-6;";
    if (hinfo.err & ERR_THIN) m += " lattice too thin for the cutoff;";
    if (hinfo.err & ERR_FAR) m += " position too far from the origin cell;";
    if (hinfo.err & ERR_PTR) m += " atom_ptr decreasing;";
    return fail(CHGNET_EINVAL, m);
  }
  graph->n_edges = hinfo.n_edges;
  graph->n_bonds = hinfo.n_bonds;
  graph->n_angles = hinfo.n_angles;
  if (hinfo.max_count > kMaxEdgesPerAtom)
    return fail(CHGNET_EINVAL, "build_graph: more than 8192 edges on one atom");
  if (hinfo.n_edges >= INT_MAX || hinfo.n_angles >= INT_MAX)
    return fail(CHGNET_EINVAL, "build_graph: graph larger than 2^31 entries");
  if (hinfo.n_edges > graph->cap_edges || hinfo.n_bonds > graph->cap_bonds || hinfo.n_angles > graph->cap_angles)
    return fail(CHGNET_ECAPACITY, "build_graph: capacity too small (required sizes written to the graph)");
  auto fill_edges = [&]() -> int {
    if (wide && hinfo.max_count <= kWaveKeys) {
      KLAUNCH(st, "k_fill", k_fill<1><<<(unsigned)cdiv(N, 4), kSearchThreads, sizeof(unsigned long long) * 4 * kWaveKeys, st>>>(
                                A, 0, graph->edge_ptr, graph->bond_ptr, graph->edge_dst, graph->edge_img, graph->bond_edge));
    } else {
      int sort_size = 64;
      while (sort_size < hinfo.max_count) sort_size <<= 1;
      KLAUNCH(st, "k_fill", k_fill<4><<<N, kSearchThreads, sizeof(unsigned long long) * sort_size, st>>>(
                                A, sort_size, graph->edge_ptr, graph->bond_ptr, graph->edge_dst, graph->edge_img, graph->bond_edge));
    }
    return CHGNET_OK;
  };
  if (candidates) {
    if (hinfo.n_edges > 0 && (!graph->edge_dst || !graph->edge_img))
      return fail(CHGNET_EINVAL, "md: candidate arrays are required");
    return fill_edges();
  }
  if (hinfo.n_edges > 0 && (!graph->edge_dst || !graph->edge_img || !graph->edge_rev))
    return fail(CHGNET_EINVAL, "graph: edge arrays are required");
  if (!graph->angle_ptr || (hinfo.n_bonds > 0 && !graph->bond_edge))
    return fail(CHGNET_EINVAL, "graph: bond_edge and angle_ptr are required");

  CHG_TRY(fill_edges());
  KLAUNCH(st, "k_rev_angles", k_rev_angles<<<2 * cdiv(N, 4), 256, 0, st>>>(N, graph->edge_ptr, graph->edge_dst, graph->edge_img,
                                                                       graph->edge_rev, graph->bond_ptr, g.angle_base,
                                                                       graph->angle_ptr, graph->angle_b2));
  return CHGNET_OK;
}

// ---------------------------------------------------------------------------
// Molecular dynamics: reuse of a candidate list (Verlet skin). The list holds
// every pair within r + skin of the positions at its build, in the canonical
// (j, n) order of each source atom. While no atom has moved more than
// (skin - 0.01 A) / 2 since then, every pair now within r is on the list, and
// filtering it with the exact cutoff test at the current positions gives the
// same graph, in the same order, as a full search.
// ---------------------------------------------------------------------------
struct CandArgs {
  int N, S;
  float rc2_atom, rc2_bond;
  const int* atom_ptr;
  const float* pos;
  const float* lattice;
  const int* cand_ptr;
  const int* cand_dst;
  const int* cand_img;
  const float* ref;  // positions at the list's build
};

// Cutoff test of candidate c of atom i at the current positions.
__device__ __forceinline__ float cand_d2(const CandArgs& A, int i, const float* L, const float (&ri)[3], int c,
                                         int& j) {
  j = A.cand_dst[c];
  const float rj[3] = {A.pos[3 * j], A.pos[3 * j + 1], A.pos[3 * j + 2]};
  return pair_d2(i, j, ri, rj, A.cand_img[3 * c], A.cand_img[3 * c + 1], A.cand_img[3 * c + 2], L);
}

// Edges and bonds of each atom among its candidates, and its squared
// displacement since the list was built; one wavefront per atom.
__global__ void __launch_bounds__(256) k_cand_count(CandArgs A, int* __restrict__ edge_count, int* __restrict__ bond_count,
                                                    float* __restrict__ disp2) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= A.N) return;
  const int s = find_struct(A.atom_ptr, A.S, i);
  float L[9];
  for (int k = 0; k < 9; ++k) L[k] = A.lattice[9 * s + k];
  const float ri[3] = {A.pos[3 * i], A.pos[3 * i + 1], A.pos[3 * i + 2]};
  int ne = 0, nb = 0;
  for (int c = A.cand_ptr[i] + lane; c < A.cand_ptr[i + 1]; c += 64) {
    int j;
    const float dd = cand_d2(A, i, L, ri, c, j);
    ne += dd < A.rc2_atom ? 1 : 0;
    nb += dd < A.rc2_bond ? 1 : 0;
  }
  for (int off = 32; off > 0; off >>= 1) {
    ne += __shfl_xor(ne, off, 64);
    nb += __shfl_xor(nb, off, 64);
  }
  if (lane == 0) {
    edge_count[i] = ne;
    bond_count[i] = nb;
    const float dx = ri[0] - A.ref[3 * i], dy = ri[1] - A.ref[3 * i + 1], dz = ri[2] - A.ref[3 * i + 2];
    // a position that is not a number has moved too far (a maximum would drop
    // it): the list is then built again, which refuses it
    const float d2 = dx * dx + dy * dy + dz * dz;
    disp2[i] = d2 <= FLT_MAX ? d2 : INFINITY;
  }
}

// The kept candidates of each atom in list order (one wavefront per atom,
// 64 candidates per round, compacted by ballot): edge arrays and bond list.
__global__ void __launch_bounds__(256) k_cand_fill(CandArgs A, const int* __restrict__ edge_ptr,
                                                   const int* __restrict__ bond_ptr, int* __restrict__ edge_dst,
                                                   int* __restrict__ edge_img, int* __restrict__ bond_edge) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= A.N) return;
  const int s = find_struct(A.atom_ptr, A.S, i);
  float L[9];
  for (int k = 0; k < 9; ++k) L[k] = A.lattice[9 * s + k];
  const float ri[3] = {A.pos[3 * i], A.pos[3 * i + 1], A.pos[3 * i + 2]};
  int e = edge_ptr[i], b = bond_ptr[i];
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int c0 = A.cand_ptr[i]; c0 < A.cand_ptr[i + 1]; c0 += 64) {
    const int c = c0 + lane;
    bool keep = false, bond = false;
    int j = 0;
    if (c < A.cand_ptr[i + 1]) {
      const float dd = cand_d2(A, i, L, ri, c, j);
      keep = dd < A.rc2_atom;
      bond = dd < A.rc2_bond;
    }
    const unsigned long long mk = __ballot(keep), mb = __ballot(bond);
    if (keep) {
      const int k = e + __popcll(mk & below);
      edge_dst[k] = j;
      edge_img[3 * k] = A.cand_img[3 * c];
      edge_img[3 * k + 1] = A.cand_img[3 * c + 1];
      edge_img[3 * k + 2] = A.cand_img[3 * c + 2];
      if (bond) bond_edge[b + __popcll(mb & below)] = k;
    }
    e += __popcll(mk);
    b += __popcll(mb);
  }
}

// Scratch of the allocation-free graph build: one array per GPU, held until
// the process ends. Host code never passes `scratch` itself to a kernel (in
// host code the name is a stand-in, not a device address); it uses the
// address hipGetSymbolAddress returns on each device.
constexpr size_t kNoAllocScratchBytes = size_t(8) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
int scratch_address(void** out) {
  int dev = -1;
  CHG_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(CHGNET_EINVAL, "build_graph_noalloc: device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    CHG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(CHGNET_EHIP, "build_graph_noalloc: no device address for the scratch array");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return CHGNET_OK;
}

}  // namespace

int build_graph(const chgnet_hparams* hp, const chgnet_batch* batch, chgnet_graph* graph, void* ws, size_t ws_bytes,
                hipStream_t st) {
  return build_graph_impl(hp, batch, graph, ws, ws_bytes, st, true);
}

int build_graph_noalloc(const chgnet_hparams* hp, const chgnet_batch* batch, chgnet_graph* graph, hipStream_t st) {
  CHG_TRY(validate_hparams(hp));
  CHG_TRY(validate_batch(batch));
  const size_t need = graph_scratch_bytes(batch->n_atoms, batch->n_struct);
  if (need > kNoAllocScratchBytes)
    return fail(CHGNET_EINVAL, "build_graph_noalloc: the batch needs " + std::to_string(need) +
                                   " bytes of graph scratch, more than the static " +
                                   std::to_string(kNoAllocScratchBytes) + " (use chgnet_build_graph with a workspace)");
  void* p = nullptr;
  CHG_TRY(scratch_address(&p));
  return build_graph_impl(hp, batch, graph, p, kNoAllocScratchBytes, st, false);
}

// Candidate list of every pair within r_atom + skin of the batch's current
// positions into s->cand_* (bonds are not kept), and those positions into
// s->ref_pos. graph->bond_ptr serves as scratch.
int md_build_candidates(const chgnet_hparams* hp, const chgnet_batch* batch, chgnet_md_state* s, chgnet_graph* graph,
                        void* ws, size_t ws_bytes, hipStream_t st) {
  chgnet_hparams hc = *hp;
  hc.r_atom = hp->r_atom + s->skin;
  hc.r_bond = hc.r_atom;
  chgnet_graph cg{};
  cg.cap_edges = s->cap_cand;
  cg.edge_ptr = s->cand_ptr;
  cg.edge_dst = s->cand_dst;
  cg.edge_img = s->cand_img;
  cg.bond_ptr = graph->bond_ptr;
  const int code = build_graph_impl(&hc, batch, &cg, ws, ws_bytes, st, true, true);
  s->n_cand = cg.n_edges;
  if (code != CHGNET_OK) return code;
  CHG_HIP(hipMemcpyAsync(s->ref_pos, batch->pos, sizeof(float) * 3 * batch->n_atoms, hipMemcpyDeviceToDevice, st));
  s->n_builds += 1;
  return CHGNET_OK;
}

// The graph of the batch's current positions from the candidate list. Sets
// *stale (and builds nothing) when some atom has moved too far since the
// list was built; otherwise as chgnet_build_graph (one wait for the sizes).
int md_filter_graph(const chgnet_hparams* hp, const chgnet_batch* batch, const chgnet_md_state* s,
                    chgnet_graph* graph, void* ws, size_t ws_bytes, hipStream_t st, bool* stale) {
  *stale = false;
  const int N = batch->n_atoms, S = batch->n_struct;
  Arena ar{static_cast<char*>(ws), ws_bytes, 0};
  GraphScratch g;
  carve(ar, N, S, g);
  if (!ws || !ar.ok()) return fail(CHGNET_EWORKSPACE, "workspace too small for the graph build");
  CandArgs A{N, S, hp->r_atom * hp->r_atom, hp->r_bond * hp->r_bond, batch->atom_ptr, batch->pos, batch->lattice,
             s->cand_ptr, s->cand_dst, s->cand_img, s->ref_pos};
  float* disp2 = reinterpret_cast<float*>(g.bin_count);  // N of its N + S + 2 entries; the bins are not used here
  KLAUNCH(st, "k_cand_count", k_cand_count<<<(unsigned)cdiv(N, 4), 256, 0, st>>>(A, g.edge_count, g.bond_count, disp2));
  GraphInfo* pinned = nullptr;
  CHG_TRY(pinned_info(pinned));
  KLAUNCH(st, "k_scan_counts", k_scan_counts<<<1, 1024, 0, st>>>(N, g.edge_count, g.bond_count, graph->edge_ptr,
                                                                   graph->bond_ptr, g.angle_base, disp2, g.ginfo, pinned));
  CHG_HIP(hipStreamSynchronize(st));
  const GraphInfo hinfo = *pinned;
  // the list covers every pair within r of the current positions while twice
  // the largest displacement stays below the skin (0.01 A spares fp32
  // rounding of coordinates up to 10^4 A)
  const float half = 0.5f * (s->skin - 0.01f);
  float md2;
  std::memcpy(&md2, &hinfo.max_disp2, sizeof(float));
  if (!(md2 < half * half)) {
    *stale = true;
    return CHGNET_OK;
  }
  graph->n_edges = hinfo.n_edges;
  graph->n_bonds = hinfo.n_bonds;
  graph->n_angles = hinfo.n_angles;
  if (hinfo.max_count > kMaxEdgesPerAtom) return fail(CHGNET_EINVAL, "build_graph: more than 8192 edges on one atom");
  if (hinfo.n_edges >= INT_MAX || hinfo.n_angles >= INT_MAX)
    return fail(CHGNET_EINVAL, "build_graph: graph larger than 2^31 entries");
  if (hinfo.n_edges > graph->cap_edges || hinfo.n_bonds > graph->cap_bonds || hinfo.n_angles > graph->cap_angles)
    return fail(CHGNET_ECAPACITY, "build_graph: capacity too small (required sizes written to the graph)");
  KLAUNCH(st, "k_cand_fill", k_cand_fill<<<(unsigned)cdiv(N, 4), 256, 0, st>>>(A, graph->edge_ptr, graph->bond_ptr,
                                                                              graph->edge_dst, graph->edge_img,
                                                                              graph->bond_edge));
  KLAUNCH(st, "k_rev_angles", k_rev_angles<<<2 * cdiv(N, 4), 256, 0, st>>>(N, graph->edge_ptr, graph->edge_dst,
                                                                            graph->edge_img, graph->edge_rev,
                                                                            graph->bond_ptr, g.angle_base,
                                                                            graph->angle_ptr, graph->angle_b2));
  return CHGNET_OK;
}

}  // namespace chg
