// Learned coarse-mesh correction: neighbour descriptor, a 128-64-64-64-32
// SiLU MLP on BF16 MFMA with FP32 accumulation, the equivariant force head,
// and training (loss, backward, Adam) - all as gfx950 kernels.
//
//   T_i[k, a] = sum_{j: r_ij < rc} q_j T_k(2 r_ij / rc - 1) s(r_ij) u_a(i -> j),
//               u = (1, unit vector), s(r) = (1 + cos(pi r / rc)) / 2, k < 32;
//   D_i[4k + l] = sum_a T_i[k, a] T_i[l, a] (l < 4);  x_i = (D_i - mu) * inv_sigma;
//   h1 = silu(x W1 + b1), h2 = silu(h1 W2 + b2), h3 = silu(h2 W3 + b3),
//   c = h3 W4 + b4;  dF_i = s_out q_i sum_k c_ik T_i[k, 1:4].
//
// Packed parameter vector (FP32 master copy, the layout of the C ABI):
//   W1[128][64] b1[64] W2[64][64] b2[64] W3[64][64] b3[64] W4[64][32] b4[32]
//   mu[128] inv_sigma[128]                                   (18912 floats)
#pragma once

#include "cell_walk.hpp"
#include "pppm_kernels.hpp"

namespace dplr {
namespace mlp {

constexpr int kIn = 128, kH = 64, kOut = 32;
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kIn * kH;
constexpr int kOffW2 = kOffB1 + kH, kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH * kH;
constexpr int kOffW4 = kOffB3 + kH, kOffB4 = kOffW4 + kH * kOut;
constexpr int kNTrain = kOffB4 + kOut;                // trainable parameters
constexpr int kOffMu = kNTrain, kOffIsd = kOffMu + kIn;
constexpr int kNParams = kOffIsd + kIn;               // packed total
constexpr int kNWeights = kIn * kH + 2 * kH * kH + kH * kOut;  // bf16 weight copy
constexpr int kRows = 128;                            // particles per MLP block (4 waves x 32)
constexpr int kMlpThreads = 256;                      // threads of the training forward's blocks

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ unsigned short f2bf(float f) {
  // round to nearest even
  unsigned u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)(u >> 16);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }

// silu with the hardware reciprocal (1 ulp): the result is rounded to bf16
// before it is used, so the last FP32 bits do not matter
__device__ __forceinline__ float silu(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

__device__ __forceinline__ float mul_rounded(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

// row / column of accumulator register r of this lane in the 32 x 32 tile
__device__ __forceinline__ int acc_row(int r) { return 8 * (r >> 2) + 4 * ((threadIdx.x & 63) >> 5) + (r & 3); }
__device__ __forceinline__ int acc_col() { return threadIdx.x & 31; }

__device__ __forceinline__ void zero(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.0f;
}

// ---------------------------------------------------------------------------
// Cell list: cells of edge >= rc per axis (at least 3 per axis).
// ---------------------------------------------------------------------------
struct CellGeo {
  int nc[3];
  float L[3], invL[3], cinv[3];  // box, 1/box, cells per Angstrom
  float rc;
  int ncells;
};

__device__ __forceinline__ float wrapf(float v, float L, float invL) {
  v -= L * floorf(v * invL);
  if (v >= L) v -= L;
  if (!(v >= 0.0f && v < L)) v = 0.0f;
  return v;
}

__device__ __forceinline__ int cell_of(float x, float y, float z, const CellGeo& c) {
  int cx = min((int)(x * c.cinv[0]), c.nc[0] - 1);
  int cy = min((int)(y * c.cinv[1]), c.nc[1] - 1);
  int cz = min((int)(z * c.cinv[2]), c.nc[2] - 1);
  return (cz * c.nc[1] + cy) * c.nc[0] + cx;
}

// Counts the particles of every cell and keeps each one's arrival number in its
// cell (rank), so that the scatter needs no atomics.  Neighbouring indices are
// neighbours in space more often than not (the atoms of a molecule), so a run
// of lanes in one cell shares one atomic.
__global__ void __launch_bounds__(256) k_cell_count(const float* __restrict__ ion_pos, const float* __restrict__ wc_pos,
                                                    int64_t n_ion, int64_t n, int* __restrict__ count,
                                                    int* __restrict__ rank, CellGeo c) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  int cell = -1;
  if (i < n) {
    const float* r = (i < n_ion) ? ion_pos + 3 * i : wc_pos + 3 * (i - n_ion);
    const float x = wrapf(r[0], c.L[0], c.invL[0]), y = wrapf(r[1], c.L[1], c.invL[1]),
                z = wrapf(r[2], c.L[2], c.invL[2]);
    cell = cell_of(x, y, z, c);
  }
  const int before = __shfl_up(cell, 1, 64);
  const uint64_t heads = __ballot(lane == 0 || before != cell);  // first lanes of the runs
  const int head = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
  const uint64_t after = lane == 63 ? 0ull : heads >> (lane + 1);
  const int len = after ? __ffsll((unsigned long long)after) : 64 - lane;  // of the run, at its head
  int first = 0;
  if (head == lane && cell >= 0) first = atomicAdd(count + cell, len);
  first = __shfl(first, head, 64);
  if (i < n) rank[i] = first + lane - head;
}

// Exclusive scan of the cell counts by several blocks: block b adds up the
// counts before its tile by itself (reads that stream from L2), then scans the
// tile; the last one also writes start[ncells].  Its reads grow with the square
// of the cell count, those of one block with a carried sum (k_bin_scan) do not:
// 6.2 and 27 us at 32,768 cells, 14.5 and 113 at 140,608, 77 and 779 at 10^6, 2,890
// and 6,470 at 8.4 x 10^6, where the line lies: twice as many cells would be four
// times the one and twice the other.
constexpr int kScanTile = 2048, kScanCells = 1 << 23;
__global__ void __launch_bounds__(1024) k_cell_scan(const int* __restrict__ count, int* __restrict__ start,
                                                    int ncells) {
  __shared__ int red[16];
  __shared__ int wsum[17];
  __shared__ int vals[kScanTile];
  const int t = threadIdx.x, b0 = blockIdx.x * kScanTile, nt = min(kScanTile, ncells - b0);
  int s = 0;
  for (int e = t; e < b0 / 4; e += 1024) {
    const int4 v = reinterpret_cast<const int4*>(count)[e];
    s += v.x + v.y + v.z + v.w;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((t & 63) == 0) red[t >> 6] = s;
  const int total = block_exclusive_scan(count + b0, vals, nt, wsum);  // contains barriers
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) base += red[w];
  for (int e = t; e < nt; e += 1024) start[b0 + e] = base + vals[e];
  if (t == 0 && b0 + nt == ncells) start[ncells] = base + total;
}

__global__ void __launch_bounds__(256) k_cell_scatter(const float* __restrict__ ion_pos, const float* __restrict__ wc_pos,
                                                      const float* __restrict__ ion_q, const float* __restrict__ wc_q,
                                                      int64_t n_ion, int64_t n, const int* __restrict__ start,
                                                      const int* __restrict__ rank, float4* __restrict__ cpos,
                                                      int* __restrict__ cidx, CellGeo c) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float* r = (i < n_ion) ? ion_pos + 3 * i : wc_pos + 3 * (i - n_ion);
  const float x = wrapf(r[0], c.L[0], c.invL[0]), y = wrapf(r[1], c.L[1], c.invL[1]),
              z = wrapf(r[2], c.L[2], c.invL[2]);
  const float q = (i < n_ion) ? ion_q[i] : wc_q[i - n_ion];
  const int slot = start[cell_of(x, y, z, c)] + rank[i];
  cpos[slot] = make_float4(x, y, z, q);
  cidx[slot] = (int)i;
}

// The scatter leaves each cell's particles in arrival order; this puts
// them in order of original index (rank = number of the cell's particles
// with a smaller index), so the cell order and every sum over neighbours
// taken in it are the same on every call.  One thread per particle; a cell
// holds tens of particles, so the O(n^2) ranking per cell is cheap.  Also clears
// the cell counts for the next call.
__global__ void k_cell_order(const float4* __restrict__ cpos_in, const int* __restrict__ cidx_in,
                             const int* __restrict__ start, int n,
                             float4* __restrict__ cpos, int* __restrict__ cidx, int* __restrict__ count,
                             CellGeo c) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  for (int k = e; k < c.ncells; k += gridDim.x * blockDim.x) count[k] = 0;
  if (e >= n) return;
  const float4 p = cpos_in[e];
  const int id = cidx_in[e];
  const int cell = cell_of(p.x, p.y, p.z, c);
  const int j0 = start[cell], j1 = start[cell + 1];
  int rank = 0;
  for (int j = j0; j < j1; ++j) rank += cidx_in[j] < id;
  cpos[j0 + rank] = p;
  cidx[j0 + rank] = id;
}

// Runtime statistics of the learned form's inputs and outputs, read by the
// fallback guard (dplr_lr_mlp_read_stats).  Maxima of non-negative floats are
// kept as their bit patterns (whose unsigned order is the float order), so
// every field is an integer reduction or a fixed-order FP64 sum: the values do
// not depend on the order of the contributions.
struct Stats {
  unsigned max_corr_bits;   // max |dF_i| of the last forward
  unsigned max_force_bits;  // max |F_i| of the forces the last forward added to
  int min_nbr, max_nbr;     // neighbour counts within the cutoff, last forward
  int unseen;               // charges outside the training set, last check
  int audit_valid;
  double audit_num, audit_den;  // sum |F - F_ref|^2, sum |F_ref|^2 of the audits
};

// Charges not in the training set (exact float comparison with the set).
constexpr int kMaxTrainCharges = 16;
struct ChargeSet {
  int n;
  float q[kMaxTrainCharges];
};

__global__ void k_check_charges(const float* __restrict__ ion_q, const float* __restrict__ wc_q, int64_t n_ion,
                                int64_t n, ChargeSet cs, Stats* st, int reset) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (reset) {  // single-block launch for an empty input
    if (i == 0) st->unseen = 0;
    return;
  }
  int bad = 0;
  if (i < n) {
    const float q = (i < n_ion) ? ion_q[i] : wc_q[i - n_ion];
    bool seen = false;
    for (int k = 0; k < cs.n; ++k) seen |= (q == cs.q[k]);
    bad = seen ? 0 : 1;
  }
  for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off, 64);
  if ((threadIdx.x & 63) == 0 && bad) atomicAdd(&st->unseen, bad);
}

// Audit sums over both particle sets: per-block FP64 partials (fixed order
// inside the block), then one block adds them in block order.
__global__ void __launch_bounds__(256) k_audit_partials(const float* __restrict__ fi, const float* __restrict__ ri,
                                                        int64_t n_ion, const float* __restrict__ fw,
                                                        const float* __restrict__ rw, int64_t n,
                                                        double* __restrict__ part) {
  __shared__ double red[2][256];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double num = 0.0, den = 0.0;
  if (i < n) {
    const float* f = (i < n_ion) ? fi + 3 * i : fw + 3 * (i - n_ion);
    const float* r = (i < n_ion) ? ri + 3 * i : rw + 3 * (i - n_ion);
    for (int a = 0; a < 3; ++a) {
      const double d = (double)f[a] - (double)r[a];
      num += d * d;
      den += (double)r[a] * (double)r[a];
    }
  }
  red[0][threadIdx.x] = num;
  red[1][threadIdx.x] = den;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      red[0][threadIdx.x] += red[0][threadIdx.x + h];
      red[1][threadIdx.x] += red[1][threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = red[0][0];
    part[2 * blockIdx.x + 1] = red[1][0];
  }
}

__global__ void k_audit_finish(const double* __restrict__ part, int nblk, Stats* st, int accumulate) {
  if (threadIdx.x != 0) return;
  double num = 0.0, den = 0.0;
  for (int b = 0; b < nblk; ++b) {
    num += part[2 * b];
    den += part[2 * b + 1];
  }
  st->audit_num = accumulate ? st->audit_num + num : num;
  st->audit_den = accumulate ? st->audit_den + den : den;
  st->audit_valid = 1;
}

// Input normalisation from training descriptors: per-block partial sums of
// D_f and D_f^2 and the block maximum of |D| (f < 128), from T [n][128];
// then the block partials are added in block order into acc[2][128] (+ count
// and max), and finish turns them into mu = mean, inv_sigma =
// 1 / (std + 1e-6 (max |D| + 1)) in the parameter vector.
__global__ void __launch_bounds__(128) k_norm_partials(const float* __restrict__ T, int n, int rows_per_block,
                                                       double* __restrict__ part) {
  const int f = threadIdx.x;  // feature 4k + l
  const int k = f >> 2, l = f & 3;
  const int r0 = blockIdx.x * rows_per_block, r1 = min(n, r0 + rows_per_block);
  double s1 = 0.0, s2 = 0.0;
  float mx = 0.0f;
  for (int r = r0; r < r1; ++r) {
    const float4 tk = reinterpret_cast<const float4*>(T + (size_t)r * 128)[k];
    const float4 tl = reinterpret_cast<const float4*>(T + (size_t)r * 128)[l];
    const float d = tk.x * tl.x + tk.y * tl.y + tk.z * tl.z + tk.w * tl.w;
    s1 += d;
    s2 += (double)d * d;
    mx = fmaxf(mx, fabsf(d));
  }
  double* p = part + (size_t)blockIdx.x * 3 * 128;
  p[f] = s1;
  p[128 + f] = s2;
  p[256 + f] = mx;
}

__global__ void __launch_bounds__(128) k_norm_reduce(const double* __restrict__ part, int nblk, int rows,
                                                     double* __restrict__ acc) {
  // acc: [0,128) sum, [128,256) sum of squares, [256] max |D|, [257] count
  const int f = threadIdx.x;
  double s1 = 0.0, s2 = 0.0, mx = 0.0;
  for (int b = 0; b < nblk; ++b) {
    const double* p = part + (size_t)b * 3 * 128;
    s1 += p[f];
    s2 += p[128 + f];
    mx = fmax(mx, p[256 + f]);
  }
  acc[f] += s1;
  acc[128 + f] += s2;
  __shared__ double m[128];
  m[f] = mx;
  __syncthreads();
  if (f == 0) {
    double g = acc[256];
    for (int i = 0; i < 128; ++i) g = fmax(g, m[i]);
    acc[256] = g;
    acc[257] += (double)rows;
  }
}

__global__ void __launch_bounds__(128) k_norm_finish(double* __restrict__ acc, float* __restrict__ params) {
  const int f = threadIdx.x;
  const double cnt = acc[257];
  if (cnt > 0.0) {
    const double mu = acc[f] / cnt;
    const double var = fmax(acc[128 + f] / cnt - mu * mu, 0.0);
    params[kOffMu + f] = (float)mu;
    params[kOffIsd + f] = (float)(1.0 / (sqrt(var) + 1e-6 * (acc[256] + 1.0)));
  }
  __syncthreads();
  acc[f] = 0.0;
  acc[128 + f] = 0.0;
  if (f == 0) {
    acc[256] = 0.0;
    acc[257] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Descriptor: four lanes per (cell-sorted) particle, one wave (16 particles) a
// block.  Lane g owns the radial orders k = g + 4 m, m < 8, advanced with the
// stride-4 Chebyshev recurrence T_{k+4} = 2 T_4 T_k - T_{k-4}.  Two phases:
// the four lanes scan the candidates together (candidate t + g), and the ones
// inside the cutoff are appended to the particle's LDS list in candidate order
// (ballot + prefix count, so the order is deterministic); then the pair
// quantities are formed once per pair and every lane runs its orders over the
// whole list (accumulate_pairs).  Writes T [n][128] (FP32, index 4k + a) and the
// normalised MLP input x [n][128] (bf16).
//
// The kernel is bound by VALU issue.  Per pair and particle, T[k, a] += w T_k u_a
// is a 32 x 4 outer product: eight v_mfma_f32_4x4x1 (16 independent 4 x 4 outer
// products each, one per particle of the wave; lane g gives w T_k of its order
// and u_g) take the 32 multiply-adds per lane off the VALU, with the same
// single-precision fused multiply-adds in the same order.  The three cells of a
// neighbour row are consecutive in memory, so the scan walks 9 ranges instead
// of 27, and the periodic image follows from the cell instead of a rounding per
// candidate and axis.
// Matrix instructions ignore the execution mask, so all loops are uniform over
// the wave and a particle that is done contributes w = 0.
// ---------------------------------------------------------------------------
constexpr int kDescThreads = 64;
constexpr int kDescParts = kDescThreads / kDescLanes;
// A list takes another chunk while it holds at most kNbrMax neighbours: 78 entries
// and a spare one, the most with which eight blocks of k_correction fit the LDS
// of a compute unit.  (Water has 36 neighbours on average.)
constexpr int kNbrMax = 62;
constexpr int kNbrList = kNbrMax + kScanChunk + 1;
static_assert(kScanChunk <= 32, "one word of candidate bits per chunk");

// Pairs per round of the accumulation: every lane of a particle forms one
// pair's quantities (once per pair), and then every lane runs its eight orders
// over all of them.  What lane g needs of a pair lies in one 16-byte slot of its
// own, the starts of its recurrence included, so that a pair costs a lane two LDS
// reads and no selection by g.
constexpr int kPairChunk = kDescLanes;
struct PairSlots {
  float lane[kPairChunk][kDescLanes][4];  // component g of (1, unit vector), T_g, T_{4-g}, unused
  float wt[kPairChunk][2];                // weight, 2 T_4
  float pad[8];  // 80 words a particle: the reads of four particles fall on distinct banks
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// acc[m][r] of lane a (a > 0): T[k = r + 4 m][a]; T0[m] of lane g: T[k = g + 4 m][0],
// whose term is the unrounded product w T_k (fused), where the vector components
// take the rounded one.
__device__ __forceinline__ void accumulate_pairs(f32x4 (&acc)[8], float (&T0)[8], const float4 pi,
                                                 const float4* __restrict__ cpos, const int* list, int cnt, int g,
                                                 const CellGeo& c, PairSlots& S) {
  const float inv_rc = 1.0f / c.rc;
  int most = cnt;  // of the wave's 16 particles
#pragma unroll
  for (int off = kDescLanes; off < 64; off <<= 1) most = max(most, __shfl_xor(most, off, 64));
  const int rounds = __builtin_amdgcn_readfirstlane((most + kPairChunk - 1) / kPairChunk);
#pragma unroll 1
  for (int round = 0; round < rounds; ++round) {
    const int t0 = round * kPairChunk;
    float w = 0.0f, u1 = 0.0f, u2 = 0.0f, u3 = 0.0f, x = 0.0f;
    if (t0 + g < cnt) {
      const float4 pj = cpos[list[t0 + g]];
      float d0 = pj.x - pi.x, d1 = pj.y - pi.y, d2 = pj.z - pi.z;
      d0 -= c.L[0] * rintf(d0 * c.invL[0]);
      d1 -= c.L[1] * rintf(d1 * c.invL[1]);
      d2 -= c.L[2] * rintf(d2 * c.invL[2]);
      const float r2 = d0 * d0 + d1 * d1 + d2 * d2;
      const float r = sqrtf(r2), ir = 1.0f / r;
      const float sw = 0.5f * (1.0f + __cosf(3.14159265358979f * r * inv_rc));
      w = pj.w * sw;
      u1 = d0 * ir;
      u2 = d1 * ir;
      u3 = d2 * ir;
      x = 2.0f * r * inv_rc - 1.0f;
    }
    const float t2 = 2.0f * x * x - 1.0f, t3 = 2.0f * x * t2 - x, t4 = 2.0f * x * t3 - t2;
    *reinterpret_cast<float4*>(S.lane[g][0]) = make_float4(1.0f, 1.0f, t4, 0.0f);
    *reinterpret_cast<float4*>(S.lane[g][1]) = make_float4(u1, x, t3, 0.0f);
    *reinterpret_cast<float4*>(S.lane[g][2]) = make_float4(u2, t2, t2, 0.0f);
    *reinterpret_cast<float4*>(S.lane[g][3]) = make_float4(u3, t3, x, 0.0f);
    *reinterpret_cast<float2*>(S.wt[g]) = make_float2(w, 2.0f * t4);
    wave_lds_fence();  // the round's slots written
    // unrolled: as a loop the compiler copies all 40 sums in and out of it every
    // round; the barriers keep it from holding all four pairs' slots at once
    float2 wt_next = *reinterpret_cast<const float2*>(S.wt[0]);
    float4 v_next = *reinterpret_cast<const float4*>(S.lane[0][g]);
#pragma unroll
    for (int t = 0; t < kPairChunk; ++t) {
      const float2 wt = wt_next;
      const float4 v = v_next;
      if (t + 1 < kPairChunk) {
        wt_next = *reinterpret_cast<const float2*>(S.wt[t + 1]);
        v_next = *reinterpret_cast<const float4*>(S.lane[t + 1][g]);
      }
      __builtin_amdgcn_sched_barrier(0);
      float cur = v.y, prev = v.z;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        if (m > 0) {
          const float nxt = wt.y * cur - prev;
          prev = cur;
          cur = nxt;
        }
        T0[m] = fmaf(wt.x, cur, T0[m]);
        acc[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(wt.x * cur, v.x, acc[m], 0, 0, 0);
      }
    }
    wave_lds_fence();  // all four lanes done before the next round
  }
}

// quad_perm data movement: lane g of a quad takes the value of lane (ctrl >> 2g) & 3
template <int CTRL>
__device__ __forceinline__ float quad_perm(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

template <int CTRL>
__device__ __forceinline__ unsigned quad_perm_u(unsigned v) {
  return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}

// 4 x 4 transpose over the quad: lane g, element r <-> lane r, element g
__device__ __forceinline__ void quad_transpose(float (&v)[4], int g) {
  constexpr int kXor1 = 0xB1, kXor2 = 0x4E;  // [1,0,3,2], [2,3,0,1]
  const bool b0 = g & 1, b1 = g & 2;
#pragma unroll
  for (int r = 0; r < 4; r += 2) {
    const float got = quad_perm<kXor1>(b0 ? v[r] : v[r + 1]);
    v[r] = b0 ? got : v[r];
    v[r + 1] = b0 ? v[r + 1] : got;
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const float got = quad_perm<kXor2>(b1 ? v[r] : v[r + 2]);
    v[r] = b1 ? got : v[r];
    v[r + 2] = b1 ? v[r + 2] : got;
  }
}

// Row k = g + 4 m of the descriptor in lane g (all four lanes call it).
__device__ __forceinline__ void descriptor_row(float (&T)[4], const f32x4& acc, float T0, int g) {
#pragma unroll
  for (int r = 0; r < 4; ++r) T[r] = acc[r];
  quad_transpose(T, g);
  T[0] = T0;
}

// Lists the next neighbours of the particle at pi (on: there is one; this is lane
// g of its four), from chunk `chunk` of segment q on, until its candidates end
// (q = kSegments) or a list of the wave is full, and returns how many.  The whole
// wave calls it.
__device__ __forceinline__ int scan_neighbours(const float4 pi, bool on, int g, const float4* __restrict__ cpos,
                                               const int* __restrict__ start, const CellGeo& c, int& q, int& chunk,
                                               int* list) {
  const float rc2 = c.rc * c.rc;
  CellWalk w{start, c.nc[0], c.nc[1], c.nc[2], min((int)(pi.x * c.cinv[0]), c.nc[0] - 1),
             min((int)(pi.y * c.cinv[1]), c.nc[1] - 1), min((int)(pi.z * c.cinv[2]), c.nc[2] - 1), on, 0, 0, 0, 0};
  // cells before 0 or past the end are one box length away
  auto shifts = [&](int q, float& sx, float& sy, float& sz) {
    const int y = w.row_y(q), z = w.row_z(q);
    sx = q & 1 ? (w.cx == w.nx - 1 ? -c.L[0] : 0.0f) : (w.cx == 0 ? c.L[0] : 0.0f);
    sy = y < 0 ? c.L[1] : y >= w.ny ? -c.L[1] : 0.0f;
    sz = z < 0 ? c.L[2] : z >= w.nz ? -c.L[2] : 0.0f;
  };
  const int dq = __any(w.at_end()) ? 1 : 2;  // second ranges only where a particle of the wave has one
  int cnt = 0;
  float sx, sy, sz;
  w.begin(q, chunk, dq);
  shifts(q, sx, sy, sz);
  // candidates j0 + 4 u + g, u < kScan, of the next chunk (those past the range are
  // masked below; the array has kScanPad spare entries for the last range's)
  float3 pj[kScan];
  auto fetch = [&]() {
    const float4* src = cpos + w.j0 + g;
#pragma unroll
    for (int u = 0; u < kScan; ++u) pj[u] = *reinterpret_cast<const float3*>(src + kDescLanes * u);
  };
  fetch();
  while (q < kSegments && !__any(cnt > kNbrMax)) {
    const int jc = w.j0 + g;
    const int left = w.left();
    // bit 4 u + g of the particle's word: candidate 4 u + g is inside the cutoff
    // (and not at the particle's own place: not itself)
    unsigned bits = 0u;
    auto test = [&](int u, float d0, float d1, float d2) {
      const float r2 = d0 * d0 + d1 * d1 + d2 * d2;
      bits |= (r2 < rc2 && r2 > 0.0f) ? 1u << (kDescLanes * u) : 0u;
    };
    if (__any(sx != 0.0f || sy != 0.0f || sz != 0.0f)) {
#pragma unroll
      for (int u = 0; u < kScan; ++u) test(u, (pj[u].x - pi.x) - sx, (pj[u].y - pi.y) - sy, (pj[u].z - pi.z) - sz);
    } else {
#pragma unroll
      for (int u = 0; u < kScan; ++u) test(u, pj[u].x - pi.x, pj[u].y - pi.y, pj[u].z - pi.z);
    }
    // the next chunk's candidates arrive while this one's are listed
    w.advance();
    ++chunk;
    if (!__any(w.j0 < w.j1)) {
      q += dq;
      chunk = 0;
      w.next_segment(q + dq);
      shifts(min(q, kSegments - 1), sx, sy, sz);
    }
    fetch();
    bits <<= g;
    unsigned word = bits | quad_perm_u<0xB1>(bits);
    word |= quad_perm_u<0x4E>(word);
    word &= (1u << left) - 1u;  // what lies past the range is dropped
    // each lane lists its own candidates at their places in candidate order
    // (the others go to a spare entry)
    int place = cnt + __popc(word & ((1u << g) - 1u));
    const unsigned own = word >> g;
#pragma unroll
    for (int u = 0; u < kScan; ++u) {
      list[own & (1u << (kDescLanes * u)) ? place : kNbrList - 1] = jc + kDescLanes * u;
      place += __popc(own & (0xfu << (kDescLanes * u)));
    }
    cnt += __popc(word);
  }
  return cnt;
}

// The descriptor of particle i into acc and T0 of its four lanes (of which this
// is lane g); list and S: the particle's LDS.  Returns the neighbour count.
// The whole wave calls it.  More neighbours than a list holds are taken in rounds, each
// of which goes on where the one before stopped (a scan of all candidates in every
// round took 16.7 ms for 20,000 particles in a droplet of 4 A; this way 2.3);
// the sums wait in the particle's row of T meanwhile, so that they are not live
// during a scan (they would cost it a third of its registers).
__device__ __forceinline__ int describe(f32x4 (&acc)[8], float (&T0)[8], const float4 pi, int i, bool on, int g,
                                        const float4* __restrict__ cpos, const int* __restrict__ start,
                                        const CellGeo& c, float* __restrict__ Tbuf, int* list, PairSlots& S) {
  float4* rows = reinterpret_cast<float4*>(Tbuf + (size_t)i * 128);
  int total = 0, q = 0, chunk = 0;
  do {
    const bool first = q + chunk == 0;
    const int cnt = scan_neighbours(pi, on, g, cpos, start, c, q, chunk, list);
    wave_lds_fence();
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      acc[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      T0[m] = 0.0f;
    }
    if (!first) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const float4 r = on ? rows[g + 4 * m] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float T[4] = {r.x, r.y, r.z, r.w};
        T0[m] = T[0];
        quad_transpose(T, g);
        acc[m] = f32x4{T[0], T[1], T[2], T[3]};
      }
    }
    accumulate_pairs(acc, T0, pi, cpos, list, cnt, g, c, S);
    total += cnt;
    if (q < kSegments) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        float T[4];
        descriptor_row(T, acc[m], T0[m], g);
        if (on) rows[g + 4 * m] = make_float4(T[0], T[1], T[2], T[3]);
      }
    }
  } while (q < kSegments);
  return total;
}

// Calls out(k, T, x) for the lane's rows k = g + 4 m: T[k][0..3] and the four
// network inputs 4k + l from the invariants D[4k + l] = sum_a T[k][a] T[l][a].
template <typename Out>
__device__ __forceinline__ void descriptor_inputs(const f32x4 (&acc)[8], const float (&T0)[8], int g,
                                                  const float* __restrict__ params, Out out) {
  const float4* mu = reinterpret_cast<const float4*>(params + kOffMu);
  const float4* isd = reinterpret_cast<const float4*>(params + kOffIsd);
  float Tl[4][4];  // T[l] is order 0 of lane l
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    float T[4];
    descriptor_row(T, acc[m], T0[m], g);
    if (m == 0) {
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        Tl[0][a] = quad_perm<0x00>(T[a]);
        Tl[1][a] = quad_perm<0x55>(T[a]);
        Tl[2][a] = quad_perm<0xAA>(T[a]);
        Tl[3][a] = quad_perm<0xFF>(T[a]);
      }
    }
    const int k = g + 4 * m;
    const float4 mk = mu[k], sk = isd[k];
    const float mv[4] = {mk.x, mk.y, mk.z, mk.w}, sv[4] = {sk.x, sk.y, sk.z, sk.w};
    bf16x4 x;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      const float d = T[0] * Tl[l][0] + T[1] * Tl[l][1] + T[2] * Tl[l][2] + T[3] * Tl[l][3];
      x[l] = (__bf16)((d - mv[l]) * sv[l]);
    }
    out(k, T, x);
  }
}

__global__ void __launch_bounds__(kDescThreads, 4) k_descriptor(const float4* __restrict__ cpos,
                                                                const int* __restrict__ start, int n,
                                                                const float* __restrict__ params,
                                                                float* __restrict__ Tout,
                                                                unsigned short* __restrict__ X, CellGeo c) {
  __shared__ int lists[kDescParts][kNbrList];
  __shared__ __align__(16) PairSlots slots[kDescParts];
  const int g = threadIdx.x & (kDescLanes - 1), p = threadIdx.x / kDescLanes;
  const int i = blockIdx.x * kDescParts + p;
  const bool on = i < n;
  f32x4 acc[8];
  float T0[8];
  (void)describe(acc, T0, cpos[min(i, n - 1)], i, on, g, cpos, start, c, Tout, lists[p], slots[p]);
  float4* to = reinterpret_cast<float4*>(Tout + (size_t)i * 128);
  bf16x4* xo = reinterpret_cast<bf16x4*>(X + (size_t)i * 128);
  descriptor_inputs(acc, T0, g, params, [&](int k, const float (&T)[4], const bf16x4& x) {
    if (on) {
      to[k] = make_float4(T[0], T[1], T[2], T[3]);
      xo[k] = x;
    }
  });
}

// ---------------------------------------------------------------------------
// LDS operand layout for the MFMA tiles: every matrix is stored with the
// contraction index k contiguous and rows padded by 4 bf16 (8 bytes), so a
// lane's eight k values are two 64-bit LDS reads and the 32 rows a half-wave
// reads fall on distinct banks (row pitch / 8 bytes is odd).
// ---------------------------------------------------------------------------
constexpr int kPadIn = kIn + 4;     // 132: rows of 128 bf16
constexpr int kPadH = kH + 4;       // 68: rows of 64 bf16
constexpr int kPadO = kOut + 4;     // 36: rows of 32 bf16

// acc (32 x 32) += A (32 x K) * B (K x 32) with both operands k-contiguous:
// A(m, k) = A[m * lda + k], B(k, n) = B[n * ldb + k].  One gfx950
// v_mfma_f32_32x32x16_bf16 per 16 values of k: lane l supplies
// A(l % 32, 8 (l / 32) + i) and B(8 (l / 32) + i, l % 32), i < 8, read as two
// 8-byte LDS loads (rows are 8-byte aligned); K is a multiple of 16.
__device__ __forceinline__ void mfma_tile_kc(f32x16& acc, const unsigned short* A, int lda,
                                             const unsigned short* B, int ldb, int K) {
  const int l = threadIdx.x & 63;
  const int mn = l & 31, kh = (l >> 5) * 8;
  const unsigned short* pa = A + mn * lda + kh;
  const unsigned short* pb = B + mn * ldb + kh;
#pragma unroll 4
  for (int k0 = 0; k0 < K; k0 += 16) {
    const bf16x4 a0 = *reinterpret_cast<const bf16x4*>(pa + k0);
    const bf16x4 a1 = *reinterpret_cast<const bf16x4*>(pa + k0 + 4);
    const bf16x4 b0 = *reinterpret_cast<const bf16x4*>(pb + k0);
    const bf16x4 b1 = *reinterpret_cast<const bf16x4*>(pb + k0 + 4);
    const bf16x8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
    const bf16x8 b = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
  }
}

// The same for two B tiles sharing A: acc0 += A B0, acc1 += A B1.
__device__ __forceinline__ void mfma_tile_kc2(f32x16& acc0, f32x16& acc1, const unsigned short* A, int lda,
                                              const unsigned short* B0, const unsigned short* B1, int ldb, int K) {
  const int l = threadIdx.x & 63;
  const int mn = l & 31, kh = (l >> 5) * 8;
  const unsigned short* pa = A + mn * lda + kh;
  const unsigned short* p0 = B0 + mn * ldb + kh;
  const unsigned short* p1 = B1 + mn * ldb + kh;
#pragma unroll 4
  for (int k0 = 0; k0 < K; k0 += 16) {
    const bf16x4 a0 = *reinterpret_cast<const bf16x4*>(pa + k0);
    const bf16x4 a1 = *reinterpret_cast<const bf16x4*>(pa + k0 + 4);
    const bf16x4 b00 = *reinterpret_cast<const bf16x4*>(p0 + k0);
    const bf16x4 b01 = *reinterpret_cast<const bf16x4*>(p0 + k0 + 4);
    const bf16x4 b10 = *reinterpret_cast<const bf16x4*>(p1 + k0);
    const bf16x4 b11 = *reinterpret_cast<const bf16x4*>(p1 + k0 + 4);
    const bf16x8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
    const bf16x8 b0 = __builtin_shufflevector(b00, b01, 0, 1, 2, 3, 4, 5, 6, 7);
    const bf16x8 b1 = __builtin_shufflevector(b10, b11, 0, 1, 2, 3, 4, 5, 6, 7);
    acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b0, acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b1, acc1, 0, 0, 0);
  }
}

// weight offsets in the padded LDS copies
constexpr int kLW1t = 0, kLW2t = kLW1t + kH * kPadIn, kLW3t = kLW2t + kH * kPadH,
              kLW4t = kLW3t + kH * kPadH, kLWt = kLW4t + kOut * kPadH;  // [out][in] copies

// ---------------------------------------------------------------------------
// The correction of 32 particles per block in one pass: descriptor, network and
// force head, with nothing but the forces written.  (As two kernels the
// descriptor and the network input, 768 bytes a particle, went through memory:
// at 288,768 particles the descriptor kernel spent 85 of its 218 us writing them
// and the network kernel 89 us mostly reading them; this kernel takes 213.)
// What is left is VALU issue: of 222 us, when full lists began their scan anew,
// about 83 were scan, 88 pairs and 22 network, the rest the inputs and the head.
// Two waves hold 16 particles each for the descriptor; for the network, wave w
// computes features 32 w .. 32 w + 31 of all 32 particles: weights as the A
// operand in fragment order straight from L2 (36 KB, read by every block; LDS
// would cost the scan its occupancy), activations as the B operand from LDS, so
// that a lane ends with four consecutive features of one particle and writes
// them as 8 bytes.  The order of every sum that is rounded to bf16 is that of
// k_mlp_fwd.
// ---------------------------------------------------------------------------
constexpr int kCorrThreads = 128;
constexpr int kCorrRows = 32;  // particles per block
constexpr int kFrags[4] = {16, 8, 8, 4};
constexpr int kFragOfs[4] = {0, 16, 24, 32};  // 36 fragments of 64 lanes x 8 values

union CorrLds {
  struct {
    int lists[kCorrRows][kNbrList];
    PairSlots slots[kCorrRows];
  } d;
  struct {
    union {
      unsigned short x[kCorrRows][kPadIn];  // network input, then the second hidden layer,
      unsigned short h1[kCorrRows][kPadH];
      float c[kCorrRows][kOut + 4];         // then the head's coefficients
    };
    unsigned short h0[kCorrRows][kPadH];    // first and third hidden layer
  } m;
};

// Per-block statistics of the forward, reduced by k_forward_stats.
struct FwdPart {
  int lo, hi;            // neighbour counts
  unsigned corr, force;  // max |dF|, max |F| (float bits)
};

// One hidden layer's tile: out(32 particles x 32 features of this wave) =
// silu(in W + b), bf16.
template <int K>
__device__ __forceinline__ void corr_layer(const unsigned short* in, int ldin, const unsigned short* __restrict__ frag,
                                           const float* __restrict__ bias, unsigned short* out) {
  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6, kh = l >> 5, n = l & 31;
  const bf16x8* A = reinterpret_cast<const bf16x8*>(frag) + (size_t)wave * (K / 16) * 64 + l;
  const unsigned short* B = in + n * ldin + 8 * kh;
  f32x16 acc;
  zero(acc);
#pragma unroll
  for (int s = 0; s < K / 16; ++s) {
    const bf16x8 a = A[64 * s];
    const bf16x4 b0 = *reinterpret_cast<const bf16x4*>(B + 16 * s);
    const bf16x4 b1 = *reinterpret_cast<const bf16x4*>(B + 16 * s + 4);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7), acc, 0,
                                                  0, 0);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int f = 32 * wave + 8 * q + 4 * kh;
    const float4 bv = *reinterpret_cast<const float4*>(bias + f);
    const float z[4] = {acc[4 * q] + bv.x, acc[4 * q + 1] + bv.y, acc[4 * q + 2] + bv.z, acc[4 * q + 3] + bv.w};
    bf16x4 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (__bf16)silu(z[e]);
    *reinterpret_cast<bf16x4*>(out + n * kPadH + f) = h;
  }
}

__global__ void __launch_bounds__(kCorrThreads, 4) k_correction(const float4* __restrict__ cpos,
                                                                const int* __restrict__ cidx,
                                                                const int* __restrict__ start, int n, int64_t n_ion,
                                                                float* __restrict__ Tbuf,
                                                                const unsigned short* __restrict__ wf,
                                                                const float* __restrict__ params, float s_out,
                                                                float* __restrict__ ion_dF, float* __restrict__ wc_dF,
                                                                int accumulate, CellGeo c,
                                                                FwdPart* __restrict__ part) {
  __shared__ __align__(16) CorrLds S;
  __shared__ FwdPart wpart[kCorrThreads / 64];
  const int g = threadIdx.x & (kDescLanes - 1), p = threadIdx.x / kDescLanes;
  const int i = blockIdx.x * kCorrRows + p;
  const bool on = i < n;
  f32x4 acc[8];
  float T0[8];
  const float4 pi = cpos[min(i, n - 1)];
  const int total = describe(acc, T0, pi, i, on, g, cpos, start, c, Tbuf, S.d.lists[p], S.d.slots[p]);
  __syncthreads();  // both waves are done with the lists
  descriptor_inputs(acc, T0, g, params, [&](int k, const float (&)[4], const bf16x4& x) {
    *reinterpret_cast<bf16x4*>(&S.m.x[p][4 * k]) = x;
  });
  __syncthreads();
  corr_layer<kIn>(&S.m.x[0][0], kPadIn, wf + kFragOfs[0] * 512, params + kOffB1, &S.m.h0[0][0]);
  __syncthreads();
  corr_layer<kH>(&S.m.h0[0][0], kPadH, wf + kFragOfs[1] * 512, params + kOffB2, &S.m.h1[0][0]);
  __syncthreads();
  corr_layer<kH>(&S.m.h1[0][0], kPadH, wf + kFragOfs[2] * 512, params + kOffB3, &S.m.h0[0][0]);
  __syncthreads();
  // output layer: c = h3 W4 + b4, one tile, by the waves in turn from block to block
  if ((int)(threadIdx.x >> 6) == (int)(blockIdx.x & 1)) {
    const int l = threadIdx.x & 63, kh = l >> 5, r = l & 31;
    const bf16x8* A = reinterpret_cast<const bf16x8*>(wf + kFragOfs[3] * 512) + l;
    const unsigned short* B = &S.m.h0[r][8 * kh];
    f32x16 o;
    zero(o);
#pragma unroll
    for (int s = 0; s < kH / 16; ++s) {
      const bf16x4 b0 = *reinterpret_cast<const bf16x4*>(B + 16 * s);
      const bf16x4 b1 = *reinterpret_cast<const bf16x4*>(B + 16 * s + 4);
      o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[64 * s], __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7),
                                                  o, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int f = 8 * q + 4 * kh;
      const float4 bv = *reinterpret_cast<const float4*>(params + kOffB4 + f);
      *reinterpret_cast<float4*>(&S.m.c[r][f]) =
          make_float4(o[4 * q] + bv.x, o[4 * q + 1] + bv.y, o[4 * q + 2] + bv.z, o[4 * q + 3] + bv.w);
    }
  }
  __syncthreads();
  // head: dF = s_out q sum_k c_k T[k, 1:4], each lane over its orders, then the quad
  // (the rows are put together again: kept from above they would be 32 more
  // registers through the network)
  float f0 = 0.0f, f1 = 0.0f, f2 = 0.0f;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    float T[4];
    asm volatile("" : "+v"(acc[m]));
    descriptor_row(T, acc[m], T0[m], g);
    const float cc = S.m.c[p][g + 4 * m];
    f0 += cc * T[1];
    f1 += cc * T[2];
    f2 += cc * T[3];
  }
  f0 += quad_perm<0xB1>(f0);
  f1 += quad_perm<0xB1>(f1);
  f2 += quad_perm<0xB1>(f2);
  f0 += quad_perm<0x4E>(f0);
  f1 += quad_perm<0x4E>(f1);
  f2 += quad_perm<0x4E>(f2);
  int lo = 0x7fffffff, hi = 0;
  unsigned mcorr = 0u, mforce = 0u;
  if (on && g == 0) {
    const float sq = s_out * pi.w;
    f0 *= sq; f1 *= sq; f2 *= sq;
    const int src = cidx[i];
    float* out = (src < n_ion) ? ion_dF + 3 * (int64_t)src : wc_dF + 3 * ((int64_t)src - n_ion);
    mcorr = __float_as_uint(sqrtf(f0 * f0 + f1 * f1 + f2 * f2));
    if (accumulate) {
      mforce = __float_as_uint(sqrtf(out[0] * out[0] + out[1] * out[1] + out[2] * out[2]));
      f0 += out[0]; f1 += out[1]; f2 += out[2];
    }
    out[0] = f0; out[1] = f1; out[2] = f2;
    lo = hi = total;
  }
  // the block's statistics
  for (int off = 32; off >= kDescLanes; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
    mcorr = max(mcorr, (unsigned)__shfl_xor((int)mcorr, off, 64));
    mforce = max(mforce, (unsigned)__shfl_xor((int)mforce, off, 64));
  }
  if ((threadIdx.x & 63) == 0) wpart[threadIdx.x >> 6] = FwdPart{lo, hi, mcorr, mforce};
  __syncthreads();
  if (threadIdx.x == 0) {
    const FwdPart a = wpart[0], b = wpart[1];
    part[blockIdx.x] = FwdPart{a.lo < b.lo ? a.lo : b.lo, a.hi > b.hi ? a.hi : b.hi,
                               a.corr > b.corr ? a.corr : b.corr, a.force > b.force ? a.force : b.force};
  }
}

// Statistics of the forward from the block partials (integer minima and
// maxima: independent of the order; nblk = 0 for an input of no particles).
__global__ void __launch_bounds__(1024) k_forward_stats(const FwdPart* __restrict__ part, int nblk,
                                                        Stats* __restrict__ st) {
  __shared__ FwdPart w[16];
  FwdPart a{0x7fffffff, 0, 0u, 0u};
  auto add = [&](const FwdPart& b) {
    a.lo = min(a.lo, b.lo);
    a.hi = max(a.hi, b.hi);
    a.corr = a.corr > b.corr ? a.corr : b.corr;
    a.force = a.force > b.force ? a.force : b.force;
  };
  for (int k = threadIdx.x; k < nblk; k += blockDim.x) add(part[k]);
  for (int off = 32; off > 0; off >>= 1)
    add(FwdPart{(int)__shfl_xor(a.lo, off, 64), (int)__shfl_xor(a.hi, off, 64),
                (unsigned)__shfl_xor((int)a.corr, off, 64), (unsigned)__shfl_xor((int)a.force, off, 64)});
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 16; ++k) add(w[k]);
    st->max_corr_bits = a.corr;
    st->max_force_bits = a.force;
    st->min_nbr = a.lo;
    st->max_nbr = a.hi;
  }
}

// ---------------------------------------------------------------------------
// MLP forward + force head of a training step.  Persistent blocks of 4 waves
// stage the weights (bf16, [out][in]) and biases once, then walk tiles of 128
// particles; wave w owns rows 32w..32w+31 of a tile.  Activations go layer to
// layer through LDS.  The pre-activations z1..z3 and activations h1..h3 are
// stored, and the head forms the loss and dL/dc.
// ---------------------------------------------------------------------------
struct FwdLds {
  unsigned short wt[kLWt];
  float b[kH * 3 + kOut];
  unsigned short x[kRows][kPadIn];
  unsigned short h[2][kRows][kPadH];
  float c[kRows][kOut + 1];
  double lred[4];
};

__global__ void __launch_bounds__(256) k_mlp_fwd(const unsigned short* __restrict__ X, const float* __restrict__ Tin,
                                                 const float4* __restrict__ cpos, const int* __restrict__ cidx,
                                                 int n, int64_t n_ion, const unsigned short* __restrict__ wt_g,
                                                 const float* __restrict__ params, float s_out,
                                                 const float* __restrict__ ion_tgt, const float* __restrict__ wc_tgt,
                                                 const float* __restrict__ ion_base, const float* __restrict__ wc_base,
                                                 float* __restrict__ Z, unsigned short* __restrict__ H,
                                                 float* __restrict__ dC, double* __restrict__ loss_part, float gscale) {
  extern __shared__ __align__(16) unsigned char smem[];
  FwdLds& S = *reinterpret_cast<FwdLds*>(smem);
  const int tid = threadIdx.x, wave = tid >> 6;
  // weights: global [out][in] (dense) -> LDS rows padded, in 16-byte chunks
  // of 8 values whose loads are all in flight before the first LDS store (a
  // loop with a run-time trip count would wait for each load in turn)
  {
    const int cols[4] = {kIn, kH, kH, kH};
    const int gofs[4] = {0, kIn * kH, kIn * kH + kH * kH, kIn * kH + 2 * kH * kH};
    const int lofs[4] = {kLW1t, kLW2t, kLW3t, kLW4t}, pitch[4] = {kPadIn, kPadH, kPadH, kPadH};
    constexpr int kChunks = kNWeights / 8, kPer = (kChunks + kMlpThreads - 1) / kMlpThreads;
    uint4 wv[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int c = tid + u * kMlpThreads;
      if (c < kChunks) wv[u] = reinterpret_cast<const uint4*>(wt_g)[c];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int c = tid + u * kMlpThreads;
      if (c < kChunks) {
        const int e = 8 * c;
        const int L = e < gofs[1] ? 0 : e < gofs[2] ? 1 : e < gofs[3] ? 2 : 3;
        const int el = e - gofs[L], r = el / cols[L], col = el - r * cols[L];
        uint2* dst = reinterpret_cast<uint2*>(S.wt + lofs[L] + r * pitch[L] + col);  // 8-byte aligned
        dst[0] = make_uint2(wv[u].x, wv[u].y);
        dst[1] = make_uint2(wv[u].z, wv[u].w);
      }
    }
  }
  for (int e = tid; e < kH; e += blockDim.x) {
    S.b[e] = params[kOffB1 + e];
    S.b[kH + e] = params[kOffB2 + e];
    S.b[2 * kH + e] = params[kOffB3 + e];
  }
  for (int e = tid; e < kOut; e += blockDim.x) S.b[3 * kH + e] = params[kOffB4 + e];

  const int wr = wave * 32;  // this wave's first row in the tile
  const unsigned short* wl[4] = {S.wt + kLW1t, S.wt + kLW2t, S.wt + kLW3t, S.wt + kLW4t};
  const int ldw[4] = {kPadIn, kPadH, kPadH, kPadH};
  double lsum = 0.0;
  const int ntiles = (n + kRows - 1) / kRows;
  // A tile's inputs travel in 16-byte chunks held in registers: the next
  // tile's loads are issued while the current tile computes (the block's
  // barriers wait on LDS only, so the loads stay in flight across them).
  constexpr int kXc = kRows * kIn / 8, kXper = kXc / kMlpThreads;
  uint4 xv[kXper];
  auto load_x = [&](int tile) {
#pragma unroll
    for (int u = 0; u < kXper; ++u) {
      const int c = tid + u * kMlpThreads, r = c / (kIn / 8), c8 = c % (kIn / 8);
      const int row = tile * kRows + r;
      xv[u] = make_uint4(0u, 0u, 0u, 0u);
      if (tile < ntiles && row < n) xv[u] = reinterpret_cast<const uint4*>(X + (size_t)row * kIn)[c8];
    }
  };
  load_x(blockIdx.x);
  // head: two threads per particle (hp = particle in the tile, hk = which
  // half of the 32 radial orders); the particle's descriptor rows are loaded
  // at the start of the tile, so that they arrive during the layers
  const int hp = tid >> 1, hk = tid & 1;
  constexpr int kHalf = kOut / 2;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int row0 = tile * kRows;
    const bool hon = row0 + hp < n;
    float4 tq[kHalf];
    if (hon) {
      const float4* Tp = reinterpret_cast<const float4*>(Tin + (size_t)(row0 + hp) * 128) + hk * kHalf;
#pragma unroll
      for (int k = 0; k < kHalf; ++k) tq[k] = Tp[k];
    }
    __syncthreads();  // previous tile done with S.x / S.c; weights staged
#pragma unroll
    for (int u = 0; u < kXper; ++u) {
      const int c = tid + u * kMlpThreads, r = c / (kIn / 8), c8 = c % (kIn / 8);
      uint2* dst = reinterpret_cast<uint2*>(&S.x[r][8 * c8]);  // 8-byte aligned rows
      dst[0] = make_uint2(xv[u].x, xv[u].y);
      dst[1] = make_uint2(xv[u].z, xv[u].w);
    }
    __syncthreads();
    load_x(tile + gridDim.x);
    // hidden layers
#pragma unroll
    for (int layer = 0; layer < 3; ++layer) {
      const int K = layer == 0 ? kIn : kH;
      const unsigned short* A = layer == 0 ? &S.x[wr][0] : &S.h[(layer - 1) & 1][wr][0];
      const int lda = layer == 0 ? kPadIn : kPadH;
      unsigned short* Hout = &S.h[layer & 1][wr][0];
      // both 32-column tiles of the layer in one pass over k (two independent
      // accumulation chains in flight)
      static_assert(kH == 64, "two 32-column tiles per hidden layer");
      f32x16 acc2[2];
      zero(acc2[0]);
      zero(acc2[1]);
      mfma_tile_kc2(acc2[0], acc2[1], A, lda, wl[layer], wl[layer] + 32 * ldw[layer], ldw[layer], K);
#pragma unroll
      for (int nt = 0; nt < kH / 32; ++nt) {
        const f32x16& acc = acc2[nt];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = acc_row(r), col = nt * 32 + acc_col();
          const float z = acc[r] + S.b[layer * kH + col];
          const float h = silu(z);
          const unsigned short hb = f2bf(h);
          Hout[row * kPadH + col] = hb;
          if (row0 + wr + row < n) {
            Z[((size_t)layer * n + row0 + wr + row) * kH + col] = z;
            H[((size_t)layer * n + row0 + wr + row) * kH + col] = hb;
          }
        }
      }
      __syncthreads();
    }
    // output layer: c = h3 W4 + b4
    {
      f32x16 acc;
      zero(acc);
      mfma_tile_kc(acc, &S.h[0][wr][0], kPadH, wl[3], ldw[3], kH);
#pragma unroll
      for (int r = 0; r < 16; ++r) S.c[wr + acc_row(r)][acc_col()] = acc[r] + S.b[3 * kH + acc_col()];
    }
    __syncthreads();

    // head: dF = s_out q sum_k c_k T[k, 1:4], each thread over its half of k
    // (in order), the halves added in the order (0, 1)
    {
      float f0 = 0.f, f1 = 0.f, f2 = 0.f;
      if (hon) {
#pragma unroll
        for (int k = 0; k < kHalf; ++k) {
          const float cc = S.c[hp][hk * kHalf + k];
          f0 += cc * tq[k].y;
          f1 += cc * tq[k].z;
          f2 += cc * tq[k].w;
        }
      }
      const float o0 = __shfl_xor(f0, 1, 64), o1 = __shfl_xor(f1, 1, 64), o2 = __shfl_xor(f2, 1, 64);
      // both threads of the pair form the same sums: half 0 first
      f0 = hk == 0 ? f0 + o0 : o0 + f0;
      f1 = hk == 0 ? f1 + o1 : o1 + f1;
      f2 = hk == 0 ? f2 + o2 : o2 + f2;
      if (hon) {
        const int slot = row0 + hp;
        const float q = cpos[slot].w;
        const float sq = s_out * q;
        // the prediction is a rounded FP32 force (not fused into the error below)
        f0 = mul_rounded(f0, sq); f1 = mul_rounded(f1, sq); f2 = mul_rounded(f2, sq);
        const int src = cidx[slot];
        // target: the residual target - base (fine minus coarse forces) when a base is given
        const int64_t o3 = (src < n_ion) ? 3 * (int64_t)src : 3 * ((int64_t)src - n_ion);
        const float* tg = ((src < n_ion) ? ion_tgt : wc_tgt) + o3;
        const float* bs = (src < n_ion) ? ion_base : wc_base;
        float t0 = tg[0], t1 = tg[1], t2 = tg[2];
        if (bs) { t0 -= bs[o3]; t1 -= bs[o3 + 1]; t2 -= bs[o3 + 2]; }
        const float e0 = f0 - t0, e1 = f1 - t1, e2 = f2 - t2;
        if (hk == 0) lsum += (double)e0 * e0 + (double)e1 * e1 + (double)e2 * e2;
        // dL/d dF = gscale * e (gscale = 2 / (3 n)); dL/dc_k = s_out q (g . T[k, 1:4])
        const float g0 = gscale * e0 * sq, g1 = gscale * e1 * sq, g2 = gscale * e2 * sq;
#pragma unroll
        for (int k = 0; k < kHalf; ++k)
          dC[(size_t)slot * kOut + hk * kHalf + k] = g0 * tq[k].y + g1 * tq[k].z + g2 * tq[k].w;
      }
    }
  }
  // deterministic block sum of the squared errors (the even threads hold them)
  for (int off = 32; off > 0; off >>= 1) lsum += __shfl_down(lsum, off, 64);
  __syncthreads();
  if ((tid & 63) == 0) S.lred[wave] = lsum;
  __syncthreads();
  if (tid == 0) loss_part[blockIdx.x] = S.lred[0] + S.lred[1] + S.lred[2] + S.lred[3];
}

// ---------------------------------------------------------------------------
// MLP backward.  A block of 4 waves walks tiles of 64 particles and keeps the
// gradients of all weights in registers over its tiles (18 tiles of 32 x 32, at
// most 5 a wave), so one partial gradient per block is written, to
// gpart[block][kNTrain] (summed by k_grad_update).  Per tile the layer inputs are
// staged transposed (features x particles) and dz in both layouts:
//   dW = act^T dz          contracts over the particles,
//   dh^T = W dz^T          contracts over the layer's outputs; a lane ends with
//                          four consecutive features of one particle.
// dz / dz^T are double-buffered across layers.  All global loads of a tile are
// 16 bytes a lane and issued before the first layer, the pre-activations
// included.  (Blocks of 128 particles with 2-byte loads took 71 us at 4,512
// particles, where 36 of them were all there were.)
// ---------------------------------------------------------------------------
constexpr int kBwdRows = 64;
constexpr int kBwdThreads = 256;
constexpr int kPadT = kBwdRows + 4;  // transposed tiles: rows of 64 particles
constexpr int kBW2 = 0, kBW3 = kBW2 + kH * kPadH, kBW4 = kBW3 + kH * kPadH, kBW = kBW4 + kH * kPadO;

struct BwdLds {
  unsigned short w[kBW];              // W2, W3, W4 as [in][out]
  unsigned short xT[kIn][kPadT];      // network input, transposed
  unsigned short hT[3][kH][kPadT];    // hidden layers, transposed
  unsigned short dz[2][kBwdRows][kPadH];  // gradient at the layer output (bf16)
  unsigned short dzT[2][kH][kPadT];   // the same, transposed
};

// 8 consecutive features f.. of particle r into a transposed tile
__device__ __forceinline__ void put_transposed(unsigned short (*tile)[kPadT], int f, int r, uint4 v) {
  const unsigned u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    tile[f + 2 * e][r] = (unsigned short)u[e];
    tile[f + 2 * e + 1][r] = (unsigned short)(u[e] >> 16);
  }
}

__global__ void __launch_bounds__(kBwdThreads) k_mlp_bwd(const unsigned short* __restrict__ X,
                                                         const float* __restrict__ Z,
                                                         const unsigned short* __restrict__ H,
                                                         const float* __restrict__ dC, int n,
                                                         const unsigned short* __restrict__ w_g,
                                                         float* __restrict__ gpart) {
  extern __shared__ __align__(16) unsigned char smem[];
  BwdLds& S = *reinterpret_cast<BwdLds*>(smem);
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63, kh = l >> 5;
  // weights, 8 outputs of one input at a time
  {
    constexpr int kChunks = (2 * kH * kH + kH * kOut) / 8;
#pragma unroll
    for (int c = tid; c < kChunks; c += kBwdThreads) {
      const uint4 v = reinterpret_cast<const uint4*>(w_g + kIn * kH)[c];
      const int e = 8 * c;
      int r, col, at;
      if (e < 2 * kH * kH) { r = (e / kH) % kH; col = e % kH; at = (e < kH * kH ? kBW2 : kBW3) + r * kPadH + col; }
      else { r = (e - 2 * kH * kH) / kOut; col = e % kOut; at = kBW4 + r * kPadO + col; }
      uint2* dst = reinterpret_cast<uint2*>(S.w + at);
      dst[0] = make_uint2(v.x, v.y);
      dst[1] = make_uint2(v.z, v.w);
    }
  }
  f32x16 g1[2], g2, g3, g4;  // this wave's tiles of dW1 (2 of 8), dW2, dW3 (1 of 4), dW4 (waves 0, 1)
  zero(g1[0]); zero(g1[1]); zero(g2); zero(g3); zero(g4);
  float gb[4] = {0.f, 0.f, 0.f, 0.f};  // bias sums of output tid / 4, a quarter of the particles
  // dh tile of this wave: inputs 32 (wave % 2).., particles 32 (wave / 2)..
  const int f0 = 32 * (wave & 1), r0 = 32 * (wave >> 1);
  const int ntiles = (n + kBwdRows - 1) / kBwdRows;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int row0 = tile * kBwdRows;
    // loads: particle tid % 64 and its features (tid / 64) * 8 + 32 u ..; the
    // pre-activations of the dh tile
    const int lr = tid & 63, row = min(row0 + lr, n - 1);
    const bool in = row0 + lr < n;
    uint4 xv[4], hv[3][2];
    float4 cv[2], zv[3][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) xv[u] = reinterpret_cast<const uint4*>(X + (size_t)row * kIn)[wave + 4 * u];
#pragma unroll
    for (int L = 0; L < 3; ++L)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        hv[L][u] = reinterpret_cast<const uint4*>(H + ((size_t)L * n + row) * kH)[wave + 4 * u];
#pragma unroll
    for (int u = 0; u < 2; ++u) cv[u] = reinterpret_cast<const float4*>(dC + (size_t)row * kOut)[2 * wave + u];
    const int zrow = min(row0 + r0 + (l & 31), n - 1);
    const bool zin = row0 + r0 + (l & 31) < n;
#pragma unroll
    for (int L = 0; L < 3; ++L)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        zv[L][q] = *reinterpret_cast<const float4*>(Z + ((size_t)L * n + zrow) * kH + f0 + 8 * q + 4 * kh);
    __syncthreads();  // the previous tile is done with the staged arrays
    // particles past n: their dz is zero, whatever the inputs hold
#pragma unroll
    for (int u = 0; u < 4; ++u) put_transposed(S.xT, 8 * (wave + 4 * u), lr, xv[u]);
#pragma unroll
    for (int L = 0; L < 3; ++L)
#pragma unroll
      for (int u = 0; u < 2; ++u) put_transposed(S.hT[L], 8 * (wave + 4 * u), lr, hv[L][u]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float c4[4] = {cv[u].x, cv[u].y, cv[u].z, cv[u].w};
      unsigned short b4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        b4[e] = in ? f2bf(c4[e]) : (unsigned short)0;
        S.dzT[0][8 * wave + 4 * u + e][lr] = b4[e];
      }
      *reinterpret_cast<ushort4*>(&S.dz[0][lr][8 * wave + 4 * u]) = make_ushort4(b4[0], b4[1], b4[2], b4[3]);
    }
    __syncthreads();
    // bias gradient of the layer whose dz is in buffer `cur`: output tid / 4
    auto bias = [&](int cur, int no, float& sum) {
      const int col = tid >> 2;
      if (col < no) {
        const unsigned short* z = &S.dzT[cur][col][(tid & 3) * 16];
        float s = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) s += bf2f(z[r]);
        sum += s;
      }
    };
    // dh of the layer below: (inputs x particles) = W dz^T, times silu'(z), into
    // buffer `nxt`
    auto back = [&](int cur, int nxt, const unsigned short* W, int pitch, int K, const float4 (&z)[4]) {
      f32x16 a;
      zero(a);
      mfma_tile_kc(a, W + f0 * pitch, pitch, &S.dz[cur][r0][0], kPadH, K);
      const int r = r0 + (l & 31);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float z4[4] = {z[q].x, z[q].y, z[q].z, z[q].w};
        const int f = f0 + 8 * q + 4 * kh;
        unsigned short b4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          b4[e] = zin ? f2bf(a[4 * q + e] * dsilu(z4[e])) : (unsigned short)0;
          S.dzT[nxt][f + e][r] = b4[e];
        }
        *reinterpret_cast<ushort4*>(&S.dz[nxt][r][f]) = make_ushort4(b4[0], b4[1], b4[2], b4[3]);
      }
    };
    // output layer
    if (wave < 2) mfma_tile_kc(g4, &S.hT[2][32 * wave][0], kPadT, &S.dzT[0][0][0], kPadT, kBwdRows);
    bias(0, kOut, gb[3]);
    back(0, 1, S.w + kBW4, kPadO, 32, zv[2]);
    __syncthreads();
    // third and second hidden layer: dW tile (inputs 32 (wave / 2).., outputs 32 (wave % 2)..)
    mfma_tile_kc(g3, &S.hT[1][32 * (wave >> 1)][0], kPadT, &S.dzT[1][32 * (wave & 1)][0], kPadT, kBwdRows);
    bias(1, kH, gb[2]);
    back(1, 0, S.w + kBW3, kPadH, 64, zv[1]);
    __syncthreads();
    mfma_tile_kc(g2, &S.hT[0][32 * (wave >> 1)][0], kPadT, &S.dzT[0][32 * (wave & 1)][0], kPadT, kBwdRows);
    bias(0, kH, gb[1]);
    back(0, 1, S.w + kBW2, kPadH, 64, zv[0]);
    __syncthreads();
    // first hidden layer: inputs 32 wave .., both halves of the outputs
    mfma_tile_kc2(g1[0], g1[1], &S.xT[32 * wave][0], kPadT, &S.dzT[1][0][0], &S.dzT[1][32][0], kPadT, kBwdRows);
    bias(1, kH, gb[0]);
  }
  float* gp = gpart + (size_t)blockIdx.x * kNTrain;
  auto put = [&](const f32x16& a, int ofs, int i0, int o0, int no) {
#pragma unroll
    for (int r = 0; r < 16; ++r) gp[ofs + (i0 + acc_row(r)) * no + o0 + acc_col()] = a[r];
  };
  put(g1[0], kOffW1, 32 * wave, 0, kH);
  put(g1[1], kOffW1, 32 * wave, 32, kH);
  put(g2, kOffW2, 32 * (wave >> 1), 32 * (wave & 1), kH);
  put(g3, kOffW3, 32 * (wave >> 1), 32 * (wave & 1), kH);
  if (wave < 2) put(g4, kOffW4, 32 * wave, 0, kOut);
  const int offB[4] = {kOffB1, kOffB2, kOffB3, kOffB4};
#pragma unroll
  for (int L = 0; L < 4; ++L) {
    float s = gb[L];
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    if ((tid & 3) == 0 && (tid >> 2) < (L == 3 ? kOut : kH)) gp[offB[L] + (tid >> 2)] = s;
  }
}

// Stores the bf16 copies of weight e (dense index over the four layers): [in][out],
// [out][in], and in the order in which k_correction's waves read them as MFMA
// fragments (lane l of fragment (tile of 32 outputs, step of 16 inputs) holds
// output l % 32, inputs 8 (l / 32) + 0..7).
struct WeightCopies {
  unsigned short *w, *wt, *wf;
};
__device__ __forceinline__ void store_weight(const WeightCopies& W, int e, float value) {
  int off = 0, ni = kIn, no = kH;
  if (e < kIn * kH) { off = 0; ni = kIn; no = kH; }
  else if (e < kIn * kH + kH * kH) { off = kIn * kH; ni = kH; no = kH; }
  else if (e < kIn * kH + 2 * kH * kH) { off = kIn * kH + kH * kH; ni = kH; no = kH; }
  else { off = kIn * kH + 2 * kH * kH; ni = kH; no = kOut; }
  const int loc = e - off, i = loc / no, o = loc % no;
  const unsigned short b = f2bf(value);
  W.w[e] = b;
  W.wt[off + o * ni + i] = b;
  const int frag = (o >> 5) * (ni / 16) + (i >> 4), lane = (o & 31) + 32 * ((i >> 3) & 1);
  W.wf[off + (frag * 64 + lane) * 8 + (i & 7)] = b;
}
// dense weight index of parameter p, or -1 (a bias)
__device__ __forceinline__ int weight_of_param(int p) {
  if (p < kOffB1) return p;
  if (p >= kOffW2 && p < kOffB2) return p - kOffW2 + kIn * kH;
  if (p >= kOffW3 && p < kOffB3) return p - kOffW3 + kIn * kH + kH * kH;
  if (p >= kOffW4 && p < kOffB4) return p - kOffW4 + kIn * kH + 2 * kH * kH;
  return -1;
}

// The gradient from the per-block partials (fixed order: four quarters of the
// blocks, then the quarters), the mean loss, and, with an update, Adam on the
// FP32 master parameters and their bf16 copies.  64 parameters per block of 256.
struct AdamStep {
  int on;
  float lr, b1, b2, eps, c1, c2;
};
__global__ void __launch_bounds__(256) k_grad_update(const float* __restrict__ gpart, int nblk,
                                                     float* __restrict__ grad_out,
                                                     const double* __restrict__ loss_part, int nloss,
                                                     double loss_scale, double* __restrict__ loss, AdamStep ad,
                                                     float* __restrict__ params, float* __restrict__ m,
                                                     float* __restrict__ v, WeightCopies W) {
  __shared__ float part[4][64];
  const int lane = threadIdx.x & 63, quarter = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  const int per = (nblk + 3) / 4, b0 = min(nblk, quarter * per), b1 = min(nblk, b0 + per);
  float s = 0.0f;
  if (p < kNTrain) {
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += gpart[(size_t)b * kNTrain + p];
  }
  part[quarter][lane] = s;
  __syncthreads();
  if (quarter == 0 && p < kNTrain) {
    const float g = part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane];
    if (grad_out) grad_out[p] = g;
    if (ad.on) {
      const float mm = ad.b1 * m[p] + (1.0f - ad.b1) * g;
      const float vv = ad.b2 * v[p] + (1.0f - ad.b2) * g * g;
      m[p] = mm;
      v[p] = vv;
      const float x = params[p] - ad.lr * (mm / ad.c1) / (sqrtf(vv / ad.c2) + ad.eps);
      params[p] = x;
      const int e = weight_of_param(p);
      if (e >= 0) store_weight(W, e, x);
    }
  }
  if (blockIdx.x == 0 && quarter == 1 && loss) {  // one wave adds the loss partials
    double t = 0.0;
    for (int b = lane; b < nloss; b += 64) t += loss_part[b];
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    if (lane == 0) *loss = t * loss_scale;
  }
}

__global__ void k_weights_to_bf16(const float* __restrict__ params, WeightCopies W) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= kNTrain) return;
  const int e = weight_of_param(p);
  if (e >= 0) store_weight(W, e, params[p]);
}

}  // namespace mlp
}  // namespace dplr
