// ffs_surrogate: gfx950 kernels of the learned offspring pre-screen (the
// DeepSets surrogate declared in include/ffs_surrogate.h).
//
// Mapping onto CDNA4
//   * The only chromosome-dependent input is a job's rank, which takes n
//     values, so layers 1 and 2 run once per (job, rank) pair: a Q = n^2 row
//     table. Its products with W2 (forward) and the two backward products run
//     on the matrix cores: v_mfma_f32_32x32x16_bf16, 64 x 64 output tiles per
//     256-thread workgroup (2 x 2 waves of 32 x 32), K staged through LDS in
//     slices of 32. Layer-1 activations and the layer-2 output gradient are
//     built in the loaders straight into LDS as bf16, never stored.
//   * A batch's forward is a gather of table rows per chromosome; its
//     backward aggregates the output gradient per table row (the gradient of
//     every row of a chromosome is the same vector w3 * dy / n, masked), so
//     dW2 and dH1 are products over the Q table rows, not over batch x n.
//   * No float atomics: every sum runs in a fixed order (per-lane sequential,
//     fixed lane trees, per-block partials reduced in block order), so each
//     call repeats bit for bit.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>

#include "ffs_surrogate.h"

namespace {

constexpr int H = FFS_SG_HIDDEN;
constexpr int kW1 = 0;                  // [4][H]
constexpr int kB1 = 4 * H;              // [H]
constexpr int kW2 = 5 * H;              // [H][H]
constexpr int kB2 = 5 * H + H * H;      // [H]
constexpr int kW3 = 6 * H + H * H;      // [H]
constexpr int kB3 = 7 * H + H * H;      // [1]
static_assert(kB3 + 1 == FFS_SG_PARAMS, "parameter layout");

constexpr int BM = 64, BN = 64, BK = 32, LDK = BK + 8;  // LDS row stride in bf16 elements
constexpr int kChunk = 256;                               // table rows per dW2 partial
constexpr int kRowChunk = 32;                             // table rows per db2 partial
constexpr int kBatchChunk = 64;                           // chromosomes per head partial
constexpr int kDChunk = 256;                              // chromosomes per D partial
constexpr int kHeaderBytes = 256;  // head of the training workspace: status word first, as ffs_status reads it

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef u32x4 u32x4_any __attribute__((aligned(2)));  // in a caller's bf16 array

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// float32 -> bfloat16, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ uint32_t bf16_bits(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ u32x4 pack8(const float *v) {
  u32x4 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) r[j] = bf16_bits(v[2 * j]) | (bf16_bits(v[2 * j + 1]) << 16);
  return r;
}

// Layer 1 before the ReLU of a unit: c_k + rank * W1[0], float32.
__device__ __forceinline__ float layer1(float c, float rank, float w) {
  return __fadd_rn(c, __fmul_rn(rank, w));
}

__device__ __forceinline__ float rank_of(int v, int n) { return __fdiv_rn((float)v, (float)n); }

// Layer-2 output gradient of a table row (before its bf16 rounding) at a unit, from the
// row's activation there, its D and the unit's w3.
__device__ __forceinline__ float out_grad(float h2, float d, float w3, float fn) {
  return h2 > 0.f ? __fdiv_rn(__fmul_rn(d, w3), fn) : 0.f;
}

struct TileLds {
  uint16_t a[BM * LDK];
  uint16_t b[BN * LDK];
};

// acc (this wave's 32 x 32 part of a 64 x 64 tile) += A[64 x K] B[K x 64]. Each thread
// fills one 8-wide slice of A (row r, from column k on) and of B (column r, from row k
// on) per K slice: la(r, k) and lb(r, k) load what a slice needs into registers, and
// fa and fb make the 8 bf16 values of it. Few blocks share a compute unit here (160 on
// 256 for 50 jobs), so the loads of a slice are issued before the slice before it is
// multiplied: what bounds a slice is the loaders' arithmetic, not their latency.
template <class LA, class LB, class FA, class FB>
__device__ __forceinline__ void mma_tile(int k_total, LA la, LB lb, FA fa, FB fb, TileLds &s,
                                         f32x16 &acc) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, wm = w >> 1, wn = w & 1;
  const int r = t >> 2, kc = (t & 3) * 8;
  const int arow = (wm * 32 + (lane & 31)) * LDK, brow = (wn * 32 + (lane & 31)) * LDK;
  const int koff = 8 * (lane >> 5);
  auto ra = la(r, kc);
  auto rb = lb(r, kc);
  for (int k0 = 0; k0 < k_total; k0 += BK) {
    *(u32x4 *)&s.a[r * LDK + kc] = fa(ra);
    *(u32x4 *)&s.b[r * LDK + kc] = fb(rb);
    const int kn = min(k0 + BK, k_total - BK) + kc;
    ra = la(r, kn);
    rb = lb(r, kn);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      const u32x4 av = *(const u32x4 *)&s.a[arow + kk + koff];
      const u32x4 bv = *(const u32x4 *)&s.b[brow + kk + koff];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                    __builtin_bit_cast(bf16x8, bv), acc, 0, 0, 0);
    }
    __syncthreads();
  }
}

struct F8 {
  float v[8];
};
__device__ __forceinline__ F8 load8(const float *p) {
  F8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.v[j] = p[j];
  return r;
}

// Tile coordinates of accumulator element e of this lane.
__device__ __forceinline__ int acc_row(int e) {
  const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) >> 1;
  return wm * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
}
__device__ __forceinline__ int acc_col() {
  const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) & 1;
  return wn * 32 + (lane & 31);
}

// ---------------------------------------------------------------------------
// Features, layer-1 constants, bf16 copies.
// ---------------------------------------------------------------------------
// One block. The least processing times of a job's unfrozen stages are added in LDS, a
// thread each (whole numbers: any order gives the same sum), so that the loads of all
// stages are in flight at once: 14.7 -> 7.4 us for 200 jobs of 10 stages.
__global__ __launch_bounds__(1024) void features_kernel(ffs_instance in, float *feats) {
  __shared__ unsigned long long sum[FFS_SG_MAX_GENES];
  __shared__ int32_t smax;
  const int n = in.n_active, g = in.n_stages, om = in.o_max;
  for (int k = threadIdx.x; k < n; k += blockDim.x) sum[k] = 0;
  if (threadIdx.x == 0) smax = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < n * g; i += blockDim.x) {
    const int k = i / g, s = i % g, j = in.active[k];
    if (s < in.first_stage[j]) continue;
    const int32_t *row = in.proc + ((size_t)j * g + s) * om;
    const int nm = in.n_machines[s];
    int32_t best = row[0];
#pragma unroll 4
    for (int m = 1; m < nm; ++m) best = row[m] < best ? row[m] : best;
    atomicAdd(&sum[k], (unsigned long long)(int64_t)best);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < n; k += blockDim.x) atomicMax(&smax, (int32_t)sum[k]);
  __syncthreads();
  const float scale = (float)(smax > 1 ? smax : 1);
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    const int j = in.active[k];
    const int64_t tot = (int64_t)sum[k];
    const int64_t ready = in.ready[j];
    const int64_t start = ready > in.rs ? ready : in.rs;
    const int64_t slack = (int64_t)in.due[j] - start - tot;
    const int64_t rel = ready - in.rs > 0 ? ready - in.rs : 0;
    feats[4 * k + 0] = __fdiv_rn((float)tot, scale);
    feats[4 * k + 1] = __fdiv_rn((float)slack, scale);
    feats[4 * k + 2] = __fdiv_rn((float)rel, scale);
    feats[4 * k + 3] = 0.f;
  }
}

// c_k = ((b1 + f0 W1[1]) + f1 W1[2]) + f2 W1[3], float32 in this order.
// status: null, or the status word of a training step, cleared.
__global__ __launch_bounds__(256) void ctab_kernel(const float *theta, const float *feats, int n,
                                                   float *ctab, int32_t *status) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0 && status) status[0] = 0;
  if (i >= n * H) return;
  const int k = i / H, h = i % H;
  float c = __fadd_rn(theta[kB1 + h], __fmul_rn(feats[4 * k + 0], theta[kW1 + H + h]));
  c = __fadd_rn(c, __fmul_rn(feats[4 * k + 1], theta[kW1 + 2 * H + h]));
  c = __fadd_rn(c, __fmul_rn(feats[4 * k + 2], theta[kW1 + 3 * H + h]));
  ctab[i] = c;
}

__global__ __launch_bounds__(256) void refresh_kernel(const float *theta, uint16_t *w2b,
                                                      uint16_t *w2tb) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= H * H) return;
  const uint16_t b = (uint16_t)bf16_bits(theta[kW2 + i]);
  w2b[i] = b;
  w2tb[(i % H) * H + i / H] = b;
}

// ---------------------------------------------------------------------------
// Table forward: a2 = h1 . bf16(W2) + b2 for the Q = n^2 (job, rank) rows.
// SCORE: per-row dot products with w3 (4 column-block partials per row).
// TRAIN: h2 = max(a2, 0) stored, float32 [Q][H].
// Block (x, y) of ceil(Q / 64) x H / 64, 256 threads.
// ---------------------------------------------------------------------------
template <bool TRAIN>
__device__ void table_fwd(int x, int y, const float *theta, const float *ctab, const uint16_t *w2tb,
                          int n, float *h2_out, float *r_part) {
  __shared__ __align__(16) TileLds s;
  __shared__ float red[2][2][32];
  const int Q = n * n, m0 = x * BM, n0 = y * BN;
  // this thread's row of A (a row past the table: the last one, its products unused)
  const int qa = min(m0 + (int)(threadIdx.x >> 2), Q - 1);
  const float *ca = ctab + (size_t)(qa / n) * H;
  const float rank = rank_of(qa % n + 1, n);
  struct A {
    F8 c, w;
  };
  auto la = [&](int, int k) { return A{load8(ca + k), load8(theta + kW1 + k)}; };
  auto fa = [&](const A &a) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = fmaxf(layer1(a.c.v[j], rank, a.w.v[j]), 0.f);
    return pack8(v);
  };
  auto lb = [&](int c, int k) {  // B[h][o] = W2[h][o], from the transpose
    return (u32x4) * (const u32x4_any *)(w2tb + (size_t)(n0 + c) * H + k);
  };
  auto fb = [&](u32x4 b) { return b; };
  f32x16 acc = {};
  mma_tile(H, la, lb, fa, fb, s, acc);
  const int col = n0 + acc_col();
  const float b2 = theta[kB2 + col], w3 = theta[kW3 + col];
  const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) >> 1, wn = (threadIdx.x >> 6) & 1;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int q = m0 + acc_row(e);
    const float h2 = fmaxf(__fadd_rn(acc[e], b2), 0.f);
    if (TRAIN) {
      if (q < Q) h2_out[(size_t)q * H + col] = h2;
    } else {
      float p = __fmul_rn(w3, h2);
      // sum over the 32 columns of this wave (lanes with the same lane >> 5)
      for (int off = 1; off < 32; off <<= 1) p += __shfl_xor(p, off);
      if ((lane & 31) == 0) red[wm][wn][8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)] = p;
    }
  }
  if (!TRAIN) {
    __syncthreads();
    const int t = threadIdx.x;
    if (t < BM) {
      const int q = m0 + t;
      if (q < Q) r_part[(size_t)y * Q + q] = red[t >> 5][0][t & 31] + red[t >> 5][1][t & 31];
    }
  }
}

__global__ __launch_bounds__(256) void table_fwd_kernel(const float *theta, const float *ctab,
                                                        const uint16_t *w2tb, int n, float *r_part) {
  table_fwd<false>(blockIdx.x, blockIdx.y, theta, ctab, w2tb, n, nullptr, r_part);
}

__global__ __launch_bounds__(256) void table_sum_kernel(const float *r_part, int Q, float *table) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Q) return;
  float s = r_part[q];
  for (int b = 1; b < H / BN; ++b) s += r_part[(size_t)b * Q + q];
  table[q] = s;
}

// ---------------------------------------------------------------------------
// A training step. Seven launches, each of all work that can run together: the
// layer-1 constants; the table forward and the input check; the batch forward; the
// partials of D and of the head; D; the three backward products; the sums of their
// partials and Adam. A step of 4096 chromosomes of 50 jobs is bound by the latency of
// its launches and of sums read one part after the other, not by its 20 MB or its
// 2 GFLOP, so every such loop has several parts in flight, in the old order.
//
// Measured: 220 -> 77 us (17 launches and 2 copies before, bits the same).
// ---------------------------------------------------------------------------
// Input check: every gene in 1..n and every target finite, else bit 0 of the status
// word; the later kernels of the step then do nothing. Block c of ceil(B n / kCheck).
constexpr int kCheck = 4096;
__device__ void validate(int c, const int32_t *prio, const float *target, int n, int B,
                         int32_t *status) {
  const size_t total = (size_t)B * n, i0 = (size_t)c * kCheck + threadIdx.x;
  bool bad = false;
#pragma unroll
  for (int j = 0; j < kCheck / 256; ++j) {
    const size_t i = i0 + 256 * j;
    const int v = i < total ? prio[i] : 1;
    bad |= v < 1 || v > n;
    if (i < (size_t)B) bad |= !(fabsf(target[i]) <= 3.0e38f);  // NaN or infinite (B <= B n)
  }
  if (bad) atomicOr(status, 1);
}

__global__ __launch_bounds__(1) void clear_status_kernel(int32_t *status) { status[0] = 0; }

// grid: blocks x H / 64 tiles of the table, then the blocks of the check.
__global__ __launch_bounds__(256) void train_fwd_kernel(const float *theta, const float *ctab,
                                                        const uint16_t *w2tb, int n, int blocks,
                                                        float *h2, const int32_t *prio,
                                                        const float *target, int B,
                                                        int32_t *status) {
  const int tiles = blocks * (H / BN), i = blockIdx.x;
  if (i < tiles) table_fwd<true>(i % blocks, i / blocks, theta, ctab, w2tb, n, h2, nullptr);
  else validate(i - tiles, prio, target, n, B, status);
}

// ---------------------------------------------------------------------------
// Training targets: ln obj standardised within each group of `group`
// consecutive chromosomes (one population), mean and population standard
// deviation in float64; a constant group gets 0. One block per group: thread t < 256
// sums its run of consecutive entries [g0 + t*c, g0 + (t+1)*c) in index order,
// c = ceil(group / 256), and the 256 partial sums are added by a fixed pairwise tree,
// so every run gives the same bits. The logarithms, the larger part of the work, are
// taken once each by all 1024 threads and kept in LDS where the group fits (`logs`, the
// 64 KB that a kernel's own arrays may take less the sums; two blocks of 1024 threads
// fill a compute unit anyway); a larger group takes them again in each of the three
// passes. 4096 entries: 20.7 -> 10.5 us; with its launches, 7456: 31.7 -> 16.1.
// ---------------------------------------------------------------------------
constexpr int kTargetThreads = 1024, kTargetSums = 256;
constexpr int kTargetLogs = (65536 - kTargetSums * 8) / 8 / 17 * 16;  // 7456, one in 17 left out
__device__ __forceinline__ double block_sum_fixed(double v, double *buf) {
  const int t = threadIdx.x;
  if (t < kTargetSums) buf[t] = v;
  __syncthreads();
  for (int w = kTargetSums / 2; w >= 1; w >>= 1) {
    if (t < w) buf[t] += buf[t + w];
    __syncthreads();
  }
  const double out = buf[0];
  __syncthreads();
  return out;
}

__global__ __launch_bounds__(kTargetThreads) void targets_kernel(const int64_t *obj, int count,
                                                                 int group, float *target,
                                                                 int32_t *status) {
  // (an entry left out after 16: the runs of a full group would all start in one bank)
  __shared__ double buf[kTargetSums], logs[kTargetLogs + kTargetLogs / 16];
  auto place = [](int x) { return x + (x >> 4); };
  const int g0 = blockIdx.x * group;
  const int g1 = g0 + group < count ? g0 + group : count;
  const bool kept = g1 - g0 <= kTargetLogs;
  auto log_of = [&](int i) { return log((double)(obj[i] > 0 ? obj[i] : 1)); };
  bool bad = false;
  for (int i = g0 + threadIdx.x; i < g1; i += kTargetThreads) {
    bad |= obj[i] <= 0;
    if (kept) logs[place(i - g0)] = log_of(i);
  }
  if (bad) atomicOr(status, 1);
  __syncthreads();
  auto value = [&](int i) { return kept ? logs[place(i - g0)] : log_of(i); };
  const int c = (g1 - g0 + kTargetSums - 1) / kTargetSums;
  const bool sums = threadIdx.x < kTargetSums;
  const int a = sums ? min(g0 + (int)threadIdx.x * c, g1) : g1, b = min(a + c, g1);
  double s = 0.0;
#pragma unroll 4
  for (int i = a; i < b; ++i) s += value(i);
  const double mean = block_sum_fixed(s, buf) / (double)(g1 - g0);
  double v = 0.0;
#pragma unroll 4
  for (int i = a; i < b; ++i) {
    const double d = value(i) - mean;
    v += d * d;
  }
  const double sd = sqrt(block_sum_fixed(v, buf) / (double)(g1 - g0));
  for (int i = g0 + threadIdx.x; i < g1; i += kTargetThreads) {
    const double d = value(i) - mean;
    target[i] = sd > 0.0 ? (float)(d / sd) : 0.f;
  }
}

// ---------------------------------------------------------------------------
// Batch forward (pool order): z_b = (sum over k of h2[k][prio_bk]) / n,
// y_b = b3 + z_b . w3, dy_b = 2 (y_b - t_b) / B.
// One wave per chromosome, 4 units per lane.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void batch_fwd_kernel(const float *theta, const float *h2,
                                                       const int32_t *prio, const float *target,
                                                       int n, int B, float *z, float *dy,
                                                       float *sq, const int32_t *status) {
  if (status[0]) return;
  const int b = blockIdx.x, lane = threadIdx.x;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int genes = prio[(size_t)b * n + min(k0 + lane, n - 1)], m = min(n - k0, 64);
#pragma unroll 8
    for (int k = 0; k < m; ++k) {
      const int q = (k0 + k) * n + __builtin_amdgcn_readlane(genes, k) - 1;
      const float *row = h2 + (size_t)q * H;
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] += row[lane + 64 * j];
    }
  }
  float part = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float zv = __fdiv_rn(acc[j], (float)n);
    z[(size_t)b * H + lane + 64 * j] = zv;
    part += __fmul_rn(theta[kW3 + lane + 64 * j], zv);
  }
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
  part = __shfl(part, 0);
  if (lane == 0) {
    const float y = __fadd_rn(theta[kB3], part);
    const float t = target[b];
    const float d = __fsub_rn(y, t);
    dy[b] = __fdiv_rn(__fmul_rn(2.f, d), (float)B);
    sq[b] = __fmul_rn(d, d);
  }
}

// Partials of D[k][v-1] = sum of dy_b over the chromosomes whose gene k is v:
// block (k, c) sums chromosomes [c * kDChunk, (c + 1) * kDChunk) in b order into
// part[c][k * n + v - 1]; the chunks are then added in chunk order.
struct DtableLds {
  int32_t vals[kDChunk];
  float dys[kDChunk];
};
__device__ void dtable(int k, int c, const int32_t *prio, const float *dy, int n, int B, float *part,
                       DtableLds &s) {
  const int b0 = c * kDChunk, nb = B - b0 < kDChunk ? B - b0 : kDChunk;
  for (int i = threadIdx.x; i < kDChunk; i += blockDim.x) {
    s.vals[i] = i < nb ? prio[(size_t)(b0 + i) * n + k] : 0;  // 0: no gene
    s.dys[i] = i < nb ? dy[b0 + i] : 0.f;
  }
  __syncthreads();
  for (int v = threadIdx.x + 1; v <= n; v += blockDim.x) {
    float d = 0.f;
#pragma unroll 16
    for (int i = 0; i < kDChunk; ++i) d += s.vals[i] == v ? s.dys[i] : 0.f;
    part[(size_t)c * n * n + k * n + v - 1] = d;
  }
}

// Partials of dw3, db3 and the loss over chromosomes [c * kBatchChunk, ...),
// b in order: part[c][0..H) = dw3, part[c][H] = db3, part[c][H + 1] = sum of squares.
__device__ void head(int c, const float *dy, const float *z, const float *sq, int B, float *part) {
  const int o = threadIdx.x;
  const int b0 = c * kBatchChunk, b1 = b0 + kBatchChunk < B ? b0 + kBatchChunk : B;
  float s = 0.f;
#pragma unroll 16
  for (int b = b0; b < b1; ++b) s += __fmul_rn(dy[b], z[(size_t)b * H + o]);
  float *out = part + (size_t)c * (H + 2);
  out[o] = s;
  if (o < 2) {  // thread 0: db3, thread 1: the loss
    const float *src = o ? sq : dy;
    float d = 0.f;
#pragma unroll 16
    for (int b = b0; b < b1; ++b) d += src[b];
    out[H + o] = d;
  }
}

// grid: n x dchunks blocks of D's partials, then the head's chunks.
__global__ __launch_bounds__(256) void parts_kernel(const int32_t *prio, const float *dy,
                                                    const float *z, const float *sq, int n, int B,
                                                    int dchunks, float *dpart, float *hpart,
                                                    const int32_t *status) {
  if (status[0]) return;
  __shared__ DtableLds s;
  const int i = blockIdx.x;
  if (i < n * dchunks) dtable(i % n, i / n, prio, dy, n, B, dpart, s);
  else head(i - n * dchunks, dy, z, sq, B, hpart);
}

// db2 partials: part[c][o] = sum of the layer-2 output gradient over rows of chunk c.
__device__ void db2_part(int c, const float *theta, const float *h2, const float *D, int n,
                         float *part) {
  const int Q = n * n, o = threadIdx.x;
  const int q1 = (c + 1) * kRowChunk < Q ? (c + 1) * kRowChunk : Q;
  const float w3 = theta[kW3 + o], fn = (float)n;
  float s = 0.f;
#pragma unroll 8
  for (int q = c * kRowChunk; q < q1; ++q) s += out_grad(h2[(size_t)q * H + o], D[q], w3, fn);
  part[(size_t)c * H + o] = s;
}

// dH1 = bf16(G) . bf16(W2)^T over the table rows, masked by a1 > 0, reduced
// straight into per-block partials of dW1 (4 rows) and db1:
// part[blockIdx.x][f][h], f = 0 rank, 1..3 features, 4 bias.
// Block (x, y) of ceil(Q / 64) x H / 64, 256 threads.
struct H1Lds {
  TileLds tile;
  float red[2][5][64];
};
__device__ void bwd_h1(int x, int y, const float *theta, const float *ctab, const float *feats,
                       const float *h2, const float *D, const uint16_t *w2b, int n, float *part,
                       H1Lds &s) {
  const int Q = n * n, m0 = x * BM, n0 = y * BN;
  const float fn = (float)n;
  // this thread's row of A (a row past the table: the last one, with a gradient of 0)
  const int ra = m0 + (int)(threadIdx.x >> 2), qa = min(ra, Q - 1);
  const float da = ra < Q ? D[qa] : 0.f;
  struct A {
    F8 h, w;
  };
  auto la = [&](int, int k) {  // A[q][o] = G[q][o]
    return A{load8(h2 + (size_t)qa * H + k), load8(theta + kW3 + k)};
  };
  auto fa = [&](const A &a) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = out_grad(a.h.v[j], da, a.w.v[j], fn);
    return pack8(v);
  };
  auto lb = [&](int c, int k) {  // B[o][h] = W2[h][o]
    return (u32x4) * (const u32x4_any *)(w2b + (size_t)(n0 + c) * H + k);
  };
  auto fb = [&](u32x4 b) { return b; };
  f32x16 acc = {};
  mma_tile(H, la, lb, fa, fb, s.tile, acc);
  const int h = n0 + acc_col();
  const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) >> 1;
  const float w1 = theta[kW1 + h];
  float p[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int q = m0 + acc_row(e);
    if (q >= Q) continue;
    const int kj = q / n;
    const float rank = rank_of(q % n + 1, n);
    const float d = layer1(ctab[kj * H + h], rank, w1) > 0.f ? acc[e] : 0.f;
    p[0] += __fmul_rn(rank, d);
    p[1] += __fmul_rn(feats[4 * kj + 0], d);
    p[2] += __fmul_rn(feats[4 * kj + 1], d);
    p[3] += __fmul_rn(feats[4 * kj + 2], d);
    p[4] += d;
  }
#pragma unroll
  for (int f = 0; f < 5; ++f) p[f] += __shfl_xor(p[f], 32);   // the two row halves of the wave
  if (lane < 32)
    for (int f = 0; f < 5; ++f) s.red[wm][f][acc_col()] = p[f];
  __syncthreads();
  const int t = threadIdx.x;
  for (int i = t; i < 5 * BN; i += blockDim.x) {
    const int f = i / BN, c = i % BN;
    part[((size_t)x * 5 + f) * H + n0 + c] = s.red[0][f][c] + s.red[1][f][c];
  }
}

// dW2 partials over one chunk of table rows: part[chunk][h][o] = sum over q of
// bf16(h1[q][h]) bf16(G[q][o]). Block (x, y, z) of H / 64 x H / 64 x chunks, 256
// threads. The chunk's ranks, jobs and D are laid out in LDS first: a division each.
struct W2Lds {
  TileLds tile;
  float rank[kChunk], d[kChunk];
  int32_t job[kChunk];
};
static_assert(kChunk == 256, "one thread per row of a chunk");
__device__ void bwd_w2(int x, int y, int z, const float *theta, const float *ctab, const float *h2,
                       const float *D, int n, float *part, W2Lds &s) {
  const int Q = n * n, m0 = x * BM, n0 = y * BN, qb = z * kChunk;
  const float fn = (float)n;
  {
    const int q = min(qb + (int)threadIdx.x, Q - 1);  // (a row past the table is not used)
    s.rank[threadIdx.x] = rank_of(q % n + 1, n);
    s.job[threadIdx.x] = q / n;
    s.d[threadIdx.x] = D[q];
  }
  __syncthreads();
  const int ht = m0 + (int)(threadIdx.x >> 2), ot = n0 + (int)(threadIdx.x >> 2);
  const float w1 = theta[kW1 + ht], w3 = theta[kW3 + ot];
  struct R {
    F8 v;
    int k;
  };
  auto la = [&](int, int k) {  // A[h][q] = h1[q][h]
    R r;
    r.k = k;
#pragma unroll
    for (int j = 0; j < 8; ++j) r.v.v[j] = ctab[s.job[k + j] * H + ht];
    return r;
  };
  auto fa = [&](const R &r) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = qb + r.k + j < Q ? fmaxf(layer1(r.v.v[j], s.rank[r.k + j], w1), 0.f) : 0.f;
    return pack8(v);
  };
  auto lb = [&](int, int k) {  // B[q][o] = G[q][o]
    R r;
    r.k = k;
#pragma unroll
    for (int j = 0; j < 8; ++j) r.v.v[j] = h2[(size_t)min(qb + k + j, Q - 1) * H + ot];
    return r;
  };
  auto fb = [&](const R &r) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = qb + r.k + j < Q ? out_grad(r.v.v[j], s.d[r.k + j], w3, fn) : 0.f;
    return pack8(v);
  };
  f32x16 acc = {};
  mma_tile(kChunk, la, lb, fa, fb, s.tile, acc);
  const int col = n0 + acc_col();
#pragma unroll
  for (int e = 0; e < 16; ++e)
    part[((size_t)z * H + m0 + acc_row(e)) * H + col] = acc[e];
}

// The backward products in one launch, the longest blocks first: chunks x 16 of dW2,
// blocks x 4 of dH1, rchunks of db2.
__global__ __launch_bounds__(256) void bwd_kernel(const float *theta, const float *ctab,
                                                  const float *feats, const float *h2,
                                                  const float *D, const uint16_t *w2b, int n,
                                                  int chunks, int blocks, float *part_w2,
                                                  float *part1, float *part_b2,
                                                  const int32_t *status) {
  if (status[0]) return;
  __shared__ union {
    W2Lds w2;
    H1Lds h1;
  } s;
  constexpr int nt = H / BM;
  int i = blockIdx.x;
  if (i < nt * nt * chunks) {
    bwd_w2(i % nt, i / nt % nt, i / (nt * nt), theta, ctab, h2, D, n, part_w2, s.w2);
    return;
  }
  i -= nt * nt * chunks;
  if (i < blocks * nt) bwd_h1(i % blocks, i / blocks, theta, ctab, feats, h2, D, w2b, n, part1, s.h1);
  else db2_part(i - blocks * nt, theta, h2, D, n, part_b2);
}

// The sum over p < n_parts of src[p * stride], p in order.
__device__ __forceinline__ float sum_parts(const float *src, int n_parts, size_t stride) {
  float s = src[0];
#pragma unroll 16
  for (int p = 1; p < n_parts; ++p) s += src[(size_t)p * stride];
  return s;
}

// D from the partials of its chunks.
__global__ __launch_bounds__(256) void dsum_kernel(const float *part, int n_parts, int Q, float *D,
                                                   const int32_t *status) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Q || status[0]) return;
  D[q] = sum_parts(part + q, n_parts, Q);
}

// Every gradient from its partials, in their order, then Adam. grad, loss: null, or
// where the step's gradients and loss (mean of squares) go.
struct GradParts {
  const float *w1, *w2, *b2, *head;  // [blocks][5][H], [chunks][H][H], [rchunks][H], [hchunks][H + 2]
  int blocks, chunks, rchunks, hchunks, B;
};
__global__ __launch_bounds__(256) void adam_kernel(GradParts P, float *theta, float *m, float *v,
                                                   float *grad, float *loss, float lr, float c1,
                                                   float c2, uint16_t *w2b, uint16_t *w2tb,
                                                   const int32_t *status) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i > FFS_SG_PARAMS || status[0]) return;
  // the partials hold dW1 and db1 together, as the parameters do; the head's dw3, db3
  // and then the loss, which is no parameter
  static_assert(kB1 == 4 * H && kB3 == kW3 + H && kB3 + 1 == FFS_SG_PARAMS, "partials' order");
  const float g = i < kW2   ? sum_parts(P.w1 + i, P.blocks, 5 * H)
                  : i < kB2 ? sum_parts(P.w2 + (i - kW2), P.chunks, (size_t)H * H)
                  : i < kW3 ? sum_parts(P.b2 + (i - kB2), P.rchunks, H)
                            : sum_parts(P.head + (i - kW3), P.hchunks, H + 2);
  if (i == FFS_SG_PARAMS) {
    if (loss) loss[0] = __fdiv_rn(g, (float)P.B);
    return;
  }
  if (grad) grad[i] = g;
  const float mi = 0.9f * m[i] + 0.1f * g;
  const float vi = 0.999f * v[i] + 0.001f * g * g;
  m[i] = mi;
  v[i] = vi;
  const float th = theta[i] - lr * (mi * c1) / (sqrtf(vi * c2) + 1e-8f);
  theta[i] = th;
  if (i >= kW2 && i < kW2 + H * H) {
    const int w = i - kW2;
    const uint16_t b = (uint16_t)bf16_bits(th);
    w2b[w] = b;
    w2tb[(w % H) * H + w / H] = b;
  }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
int grid1(int count) { return (count + 255) / 256; }

struct TableWs {
  float *ctab, *r_part;
  size_t total;
};

TableWs table_ws(void *ws, int n) {
  uint8_t *b = (uint8_t *)ws;
  TableWs L{};
  size_t off = 0;
  L.ctab = (float *)(b + off);
  off += align_up((size_t)n * H * 4, 256);
  L.r_part = (float *)(b + off);
  off += align_up((size_t)(H / BN) * n * n * 4, 256);
  L.total = off;
  return L;
}

struct TrainWs {
  int32_t *status;
  float *ctab, *h2, *D, *Dpart, *z, *dy, *sq, *head, *part1, *part_b2, *part_w2;
  size_t total;
};

TrainWs train_ws(void *ws, int n, int B) {
  uint8_t *b = (uint8_t *)ws;
  TrainWs L{};
  const size_t Q = (size_t)n * n, chunks = (Q + kChunk - 1) / kChunk, blocks = (Q + BM - 1) / BM;
  const size_t rchunks = (Q + kRowChunk - 1) / kRowChunk, dchunks = (B + kDChunk - 1) / kDChunk;
  const size_t hchunks = (B + kBatchChunk - 1) / kBatchChunk;
  size_t off = kHeaderBytes;
  L.status = (int32_t *)b;
  auto take = [&](size_t floats) {
    float *p = (float *)(b + off);
    off += align_up(floats * 4, 256);
    return p;
  };
  L.ctab = take((size_t)n * H);
  L.h2 = take(Q * H);
  L.D = take(Q);
  L.Dpart = take(dchunks * Q);
  L.z = take((size_t)B * H);
  L.dy = take(B);
  L.sq = take(B);
  L.head = take(hchunks * (H + 2));
  L.part1 = take(blocks * 5 * H);
  L.part_b2 = take(rchunks * H);
  L.part_w2 = take(chunks * H * H);
  L.total = off;
  return L;
}

bool ok(hipError_t e) { return e == hipSuccess; }

}  // namespace

extern "C" {

int sg_refresh(ffs_surrogate *m, void *stream) {
  if (!m || !m->theta || !m->w2_bf16 || !m->w2t_bf16) return FFS_E_INVAL;
  hipLaunchKernelGGL(refresh_kernel, dim3(grid1(H * H)), dim3(256), 0, (hipStream_t)stream,
                     (const float *)m->theta, m->w2_bf16, m->w2t_bf16);
  return ok(hipGetLastError()) ? FFS_OK : FFS_E_DEVICE;
}

int sg_features(const ffs_instance *inst, float *feats, void *workspace, size_t workspace_bytes,
                void *stream) {
  (void)workspace;
  (void)workspace_bytes;
  if (!inst || !feats || inst->n_active < 1 || inst->n_active > FFS_SG_MAX_GENES ||
      inst->n_stages < 1 || inst->o_max < 1 || !inst->active || !inst->proc ||
      !inst->n_machines || !inst->first_stage || !inst->ready || !inst->due)
    return FFS_E_INVAL;
  hipLaunchKernelGGL(features_kernel, dim3(1), dim3(1024), 0, (hipStream_t)stream, *inst, feats);
  return ok(hipGetLastError()) ? FFS_OK : FFS_E_DEVICE;
}

size_t sg_table_workspace_size(int32_t n_genes) {
  if (n_genes < 1 || n_genes > FFS_SG_MAX_GENES) return 0;
  return table_ws(nullptr, n_genes).total;
}

int sg_score_table(const ffs_surrogate *m, const float *feats, int32_t n, float *table,
                   void *workspace, size_t workspace_bytes, void *stream) {
  if (!m || !m->theta || !m->w2t_bf16 || !feats || !table || n < 1 || n > FFS_SG_MAX_GENES)
    return FFS_E_INVAL;
  const TableWs L = table_ws(workspace, n);
  if (!workspace || workspace_bytes < L.total) return FFS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const int Q = n * n;
  hipLaunchKernelGGL(ctab_kernel, dim3(grid1(n * H)), dim3(256), 0, s, (const float *)m->theta,
                     feats, n, L.ctab, (int32_t *)nullptr);
  hipLaunchKernelGGL(table_fwd_kernel, dim3((Q + BM - 1) / BM, H / BN), dim3(256), 0, s,
                     (const float *)m->theta, (const float *)L.ctab,
                     (const uint16_t *)m->w2t_bf16, n, L.r_part);
  hipLaunchKernelGGL(table_sum_kernel, dim3(grid1(Q)), dim3(256), 0, s, (const float *)L.r_part,
                     Q, table);
  return ok(hipGetLastError()) ? FFS_OK : FFS_E_DEVICE;
}

size_t sg_train_workspace_size(int32_t n_genes, int32_t batch) {
  if (n_genes < 1 || n_genes > FFS_SG_MAX_GENES || batch < 1 || batch > FFS_SG_MAX_BATCH) return 0;
  return train_ws(nullptr, n_genes, batch).total;
}

int sg_targets(const int64_t *obj, int32_t count, int32_t group, float *target, void *workspace,
               size_t workspace_bytes, void *stream) {
  if (!obj || !target || count < 0 || group < 1) return FFS_E_INVAL;
  if (!workspace || workspace_bytes < (size_t)kHeaderBytes) return FFS_E_WORKSPACE;
  if (count == 0) return FFS_OK;
  hipStream_t s = (hipStream_t)stream;
  int32_t *status = (int32_t *)workspace;
  hipLaunchKernelGGL(clear_status_kernel, dim3(1), dim3(1), 0, s, status);
  hipLaunchKernelGGL(targets_kernel, dim3((count + group - 1) / group), dim3(kTargetThreads), 0, s, obj,
                     count, group, target, status);
  return ok(hipGetLastError()) ? FFS_OK : FFS_E_DEVICE;
}

int sg_train_step(ffs_surrogate *m, const float *feats, int32_t n, const int32_t *prio,
                  const float *target, int32_t B, float lr, float *loss, float *grad,
                  void *workspace, size_t workspace_bytes, void *stream) {
  if (!m || !m->theta || !m->adam_m || !m->adam_v || !m->w2_bf16 || !m->w2t_bf16 || !feats ||
      !prio || !target || n < 1 || n > FFS_SG_MAX_GENES || B < 1 || B > FFS_SG_MAX_BATCH ||
      !(lr > 0.f) || m->step < 0)
    return FFS_E_INVAL;
  const TrainWs L = train_ws(workspace, n, B);
  if (!workspace || workspace_bytes < L.total) return FFS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const int Q = n * n, chunks = (Q + kChunk - 1) / kChunk, blocks = (Q + BM - 1) / BM;
  const int rchunks = (Q + kRowChunk - 1) / kRowChunk, dchunks = (B + kDChunk - 1) / kDChunk;
  const int hchunks = (B + kBatchChunk - 1) / kBatchChunk;
  const float *th = m->theta;
  const int32_t *st = L.status;
  const int checks = (int)(((size_t)B * n + kCheck - 1) / kCheck);
  hipLaunchKernelGGL(ctab_kernel, dim3(grid1(n * H)), dim3(256), 0, s, th, feats, n, L.ctab,
                     L.status);
  hipLaunchKernelGGL(train_fwd_kernel, dim3(blocks * (H / BN) + checks), dim3(256), 0, s, th,
                     (const float *)L.ctab, (const uint16_t *)m->w2t_bf16, n, blocks, L.h2, prio,
                     target, B, L.status);
  hipLaunchKernelGGL(batch_fwd_kernel, dim3(B), dim3(64), 0, s, th, (const float *)L.h2, prio,
                     target, n, B, L.z, L.dy, L.sq, st);
  hipLaunchKernelGGL(parts_kernel, dim3(n * dchunks + hchunks), dim3(256), 0, s, prio,
                     (const float *)L.dy, (const float *)L.z, (const float *)L.sq, n, B, dchunks,
                     L.Dpart, L.head, st);
  hipLaunchKernelGGL(dsum_kernel, dim3(grid1(Q)), dim3(256), 0, s, (const float *)L.Dpart, dchunks,
                     Q, L.D, st);
  hipLaunchKernelGGL(bwd_kernel, dim3(chunks * (H / BM) * (H / BN) + blocks * (H / BN) + rchunks),
                     dim3(256), 0, s, th, (const float *)L.ctab, feats, (const float *)L.h2,
                     (const float *)L.D, (const uint16_t *)m->w2_bf16, n, chunks, blocks, L.part_w2,
                     L.part1, L.part_b2, st);
  const int t = m->step + 1;
  const float c1 = (float)(1.0 / (1.0 - std::pow(0.9, t)));
  const float c2 = (float)(1.0 / (1.0 - std::pow(0.999, t)));
  const GradParts P{L.part1, L.part_w2, L.part_b2, L.head, blocks, chunks, rchunks, hchunks, B};
  hipLaunchKernelGGL(adam_kernel, dim3(grid1(FFS_SG_PARAMS + 1)), dim3(256), 0, s, P, m->theta,
                     m->adam_m, m->adam_v, grad, loss, lr, c1, c2, m->w2_bf16, m->w2t_bf16, st);
  if (!ok(hipGetLastError())) return FFS_E_DEVICE;
  m->step = t;
  return FFS_OK;
}

}  // extern "C"
