// score_f32.hip -- the window score of fp32 caches on gfx950 (the definition and
// the two passes are score.hip's; this file is its fp32 arithmetic).
//
// The products q_r . k_t come from v_mfma_f32_32x32x2_f32, which multiplies and
// accumulates in fp32: 256 flop per CU and clock, twice the scalar fma rate, so
// a 32-row x 32-key tile takes D/2 MFMAs of 64 cycles (1.9 us at d = 128) and
// its 1024 exponentials and every load hide behind it.  What bounds a call is
// therefore the number of tiles a SIMD gets, and at small sizes the launches.
//
//   pass 1  a wave keeps one 32-row tile of the window in registers and streams
//           a run of 32-key tiles past it (the next tile's rows are loaded
//           during the MFMAs of the current one; keys are shared by the waves
//           of a block through L1), with a running maximum and sum per lane;
//           it writes (max, sum) of its rows over its run.
//   pass 2  a wave keeps one 32-key tile and streams the window's row tiles past
//           it; the rows' normalisers are merged from pass 1's runs by each
//           block into LDS first.  Column sums need no exchange between waves.
//
// Neither pass stages operands in LDS: a tile is 16 KB against 4096 cycles of
// MFMA, 16 bytes per clock and CU.  The V rows' scores are further blocks of
// pass 1, so they cost no launch and their memory time overlaps with MFMA work.
// Against one thread per row with LDS operands and scalar fma (two LDS reads
// per product, 160-key runs of one wave each), 24 instances of 96 window rows
// and 1092 slots at d = 128 went from 371 to 32 us.
#include "vase_internal.hpp"
#include "vase.h"

namespace vase {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kFBlock = 256;
constexpr int kFWaves = kFBlock / kWave;
constexpr int kTile = 32;
constexpr int kGroupRows = 1024;      // window rows whose normalisers pass 2 holds in LDS
constexpr int kValueIters = 8;        // value blocks: row groups per block
constexpr float kFloor = -3.0e38f;    // finite stand-in for an empty maximum
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// 32 rows of D floats as an MFMA operand: lane l holds row l % 32, and of every
// 8 elements the 4 of its half.  Both operands permute the contraction index
// alike, so each lane loads 16 bytes at a time.
template <int D>
struct Frag {
  static constexpr int P = D / 8;
  f32x4_t p[P];
  // this lane's pieces of row row0 + l % 32; past n_rows, of row n_rows - 1
  __device__ __forceinline__ static const f32x4_t* at(const float* rows, int row0, int n_rows,
                                                      int lane) {
    const int row = min(row0 + lane % 32, n_rows - 1);
    return reinterpret_cast<const f32x4_t*>(rows + (size_t)row * D) + lane / 32;
  }
  // the same of window rows (at most 2^16), as one 32-bit lane offset from a
  // uniform base: three registers less than an address
  __device__ __forceinline__ static const f32x4_t* at_window(const float* rows, int row0, int n_rows,
                                                             int lane) {
    const uint32_t row = (uint32_t)min(row0 + lane % 32, n_rows - 1);
    return reinterpret_cast<const f32x4_t*>(reinterpret_cast<const char*>(rows) +
                                            (row * (uint32_t)(D * 4) + (uint32_t)(lane / 32) * 16u));
  }
  __device__ __forceinline__ void load(const f32x4_t* r) {
#pragma unroll
    for (int i = 0; i < P; ++i) p[i] = r[2 * i];
  }
};

// The product of a resident and a streamed tile, with the streamed one's pieces
// replaced by the next tile's (at `next`) as they are used, so that a load has
// the rest of this tile's MFMAs to arrive and takes no registers of its own.
// ROWS: the streamed tile holds the rows (else the keys).  Element e of lane l
// is row 8(e/4) + 4(l/32) + e%4, key l%32.
//
// d = 128 sums in two chains.  One chain of 64 MFMAs rounds the products more
// often than the scalar kernel did, and in calls too short to gain from the
// softmax sums' shorter chains the scores came out up to 15 % further from 64 bits
// (37 instances of 1059 slots with lse_win, mean of 6 inputs: scalar 3.45e-7, one
// chain 3.98e-7, two 3.69e-7; 14 drawn calls: two take 0.94 to 1.02 of the time).
// At d = 64 one chain stays within a tenth of the scalar kernel's error (the most in
// the smallest calls, where two do not change it: 16 instances of 160 slots, mean of
// 60 inputs, 1.51e-7, 1.64e-7, 1.64e-7), and the 16 additions would cost 3 to 5 %
// of the shorter tile's time.
template <int D, bool ROWS>
__device__ __forceinline__ f32x16_t tile_product(const Frag<D>& fixed, Frag<D>& moving,
                                                 const f32x4_t* next) {
  constexpr int kChains = D == 128 ? 2 : 1;
  f32x16_t acc[kChains] = {};
#pragma unroll
  for (int i = 0; i < Frag<D>::P; ++i) {
    f32x16_t& a = acc[i % kChains];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      a = __builtin_amdgcn_mfma_f32_32x32x2f32(ROWS ? moving.p[i][c] : fixed.p[i][c],
                                               ROWS ? fixed.p[i][c] : moving.p[i][c], a, 0, 0, 0);
    moving.p[i] = next[2 * i];
    __builtin_amdgcn_sched_barrier(0);   // keep the load here, not ahead of the MFMAs
  }
  if constexpr (kChains == 1) return acc[0];
  const f32x16_t sum = acc[0] + acc[kChains - 1];
  __builtin_amdgcn_sched_barrier(0);     // 16 registers are free before the epilogue takes its own
  return sum;
}

__device__ __forceinline__ int tile_row(int e, int half) { return 8 * (e / 4) + 4 * half + e % 4; }

// Value scores of the candidate rows of one block (kinds Range, L2 and Var).
template <int D>
__device__ __forceinline__ void value_block(const float* v, int blk, int blocks_per_inst, int N, int K,
                                            int kind, float* out, uint32_t* status) {
  constexpr int LPR = D / 4;
  constexpr int RPI = kFBlock / LPR;
  const int inst = blk / blocks_per_inst;
  const int row0 = (blk % blocks_per_inst) * RPI * kValueIters + (int)threadIdx.x / LPR;
  const int seg = (int)threadIdx.x % LPR;
  const uint4* vb = reinterpret_cast<const uint4*>(v + (size_t)inst * N * D);
  bool bad = false;
  // half of the loads in flight at a time, in a rolled loop: unrolled in full,
  // the three kinds make 30 KB of code
#pragma unroll 1
  for (int i0 = 0; i0 < kValueIters; i0 += kValueIters / 2) {
    uint4 w[kValueIters / 2];
#pragma unroll
    for (int i = 0; i < kValueIters / 2; ++i)
      w[i] = vb[(size_t)min(row0 + (i0 + i) * RPI, K - 1) * LPR + seg];
#pragma unroll
    for (int i = 0; i < kValueIters / 2; ++i) {
      const int row = row0 + (i0 + i) * RPI;
      float f[4];
      Vec16<float>::unpack(w[i], f);
      const float val = row_value_score<4, LPR>(f, kind);
      if (row < K && seg == 0) out[(size_t)inst * K + row] = val;
      if (status) bad |= row < K && any_nonfinite<4>(f);
    }
  }
  if (status) block_status(status, bad, VASE_STATUS_VALUE_ROW);
}

// part[inst][run][row] = (max, sum of exp2(x - max)) over the keys of the run,
// x = s * c.  The first key is key_base; blocks past n_score score value rows.
template <int D>
__global__ __launch_bounds__(kFBlock, 2) void score_f32_rows_kernel(
    const float* __restrict__ k, const float* __restrict__ q, const float* __restrict__ v, int N,
    int K, int R, int n_inst, int n_rt, int n_run, int run_tiles, int key_base, float c,
    float2* __restrict__ part, unsigned n_score, int value_blocks, int value_kind,
    float* __restrict__ vrange, uint32_t* __restrict__ status) {
  __shared__ float s_m[kFWaves][kTile][kTile + 1], s_l[kFWaves][kTile][kTile + 1];
  if (blockIdx.x >= n_score) {
    value_block<D>(v, (int)(blockIdx.x - n_score), value_blocks, N, K, value_kind, vrange, status);
    return;
  }
  const int lane = threadIdx.x % kWave, half = lane / 32, j = lane % 32;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t task = xcd_logical_block(blockIdx.x, n_score) * kFWaves + wave;
  const int rt = (int)(task % (uint32_t)n_rt);
  const uint32_t t1 = task / (uint32_t)n_rt;
  const int run = (int)(t1 % (uint32_t)n_run);
  const int inst = (int)(t1 / (uint32_t)n_run);
  if (inst >= n_inst) return;
  const float* ki = k + (size_t)inst * N * D;
  const int key_lo = key_base + run * run_tiles * kTile;
  const int key_hi = min(N, key_lo + run_tiles * kTile);
  Frag<D> a, b;
  b.load(Frag<D>::at(ki, key_lo, N, lane));
  a.load(Frag<D>::at(q + (size_t)inst * R * D, rt * kTile, R, lane));
  float m[16], l[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    m[e] = kFloor;
    l[e] = 0.f;
  }
  for (int key0 = key_lo; key0 < key_hi; key0 += kTile) {
    // the last tile fetches itself again
    const int next = key0 + kTile < key_hi ? key0 + kTile : key0;
    const f32x16_t acc = tile_product<D, false>(a, b, Frag<D>::at(ki, next, N, lane));
    const bool ok = key0 + j < key_hi;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float x = ok ? acc[e] * c : -INFINITY;
      const float mn = fmaxf(m[e], x);
      l[e] = l[e] * fast_exp2(m[e] - mn) + fast_exp2(x - mn);
      m[e] = mn;
    }
  }
  // over the 32 keys of each row: through LDS, two lanes a row, in rolled loops.
  // A small call runs this code once per launch, from a cold instruction cache:
  // unrolled as lane exchanges it was 10 KB and 10 us of a one-tile launch.
  float(&sm)[kTile][kTile + 1] = s_m[wave];
  float(&sl)[kTile][kTile + 1] = s_l[wave];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    sm[tile_row(e, half)][j] = m[e];
    sl[tile_row(e, half)][j] = l[e];
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  float mr = kFloor, lr = 0.f;
#pragma unroll 4
  for (int i = 0; i < kTile / 2; ++i) mr = fmaxf(mr, sm[j][half * (kTile / 2) + i]);
  mr = fmaxf(mr, __shfl_xor(mr, 32, kWave));
#pragma unroll 4
  for (int i = 0; i < kTile / 2; ++i) {
    const int t = half * (kTile / 2) + i;
    lr += sl[j][t] * fast_exp2(sm[j][t] - mr);
  }
  lr += __shfl_xor(lr, 32, kWave);
  const int row = rt * kTile + j;
  if (half == 0 && row < R) part[((size_t)inst * n_run + run) * R + row] = make_float2(mr, lr);
}

// col[inst][slab][key] = sum over the slab's rows of exp2(s * c - lse2_r), with
// lse2_r merged from the runs (and lse_win's persistent part, when given).  168
// registers at d = 128 are the last that leave a SIMD three waves (two: 933
// instances of 311 slots and 12 rows 76 -> 81 us).
template <int D>
__global__ __launch_bounds__(kFBlock, D == 128 ? 3 : 2) void score_f32_cols_kernel(
    const float* __restrict__ k, const float* __restrict__ q, const float2* __restrict__ part,
    const float* __restrict__ lse_win, int N, int K, int R, int n_run, int n_slab, int slab_tiles,
    int n_kg, float c, float* __restrict__ col, uint32_t* __restrict__ status) {
  __shared__ float lse[kGroupRows];
  const int lane = threadIdx.x % kWave, half = lane / 32, j = lane % 32;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int kg = (int)(lb % (uint32_t)n_kg);
  const uint32_t t1 = lb / (uint32_t)n_kg;
  const int slab = (int)(t1 % (uint32_t)n_slab);
  const int inst = (int)(t1 / (uint32_t)n_slab);
  const int key0 = (kg * kFWaves + wave) * kTile;
  const bool active = key0 < K;
  const int row_lo = slab * slab_tiles * kTile;
  const int row_hi = min(R, row_lo + slab_tiles * kTile);
  const float* qi = q + (size_t)inst * R * D;
  Frag<D> a, b;
  if (active) {
    b.load(Frag<D>::at(k + (size_t)inst * N * D, key0, N, lane));
    a.load(Frag<D>::at_window(qi, row_lo, R, lane));
  }
  bool row_bad = false;
  float sum = 0.f;
  for (int g0 = row_lo; g0 < row_hi; g0 += kGroupRows) {
    const int g1 = min(row_hi, g0 + kGroupRows);
    if (g0 != row_lo) __syncthreads();
    // whole tiles: rows past the window's end get +inf, which gives p = 0
    for (int r = g0 + threadIdx.x; r < g0 + (g1 - g0 + kTile - 1) / kTile * kTile; r += kFBlock) {
      float l2 = INFINITY;
      if (r < g1) {
        const float2* p = part + (size_t)inst * n_run * R + r;
        float mm = kFloor, ll = 0.f;
        for (int i = 0; i < n_run; ++i) mm = fmaxf(mm, p[(size_t)i * R].x);
        for (int i = 0; i < n_run; ++i) {
          const float2 x = p[(size_t)i * R];
          ll += x.y * fast_exp2(x.x - mm);
        }
        l2 = mm + fast_log2(ll);
        if (lse_win) {
          const float w = lse_win[(size_t)inst * R + r] * kLog2e;
          const float m = fmaxf(l2, w);
          l2 = m + fast_log2(fast_exp2(l2 - m) + fast_exp2(w - m));
        }
        row_bad |= !(l2 > -INFINITY && l2 < INFINITY);
      }
      lse[r - g0] = l2;
    }
    __syncthreads();
    if (!active) continue;
    for (int r0 = g0; r0 < g1; r0 += kTile) {
      const int next = r0 + kTile < row_hi ? r0 + kTile : r0;
      const f32x16_t acc = tile_product<D, true>(b, a, Frag<D>::at_window(qi, next, R, lane));
      float s[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 z = *reinterpret_cast<const float4*>(&lse[r0 - g0 + 8 * i + 4 * half]);
        s[i] = (fast_exp2(__builtin_fmaf(acc[4 * i], c, -z.x)) +
                fast_exp2(__builtin_fmaf(acc[4 * i + 1], c, -z.y))) +
               (fast_exp2(__builtin_fmaf(acc[4 * i + 2], c, -z.z)) +
                fast_exp2(__builtin_fmaf(acc[4 * i + 3], c, -z.w)));
      }
      sum += (s[0] + s[1]) + (s[2] + s[3]);
    }
  }
  sum += __shfl_xor(sum, 32, kWave);
  int key = key0;
  asm volatile("" : "+s"(key));          // formed here, not kept from the loads on
  if (active && half == 0 && key + j < K)
    col[((size_t)inst * n_slab + slab) * K + key + j] = sum;
  // every key group merges the same normalisers: one of them reports
  if (status && kg == 0) block_status(status, row_bad, VASE_STATUS_ROW_NORM);
}

template <int D>
hipError_t launch_d(const float* k, const float* v, const float* q, int n_inst, int N, int K, int R,
                    float c, int kind, const float* lse_win, const ScorePlan& pl, float2* part,
                    float* col, float* vrange, hipStream_t stream, uint32_t* status) {
  const int n_rt = (R + kTile - 1) / kTile;
  // row statistics over all N slots, or over the buffer only when lse_win is given
  const int key_base = lse_win ? K : 0;
  const int tiles = (N - key_base + kTile - 1) / kTile;
  const int n_run = lse_win ? (tiles < pl.n_chunk1 ? tiles : pl.n_chunk1) : pl.n_chunk1;
  const int run_tiles = (tiles + n_run - 1) / n_run;
  const int runs = (tiles + run_tiles - 1) / run_tiles;
  const unsigned n_score =
      (unsigned)(((long long)n_inst * runs * n_rt + kFWaves - 1) / kFWaves);
  constexpr int kValueRows = kFBlock / (D / 4) * kValueIters;
  const int vb = kind <= VASE_VALUE_VAR ? (K + kValueRows - 1) / kValueRows : 0;
  hipLaunchKernelGGL((score_f32_rows_kernel<D>), dim3(n_score + (unsigned)(vb * n_inst)),
                     dim3(kFBlock), 0, stream, k, q, v, N, K, R, n_inst, n_rt, runs, run_tiles,
                     key_base, c, part, n_score, vb, kind, vrange, status);
  const int n_kg = (K + kTile * kFWaves - 1) / (kTile * kFWaves);
  hipLaunchKernelGGL((score_f32_cols_kernel<D>), dim3((unsigned)(n_inst * pl.n_slab * n_kg)),
                     dim3(kFBlock), 0, stream, k, q, part, lse_win, N, K, R, runs, pl.n_slab,
                     pl.rows_per_slab / kTile, n_kg, c, col, status);
  return hipGetLastError();
}

}  // namespace

// Runs per instance of pass 1 and row slabs of pass 2.  A SIMD works through its
// waves' tiles one after the other, so a pass takes about
// ceil(waves / 1024 SIMDs) x (tiles per wave + the wave's own operand load and
// reduction, about half a tile).  A run costs every pass-2 block one more
// partial to merge (R x 8 bytes, about a twentieth of a tile at R = 256).  Up to
// 24 runs and 8 slabs: with 64 and 16, calls of up to 8192 candidates take 0.86 to
// 1.08 of the time (one instance of 8320 slots: 8 rows 44 -> 38 us, 128 rows 50 ->
// 45; one of 2176 and 512 rows 34 -> 37); a single much longer instance would
// gain (50128 slots and 32 rows: 173 -> 93 us; one thread per row took 839).
// `part_bytes`: room for the partials, of which what the runs leave takes the
// column sums of further slabs.
void score_f32_split(int n_inst, int N, int K, int R, size_t part_bytes, ScorePlan& pl) {
  constexpr long long kSimds = 1024;
  constexpr int kMaxRuns = 24, kMaxSlabs = 8;
  auto cost = [](long long waves, int tiles) {
    return (double)((waves + kSimds - 1) / kSimds) * (tiles + 0.5);
  };
  const int n_rt = (R + kTile - 1) / kTile, n_kt = (N + kTile - 1) / kTile;
  double best = 0;
  for (int runs = 1; runs <= kMaxRuns && runs <= n_kt; ++runs) {
    const int tiles = (n_kt + runs - 1) / runs;
    const double t = cost((long long)n_inst * n_rt * runs, tiles) + 0.05 * runs;
    if (runs == 1 || t < best) {
      best = t;
      pl.n_chunk1 = (n_kt + tiles - 1) / tiles;
    }
  }
  pl.off_part = 0;
  pl.off_col = ((size_t)n_inst * pl.n_chunk1 * R * sizeof(float2) + 255) & ~(size_t)255;
  const size_t spare = part_bytes - pl.off_col;
  const long long kt2 = (long long)n_inst * ((K + kTile - 1) / kTile);
  for (int slabs = 1; slabs <= kMaxSlabs && slabs <= n_rt; ++slabs) {
    const int tiles = (n_rt + slabs - 1) / slabs;
    const int n = (n_rt + tiles - 1) / tiles;
    if ((size_t)n_inst * (n - 1) * K * sizeof(float) > spare) break;
    const double t = cost(kt2 * n, tiles);
    if (slabs == 1 || t < best) {
      best = t;
      pl.n_slab = n;
      pl.rows_per_slab = tiles * kTile;
    }
  }
}

hipError_t launch_score_f32(const void* k, const void* v, const void* q, int n_inst, int N, int K,
                            int R, int d, float c, int kind, const float* lse_win,
                            const ScorePlan& pl, char* ws, float* vrange, hipStream_t stream,
                            uint32_t* status) {
  float2* part = reinterpret_cast<float2*>(ws + pl.off_part);
  float* col = reinterpret_cast<float*>(ws + pl.off_col);
  const float *kk = static_cast<const float*>(k), *vv = static_cast<const float*>(v),
              *qq = static_cast<const float*>(q);
  return d == 128 ? launch_d<128>(kk, vv, qq, n_inst, N, K, R, c, kind, lse_win, pl, part, col, vrange,
                                  stream, status)
                  : launch_d<64>(kk, vv, qq, n_inst, N, K, R, c, kind, lse_win, pl, part, col, vrange,
                                 stream, status);
}

}  // namespace vase
