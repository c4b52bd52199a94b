// dkv.hip -- VaSE-DKV scoring on gfx950 (Sec. 3.2 of the paper, with CurDKV's
// product score, Eq. 4).
//
// At every eviction step each head instance draws a Gaussian projection
// G_t in R^{d x r} (entries N(0, 1/r)), independent of earlier steps, and
// scores candidate slot i < K by
//     s_i = ||G_t^T k_i||^2 * ||G_t^T v_i||^2.
// Survivors are then the K - B highest scores (vase_select in deterministic
// mode with N_v = 0), and compaction and decode follow as for VaSE-AttnV.
//
// dkv_projection_kernel draws G_t (rng.hpp; this unit is compiled with
// -ffp-contract=off).  The score streams the K candidate key and value rows
// of each instance once, so it is bound by HBM: for bf16 caches the
// projections run on MFMA (v_mfma_f32_32x32x16_bf16) with G^T as the A
// operand, split into a bf16 head and tail (G ~ G_hi + G_lo to 2^-16) so that
// the bf16 rows meet an almost fp32 projection; the accumulator then holds
// 16 projection coordinates x 1 row per lane and the squared norm is a sum
// inside the lane plus one exchange.  fp32 caches take the fp32 MFMA.
#include "vase_internal.hpp"
#include "vase.h"

#pragma clang fp contract(off)

#include "rng.hpp"

namespace vase {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kDkvBlock = 256;

__global__ __launch_bounds__(kDkvBlock) void dkv_projection_kernel(int n_inst, uint32_t inst_base,
                                                                 int dr, int r, uint32_t k0,
                                                                 uint32_t k1, uint32_t round,
                                                                 float* __restrict__ g) {
  const size_t i = (size_t)blockIdx.x * kDkvBlock + threadIdx.x;
  if (i >= (size_t)n_inst * dr) return;
  const uint32_t inst = (uint32_t)(i / (size_t)dr);
  const uint32_t e = (uint32_t)(i % (size_t)dr);
  const float scale = 1.0f / __builtin_sqrtf((float)r);
  g[i] = dkv_gaussian_entry(e, inst_base + inst, round, k0, k1, scale);
}

// bf16 head and tail of x: x ~ hi + lo with |x - hi - lo| <= 2^-16 |x|.
__device__ __forceinline__ void split_bf16(float x, __bf16& hi, __bf16& lo) {
  hi = (__bf16)x;
  lo = (__bf16)(x - (float)hi);
}

// One block: `tiles` consecutive 32-row tiles of one instance, wave w taking
// tiles w, w + 4, ...  With dlog given, the rows run to N (the buffer included)
// and the block also writes the decode queries' logits dlog[inst][h][row] =
// qdec[inst][h] . k_row (h < G) from the key rows it holds: the G queries are the
// A operand of one more 32x32x16 MFMA chain per tile.  (As spare rows of the
// projection's head operand they would be free, but the tail chain would add
// 0 * k to them, which is not 0 for an infinite k.)
template <int D>
__global__ __launch_bounds__(kDkvBlock) void dkv_score_mfma_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, const float* __restrict__ g,
    int N, int K, int r, int blocks_per_inst, int tiles, float* __restrict__ out,
    const uint16_t* __restrict__ qdec, int G, float* __restrict__ dlog) {
  constexpr int KS = D / 16;
  __shared__ bf16x8_t sa[3][KS][kWave];   // [G^T head, G^T tail, decode queries][step][lane]
  // blocks in dispatch order: what is resident covers one stretch of memory (an
  // eighth of the instances to each XCD: 272 against 263 us)
  const int inst = (int)(blockIdx.x / (unsigned)blocks_per_inst);
  const int rb = (int)(blockIdx.x % (unsigned)blocks_per_inst);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, half = lane / 32;
  // A operands, the same for every wave: G^T (32 projection columns x D, columns
  // >= r zero), head and tail, and the decode queries, staged once per block as
  // per-lane fragments read at each step (in registers they would take 96
  // VGPRs).  The contraction index is permuted identically in both operands:
  // lane half h, step ks holds elements [16*ks + 8*h, +8), so that the two lanes
  // of a row read 32 adjacent bytes in one load.
  const float* gi = g + (size_t)inst * D * r;
  const uint16_t* qi = dlog ? qdec + (size_t)inst * G * D : nullptr;
  const int col = lane % 32;
#pragma unroll
  for (int i = 0; i < (KS * kWave + kDkvBlock - 1) / kDkvBlock; ++i) {
    const int t = (int)threadIdx.x + i * kDkvBlock;
    const int ks = t / kWave, c = t % 32, d0 = 16 * ks + 8 * (t % kWave / 32);
    bf16x8_t fh = {}, fl = {};
    if (c < r) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        __bf16 hi, lo;
        split_bf16(gi[(d0 + e) * r + c], hi, lo);
        fh[e] = hi;
        fl[e] = lo;
      }
    }
    sa[0][ks][t % kWave] = fh;
    sa[1][ks][t % kWave] = fl;
    if (dlog)
      sa[2][ks][t % kWave] = *reinterpret_cast<const bf16x8_t*>(qi + (size_t)min(c, G - 1) * D + d0);
  }
  __syncthreads();
  const int rows = dlog ? N : K;
  const uint16_t* kinst = k + (size_t)inst * N * D;
  const uint16_t* vinst = v + (size_t)inst * N * D;
  float* oinst = out + (size_t)inst * K;
  const int row_base = rb * tiles * 32;
  const int nt = min(tiles, (rows - row_base + 31) / 32);
  // All 2*KS loads of a tile are issued before its first MFMA, a row's pieces
  // one after the other: the four loads of a 128-byte line meet it in L1 (loads
  // that skip L1 take 369 us for 264).  Rows past the last re-read it and are not
  // stored.  12 waves of 16 KB keep 49 MB in flight over the chip, so what is
  // left above the copy rate is how the memory takes this pattern: 1.28 GB (576
  // instances of 4224 rows, with logits) 293 -> 263 us, 4.9 TB/s; 8 instances
  // of 2176 rows, which fill the chip with blocks of 4 tiles, 24.7 -> 8.4 us.
  for (int t = wave; t < nt; t += kDkvBlock / kWave) {
    const int row = row_base + t * 32 + col;
    const int rr = min(row, rows - 1);
    const bf16x8_t* kr = reinterpret_cast<const bf16x8_t*>(kinst + (size_t)rr * D + 8 * half);
    const bf16x8_t* vr = reinterpret_cast<const bf16x8_t*>(vinst + (size_t)rr * D + 8 * half);
    bf16x8_t kb[KS], vb[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kb[ks] = kr[2 * ks];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) vb[ks] = vr[2 * ks];
    __builtin_amdgcn_sched_barrier(0);
    f32x16_t pk = f32x16_t{}, pv = f32x16_t{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8_t ghi = sa[0][ks][lane], glo = sa[1][ks][lane];
      pk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ghi, kb[ks], pk, 0, 0, 0);
      pv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ghi, vb[ks], pv, 0, 0, 0);
      pk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(glo, kb[ks], pk, 0, 0, 0);
      pv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(glo, vb[ks], pv, 0, 0, 0);
    }
    // lane holds projection coordinates 8(e/4) + 4h + e%4 of row `col`
    float lk = 0.f, lv = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      lk = __builtin_fmaf(pk[e], pk[e], lk);
      lv = __builtin_fmaf(pv[e], pv[e], lv);
    }
    lk += __shfl_xor(lk, 32, kWave);
    lv += __shfl_xor(lv, 32, kWave);
    if (half == 0 && row < K) oinst[row] = lk * lv;
    if (dlog) {
      pk = f32x16_t{};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        pk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa[2][ks][lane], kb[ks], pk, 0, 0, 0);
      // lane holds head 8(e/4) + 4h + e%4 of row `col`
      if (row < N) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int h = 8 * (e / 4) + 4 * half + e % 4;
          if (h < G) dlog[((size_t)inst * G + h) * N + row] = pk[e];
        }
      }
    }
  }
}

// fp32 caches: the same tiles with v_mfma_f32_32x32x2_f32, which multiplies and
// accumulates in fp32.  A lane holds 4 of every 8 elements of its row and of its
// projection column, the contraction index permuted alike in both.  A tile takes
// 2 x D/2 MFMAs of 64 cycles (3.4 us at d = 128 on one SIMD) against 32 KB from
// memory, so both are near their rates.  One thread per row, which went over the
// row once per projection column, took 6581 us for 288 instances of 4096 rows
// at r = 20 (1.21 GB); this takes 228 (5.3 TB/s); 8 instances of 2048 rows 141 -> 9.4 us.
template <int D>
__global__ __launch_bounds__(kDkvBlock, 2) void dkv_score_f32_kernel(
    const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ g, int N,
    int K, int r, int blocks_per_inst, int tiles, float* __restrict__ out) {
  constexpr int P = D / 8;
  __shared__ f32x4_t sa[P][kWave];        // G^T, columns >= r zero
  const int inst = (int)(blockIdx.x / (unsigned)blocks_per_inst);
  const int rb = (int)(blockIdx.x % (unsigned)blocks_per_inst);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, half = lane / 32;
  const int col = lane % 32;
  const float* gi = g + (size_t)inst * D * r;
#pragma unroll
  for (int i = wave; i < P; i += kDkvBlock / kWave) {
    f32x4_t x = {0.f, 0.f, 0.f, 0.f};
    if (col < r) {
#pragma unroll
      for (int c = 0; c < 4; ++c) x[c] = gi[(8 * i + 4 * half + c) * r + col];
    }
    sa[i][lane] = x;
  }
  __syncthreads();
  const float* kinst = k + (size_t)inst * N * D;
  const float* vinst = v + (size_t)inst * N * D;
  float* oinst = out + (size_t)inst * K;
  const int row_base = rb * tiles * 32;
  const int nt = min(tiles, (K - row_base + 31) / 32);
  for (int t = wave; t < nt; t += kDkvBlock / kWave) {
    const int row = row_base + t * 32 + col;
    const size_t at = (size_t)min(row, K - 1) * D + 4 * half;   // rows past the last re-read it
    const f32x4_t* kr = reinterpret_cast<const f32x4_t*>(kinst + at);
    const f32x4_t* vr = reinterpret_cast<const f32x4_t*>(vinst + at);
    f32x4_t kb[P], vb[P];
#pragma unroll
    for (int i = 0; i < P; ++i) kb[i] = kr[2 * i];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < P; ++i) vb[i] = vr[2 * i];
    __builtin_amdgcn_sched_barrier(0);
    f32x16_t pk = f32x16_t{}, pv = f32x16_t{};
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const f32x4_t a = sa[i][lane];
#pragma unroll
      for (int c = 0; c < 4; ++c) pk = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c], kb[i][c], pk, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const f32x4_t a = sa[i][lane];
#pragma unroll
      for (int c = 0; c < 4; ++c) pv = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c], vb[i][c], pv, 0, 0, 0);
    }
    // lane holds projection coordinates 8(e/4) + 4h + e%4 of row `col`; the
    // padding ones are left out (0 times an infinite element is no 0)
    float lk = 0.f, lv = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const bool proj = 8 * (e / 4) + 4 * half + e % 4 < r;
      lk = proj ? __builtin_fmaf(pk[e], pk[e], lk) : lk;
      lv = proj ? __builtin_fmaf(pv[e], pv[e], lv) : lv;
    }
    lk += __shfl_xor(lk, 32, kWave);
    lv += __shfl_xor(lv, 32, kWave);
    if (half == 0 && row < K) oinst[row] = lk * lv;
  }
}

}  // namespace

hipError_t launch_dkv_projection(int n_inst, uint32_t inst_base, int d, int r, uint64_t seed,
                                 uint32_t round, float* g, hipStream_t stream) {
  const size_t total = (size_t)n_inst * d * r;
  const unsigned grid = (unsigned)((total + kDkvBlock - 1) / kDkvBlock);
  hipLaunchKernelGGL(dkv_projection_kernel, dim3(grid), dim3(kDkvBlock), 0, stream, n_inst,
                     inst_base, d * r, r, (uint32_t)seed, (uint32_t)(seed >> 32), round, g);
  return hipGetLastError();
}

hipError_t launch_dkv_score(const void* k, const void* v, const float* g, int dtype, int n_inst,
                            int K, int B, int d, int r, float* out, const void* q_dec, int G,
                            float* dec_logits, hipStream_t stream) {
  const int N = K + B;
  // Blocks evenly split, so that none is a remainder, down to one tile a wave.
  // bf16: up to 384 instances as many as fill the 768 places (three blocks to a
  // CU) and not a few more, which would run a round by themselves (159 instances
  // of 3035 rows: 5 blocks each 47.7 us, 4 44.5; 51 of 6787: 16 37.3, 15 30.5);
  // beyond, two.  Where such blocks are longer than 32 tiles the call runs for many
  // times a block anyway, and blocks of 8 tiles even out its end (200 instances of
  // 5049 rows: 4 long blocks each 137 us, 19 118; 477 of 5607: 291 and 270).
  // fp32, whose blocks stage twice the G: 23 of 6083 rows took 518 us for 373
  // instances, 5 465; but from 512 instances on two rounds of them (797 of 715 rows,
  // d = 64: one each 70 us, two 64).
  const int nt = ((dec_logits ? N : K) + 31) / 32;
  int want;
  if (dtype == VASE_BF16) {
    want = n_inst <= 384 ? 768 / n_inst : (768 + n_inst - 1) / n_inst;
    if (nt > 32 * want) want = nt / 8;
  } else {
    const int places = n_inst < 512 ? 768 : 1536;
    want = (places + n_inst - 1) / n_inst;
    want = want > nt / 32 ? want : nt / 32;
  }
  want = want < nt / 4 ? want : nt / 4;
  const int tiles = want > 1 ? (nt + want - 1) / want : nt;
  const int bpi = (nt + tiles - 1) / tiles;
  const unsigned grid = (unsigned)(n_inst * bpi);
  if (dtype == VASE_BF16) {
    const uint16_t* qd = static_cast<const uint16_t*>(q_dec);
    auto kernel = d == 128 ? dkv_score_mfma_kernel<128> : dkv_score_mfma_kernel<64>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kDkvBlock), 0, stream,
                       static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v), g, N, K, r,
                       bpi, tiles, out, qd, G, dec_logits);
  } else {
    auto kernel = d == 128 ? dkv_score_f32_kernel<128> : dkv_score_f32_kernel<64>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kDkvBlock), 0, stream, static_cast<const float*>(k),
                       static_cast<const float*>(v), g, N, K, r, bpi, tiles, out);
  }
  return hipGetLastError();
}

}  // namespace vase
