// compact.hip -- in-place stable compaction of the K survivors (gfx950).
//
// After selection, the cache keeps K of its N = K + B slots.  The survivor map
// src is strictly increasing with src[j] >= j, so every row moves towards lower
// slots by at most B.  The destination range [0, K) of an instance is cut into
// parts of T rows, one workgroup each:
//
//   * rows that part p reads but part p+1 overwrites (the source range
//     [(p+1)T, src[(p+1)T - 1]], at most B rows) are first copied to a staging
//     workspace by a separate kernel, so parts never race with each other;
//   * inside a part, chunks of rows are processed in ascending order, and each
//     chunk's loads complete (s_waitcnt + barrier) before any of its stores:
//     later chunks only read rows at or above their own destination, which no
//     earlier store touches.
//
// Rows in the unmoved prefix (src[j] == j) are skipped; src[j] - j is
// non-decreasing, so compact_move_kernel finds that prefix by binary search.
#include "vase_internal.hpp"
#include "vase.h"

namespace vase {
namespace {

constexpr int kCompBlock = 256;

// first j in [lo, hi) with src[j] != j, or hi
__device__ __forceinline__ int first_moved(const int32_t* s, int lo, int hi) {
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (s[mid] > mid) hi = mid; else lo = mid + 1;
  }
  return lo;
}

__device__ __forceinline__ int clamp_slot(int s, int N) { return s < 0 ? 0 : (s >= N ? N - 1 : s); }

__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

// Stage the rows [(p+1)T, src[(p+1)T-1]] of part p (p < n_part-1) into ws.
// ws layout: [inst][n_part-1][2][B][row_u4] uint4.
template <int ROW_U4>
__global__ __launch_bounds__(kCompBlock) void compact_stage_kernel(
    const uint4* __restrict__ k, const uint4* __restrict__ v, const int32_t* __restrict__ src,
    int K, int B, int T, int n_part, uint4* __restrict__ ws) {
  const int p = blockIdx.x, inst = blockIdx.y;
  const int N = K + B;
  const int32_t* s = src + (size_t)inst * K;
  const int lo = (p + 1) * T;
  const int last = clamp_slot(s[min((p + 1) * T, K) - 1], N);
  const int cnt = min(last - lo + 1, B);
  if (cnt <= 0) return;
  const uint4* kb = k + (size_t)inst * N * ROW_U4;
  const uint4* vb = v + (size_t)inst * N * ROW_U4;
  uint4* wk = ws + (((size_t)inst * (n_part - 1) + p) * 2 + 0) * (size_t)B * ROW_U4;
  uint4* wv = ws + (((size_t)inst * (n_part - 1) + p) * 2 + 1) * (size_t)B * ROW_U4;
  for (int e = threadIdx.x; e < cnt * ROW_U4; e += kCompBlock) {
    const size_t off = (size_t)lo * ROW_U4 + e;
    wk[e] = kb[off];
    wv[e] = vb[off];
  }
}

template <int ROW_U4, int CHUNK>
__global__ __launch_bounds__(kCompBlock) void compact_move_kernel(
    uint4* __restrict__ k, uint4* __restrict__ v, const int32_t* __restrict__ src, int K, int B,
    int T, int n_part, const uint4* __restrict__ ws) {
  constexpr int kRowsPerPass = kCompBlock / ROW_U4;   // rows covered by one block-wide load
  constexpr int kPasses = CHUNK / kRowsPerPass;
  static_assert(CHUNK % kRowsPerPass == 0, "chunk must be a multiple of rows per pass");
  __shared__ int s_start;
  const int p = blockIdx.x, inst = blockIdx.y;
  const int N = K + B;
  const int32_t* s = src + (size_t)inst * K;
  const int j_lo = p * T;
  const int j_hi = min(K, (p + 1) * T);
  const int stage_lo = (p + 1) * T;     // rows >= stage_lo come from the staging area
  if (threadIdx.x == 0) s_start = first_moved(s, j_lo, j_hi);
  __syncthreads();
  const int start = s_start;
  uint4* kb = k + (size_t)inst * N * ROW_U4;
  uint4* vb = v + (size_t)inst * N * ROW_U4;
  const uint4* wk = nullptr;
  const uint4* wv = nullptr;
  if (p + 1 < n_part) {
    wk = ws + (((size_t)inst * (n_part - 1) + p) * 2 + 0) * (size_t)B * ROW_U4;
    wv = ws + (((size_t)inst * (n_part - 1) + p) * 2 + 1) * (size_t)B * ROW_U4;
  }
  const int col = threadIdx.x % ROW_U4;
  const int row0 = threadIdx.x / ROW_U4;
  for (int c0 = start; c0 < j_hi; c0 += CHUNK) {
    uint4 rk[kPasses], rv[kPasses];
#pragma unroll
    for (int u = 0; u < kPasses; ++u) {
      // rows past the part's end load a valid row and are not stored
      const int j = min(c0 + row0 + u * kRowsPerPass, j_hi - 1);
      const int sj = clamp_slot(s[j], N);
      const bool staged = wk != nullptr && sj >= stage_lo;
      const size_t off = staged ? (size_t)min(sj - stage_lo, B - 1) * ROW_U4 + col
                                : (size_t)sj * ROW_U4 + col;
      rk[u] = (staged ? wk : kb)[off];
      rv[u] = (staged ? wv : vb)[off];
    }
    wait_vmem();
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPasses; ++u) {
      const int j = c0 + row0 + u * kRowsPerPass;
      if (j < j_hi) {
        const size_t off = (size_t)j * ROW_U4 + col;
        kb[off] = rk[u];
        vb[off] = rv[u];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Compaction fused with one decode-attention step (Eq. 1) over the compacted
// cache: a workgroup takes one part [p T, (p+1) T) of an instance's destination
// rows, reads every survivor row of it exactly once (rows in place are read but
// not written), stores the rows that move, and accumulates the G query heads'
// online softmax over the rows it holds in registers, so that the decode and
// the value scores cost no further pass over the cache.  With one part per
// instance it writes the outputs itself; else the partials (m, l, o) of the
// parts go to the decode's combine, and rows from the next part's range are
// read from their staged copies, as in compact_move_kernel.
//
// Bound by HBM: 2 rows read and up to 2 written per slot.  Rows go in chunks, in
// ascending order.  A chunk's stores wait until every thread's loads of that
// chunk have completed (vmcnt, then a barrier): a row may be read and
// overwritten within one chunk.  The loads of the next two chunks are in flight
// meanwhile: they read rows src[j] >= j at or above the next chunk's first row,
// which no store of this or an earlier chunk touches.  The survivor map sits in
// LDS (kMapRows of it at a time), so no load waits for an index; the three
// register stages rotate by name, since a stage that is copied to another one
// has to have arrived first.  That holds within a turn of the three-chunk loop:
// at its head, where the exits from its middle join, the compiler waits for
// everything (vmcnt(0)), so two steps of three overlap with the loads ahead and
// the pipeline drains, stores included, once in every three chunks.
//
// Against staging, moving, scoring and decoding in launches of their own, which
// went over the cache three times, a call repeated on the same buffers (d = 128,
// G = 4, B = 128, with value scores): 64 bf16 instances of 4096 rows (268 MB to
// move) 129 -> 59 us, 576 934 -> 560, 512 fp32 instances 1555 -> 882.  Kernel
// times of the 64: staging 7, this kernel 48, combine 4.  From 1024 bf16
// instances on, which were one part each before too, 2304 take 1953 us either way.
// ---------------------------------------------------------------------------
constexpr int kMapRows = 4096;

// PARTS: several parts per instance.  One part reads no staged row, and choosing
// between cache and staging per row costs short instances 2 to 3 % (285 rows,
// G = 6, fp32: 32.3 us for 31.4).
template <typename T, int D, int G, bool CARRY, bool PARTS>
__global__ __launch_bounds__(kCompBlock) void compact_decode_kernel(
    uint4* k, uint4* v, const int32_t* __restrict__ src, int K, int B, int rows_per_part,
    int n_part, const uint4* __restrict__ stage, const T* __restrict__ q, T* __restrict__ out,
    float* __restrict__ part, float scale_log2, int value_kind, float* __restrict__ vrange) {
  constexpr int VEC = Vec16<T>::n;            // elements per 16-byte piece
  constexpr int ROW_U4 = D / VEC;             // pieces (lanes) per row
  constexpr int kRowsPerPass = kCompBlock / ROW_U4;
  constexpr int kPasses = 2;
  constexpr int CHUNK = kRowsPerPass * kPasses;
  constexpr int kWaves = kCompBlock / kWave;
  static_assert(kMapRows % CHUNK == 0, "whole chunks per map segment");
  __shared__ float s_o[kWaves][G][D];
  __shared__ float s_ml[kWaves][G][2];
  __shared__ int s_src[kMapRows];
  const int p = PARTS ? (int)(blockIdx.x % (unsigned)n_part) : 0;
  const int inst = PARTS ? (int)(blockIdx.x / (unsigned)n_part) : (int)blockIdx.x;
  const int N = K + B;
  const int32_t* s = src + (size_t)inst * K;
  const int j_lo = p * rows_per_part, j_hi = min(K, j_lo + rows_per_part);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int col = threadIdx.x % ROW_U4;
  const int row0 = threadIdx.x / ROW_U4;
  uint4* kb = k + (size_t)inst * N * ROW_U4;
  uint4* vb = v + (size_t)inst * N * ROW_U4;
  // source rows at or above stage_lo come from the staging area
  const bool last_part = p + 1 == n_part;
  const int stage_lo = last_part ? N : j_hi;
  const uint4* wk = stage + ((size_t)inst * (n_part - 1) + p) * 2 * (size_t)B * ROW_U4;
  float qf[G][VEC];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint4 w = reinterpret_cast<const uint4*>(q + ((size_t)inst * G + g) * D)[col];
    Vec16<T>::unpack(w, qf[g]);
#pragma unroll
    for (int e = 0; e < VEC; ++e) qf[g][e] *= scale_log2;
  }
  float m[G], l[G], o[G][VEC];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -1.0e30f;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < VEC; ++e) o[g][e] = 0.f;
  }
  struct Rows {
    uint4 k[kPasses], v[kPasses];
  };
  Rows ra, rb, rc;
  for (int seg = j_lo; seg < j_hi; seg += kMapRows) {
    const int seg_hi = min(j_hi, seg + kMapRows);
    __syncthreads();                                   // the last segment's map is read
    for (int i = seg + threadIdx.x; i < seg_hi; i += kCompBlock) s_src[i - seg] = clamp_slot(s[i], N);
    __syncthreads();
    auto load = [&](int c0, Rows& r) {
#pragma unroll
      for (int u = 0; u < kPasses; ++u) {
        const int sj = s_src[min(c0 + row0 + u * kRowsPerPass, seg_hi - 1) - seg];
        const bool staged = PARTS && sj >= stage_lo;
        const size_t off = (size_t)(staged ? min(sj - stage_lo, B - 1) : sj) * ROW_U4 + col;
        r.k[u] = (staged ? wk : kb)[off];
        r.v[u] = (staged ? wk + (size_t)B * ROW_U4 : vb)[off];
      }
    };
    const int last = seg + (seg_hi - 1 - seg) / CHUNK * CHUNK;   // first row of the last chunk
    bool moved = false;                                  // the chunk before was stored
    // chunk c0 is in `cur`; two chunks ahead go to `next` (the last repeats)
    auto step = [&](int c0, const Rows& cur, Rows& next) {
      const bool full = c0 + CHUNK <= seg_hi;
      const int j_end = min(c0 + CHUNK, seg_hi) - 1;
      // one part: read ahead of the wait (285 rows a call 0.4 us less, but 1 % more in parts)
      int src_end = PARTS ? 0 : s_src[j_end - seg];
      load(min(c0 + 2 * CHUNK, last), next);
      // this thread's loads of chunk c0 are done: only the next two chunks'
      // 4*kPasses loads may remain, and what the chunk before (a full one)
      // stored between them; then every thread's are
      constexpr int kLoads = 4 * kPasses, kScores = CARRY ? kPasses : 0;
      if (c0 == seg) __builtin_amdgcn_s_waitcnt(0x0f70 | kLoads);
      else if (!moved) __builtin_amdgcn_s_waitcnt(0x0f70 | (kLoads + kScores));
      else __builtin_amdgcn_s_waitcnt(0x0f70 | (kLoads + kScores + 2 * kPasses));
      __syncthreads();
      // store the chunk unless every row is in place: src[j] - j never falls
      if (PARTS) src_end = s_src[j_end - seg];
      moved = __builtin_amdgcn_readfirstlane(src_end) != j_end;
      if (moved) {
#pragma unroll
        for (int u = 0; u < kPasses; ++u) {
          const int j = c0 + row0 + u * kRowsPerPass;
          if (full || j < seg_hi) {
            const size_t off = (size_t)j * ROW_U4 + col;
            kb[off] = cur.k[u];
            vb[off] = cur.v[u];
          }
        }
      }
      // decode: scores of the rows, one online-softmax update per chunk
      float sc[kPasses][G];
#pragma unroll
      for (int u = 0; u < kPasses; ++u) {
        float kf[VEC];
        Vec16<T>::unpack(cur.k[u], kf);
        const bool ok = c0 + row0 + u * kRowsPerPass < seg_hi;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          float acc = 0.f;
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc = __builtin_fmaf(qf[g][e], kf[e], acc);
          acc = lanes_sum<ROW_U4>(acc);
          sc[u][g] = ok ? acc : -INFINITY;
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float mn = m[g];
#pragma unroll
        for (int u = 0; u < kPasses; ++u) mn = fmaxf(mn, sc[u][g]);
        const float alpha = __builtin_amdgcn_exp2f(m[g] - mn);
        l[g] *= alpha;
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[g][e] *= alpha;
        m[g] = mn;
      }
#pragma unroll
      for (int u = 0; u < kPasses; ++u) {
        float vf[VEC];
        Vec16<T>::unpack(cur.v[u], vf);
        if (CARRY) {
          // the value score of compacted row j, which the next round's candidates
          // keep unchanged (only the buffer slots are written until then)
          const float val = row_value_score<VEC, ROW_U4>(vf, value_kind);
          const int j = c0 + row0 + u * kRowsPerPass;
          if (col == 0 && j < seg_hi) vrange[(size_t)inst * K + j] = val;
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float pr = __builtin_amdgcn_exp2f(sc[u][g] - m[g]);
          l[g] += pr;
#pragma unroll
          for (int e = 0; e < VEC; ++e) o[g][e] = __builtin_fmaf(pr, vf[e], o[g][e]);
        }
      }
    };
    load(seg, ra);
    __builtin_amdgcn_sched_barrier(0);
    load(min(seg + CHUNK, last), rb);
    __builtin_amdgcn_sched_barrier(0);
    for (int c0 = seg; c0 < seg_hi; c0 += 3 * CHUNK) {
      step(c0, ra, rc);
      if (c0 + CHUNK >= seg_hi) break;
      step(c0 + CHUNK, rb, ra);
      if (c0 + 2 * CHUNK >= seg_hi) break;
      step(c0 + 2 * CHUNK, rc, rb);
    }
  }
  // merge the row groups of each wave (lane bits above log2(ROW_U4)), fixed order
#pragma unroll
  for (int off = ROW_U4; off < kWave; off <<= 1) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float m2 = __shfl_xor(m[g], off, kWave);
      const float l2 = __shfl_xor(l[g], off, kWave);
      const float mn = fmaxf(m[g], m2);
      const float a1 = __builtin_amdgcn_exp2f(m[g] - mn), a2 = __builtin_amdgcn_exp2f(m2 - mn);
      l[g] = l[g] * a1 + l2 * a2;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float o2 = __shfl_xor(o[g][e], off, kWave);
        o[g][e] = o[g][e] * a1 + o2 * a2;
      }
      m[g] = mn;
    }
  }
  if (lane < ROW_U4) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) s_o[wave][g][col * VEC + e] = o[g][e];
      if (col == 0) {
        s_ml[wave][g][0] = m[g];
        s_ml[wave][g][1] = l[g];
      }
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < G * D; t += kCompBlock) {
    const int g = t / D, dd = t % D;
    float mn = s_ml[0][g][0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mn = fmaxf(mn, s_ml[w][g][0]);
    float lt = 0.f, ot = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float a = __builtin_amdgcn_exp2f(s_ml[w][g][0] - mn);
      lt += s_ml[w][g][1] * a;
      ot += s_o[w][g][dd] * a;
    }
    if (!PARTS) {
      store_out<T>(out + ((size_t)inst * G + g) * D + dd, ot / lt);
    } else {
      float* pp = part + (((size_t)inst * n_part + p) * G + g) * (kPartHead + D);
      pp[kPartHead + dd] = ot;
      if (dd == 0) *reinterpret_cast<float4*>(pp) = make_float4(mn, lt, mn, lt);
    }
  }
}

struct CompactDecodeArgs {
  uint4 *k, *v;
  const int32_t* src;
  int n_inst, K, B, G;
  const void* q;
  void* out;
  int value_kind;
  float* vrange;
  uint4* stage;
  float* part;
};

template <typename T, int D>
hipError_t launch_cd_d(const CompactDecodeArgs& a, const CompactPlan& pl, hipStream_t stream) {
  constexpr int kRowU4 = D / Vec16<T>::n;
  const float sl = 1.4426950408889634f / sqrtf((float)D);
  if (pl.n_part > 1)
    hipLaunchKernelGGL(compact_stage_kernel<kRowU4>, dim3(pl.n_part - 1, a.n_inst), dim3(kCompBlock),
                       0, stream, a.k, a.v, a.src, a.K, a.B, pl.rows_per_part, pl.n_part, a.stage);
#define VASE_CD(GG)                                                                             \
  case GG: {                                                                                    \
    auto kernel = pl.n_part > 1 ? (a.vrange ? compact_decode_kernel<T, D, GG, true, true>       \
                                            : compact_decode_kernel<T, D, GG, false, true>)     \
                                : (a.vrange ? compact_decode_kernel<T, D, GG, true, false>      \
                                            : compact_decode_kernel<T, D, GG, false, false>);   \
    hipLaunchKernelGGL(kernel, dim3((unsigned)(pl.n_part * a.n_inst)), dim3(kCompBlock), 0,     \
                       stream, a.k, a.v, a.src, a.K, a.B, pl.rows_per_part, pl.n_part, a.stage, \
                       static_cast<const T*>(a.q), static_cast<T*>(a.out), a.part, sl,          \
                       a.value_kind, a.vrange);                                                 \
    break;                                                                                      \
  }
  switch (a.G) {
    VASE_CD(1) VASE_CD(2) VASE_CD(3) VASE_CD(4) VASE_CD(5) VASE_CD(6) VASE_CD(7) VASE_CD(8)
    default: return hipErrorInvalidValue;
  }
#undef VASE_CD
  return hipGetLastError();
}

template <int ROW_U4>
hipError_t launch_rows(uint4* k, uint4* v, int n_inst, int K, int B, const int32_t* src,
                       uint4* ws, const CompactPlan& plan, hipStream_t stream) {
  if (plan.n_part > 1) {
    hipLaunchKernelGGL(compact_stage_kernel<ROW_U4>, dim3(plan.n_part - 1, n_inst),
                       dim3(kCompBlock), 0, stream, k, v, src, K, B, plan.rows_per_part,
                       plan.n_part, ws);
  }
  constexpr int kChunk = (kCompBlock / ROW_U4) * 4;
  hipLaunchKernelGGL((compact_move_kernel<ROW_U4, kChunk>), dim3(plan.n_part, n_inst),
                     dim3(kCompBlock), 0, stream, k, v, src, K, B, plan.rows_per_part,
                     plan.n_part, ws);
  return hipGetLastError();
}

}  // namespace

CompactPlan compact_plan(int dtype, int n_inst, int K, int B, int d) {
  CompactPlan pl;
  const size_t row_bytes = (size_t)d * (dtype == VASE_BF16 ? 2 : 4);
  // enough workgroups to cover the chip; parts of at least 256 rows
  int want = (1024 + n_inst - 1) / n_inst;
  int max_parts = K / 256 > 0 ? K / 256 : 1;
  pl.n_part = want < max_parts ? want : max_parts;
  if (pl.n_part < 1) pl.n_part = 1;
  pl.rows_per_part = (K + pl.n_part - 1) / pl.n_part;
  pl.n_part = (K + pl.rows_per_part - 1) / pl.rows_per_part;
  pl.bytes = pl.n_part > 1 ? (size_t)n_inst * (pl.n_part - 1) * 2 * (size_t)B * row_bytes : 0;
  return pl;
}

size_t compact_decode_least(int dtype, int n_inst, int K, int B, int d, int G) {
  const CompactPlan cp = compact_plan(dtype, n_inst, K, B, d);
  if (cp.n_part == 1 && K <= kCompactOneMaxK) return 0;
  const size_t dec = decode_plan(dtype, n_inst, K, B, d, G, K, K).bytes;
  return cp.bytes > dec ? cp.bytes : dec;
}

size_t compact_decode_bytes(int dtype, int n_inst, int K, int B, int d, int G) {
  const size_t least = compact_decode_least(dtype, n_inst, K, B, d, G);
  if (least == 0) return 0;
  const CompactPlan full = compact_decode_plan(dtype, n_inst, K, B, d, G, SIZE_MAX);
  return (long long)n_inst * full.n_part <= 256 && full.bytes > least ? full.bytes : least;
}

// Parts per instance for about 512 workgroups (two to a CU; 256 and 1024 are
// within 5 % of it from 64 to 576 instances), of at least 256 rows: each part
// but the last stages up to B rows, which are copied once more.  64 instances of
// 4096 rows and 128 staged, call time: 58 us with 8 parts, 66 with 16.  As many
// parts as the workspace holds.  The least that a call may come with holds the
// staged rows or the partials, which for few staged rows leaves one part to an
// instance; compact_decode_bytes asks for room for more where that leaves CUs
// idle (7 instances of 754 rows, B = 20, G = 7: one part 47 us, two 31).
CompactPlan compact_decode_plan(int dtype, int n_inst, int K, int B, int d, int G, size_t room) {
  const size_t row_bytes = (size_t)d * (dtype == VASE_BF16 ? 2 : 4);
  const int want = (512 + n_inst - 1) / n_inst;
  const int most = K / 256 > 0 ? K / 256 : 1;
  CompactPlan pl;
  for (int n = want < most ? want : most;; --n) {
    pl.rows_per_part = ((K + n - 1) / n + 31) / 32 * 32;
    pl.n_part = (K + pl.rows_per_part - 1) / pl.rows_per_part;
    pl.bytes = (size_t)n_inst * (pl.n_part - 1) * 2 * (size_t)B * row_bytes;
    if (pl.n_part == 1) break;
    pl.off_part = pl.bytes;
    pl.bytes += (size_t)n_inst * pl.n_part * G * (kPartHead + d) * sizeof(float);
    if (pl.bytes <= room) break;
  }
  return pl;
}

hipError_t launch_compact_decode(void* k, void* v, int dtype, int n_inst, int K, int B, int d,
                                 const int32_t* src, const void* q, int G, void* out,
                                 int value_kind, float* vrange, void* ws, const CompactPlan& pl,
                                 hipStream_t stream) {
  const CompactDecodeArgs a{static_cast<uint4*>(k), static_cast<uint4*>(v), src, n_inst, K, B, G, q,
                            out, value_kind, vrange, static_cast<uint4*>(ws),
                            reinterpret_cast<float*>(static_cast<char*>(ws) + pl.off_part)};
  hipError_t e = hipErrorInvalidValue;
  if (dtype == VASE_BF16) {
    if (d == 128) e = launch_cd_d<bf16_t, 128>(a, pl, stream);
    if (d == 64) e = launch_cd_d<bf16_t, 64>(a, pl, stream);
  } else {
    if (d == 128) e = launch_cd_d<float, 128>(a, pl, stream);
    if (d == 64) e = launch_cd_d<float, 64>(a, pl, stream);
  }
  if (e != hipSuccess || pl.n_part == 1) return e;
  return launch_decode_combine(a.part, dtype, n_inst, d, G, pl.n_part, out, stream);
}

hipError_t launch_compact(void* k, void* v, int dtype, int n_inst, int K, int B, int d,
                          const int32_t* src, void* ws, const CompactPlan& plan,
                          hipStream_t stream) {
  const int row_u4 = d * (dtype == VASE_BF16 ? 2 : 4) / 16;
  uint4* kk = static_cast<uint4*>(k);
  uint4* vv = static_cast<uint4*>(v);
  uint4* w = static_cast<uint4*>(ws);
  switch (row_u4) {
    case 8: return launch_rows<8>(kk, vv, n_inst, K, B, src, w, plan, stream);
    case 16: return launch_rows<16>(kk, vv, n_inst, K, B, src, w, plan, stream);
    case 32: return launch_rows<32>(kk, vv, n_inst, K, B, src, w, plan, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vase
