// score.hip -- pooled window-mean attention score and Range(v) on gfx950.
//
// abar_i = (1/R) sum_r exp(s_ri - lse_r),  s_ri = q_r . k_i / sqrt(d),  R = G*w rows,
// lse_r = log sum_{t<N} exp(s_rt) over all N slots (Eq. 1 rows inside Eq. 2),
// attn_i = (1/P) sum_{|j-i|<=P/2, 0<=j<K} abar_j,   vrange_i = max(v_i) - min(v_i) (Eq. 5).
//
// The row normaliser depends on every slot, so the scores are computed twice:
//   pass 1 (rows):  per row, the sum of exp2 over the slots -> lse2_r
//   pass 2 (cols):  p = exp2(s*c - lse2_r), column sums over rows
//   pool:           per slot: sum over row slabs, /R, then the P-wide box filter
// All exponentials are base 2 with c = log2(e)/sqrt(d) folded in.  No floating
// point atomics are used; every reduction has a fixed order.
// bf16 caches use MFMA on bf16 operands (v_mfma_f32_32x32x16_bf16, described
// below); fp32 caches MFMA on fp32 operands (score_f32.hip).
#include "vase_internal.hpp"
#include "vase.h"

#include <type_traits>

namespace vase {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kSBlock = 256;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
constexpr float kLog2e = 1.4426950408889634f;

// ---------------------------------------------------------------------------
// MFMA path (bf16), query-stationary.  A workgroup of W waves owns a slab of
// 64*W query rows of one instance and one range of its slots (the whole range
// when there are enough instances to fill the chip).  Each wave keeps its 64
// rows resident in VGPRs as A operands (two 32-row blocks); the slots stream
// through an LDS ring in chunks of 32 keys that all waves share as B operands
// (8 chunks deep, or 4 beside a 4-chunk ring of value rows when the pass
// scores them).  Accumulator element r of lane l holds (row 8(r/4) + 4h + r%4
// of a 32-row block, key l%32 of the chunk), h = l/32.
//
// The ring is filled by global->LDS DMA (global_load_lds_dwordx4) a ring's
// depth ahead of use, so the loads cost no VGPRs and their latency hides
// behind several chunks of MFMA work.  Completion is tracked with vmcnt by hand: the
// stream issues no other vector-memory operation, ring reads are explicit
// ds_read_b128 with their own lgkmcnt wait, and the barriers are plain
// s_barrier with the exact waits in front of them.  Column sums and Range
// collect in LDS and are written out after the stream.
//
// pass 1  m_f = midway between the largest and the smallest row maximum of a
//         32-row block over the first chunk (one offset per block, kept in a
//         scalar register); each lane sums exp2(s*c - m_f) over its keys, and
//         one transpose-reduce over the 32 lanes of a half wave gives l_r, so
//         lse2_r = m_f + log2 l_r.  That is exact while every row's sum lies in
//         [2^-90, FLT_MAX] (no term overflows, and the largest term of the row
//         is a normal number); otherwise the block computes the exact row
//         maxima and repeats the pass with one offset per row.  Attention-like
//         rows, whose maxima within a block differ by far less than 90
//         (base-2 units), never take that path.
// pass 2  p = exp2(s*c - lse2_r); each lane sums its 32 rows, one shuffle adds
//         the other half wave, and the W waves' sums meet in LDS in a fixed
//         order.  The same stream carries the value rows for Range (slab 0).
// With one range per instance both passes run in one kernel; otherwise pass 1
// writes (m_r, l_r) per range and pass 2 runs as its own kernel, whose
// workgroups first merge the ranges of their rows.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int kChunk = 32;         // keys per chunk
constexpr int kRingChunks = 8;     // LDS ring: 8 K chunks, or 4 K + 4 V chunks
constexpr int kMaxWaves = 8;
constexpr int kSlabRowsMax = 64 * kMaxWaves;
// slots per range: its column sums and Range (8 bytes per slot) share the 160
// KB of LDS with the ring (64 KB) and the row/column scratch (5 KB)
constexpr int kMaxSplitKeys = 11264;
// (instance, slab) pairs below which the slots may be split to fill the chip
constexpr int kSplitBelow = 512;

template <int D>
struct QFrag {
  static constexpr int KS = D / 16;   // k-steps of 16
  bf16x8_t a[2][KS];
  // rows row_base + [0, 64); rows >= R read as zero.  The contraction index is
  // permuted identically in both operands: lane half h, step ks holds elements
  // [16*ks + 8*h, +8) of its row (piece 2*ks + h), so that the two lanes of a
  // row read 32 adjacent bytes in one load.
  __device__ __forceinline__ void load(const uint16_t* qinst, int row_base, int R, int lane) {
    const int half = lane / 32;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const int row = row_base + f * 32 + lane % 32;
      const bool ok = row < R;
      const bf16x8_t* p =
          reinterpret_cast<const bf16x8_t*>(qinst + (size_t)(ok ? row : R - 1) * D + 8 * half);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8_t x = p[2 * ks];
        a[f][ks] = ok ? x : bf16x8_t{};
      }
    }
  }
};

// Layout of one 32-key chunk in LDS: 32 rows of D/8 16-byte pieces packed into
// 256-byte lines, the piece index XOR-swizzled by the line, so that the 16
// lanes of a B-operand read (16 rows, same piece) hit 16 bank groups.
template <int D>
struct ChunkLayout {
  static constexpr int kPieces = D / 8;
  static constexpr int kRowsPerLine = 16 / kPieces;
  static constexpr int kU4 = kChunk * kPieces;      // 16-byte pieces per chunk
  __device__ static __forceinline__ int off(int row, int p) {
    const int line = row / kRowsPerLine;
    const int lp = (row % kRowsPerLine) * kPieces + p;
    return line * 16 + (lp ^ (line & 15));
  }
  // inverse of off(): the (row, piece) stored at piece index idx
  __device__ static __forceinline__ void inv(int idx, int& row, int& p) {
    const int line = idx / 16;
    const int lp = (idx % 16) ^ (line & 15);
    row = line * kRowsPerLine + lp / kPieces;
    p = lp % kPieces;
  }
};

// DMA of one chunk (rows key0.., clamped to n_rows - 1) into an LDS slot.  The
// LDS side of global_load_lds is fixed (lane l of an instruction writes piece
// base + l), so each lane fetches the global piece that the swizzled layout
// puts there.  Per wave: kDma instructions (waves past the chunk issue none).
template <int D, int W>
struct ChunkDma {
  static constexpr int kU4 = ChunkLayout<D>::kU4;
  static constexpr int kDma = kU4 / (64 * W) > 0 ? kU4 / (64 * W) : 1;
  __device__ static __forceinline__ void issue(uint4* slot, const uint4* rows, int key0, int n_rows,
                                               int wave, int lane) {
#pragma unroll
    for (int i = 0; i < kDma; ++i) {
      const int base = (wave * kDma + i) * 64;
      if (kU4 % (64 * W) == 0 || base < kU4) {
        int row, p;
        ChunkLayout<D>::inv(base + lane, row, p);
        // byte offset from the instance's rows (an instance spans far less than
        // 4 GB), so the address is a uniform base plus one 32-bit lane offset
        const uint32_t key = (uint32_t)min(key0 + row, n_rows - 1);
        const uint32_t off = key * (uint32_t)(D * 2) + (uint32_t)p * 16u;
        __builtin_amdgcn_global_load_lds(
            static_cast<const void*>(reinterpret_cast<const char*>(rows) + off),
            (lds_void_t*)(slot + base), 16, 0, 0);
      }
    }
  }
};

// 16-byte LDS read that the compiler does not track (the ring is written by
// DMA, which the compiler would otherwise wait for in full before every read).
__device__ __forceinline__ bf16x8_t lds_read16(const uint4* p) {
  const uint32_t a = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint4*)p;
  bf16x8_t v;
  asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(a));
  return v;
}

// lds_read16 at a compile-time byte offset from a per-lane address (the
// instruction's 16-bit offset field), so that a ring slot known at compile
// time costs no address arithmetic.
template <int OFF>
__device__ __forceinline__ bf16x8_t lds_read16_at(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds_read offset field");
  bf16x8_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF));
  return v;
}

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// 4-byte LDS write, untracked for the same reason (the compiler cannot tell
// the dynamic LDS buffer from the DMA targets).  Barriers wait for it.
__device__ __forceinline__ void lds_write4(float* p, float x) {
  const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)p;
  asm volatile("ds_write_b32 %0, %1" : : "v"(a), "v"(x) : "memory");
}

// Barrier with explicit waits: this wave's ring DMA down to `VM` outstanding
// instructions and all of its LDS operations done, then s_barrier.  Compiler
// barriers keep memory operations on their side.
template <int VM>
__device__ __forceinline__ void ring_barrier() {
  static_assert(VM >= 0 && VM < 16, "vmcnt field");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070 | VM);   // vmcnt(VM) expcnt(7) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The B operand pieces of one lane: LDS byte addresses of its KS pieces in
// ring slot 0 (the piece layout is the same in every slot).
template <int D>
struct BAddr {
  static constexpr int KS = D / 16;
  uint32_t a[KS];
  __device__ __forceinline__ BAddr(const uint4* ring, int lane) {
    const int row = lane % 32, half = lane / 32;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = lds_addr(ring + ChunkLayout<D>::off(row, 2 * ks + half));
  }
};

// mfma_chunk for ring slot SLOT (a compile-time constant): the slot's offset
// goes into the LDS reads' offset field.
template <int D, int SLOT>
__device__ __forceinline__ void mfma_chunk_at(const QFrag<D>& qf, const BAddr<D>& ba,
                                              f32x16_t (&acc)[2]) {
  constexpr int KS = QFrag<D>::KS;
  constexpr int kSlotBytes = ChunkLayout<D>::kU4 * 16;
  bf16x8_t b[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) b[ks] = lds_read16_at<SLOT * kSlotBytes>(ba.a[ks]);
  acc[0] = f32x16_t{};
  acc[1] = f32x16_t{};
  // LDS reads complete in order: depth step ks waits only for its own read
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(b[ks]) : "i"(KS - 1 - ks));
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf.a[0][ks], b[ks], acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf.a[1][ks], b[ks], acc[1], 0, 0, 0);
  }
}

// acc[f] = Q_block(f) x K_chunk^T (32 rows x 32 keys each).
template <int D>
__device__ __forceinline__ void mfma_chunk(const QFrag<D>& qf, const uint4* slot, int lane,
                                           f32x16_t (&acc)[2]) {
  constexpr int KS = QFrag<D>::KS;
  const int row = lane % 32, half = lane / 32;
  bf16x8_t b[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) b[ks] = lds_read16(slot + ChunkLayout<D>::off(row, 2 * ks + half));
  // the reads above are invisible to the compiler: wait for them here, tying
  // the registers so that no MFMA can be scheduled before the wait
  if constexpr (KS == 8)
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]),
                 "+v"(b[4]), "+v"(b[5]), "+v"(b[6]), "+v"(b[7]));
  else
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
  acc[0] = f32x16_t{};
  acc[1] = f32x16_t{};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf.a[0][ks], b[ks], acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf.a[1][ks], b[ks], acc[1], 0, 0, 0);
  }
}


// Value score of the rows of a chunk held in an LDS slot, into out[key - key_lo]
// for keys below hi: Range = max - min (Eq. 5), L2 = sqrt(sum v^2) or
// Var = mean (v - mu)^2 (Appendix A), over each row's D elements.
template <int D, int W>
__device__ __forceinline__ void chunk_value(const uint4* vslot, int key0, int key_lo, int hi,
                                            int kind, float* out, bool check, bool& bad) {
  constexpr int kPieces = D / 8;
  constexpr int kU4 = ChunkLayout<D>::kU4;
  constexpr int kPer = (kU4 + 64 * W - 1) / (64 * W);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int pc = (int)threadIdx.x + i * 64 * W;   // consecutive lanes: consecutive pieces of a row
    const int pcc = pc < kU4 ? pc : kU4 - 1;
    const int row = pcc / kPieces;
    bf16x8_t w = lds_read16(vslot + ChunkLayout<D>::off(row, pcc % kPieces));
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w));
    float f[8];
    Vec16<bf16_t>::unpack(__builtin_bit_cast(uint4, w), f);
    const float val = row_value_score<8, kPieces>(f, kind);
    if (check) bad |= key0 + row < hi && any_nonfinite<8>(f);
    if (pc < kU4 && pc % kPieces == 0 && key0 + row < hi) lds_write4(out + (key0 + row - key_lo), val);
  }
}

// Transpose-reduce over the 32 lanes of each half wave: lane j ends with
// element j reduced (sum or max) over its half's lanes.
template <bool MAX>
__device__ __forceinline__ float treduce32(float (&v)[32], int lane) {
#pragma unroll
  for (int o = 16; o >= 1; o >>= 1) {
    // lanes with bit o set keep the upper half and send the lower; the swap is
    // done on the bits so that no element is picked by a lane-dependent index
    const uint32_t m = (lane & o) ? 0xffffffffu : 0u;
#pragma unroll
    for (int i = 0; i < o; ++i) {
      const uint32_t lo = __float_as_uint(v[i]), hi = __float_as_uint(v[i + o]);
      const uint32_t x = (lo ^ hi) & m;
      const float send = __uint_as_float(hi ^ x);
      const float keep = __uint_as_float(lo ^ x);
      const float got = __shfl_xor(send, o, kWave);
      v[i] = MAX ? fmaxf(keep, got) : keep + got;
    }
  }
  return v[0];
}

// slab row of element j (= 16 f + r) of a lane in half h of a wave
__device__ __forceinline__ int elem_row(int j, int half) {
  return (j / 16) * 32 + 8 * ((j % 16) / 4) + 4 * half + (j % 4);
}

// Decode-query logits of one chunk: q_dec[g] . k_key for the chunk's keys below
// hi and g < G, into dst[g * stride + key - base].  Two 16-key tiles of
// v_mfma_f32_16x16x32_bf16 with the keys as the A operand (lane l: key l % 16,
// depth [8(l/16), +8) of each 32-deep step) and the query rows as the B operand
// (column l % 16 = head, clamped to G - 1; those columns are dropped),
// accumulated over the depth steps in order, so that the logits are bit for
// bit those of a decode kernel that runs the same tiles from global memory.
// Lane l ends with keys 4(l/16) .. +3 of head l % 16.  TO_LDS: dst is LDS
// (written untracked, like the ring); else global memory.
typedef float df32x4_t __attribute__((ext_vector_type(4)));
template <int D, bool TO_LDS>
__device__ __forceinline__ void dec_logits_chunk(const uint4* slot, const uint4* qd, int G, int lane,
                                                 int key0, int hi, int base, float* dst,
                                                 int stride) {
  constexpr int KS = D / 32;
  constexpr int KP = D / 8;
  const int hm = lane % 16, hq = lane / 16;
  const int hc = min(hm, G - 1);
  if constexpr (D == 128 && TO_LDS) {
    // one 256-byte line per key row: piece p of row r sits at r*16 + (p ^ (r & 15)),
    // so depth step ks of tile t is at a per-lane base, a per-lane 64-byte step
    // (ks ^ (hm >> 2)) and a fixed 4 KB per tile (immediate offsets).  The lane
    // id is read here (volatile), so these addresses are formed at each call
    // instead of being kept live across the key loop, where they would spill.
    uint32_t ln;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
    const int lm = (int)(ln % 16u), lq = (int)(ln / 16u);
    const int lc = min(lm, G - 1);
    const uint32_t bq = lds_addr(qd) + (uint32_t)(lc * KP + lq) * 16u;
    const uint32_t a0 = lds_addr(slot) + (uint32_t)(16 * lm + (lq ^ (lm & 3))) * 16u;
    uint32_t aa[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) aa[ks] = a0 + ((uint32_t)(ks ^ (lm >> 2)) << 6);
    bf16x8_t b[KS], a[KS];
    b[0] = lds_read16_at<0>(bq);
    b[1] = lds_read16_at<64>(bq);
    b[2] = lds_read16_at<128>(bq);
    b[3] = lds_read16_at<192>(bq);
    const bool full = key0 + kChunk <= hi && stride % 4 == 0;
    const int k4 = key0 + 4 * lq;
    float* p = dst + (size_t)lc * stride + (k4 - base);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) a[ks] = t ? lds_read16_at<4096>(aa[ks]) : lds_read16_at<0>(aa[ks]);
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]),
                   "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
      df32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], b[ks], acc, 0, 0, 0);
      if (lm < G) {
        if (full) {
          asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(lds_addr(p)), "v"(acc), "i"(64 * t)
                       : "memory");
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (k4 + 16 * t + i < hi) lds_write4(p + 16 * t + i, acc[i]);
        }
      }
    }
    return;
  }
  bf16x8_t b[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) b[ks] = lds_read16(qd + hc * KP + 4 * ks + hq);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    bf16x8_t a[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = lds_read16(slot + ChunkLayout<D>::off(16 * t + hm, 4 * ks + hq));
    if constexpr (KS == 4)
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]),
                   "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
    else
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]));
    df32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], b[ks], acc, 0, 0, 0);
    if (hm < G) {
      const int key = key0 + 16 * t + 4 * hq;
      float* p = dst + (size_t)hm * stride + (key - base);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (key + i < hi) {
          if (TO_LDS) lds_write4(p + i, acc[i]);
          else p[i] = acc[i];
        }
      }
    }
  }
}

// log2(2^l2 + 2^(L log2 e)): a row's normaliser with its supplied persistent part L
__device__ __forceinline__ float add_persistent(float l2, float L) {
  const float b = L * kLog2e;
  const float m = fmaxf(l2, b);
  return m + fast_log2(fast_exp2(l2 - m) + fast_exp2(b - m));
}

// lse2 of one row from its n_part partials p[i * R] = (m, l), four in flight:
// m + log2(sum l_i 2^(m_i - m)).  Each pass-2 workgroup merges its own rows (a
// launch for it took 6.5 to 15 us).
__device__ __forceinline__ float merge_parts(const float2* p, int R, int n_part) {
  float m = -INFINITY, l = 0.f;
#pragma unroll 1
  for (int i = 0; i < n_part; i += 4) {
    float2 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u] = p[(size_t)min(i + u, n_part - 1) * R];
      if (i + u >= n_part) x[u].y = 0.f;              // a repeat adds nothing
    }
    const float mn = fmaxf(fmaxf(fmaxf(x[0].x, x[1].x), fmaxf(x[2].x, x[3].x)), m);
    l = l * fast_exp2(m - mn);
#pragma unroll
    for (int u = 0; u < 4; ++u) l += x[u].y * fast_exp2(x[u].x - mn);
    m = mn;
  }
  return m + fast_log2(l);
}

enum ScoreMode { kPass1 = 0, kPass2 = 1, kFused = 2 };

// Workgroups of score_mfma_kernel that a CU holds: 160 KB of LDS in steps of 1280
// bytes (the ring, the rows' and columns' exchange, 256 for the block votes, and
// what the launch adds), and 512 registers to a lane of a SIMD, of which the
// second pass takes 165 at d = 64 and every other one more than 170.
int score_places(int d, int waves, ScoreMode mode, size_t dynamic) {
  if (waves == 8) return 1;
  size_t lds = (size_t)kRingChunks * kChunk * d * 2 + 256 + dynamic;
  if (mode != kPass2) lds += (size_t)waves * 2 * 32 * 4;
  if (mode != kPass1) lds += (size_t)4 * kChunk * waves * 4;
  const size_t n = (size_t)160 * 1024 / ((lds + 1279) / 1280 * 1280);
  const size_t most = d == 64 && mode == kPass2 ? 3 : 2;
  return n < 1 ? 1 : n > most ? (int)most : (int)n;
}

// The ring and the stream state of one pass.  A pass that scores values (pass
// 2 with Range, L2 or Var) streams the V rows through a second ring of the
// same depth S = 4 beside the K ring; every other pass gives the whole LDS
// ring to K (S = 8), so its DMA runs further ahead.  Every chunk costs the
// same number of DMA instructions, which the vmcnt waits count.
template <int D, int W, bool WITH_V>
struct Stream {
  static constexpr int kU4 = ChunkLayout<D>::kU4;
  static constexpr int kPerChunk = ChunkDma<D, W>::kDma * (WITH_V ? 2 : 1);
  static constexpr int S = WITH_V ? kRingChunks / 2 : kRingChunks;   // ring depth in chunks
  uint4* kring;
  uint4* vring;
  const uint4* krows;
  const uint4* vrows;
  int key_lo, n_krows, n_vrows, wave, lane;
  __device__ __forceinline__ uint4* kslot(int ch) const { return kring + (ch % S) * kU4; }
  __device__ __forceinline__ uint4* vslot(int ch) const { return vring + (ch % S) * kU4; }
  __device__ __forceinline__ void fetch(int ch) const {
    const int key0 = key_lo + kChunk * ch;
    ChunkDma<D, W>::issue(kslot(ch), krows, key0, n_krows, wave, lane);
    if (WITH_V) ChunkDma<D, W>::issue(vslot(ch), vrows, key0, n_vrows, wave, lane);
  }
};

// Chunk pipeline over chunks [0, nc) with a ring of S chunks.  The first A
// chunks are fetched up front and chunk 0 goes through the MFMAs before the
// first step (init sees its products then); at step ch a wave
//   * fetches chunk ch+A into ring slot (ch+A)%S,
//   * runs side(ch+1) (value scores or decode logits of chunk ch+1, the
//     column-sum flush of an earlier chunk),
//   * issues the MFMAs of chunk ch+1 and the VALU epilogue of chunk ch (its
//     accumulators were filled at step ch-1) in one basic block,
//     (a wave whose rows all lie past the last window row skips both: it
//     only fetches and meets the other waves),
//   * after every step (S = 4, A = 4) or every odd step (S = 8, A = 6) waits
//     until its own DMA up to chunk ch+2 (S = 4) or ch+3 (S = 8) has landed and
//     meets the other waves.
// With S = 8 no wave can be more than one step ahead of another, so the slot
// (ch+6)%8 = (ch-2)%8 refilled at step ch was last read at step ch-3, and a
// barrier lies between any three consecutive steps; each barrier covers the
// chunks read in the two steps after it.  The loop is unrolled over the ring,
// so every slot and accumulator buffer is a compile-time constant.  Chunks
// past the end fetch clamped rows; their results are dropped.  The caller
// waits for the trailing DMA before the ring is used again.
template <int U, int S, typename F>
__device__ __forceinline__ bool ring_steps(F& step, int t) {
  if constexpr (U < S) {
    if (step(std::integral_constant<int, U>{}, t)) return true;
    return ring_steps<U + 1, S>(step, t);
  } else {
    return false;
  }
}

template <int D, typename St, typename Epi, typename Side, typename Init>
__device__ __forceinline__ void stream_chunks(const QFrag<D>& qf, const St& st, int nc, int lane,
                                              bool active, Epi&& epi, Side&& side, Init&& init) {
  constexpr int S = St::S;
  // an 8-deep ring meets after every other step: fetch 6 ahead, wait for 3 ahead
  constexpr bool kPair = S == 8;
  constexpr int kAhead = kPair ? S - 2 : S;
  constexpr int kWait = kPair ? 3 * St::kPerChunk : (S - 2) * St::kPerChunk;
  const BAddr<D> ba(st.kring, lane);
#pragma unroll
  for (int ch = 0; ch < kAhead; ++ch) st.fetch(ch);
  ring_barrier<kWait>();
  f32x16_t acc[2][2];
  side(0);
  if (active) {
    mfma_chunk_at<D, 0>(qf, ba, acc[0]);
    init(acc[0]);                       // sees chunk 0's products before its epilogue
  }
  ring_barrier<kWait>();
  auto step = [&](auto u_, int t) -> bool {
    constexpr int U = decltype(u_)::value;
    const int ch = t + U;
    st.fetch(ch + kAhead);
    side(ch + 1);
    if (active) {
      mfma_chunk_at<D, (U + 1) % S>(qf, ba, acc[(U + 1) % 2]);
      epi(ch, acc[U % 2]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!kPair || U % 2 == 1) ring_barrier<kWait>();
    return ch + 1 >= nc;
  };
  for (int t = 0; t < nc; t += S)
    if (ring_steps<0, S>(step, t)) break;
}

// Plain loop (one chunk at a time) for the rarely taken exact path.
template <int D, typename St, typename Epi>
__device__ __forceinline__ void simple_chunks(const QFrag<D>& qf, const St& st, int nc, int lane,
                                              Epi&& epi) {
  for (int ch = 0; ch < nc; ++ch) {
    st.fetch(ch);
    ring_barrier<0>();
    f32x16_t a[2];
    mfma_chunk<D>(qf, st.kslot(ch), lane, a);
    epi(ch, a);
    ring_barrier<0>();
  }
}

// DL: decode-query logits of pass 1: 0 none, 1 staged in LDS and written after
// the pass, 2 written from the chunk loop (when they do not fit in LDS).
// PARTIAL: the last slab holds fewer than W waves' rows (its other waves only
// stream the keys); a separate instantiation, so that full slabs carry no test
template <int D, int W, int MODE, int DL, bool PARTIAL>
__global__ __launch_bounds__(64 * W, 2) void score_mfma_kernel(
    const uint4* __restrict__ k, const uint4* __restrict__ v, const uint16_t* __restrict__ q,
    int N, int K, int R, int n_slab, int n_split, int split_keys, float c, int pool, int value_kind,
    const float* __restrict__ lse_win, float2* __restrict__ part, int n_part,
    float* __restrict__ col, float* __restrict__ vrange, float* __restrict__ attn,
    const int32_t* __restrict__ ord, const uint4* __restrict__ qdec, int G_dec,
    float* __restrict__ dlog, int dl_stride, int first_apart, uint32_t* __restrict__ status) {
  constexpr int kU4 = ChunkLayout<D>::kU4;
  __shared__ uint4 ring[kRingChunks * kU4];
  __shared__ float rowbuf[W][2][32];
  __shared__ float colbuf[4][kChunk][W];   // [chunk % 4][column][wave]
  extern __shared__ float keybuf[];   // pass 2: [split_keys] column sums, then [split_keys] Range
  constexpr int KP = D / 8;
  const uint32_t lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int split = (int)(lb % (uint32_t)n_split);
  const uint32_t t0 = lb / (uint32_t)n_split;
  const int slab = (int)(t0 % (uint32_t)n_slab);
  const int inst = (int)(t0 / (uint32_t)n_slab);
  const int lane = threadIdx.x % kWave, half = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);   // uniform per wave
  const int j = lane % 32;
  const int row_base = slab * 64 * W + wave * 64;
  // waves whose 64 rows all lie past R (the last slab of a window that is not
  // a multiple of the slab) stream the keys with the others but score nothing;
  // the column sums take the first n_act waves' partial sums
  const bool active = !PARTIAL || row_base < R;
  const int n_act = PARTIAL ? min(W, (R - slab * 64 * W + 63) / 64) : W;
  const int key_lo = split * split_keys;
  const uint4* kinst = k + (size_t)inst * N * KP;
  QFrag<D> qf;
  qf.load(q + (size_t)inst * R * D, row_base, R, lane);
  float rs[32];   // per element: exact row maxima (exact path), then lse2 (pass 2)
  // data faults for the status word: a row normaliser that is not a positive
  // finite number (this lane's row), a value row with a non-finite element
  bool row_bad = false, v_bad = false;
  auto report = [&]() {
    if (status) {
      block_status(status, row_bad, VASE_STATUS_ROW_NORM);
      block_status(status, v_bad, VASE_STATUS_VALUE_ROW);
    }
  };

  if (MODE != kPass2) {
    // pass 1 covers this range's slots, or only the buffer [K, N) when the
    // persistent part of every row's normaliser is supplied (lse_win)
    const bool single = lse_win != nullptr;
    const int lo1 = single ? K : key_lo;
    const int hi1 = single ? N : min(N, key_lo + split_keys);
    const int nc1 = (hi1 - lo1 + kChunk - 1) / kChunk;
    const Stream<D, W, false> st{ring, ring, kinst, kinst, lo1, N, N, wave, lane};
    // decode-query logits of the streamed keys (slab 0 only).  The G_dec query
    // rows wait in the pass-2 scratch, which pass 1 does not use, and, when
    // dl_stride > 0, the logits too ([G_dec][dl_stride], written out after the
    // pass): a global store inside the chunk loop would be counted by the
    // vmcnt waits that pace the ring
    float* const dl = DL != 0 && slab == 0 ? dlog + (size_t)inst * G_dec * N : nullptr;
    uint4* const qd = reinterpret_cast<uint4*>(keybuf);
    float* const dls = keybuf + G_dec * KP * 4;
    if (dl) {
      for (int i = threadIdx.x; i < G_dec * KP; i += 64 * W) qd[i] = qdec[(size_t)inst * G_dec * KP + i];
    }
    // mb[f]: one offset per 32-row block, midway between the largest and the
    // smallest row maximum over the first chunk (rows >= R left out), taken
    // from chunk 0's products when the stream has computed them
    float mb[2] = {0.f, 0.f};
    // a pass of its own sums the first chunk's terms apart, element j's in l_first:
    // where they outweigh the rest (a row that looks at the first tokens), every
    // later term would be rounded to their last place.  One sum, not the 32 terms
    // of a lane: those took the registers of d = 128 past 256 (7 to 39 spilled in
    // 10 of 12 instantiations).  Errors against 64 bits, mean of 30 inputs: 64
    // instances of 4224 slots 1.9e-7 either way, 8 of 2176 1.9e-7 for 2.0e-7.
    // One range does so where the call might have been split (first_apart), so
    // that the choice of ranges costs no accuracy: 64 instances of 8448 slots and
    // 2048 rows 1.8e-7, in about 1024 workgroups 2.6e-7, in one sum 5.5e-7.
    // Everywhere it would cost 0.4 % of the largest calls
    const bool apart = MODE == kPass1 || first_apart != 0;
    float l_first = 0.f;
    auto init1 = [&](f32x16_t (&a)[2]) {
      const bool ok = lo1 + j < hi1;
      float t[32];
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) t[f * 16 + r] = ok ? a[f][r] * c : -INFINITY;
      const float mj0 = treduce32<true>(t, lane);     // row max of element j over the chunk
      const bool rv = row_base + elem_row(j, half) < R;
      float hi = rv ? mj0 : -INFINITY, lo = rv ? mj0 : INFINITY;
#pragma unroll
      for (int o = 1; o <= 32; o <<= 1) {
        if (o == 16) continue;                        // lanes j and j^16 hold different blocks
        hi = fmaxf(hi, __shfl_xor(hi, o, kWave));
        lo = fminf(lo, __shfl_xor(lo, o, kWave));
      }
      const float mid = hi == -INFINITY ? 0.f : 0.5f * (hi + lo);
      mb[0] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mid), 0));
      mb[1] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mid), 16));
      if (apart) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            t[f * 16 + r] = ok ? fast_exp2(__builtin_fmaf(a[f][r], c, -mb[f])) : 0.f;
        l_first = treduce32<false>(t, lane);
      }
    };
    float l[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) l[i] = 0.f;
    auto epi1 = [&](int ch, f32x16_t (&a)[2]) {
      const bool ok = lo1 + kChunk * ch + j < hi1 && (!apart || ch > 0);
      const float okf = ok ? 1.f : 0.f;
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          l[f * 16 + r] = __builtin_fmaf(okf, fast_exp2(__builtin_fmaf(a[f][r], c, -mb[f])),
                                         l[f * 16 + r]);
    };
    auto side1 = [&](int ch) {
      if (DL != 0 && dl && ch < nc1 && wave == ch % W) {
        if constexpr (DL == 1)
          dec_logits_chunk<D, true>(st.kslot(ch), qd, G_dec, lane, lo1 + kChunk * ch, hi1, lo1,
                                    dls, dl_stride);
        else
          dec_logits_chunk<D, false>(st.kslot(ch), qd, G_dec, lane, lo1 + kChunk * ch, hi1, 0,
                                     dl, N);
      }
      // keep the logit tiles' registers apart from the chunk's MFMA operands
      if (DL != 0) __builtin_amdgcn_sched_barrier(0);
    };
    stream_chunks<D>(qf, st, nc1, lane, active, epi1, side1, init1);
    ring_barrier<0>();                                // trailing DMA landed
    if (DL == 1 && dl) {
      const int nk1 = hi1 - lo1;
      for (int i = threadIdx.x; i < G_dec * nk1; i += 64 * W) {
        const int g = i / nk1, t = i - g * nk1;
        dl[(size_t)g * N + lo1 + t] = dls[g * dl_stride + t];
      }
    }
    float lj = treduce32<false>(l, lane) + l_first;
    float mj = j < 16 ? mb[0] : mb[1];
    const int row = row_base + elem_row(j, half);
    // Exact as long as every term stays finite and the largest term of each row
    // stays a normal number: sums in [2^-90, FLT_MAX] guarantee both.
    const bool bad = row < R && !(lj >= 0x1p-90f && lj <= 3.0e38f);
    if (__syncthreads_or(bad)) {
      // exact row maxima first, then the sums again with one offset per row
      float mx[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) mx[i] = -INFINITY;
      auto epim = [&](int ch, f32x16_t (&a)[2]) {
        const bool ok = lo1 + kChunk * ch + j < hi1;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx[f * 16 + r] = ok ? fmaxf(mx[f * 16 + r], a[f][r] * c) : mx[f * 16 + r];
      };
      simple_chunks<D>(qf, st, nc1, lane, epim);
      rowbuf[wave][half][j] = treduce32<true>(mx, lane);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        rs[i] = rowbuf[wave][half][i];
        l[i] = 0.f;
      }
      auto epix = [&](int ch, f32x16_t (&a)[2]) {
        const float okf = lo1 + kChunk * ch + j < hi1 ? 1.f : 0.f;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            l[f * 16 + r] = __builtin_fmaf(okf, fast_exp2(__builtin_fmaf(a[f][r], c, -rs[f * 16 + r])),
                                           l[f * 16 + r]);
      };
      simple_chunks<D>(qf, st, nc1, lane, epix);
      lj = treduce32<false>(l, lane);
      mj = rowbuf[wave][half][j];
    }
    if (MODE == kPass1) {
      if (row < R) part[((size_t)inst * n_split + split) * R + row] = make_float2(mj, lj);
      return;
    }
    __syncthreads();
    float l2 = mj + fast_log2(lj);
    if (single && row < R) l2 = add_persistent(l2, lse_win[(size_t)inst * R + row]);
    row_bad = row < R && !(l2 > -INFINITY && l2 < INFINITY);
    rowbuf[wave][half][j] = row < R ? l2 : INFINITY;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; ++i) rs[i] = rowbuf[wave][half][i];
  } else {
    // merge pass 1's ranges: each lane one row of its wave
    const int row = row_base + elem_row(j, half);
    float l2 = INFINITY;                              // padded rows give p = 0
    if (row < R) {
      l2 = merge_parts(part + (size_t)inst * n_part * R + row, R, n_part);
      if (lse_win) l2 = add_persistent(l2, lse_win[(size_t)inst * R + row]);
      row_bad = split == 0 && !(l2 > -INFINITY && l2 < INFINITY);
    }
    // passed on by lane exchanges: 1 KB more of LDS (rowbuf) would leave a CU one
    // workgroup for two from 1632 slots per range on, for 1760 (4 waves, d = 128)
#pragma unroll
    for (int i = 0; i < 32; ++i) rs[i] = __shfl(l2, 32 * half + i, kWave);
  }

  // ---- pass 2: column sums over the slab's rows for slots [key_lo, hi2)
  const int hi2 = min(K, key_lo + split_keys);
  if (hi2 <= key_lo) {
    report();
    return;
  }
  const int nc2 = (hi2 - key_lo + kChunk - 1) / kChunk;
  // value scores of the candidates: not for random reservation (drawn elsewhere)
  // nor when the caller supplies them
  const bool rng = slab == 0 && value_kind <= VASE_VALUE_VAR;
  float* colsum = keybuf;
  float* vr = keybuf + split_keys;
  // column sums of chunk ch over the W waves, fixed order; colbuf rotates over
  // four chunks.  With the value rows in the stream (a barrier after every
  // step) chunk ch is flushed at step ch+1; without them (a barrier after
  // every odd step) at step ch+2.  Either way the flush follows a barrier that
  // followed every wave's epilogue of ch, and a barrier separates it from the
  // epilogue of ch+4 that writes its buffer again
  auto flush = [&](int ch) {
    if (ch >= 0 && ch < nc2 && wave == ch % W && lane < kChunk) {
      // the W waves' sums of this column sit together: one or two 16-byte reads
      float cw[W];
#pragma unroll
      for (int w = 0; w < W; w += 4)
        *reinterpret_cast<float4*>(cw + w) = *reinterpret_cast<const float4*>(&colbuf[ch % 4][lane][w]);
      float sum = cw[0];
#pragma unroll
      for (int w = 1; w < W; ++w) sum += w < n_act ? cw[w] : 0.f;
      lds_write4(colsum + kChunk * ch + lane, sum);
    }
  };
  auto epi2 = [&](int ch, f32x16_t (&a)[2]) {
    // four partial sums, each seeded with its first term
    float p0 = fast_exp2(__builtin_fmaf(a[0][0], c, -rs[0]));
    float p1 = fast_exp2(__builtin_fmaf(a[0][1], c, -rs[1]));
    float p2 = fast_exp2(__builtin_fmaf(a[0][2], c, -rs[2]));
    float p3 = fast_exp2(__builtin_fmaf(a[0][3], c, -rs[3]));
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int r = f == 0 ? 4 : 0; r < 16; r += 4) {
        const int e = f * 16 + r;
        p0 += fast_exp2(__builtin_fmaf(a[f][r], c, -rs[e]));
        p1 += fast_exp2(__builtin_fmaf(a[f][r + 1], c, -rs[e + 1]));
        p2 += fast_exp2(__builtin_fmaf(a[f][r + 2], c, -rs[e + 2]));
        p3 += fast_exp2(__builtin_fmaf(a[f][r + 3], c, -rs[e + 3]));
      }
    float cs = (p0 + p1) + (p2 + p3);
    cs += __shfl_xor(cs, 32, kWave);
    colbuf[ch % 4][j][wave] = cs;
  };
  if (rng) {
    // the value rows ride in the second half of the ring
    const Stream<D, W, true> st{ring, ring + (kRingChunks / 2) * kU4, kinst,
                                v + (size_t)inst * N * KP, key_lo, N, K, wave, lane};
    auto side2 = [&](int ch) {
      if (ch < nc2)
        chunk_value<D, W>(st.vslot(ch), key_lo + kChunk * ch, key_lo, hi2, value_kind, vr,
                          status != nullptr, v_bad);
      flush(ch - 2);
    };
    stream_chunks<D>(qf, st, nc2, lane, active, epi2, side2, [](f32x16_t (&)[2]) {});
  } else {
    const Stream<D, W, false> st{ring, ring, kinst, kinst, key_lo, N, N, wave, lane};
    stream_chunks<D>(qf, st, nc2, lane, active, epi2, [&](int ch) { flush(ch - 3); },
                     [](f32x16_t (&)[2]) {});
  }
  ring_barrier<0>();                                  // trailing DMA landed, last colbuf visible
  // the stream flushed chunks up to (last step + 1) - 2; flush the rest
  const int last_side = (nc2 - 1) + 1;                // side() of the final step
  for (int ch = max(last_side - (rng ? 1 : 2), 0); ch < nc2; ++ch) flush(ch);
  __syncthreads();
  float* vr_out = vrange + (size_t)inst * K;
  if (MODE == kFused && n_slab == 1) {
    // the workgroup holds every column sum of the instance: pool here, with
    // the same arithmetic as score_pool_kernel (mean over rows, then the
    // zero-padded box filter summed in slot order, then / P).  Under an order
    // map the filter runs over temporal ranks: rank t is slot ord[t], and the
    // outputs are indexed by rank (the map is staged in the idle ring).
    const float fr = (float)R, fp = (float)pool;
    const int h = pool / 2;
    float* attn_out = attn + (size_t)inst * K;
    int* slot_of = reinterpret_cast<int*>(ring);
    if (ord) {
      for (int i = threadIdx.x; i < K; i += 64 * W)
        slot_of[i] = min(max(ord[(size_t)inst * K + i], 0), K - 1);
      __syncthreads();
    }
    for (int i = threadIdx.x; i < K; i += 64 * W) {
      float sum = 0.f;
      for (int t = 0; t < pool; ++t) {
        const int jj = i - h + t;
        sum += (jj >= 0 && jj < K) ? colsum[ord ? slot_of[jj] : jj] / fr : 0.f;
      }
      attn_out[i] = sum / fp;
      if (rng) vr_out[i] = vr[ord ? slot_of[i] : i];
    }
    report();
    return;
  }
  float* col_out = col + ((size_t)inst * n_slab + slab) * K;
  for (int i = threadIdx.x; i < hi2 - key_lo; i += 64 * W) {
    col_out[key_lo + i] = colsum[i];
    if (rng) vr_out[key_lo + i] = vr[i];
  }
  report();
}

// ---------------------------------------------------------------------------
// pooling: abar_j = (sum over slabs of col) / R ; attn_i = box filter / P
// ---------------------------------------------------------------------------
constexpr int kPoolTile = 256;
constexpr int kMaxHalo = 127;
__global__ __launch_bounds__(kSBlock) void score_pool_kernel(const float* __restrict__ col, int K,
                                                           int n_slab, int R, int pool,
                                                           float* __restrict__ attn) {
  __shared__ float tile[kPoolTile + 2 * kMaxHalo];
  const int inst = blockIdx.y;
  const int i0 = blockIdx.x * kPoolTile;
  const int h = pool / 2;
  const float fr = (float)R, fp = (float)pool;
  for (int t = threadIdx.x; t < kPoolTile + 2 * h; t += kSBlock) {
    const int j = i0 - h + t;
    float v = 0.f;
    if (j >= 0 && j < K) {
      float s = 0.f;
      for (int sl = 0; sl < n_slab; ++sl) s += col[((size_t)inst * n_slab + sl) * K + j];
      v = s / fr;
    }
    tile[t] = v;
  }
  __syncthreads();
  const int i = i0 + threadIdx.x;
  if (i >= K) return;
  float s = 0.f;
  for (int t = 0; t < pool; ++t) s += tile[threadIdx.x + t];
  attn[(size_t)inst * K + i] = s / fp;
}

// The same under an order map, by one workgroup per instance: the slots' means
// (over the slabs, then / R) go to LDS in slot order, the map gathers them into
// temporal order there, and the box filter runs over ranks; the value scores
// that the score wrote per slot are gathered the same way.  Every global access
// is in order, so it is bound by its bytes (4 per slab, 12 for the map and the
// result, 8 more with value scores); gathering slot means from global memory
// in a kernel behind the pooling took 50 us at 512 instances of 8192
// candidates and two slabs, against 27 here.
constexpr int kPoolMapPer = 8;   // candidates per thread: K <= VASE_MAX_K at 1024 threads
template <int NT>
__global__ __launch_bounds__(NT) void score_pool_map_kernel(
    const float* __restrict__ col, const int32_t* __restrict__ ord,
    const float* __restrict__ vr_slot, int K, int n_slab, int R, int pool,
    float* __restrict__ attn, float* __restrict__ vrange) {
  extern __shared__ float pool_buf[];   // [K] by slot, [K] by rank
  float* const slot_v = pool_buf;
  float* const rank_v = pool_buf + K;
  const int inst = blockIdx.x;
  const size_t base = (size_t)inst * K;
  const float fr = (float)R, fp = (float)pool;
  // candidates past the last read the last one's, so that no load is behind a
  // branch and a thread's loads are all in flight
  int at[kPoolMapPer], o[kPoolMapPer];
#pragma unroll
  for (int u = 0; u < kPoolMapPer; ++u) {
    at[u] = min((int)threadIdx.x + u * NT, K - 1);
    o[u] = ord[base + at[u]];
  }
  float s[kPoolMapPer], vr[kPoolMapPer];
#pragma unroll
  for (int u = 0; u < kPoolMapPer; ++u) {
    s[u] = 0.f;
    vr[u] = vr_slot ? vr_slot[base + at[u]] : 0.f;
  }
  for (int sl = 0; sl < n_slab; ++sl) {
    const float* c = col + ((size_t)inst * n_slab + sl) * K;
#pragma unroll
    for (int u = 0; u < kPoolMapPer; ++u) s[u] += c[at[u]];
  }
#pragma unroll
  for (int u = 0; u < kPoolMapPer; ++u) {
    o[u] = min(max(o[u], 0), K - 1);
    if ((int)threadIdx.x + u * NT < K) slot_v[threadIdx.x + u * NT] = s[u] / fr;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPoolMapPer; ++u)
    if ((int)threadIdx.x + u * NT < K) rank_v[threadIdx.x + u * NT] = slot_v[o[u]];
  __syncthreads();
  // the box filter, its taps in order, the thread's candidates side by side
  const int h = pool / 2;
#pragma unroll
  for (int u = 0; u < kPoolMapPer; ++u) s[u] = 0.f;
  for (int t = -h; t <= h; ++t) {
#pragma unroll
    for (int u = 0; u < kPoolMapPer; ++u) {
      const int i = at[u] + t;
      const float x = rank_v[min(max(i, 0), K - 1)];
      s[u] += i >= 0 && i < K ? x : 0.f;
    }
  }
#pragma unroll
  for (int u = 0; u < kPoolMapPer; ++u) {
    const int i = threadIdx.x + u * NT;
    if (i >= K) continue;
    if (vr_slot) slot_v[i] = vr[u];
    attn[base + i] = s[u] / fp;
  }
  if (!vr_slot) return;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPoolMapPer; ++u) {
    const int i = threadIdx.x + u * NT;
    if (i < K) vrange[base + i] = slot_v[o[u]];
  }
}

// The same by one workgroup per 256 ranks, which gathers the slots' sums and value
// scores straight from memory: a scattered 4-byte read each, but no workgroup
// goes over a whole instance.
__global__ __launch_bounds__(kSBlock) void score_pool_gather_kernel(
    const float* __restrict__ col, const int32_t* __restrict__ ord,
    const float* __restrict__ vr_slot, int K, int n_slab, int R, int pool,
    float* __restrict__ attn, float* __restrict__ vrange) {
  __shared__ float mean[kSBlock + 256];   // ranks [i0 - h, i0 + kSBlock + h), h <= 127
  const int inst = blockIdx.y, i0 = blockIdx.x * kSBlock, h = pool / 2;
  const size_t base = (size_t)inst * K;
  const float fr = (float)R, fp = (float)pool;
  const float* c = col + (size_t)inst * n_slab * K;
  for (int t = threadIdx.x; t < kSBlock + 2 * h; t += kSBlock) {
    const int i = i0 - h + t;
    float s = 0.f;
    if (i >= 0 && i < K) {
      const int o = min(max(ord[base + i], 0), K - 1);
      for (int sl = 0; sl < n_slab; ++sl) s += c[(size_t)sl * K + o];
    }
    mean[t] = s / fr;
  }
  const int i = i0 + threadIdx.x;
  const float vr = vr_slot && i < K ? vr_slot[base + min(max(ord[base + i], 0), K - 1)] : 0.f;
  __syncthreads();
  if (i >= K) return;
  float sum = 0.f;
  for (int t = 0; t < pool; ++t) sum += mean[threadIdx.x + t];
  attn[base + i] = sum / fp;
  if (vr_slot) vrange[base + i] = vr;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

template <int D, int W, bool P>
void launch_mfma_w(const void* k, const void* v, const void* q, int n_inst, int N, int K, int R,
                   float c, int pool, int kind, const float* lse_win, const ScorePlan& pl, char* ws,
                   float* vrange, float* attn, const int32_t* ord, const DecLogits& dec,
                   hipStream_t stream, uint32_t* status) {
  const uint4* qd = static_cast<const uint4*>(dec.q);
  // pass 1 stages the decode queries, and the logits when they fit, in the
  // dynamic LDS that pass 2 uses
  const int dl_keys = ((pl.n_chunk1 == 1 ? N : pl.split_keys) + 3) / 4 * 4;   // 16-byte rows
  constexpr size_t kStaticLds = (size_t)kRingChunks * ChunkLayout<D>::kU4 * 16 + W * 2 * 32 * 4 +
                                4 * kChunk * W * 4;
  constexpr size_t kLdsCap = 160 * 1024 - kStaticLds - 1024;
  const size_t q_lds = (size_t)dec.G * D * 2;
  const size_t keybuf = 2 * sizeof(float) * (size_t)pl.split_keys;
  const size_t staged = q_lds + (size_t)dec.G * dl_keys * 4;
  // Staging must not cost the CU a workgroup: 350 instances of 1053 slots and 45
  // rows at d = 128 take 100 us with staged logits at one workgroup to a CU, 53 with
  // logits written from the loop at two (42 drawn calls of that kind: 0.52 to 0.93
  // of the staged time).  At as many workgroups the two are within 4 %.
  const ScoreMode mode1 = pl.n_chunk1 == 1 ? kFused : kPass1;
  const size_t floor_lds = pl.n_chunk1 == 1 && keybuf > q_lds ? keybuf : q_lds;
  const bool stage = staged <= kLdsCap && score_places(D, W, mode1, staged > floor_lds ? staged : floor_lds) ==
                                              score_places(D, W, mode1, floor_lds);
  const int dl_stride = dec.out && stage && !lse_win ? dl_keys : 0;
  const size_t dec_lds = dec.out ? q_lds + (size_t)dec.G * dl_stride * 4 : 0;
  const int dl_mode = !dec.out ? 0 : dl_stride > 0 ? 1 : 2;
  float2* part = reinterpret_cast<float2*>(ws + pl.off_part);
  float* col = reinterpret_cast<float*>(ws + pl.off_col);
  const uint4* kk = static_cast<const uint4*>(k);
  const uint4* vv = static_cast<const uint4*>(v);
  const uint16_t* qq = static_cast<const uint16_t*>(q);
  const unsigned grid = (unsigned)(n_inst * pl.n_slab * pl.n_chunk1);
  if (pl.n_chunk1 == 1) {
    auto fused = dl_mode == 0 ? score_mfma_kernel<D, W, kFused, 0, P>
                 : dl_mode == 1 ? score_mfma_kernel<D, W, kFused, 1, P>
                                : score_mfma_kernel<D, W, kFused, 2, P>;
    hipLaunchKernelGGL(fused, dim3(grid), dim3(64 * W), keybuf > dec_lds ? keybuf : dec_lds,
                       stream, kk, vv, qq, N, K, R, pl.n_slab, 1, pl.split_keys, c, pool, kind,
                       lse_win, part, 0, col, vrange, attn, ord, qd, dec.G, dec.out, dl_stride,
                       (int)(!lse_win && (long long)n_inst * pl.n_slab < kSplitBelow), status);
    return;
  }
  // pass 1: every slot range, or one range over the buffer [K, N) when the
  // persistent part of each row's normaliser is supplied
  const int n1 = lse_win ? 1 : pl.n_chunk1;
  const int keys1 = lse_win ? (N - K + kChunk - 1) / kChunk * kChunk : pl.split_keys;
  auto pass1 = dl_mode == 0 ? score_mfma_kernel<D, W, kPass1, 0, P>
               : dl_mode == 1 ? score_mfma_kernel<D, W, kPass1, 1, P>
                              : score_mfma_kernel<D, W, kPass1, 2, P>;
  hipLaunchKernelGGL(pass1, dim3((unsigned)(n_inst * pl.n_slab * n1)), dim3(64 * W), dec_lds,
                     stream, kk, vv, qq, N, K, R, pl.n_slab, n1, keys1, c, pool, kind, lse_win,
                     part, 0, col, vrange, attn, nullptr, qd, dec.G, dec.out, dl_stride, 1, nullptr);
  hipLaunchKernelGGL((score_mfma_kernel<D, W, kPass2, 0, P>), dim3(grid), dim3(64 * W), keybuf, stream,
                     kk, vv, qq, N, K, R, pl.n_slab, pl.n_chunk1, pl.split_keys, c, pool, kind,
                     lse_win, part, n1, col, vrange, attn, nullptr, nullptr, 0, nullptr, 0, 0, status);
}

template <int D>
void launch_mfma(const void* k, const void* v, const void* q, int n_inst, int N, int K, int R,
                 float c, int pool, int kind, const float* lse_win, const ScorePlan& pl, char* ws,
                 float* vrange, float* attn, const int32_t* ord, const DecLogits& dec,
                 hipStream_t stream, uint32_t* status) {
  // some waves of the last slab hold no window row
  const bool partial = pl.n_slab * pl.rows_per_slab - R >= 64;
#define VASE_MFMA_W(W, P)                                                                          \
  launch_mfma_w<D, W, P>(k, v, q, n_inst, N, K, R, c, pool, kind, lse_win, pl, ws, vrange, attn, \
                         ord, dec, stream, status)
  if (pl.waves == 4) {
    if (partial) VASE_MFMA_W(4, true);
    else VASE_MFMA_W(4, false);
  } else {
    if (partial) VASE_MFMA_W(8, true);
    else VASE_MFMA_W(8, false);
  }
#undef VASE_MFMA_W
}

}  // namespace

namespace {

// ranges that n_split equal ones of whole chunks come down to
int split_ranges(int N, int n_split) {
  const int keys = ((N + n_split - 1) / n_split + kChunk - 1) / kChunk * kChunk;
  return (N + keys - 1) / keys;
}

// What a pass takes on the chip, in us.  A workgroup of four waves leaves room for
// another on its CU, as far as LDS (and for d = 64 registers) reaches.  A chunk
// step of a CU takes `fixed` (the ring's transfers and barriers) and `rows` for
// each of its workgroups, as far as their waves hold window rows; eight waves are
// one workgroup to a CU.  A workgroup costs `own` more steps (its rows' load, the
// ring's fill, the reductions).  Fitted to 1200 drawn calls of up to 511
// (instance, slab) pairs at every number of ranges (9 % root mean square).  The
// ranges so chosen take 1 % longer than the best ones in the mean and 0.72 of the
// time of splitting every call into about 1024 workgroups, at most 1.06 of it;
// with two workgroups taken for granted some took 1.5 of it.
struct StepCost {
  double fixed, rows, own, wide_fixed, wide_rows, wide_own;   // four waves, eight waves
};
constexpr StepCost kStep128{0.50, 0.21, 5.3, 0.53, 0.20, 7.5}, kStep64{0.36, 0.16, 5.3, 0.55, 0.07, 6.0};
constexpr double kSplitLaunch = 6.3;    // the second pass and the pooling as launches of their own
constexpr double kMergePart = 0.09;     // one more partial per row for every pass-2 workgroup
constexpr double kPoolInside = 1.5e-3;  // pooling by the fused kernel, per candidate (5 taps)
constexpr double kValueShare = 0.24;    // value rows in pass 2: they add 0.6, where not carried
constexpr int kCus = 256;

// filled: the share of a workgroup's waves that hold window rows; uneven: full slabs
// and one that is not.  Workgroups of those differ, so rounds do not end together:
// a pass takes no less than its work over the CUs and half of a full workgroup.
// Without that one range looked best for 233 instances of 4869 slots and 609 rows
// (577 us, three 544), and two for 95 of 760 and 1677 (119 us, one 98).  At d = 64 a
// workgroup's time hardly depends on its rows, and the rule above does better (51
// of 7056 slots and 711 rows 173 us, 193 so).
double pass_us(long long blocks, int places, int waves, double filled, bool uneven, int d, int chunks) {
  const StepCost& c = d == 128 ? kStep128 : kStep64;
  if (waves == 8) {
    const double step = c.wide_fixed + c.wide_rows * filled;
    double steps = (double)((blocks + kCus - 1) / kCus) * step;
    if (uneven && blocks > kCus) {
      const double least = (double)blocks / kCus * step + 0.5 * (c.wide_fixed + c.wide_rows);
      steps = steps > least ? steps : least;
    }
    return steps * (chunks + c.wide_own);
  }
  const long long round = (long long)kCus * places, rest = blocks % round;
  double steps = (double)(blocks / round) * (c.fixed + c.rows * filled * places);
  if (rest) steps += c.fixed + c.rows * filled * (double)((rest + kCus - 1) / kCus);
  return steps * (chunks + c.own);
}

// Ranges per (instance, slab) for `base` of them, too few to fill the chip, from
// `least` to `most`.  The choice hangs on the sizes alone, so that a call with
// and without value rows, decode logits or an order map sums in the same order.
int pick_split(long long base, int n_slab, int waves, int R, int d, int K, int B, int least, int most,
               bool lse) {
  const double filled = (double)((R + 63) / 64) / (n_slab * waves);
  const bool uneven = d == 128 && n_slab > 1 && filled < 1;
  const int chunks = (K + B + kChunk - 1) / kChunk;
  int best_n = least;
  double best = 0;
  for (int n = least; n <= most;) {
    const int per = (chunks + n - 1) / n;
    const long long blocks = base * ((chunks + per - 1) / per);
    const size_t keybuf = 2 * sizeof(float) * (size_t)per * kChunk;
    const int p1 = n == 1 ? score_places(d, waves, kFused, keybuf) : score_places(d, waves, kPass1, 0);
    const int p2 = n == 1 ? p1 : score_places(d, waves, kPass2, keybuf);
    // with the persistent normalisers given, pass 1 is one range over the buffer
    double t = lse ? pass_us(base, p1, waves, filled, uneven, d, (B + kChunk - 1) / kChunk)
                   : pass_us(blocks, p1, waves, filled, uneven, d, per) + kMergePart * n;
    t += pass_us(blocks, p2, waves, filled, uneven, d, per) * (1 + kValueShare);
    if (n > 1) t += kSplitLaunch;
    else if (n_slab == 1) t += kPoolInside * K;
    if (n == least || t < best) {
      best = t;
      best_n = n;
    }
    if (per == 1) break;
    const int next = (chunks + per - 2) / (per - 1);   // the fewest ranges that are shorter
    n = next > n ? next : n + 1;
  }
  return best_n;
}

}  // namespace

ScorePlan score_plan(int dtype, int n_inst, int K, int B, int d, int G, int w, bool lse) {
  ScorePlan pl{};
  const int N = K + B;
  const int R = G * w;
  pl.mfma = dtype == VASE_BF16;
  if (pl.mfma) {
    // slabs of at most 512 rows; 4 or 8 waves of 64 rows per slab
    pl.n_slab = (R + kSlabRowsMax - 1) / kSlabRowsMax;
    const int need = (R + 64 * pl.n_slab - 1) / (64 * pl.n_slab);
    pl.waves = need <= 4 ? 4 : 8;
    pl.rows_per_slab = 64 * pl.waves;
    pl.n_slab = (R + pl.rows_per_slab - 1) / pl.rows_per_slab;
    // one slot range per (instance, slab) when that alone gives >= 512 workgroups
    // and the range's column sums fit in LDS; otherwise the slots are split.  The
    // workspace has room for as many ranges as give about 1024 workgroups.
    const long long base = (long long)n_inst * pl.n_slab;
    const int chunks = (N + kChunk - 1) / kChunk;
    int n_split = (N + kMaxSplitKeys - 1) / kMaxSplitKeys;
    int most = n_split;
    if (base < kSplitBelow) {
      const long long want = (1024 + base - 1) / base;
      const int more = (int)(want < chunks ? want : chunks);
      most = more > n_split ? more : n_split;
    }
    pl.n_chunk2 = split_ranges(N, most);
    pl.n_chunk1 = base < kSplitBelow ? split_ranges(N, pick_split(base, pl.n_slab, pl.waves, R, d, K, B, n_split,
                                                          pl.n_chunk2, lse))
                             : pl.n_chunk2;
    pl.split_keys = ((N + pl.n_chunk1 - 1) / pl.n_chunk1 + kChunk - 1) / kChunk * kChunk;
  } else {
    pl.waves = 0;
    pl.split_keys = 0;
    // the workspace holds partials for runs of one 32-key tile and one row slab;
    // longer runs leave room for the column sums of more slabs
    pl.n_chunk2 = (N + kChunk - 1) / kChunk;
    const size_t col = align256((size_t)n_inst * K * sizeof(float));
    const size_t part = align256((size_t)n_inst * pl.n_chunk2 * R * sizeof(float2)) +
                        align256((size_t)n_inst * R * sizeof(float));
    score_f32_split(n_inst, N, K, R, part, pl);
    pl.bytes = part + col;
    return pl;
  }
  pl.off_part = 0;
  // one workgroup that holds the instance's every row and slot pools by itself
  pl.pool_in_kernel = pl.n_chunk1 == 1 && pl.n_slab == 1;
  // row partials only where the slots may be split
  pl.off_col = pl.n_chunk2 == 1 ? 0 : align256((size_t)n_inst * pl.n_chunk2 * R * sizeof(float2));
  pl.bytes = pl.n_chunk2 == 1 && pl.n_slab == 1
                 ? 0 : pl.off_col + align256((size_t)n_inst * pl.n_slab * K * sizeof(float));
  return pl;
}

hipError_t launch_score(const void* k, const void* v, const void* q, int dtype, int n_inst, int K,
                        int B, int d, int G, int w, int pool, int value_kind, const float* lse_win,
                        float* attn, float* vrange, void* ws, const ScorePlan& pl,
                        hipStream_t stream, const int32_t* ord, const DecLogits& dec,
                        uint32_t* status, float* vr_phys) {
  const int N = K + B;
  const int R = G * w;
  const float c = 1.4426950408889634f / sqrtf((float)d);
  char* wsb = static_cast<char*>(ws);
  // where the value scores go: under a map that the pooling launch applies,
  // per slot into the workspace first
  float* vr_slot = ord && !pl.pool_in_kernel ? vr_phys : vrange;
  if (dtype == VASE_BF16) {
    if (d == 128)
      launch_mfma<128>(k, v, q, n_inst, N, K, R, c, pool, value_kind, lse_win, pl, wsb, vr_slot,
                       attn, ord, dec, stream, status);
    else
      launch_mfma<64>(k, v, q, n_inst, N, K, R, c, pool, value_kind, lse_win, pl, wsb, vr_slot,
                      attn, ord, dec, stream, status);
  } else {
    const hipError_t e = launch_score_f32(k, v, q, n_inst, N, K, R, d, c, value_kind, lse_win, pl,
                                          wsb, vr_slot, stream, status);
    if (e != hipSuccess) return e;
  }
  const float* col = reinterpret_cast<const float*>(wsb + pl.off_col);
  if (!pl.pool_in_kernel) {
    if (ord) {
      const float* vs = value_kind <= VASE_VALUE_VAR ? vr_slot : nullptr;
      // Up to 2^19 candidates in the call the scattered reads meet in the caches and
      // more workgroups win, beyond that reading everything once does (score of
      // the 16-row window with Range, gathered / staged, us): 2 instances of 4096
      // 16.0 / 21.3, 64: 31.0 / 33.9, 128: 47.0 / 47.1, 256: 79.9 / 75.9
      if ((long long)n_inst * K <= (1LL << 19)) {
        hipLaunchKernelGGL(score_pool_gather_kernel, dim3((K + kSBlock - 1) / kSBlock, n_inst),
                           dim3(kSBlock), 0, stream, col, ord, vs, K, pl.n_slab, R, pool, attn, vrange);
      } else {
        // 8 candidates per thread: four waves cover K <= 2048, sixteen the rest
        const size_t lds = 2 * sizeof(float) * (size_t)K;
        const bool wide = K > 256 * kPoolMapPer;
        hipLaunchKernelGGL(wide ? score_pool_map_kernel<1024> : score_pool_map_kernel<256>, dim3(n_inst),
                           dim3(wide ? 1024 : 256), lds, stream, col, ord, vs, K, pl.n_slab, R, pool,
                           attn, vrange);
      }
    } else {
      hipLaunchKernelGGL(score_pool_kernel, dim3((K + kPoolTile - 1) / kPoolTile, n_inst),
                         dim3(kSBlock), 0, stream, col, K, pl.n_slab, R, pool, attn);
    }
  }
  return hipGetLastError();
}

}  // namespace vase
