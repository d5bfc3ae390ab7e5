// Matrix-core kernel of tkv_quant_attn_decode (Sec. 2.1 Eq. 3 over the quantized cache
// of Sec. 4.3) for gfx950: up to H = 4 or 8 query heads of a KV head per workgroup, D = 128, 2 bits with
// quantization groups of 32 or 64, 4 bits with groups of 32, 1 bit with groups of 64 (Sec. 5.1 runs 1
// and 2 bits with groups of 64).
//
// One wave64 owns one packed block of 32 tokens at a time (half a key group when the
// quantization group is 64; "group" below means such a block).  Both contractions run on
// v_mfma_f32_16x16x32_f16 with the packed codes as the A operand:
//
//   * a b-bit code c sitting at mantissa bits [bp, bp+b) of an otherwise zero fp16 IS
//     the subnormal number c * 2^bp * 2^-24, so one v_and_b32 per register turns two
//     codes into two exact fp16 operands (no bias, no convert); the 2^bp factor is
//     compensated in the other operand;
//   * q.K-hat = sum_c code[t][c] * (q[c] s[c]) + sum_c q[c] z[c]: the scaler moves into
//     the query operand, split into fp16 hi + lo parts so the product keeps ~22 bits.
//     The 16 operand columns are H query heads x 16 / H column groups; even groups carry the
//     hi part and odd groups the lo part, so ONE MFMA per (16 tokens, 32 channels) produces
//     both partial sums and a single cross-lane add joins them.  The zero-point term does
//     not depend on the token: it is computed once per workgroup for all of its groups
//     (16 groups per MFMA) and kept in an LDS table;
//   * p.V-hat = sum_t code[t][d] * (p[t] s_v[t][u]) + sum_t p[t] z_v[t][u]: here the column
//     groups are the channel groups u, so the weights never leave the lanes that produced
//     them (the D layout of the first product is the B layout of the second); z_v and the
//     softmax denominator ride on one more MFMA.  A 16-channel block of V needs one u only:
//     with 8 heads, whose columns hold two u, four channel groups (group 32) take a second
//     set of weights for the blocks of u = 2, 3, and no MFMA more.  The weights go in as one
//     fp16 number each (the product p s_v is rounded once).
//
// Groups of 5 to 8 query heads per KV head (H = 8) cost the operand preparation of four more heads
// and a merge of twice the partials; served as two workgroups of up to 4 heads they cost the reading and unpacking of
// the codes twice.  The launch takes whichever is shorter (see its rule).  4 bits with groups of 64 and 1 bit
// with groups of 32 are not served here: they keep float32 weights (tkv_quant_attn.hip).
//
// The machine issues one vector or matrix instruction per SIMD at a time and a wave issues
// in order, so the cost of a group is close to the plain sum of its instructions: the
// design minimises instruction count first, then hides latencies with three resident
// waves per SIMD (2 bit) and a three-deep ring of direct global->LDS loads per wave.
//
// Softmax is online per wave with lazy rescaling; the waves of a workgroup and the chunks
// of a sequence are merged with log-sum-exp merges, the last workgroup of a (sequence, KV
// head) to finish doing the cross-chunk merge.
#include "tkv_common.h"
#include "tkv_quantizer.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

struct MfmaParams {
  const uint32_t* k_codes;
  const uint32_t* v_codes;
  const __half* k_scale;
  const __half* k_zero;
  const __half* v_scale;
  const __half* v_zero;
  const __half* k_resid;
  const __half* v_resid;
  const __half* q;
  float* parts;        // sequence after sequence: [Hq], chunks of the sequence * (D + 4) floats each
  uint32_t* arrivals;  // [B][Hkv << split], zero between calls
  __half* out;         // [B][Hq][D]
  float scale2;
  int32_t hq, hkv, residual, capacity;
  int32_t batch;
  int32_t tail_blocks; // blocks that a 32-token piece of the fp16 tail counts as in the split
  int32_t split;       // 0: one workgroup takes all query heads of a KV head; 1: two, of up to 4 (blockIdx.y = 2 h + part)
#ifdef TKV_PHASE
  long long* prof;  // phase time stamps (profiling builds only)
#endif
  TkvSeqLens lens;
  TkvSeqLens chunks;  // split-K chunks of every sequence, in proportion to its length: blockIdx.x runs over all of them
  // The step's new tokens, when the call also appends them (Eq. 2): the last n_add[b] tokens of
  // sequence b, rows k_new / v_new [B][n_stride][Hkv][D], are copied into the fp16 ring by the
  // workgroups that own the head's tail, which read them from here themselves.  k_new == nullptr: none.
  const __half* k_new;
  const __half* v_new;
  int32_t n_stride;
  int32_t complete;  // non-zero: they may complete a group, which this launch then quantizes
  TkvSeqLens n_add;
};

__device__ inline floatx4 mfma(uintx4 a, uintx4 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// Reinterpret one 32-bit register as two fp16.  Takes the word BY VALUE: applying
// __builtin_bit_cast directly to an element of an ext-vector (vec[j]) reads element 0
// for every j with this compiler.
__device__ inline half2_t as_half2(uint32_t w) { return __builtin_bit_cast(half2_t, w); }

__device__ inline uint32_t pack2(_Float16 lo, _Float16 hi) {
  half2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, v);
}

// v + (value of the lane H = 4 or 8 places away in the same row of 16 lanes)
template <int H>
__device__ inline float ror_add(float v) {
  const int r = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + H /* row_ror:H */, 0xF, 0xF, false);
  return v + __builtin_bit_cast(float, r);
}

// fp16 hi/lo split of a product, written so that each part is one fused multiply-add
// with an fp16 result (the compiler selects v_fma_mixlo/mixhi_f16 for this shape):
//   hi = f16(a * b), lo = f16(a * b - hi)   (the FMA makes the residual exact)
// s2 holds two fp16 scalers; the results are packed the same way.  No inline assembly:
// operands that come straight from MFMA / transcendental results have read hazards that
// only the compiler's own instructions are checked for.
__device__ inline uint32_t mix_hi_pair(float a0, float a1, uint32_t s2) {
  const half2_t s = as_half2(s2);
  return pack2((_Float16)__builtin_fmaf(a0, (float)s[0], 0.0f), (_Float16)__builtin_fmaf(a1, (float)s[1], 0.0f));
}
__device__ inline uint32_t mix_lo_pair(float a0, float a1, uint32_t s2, uint32_t hi) {
  const half2_t s = as_half2(s2), h = as_half2(hi);
  return pack2((_Float16)__builtin_fmaf(a0, (float)s[0], -(float)h[0]),
               (_Float16)__builtin_fmaf(a1, (float)s[1], -(float)h[1]));
}

// 1 bit: four MFMA operands out of one word.  Operands 1 and 3 sit four mantissa bits
// higher than operands 0 and 2: their results carry an extra 2^4.
__device__ inline void extract1(uint32_t w, uintx4 (&a)[4]) {
  const uint32_t w8 = w >> 8;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    a[0][j] = w & (0x00010001u << j);
    a[1][j] = w & (0x00100010u << j);
    a[2][j] = w8 & (0x00010001u << j);
    a[3][j] = w8 & (0x00100010u << j);
  }
}
// 2 bit: two MFMA operands (8 registers) out of one 32-bit word of packed codes.
__device__ inline void extract2(uint32_t w, uintx4& a0, uintx4& a1) {
  const uint32_t w8 = w >> 8;
  a0[0] = w & 0x00030003u;
  a0[1] = w & 0x000C000Cu;
  a0[2] = w & 0x00300030u;
  a0[3] = w & 0x00C000C0u;
  a1[0] = w8 & 0x00030003u;
  a1[1] = w8 & 0x000C000Cu;
  a1[2] = w8 & 0x00300030u;
  a1[3] = w8 & 0x00C000C0u;
}
// 4 bit: one operand per word.
__device__ inline void extract4(uint32_t w, uintx4& a) {
  const uint32_t w8 = w >> 8;
  a[0] = w & 0x000F000Fu;
  a[1] = w & 0x00F000F0u;
  a[2] = w8 & 0x000F000Fu;
  a[3] = w8 & 0x00F000F0u;
}

// SIZE bytes per lane from a descriptor's array straight to LDS, in lane order from `to` on
template <int SIZE>
__device__ inline void buffer_to_lds(__amdgpu_buffer_rsrc_t from, void* to, uint32_t lane_offset, uint32_t offset) {
  auto* lds = (__attribute__((address_space(3))) void*)to;
  static_assert(SIZE == 4 || SIZE == 16, "sizes used here");
  if constexpr (SIZE == 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(from, lds, 4, (int)lane_offset, (int)offset, 0, 0);
  else __builtin_amdgcn_raw_ptr_buffer_load_lds(from, lds, 16, (int)lane_offset, (int)offset, 0, 0);
}

// Query-side operands q s 2^(kEK - position shift) are fp16 hi + lo pairs.  kEK = 0 leaves the
// whole fp16 range to the product of query and key scaler; the parts that then fall into
// fp16's subnormal range keep an absolute precision (2^-25 per operand) that is worth less
// than 1e-5 in the logit, so nothing is gained by a larger kEK (measured 0 to 4).
constexpr int kEK = 0;
// Weight-side operands carry 2^kEP: fp16 weights p 2^(kEP - position shift) (p below
// 2^kHeadroomLog2) times the value scaler must stay below 65504, and so must the zero-point
// times 2^(position shift - kEP).  kEP = 2 keeps both finite for value scalers up to 1023 (a group's
// range up to 1023 at 1 bit, 3069 at 2, 15345 at 4) and zero-points up to 4000; the attention
// error does not depend on it (measured 0 to 6).
constexpr int kEP = 2;
constexpr int kHeadroomLog2 = 4;  // lazy rescale: weights may reach 2^kHeadroomLog2
constexpr int kRefBelowMax = 3;   // a rescale puts the reference this far under the largest logit (< headroom)
// The fp16 tail's accumulators start the block loop scaled by 2^kTailRoomLog2.  Blocks whose logits are
// further below change an output by less than 65504 * 2^-32, a subnormal number.
constexpr int kTailRoomLog2 = 32;
constexpr int kBkStride = 68;     // words per head row of the query-side operand in LDS (16 rows x 4 words: all 64 banks)
constexpr int max_gpc(int heads) { return heads <= 4 ? 512 : 256; }  // groups per chunk that the zero-point table holds
// Blocks that a 32-token piece of the fp16 tail counts as in the split (2 bit, 2000 tokens: 12.6 us per
// call with 3, 13.1 with 2; from 16384 tokens on 2 to 5 make no difference).
constexpr int kTailBlocks = 3, kTailBlocksLeast = 2;
// ... and that quantizing a group which the step's new tokens complete counts as, where a sequence has several chunks.  us per
// call of such a step, with a launch of its own for the append / here: 2 bit, 32/8 heads, 131071 tokens 35.6, 30.6; 32767 22.7,
// 18.0; 2047 17.2, 15.3; 255 14.2, 12.1; 4 bit, 131071 44.7, 38.8; 2 bit / 64, 32767 24.6, 17.6; 1 bit / 64, 98431, 32/4 heads
// 28.3, 22.9; 8 sequences of 16383 36.8, 31.6.  (Counting as 40 blocks instead of 24: the same within 2 %; as none: 2 to 4 us longer.)
constexpr int kCompleteBlocks = 24;
// Sequences of up to this many blocks (tail pieces counted as above) per wave are one workgroup's:
// no partials to write, no arrival, no merge.  us per call with 3 rounds against 1, 8 KV heads: 2 bit, one
// sequence, 200 tokens 9.1, 11.4; 520 10.8, 11.7; 896 11.0, 12.2; 16 sequences of 800 11.8, 13.7; 4 bit, 200 tokens 8.7,
// 10.3, 400 10.7, 10.4.  Over 200 to 896 tokens, 1 to 32 KV heads and all settings at most 5 % longer, at most
// 30 % shorter.  With more rounds the loop outgrows the merge (2 bit, 1000 tokens: 14.1 in one, 12.9 in several).
constexpr int kOneChunkRounds = 3;

// Results of one wave for the merge inside the workgroup; it takes the place of the start of
// the wave's own load ring once the wave has left the group loop.
template <int H>
struct MergeWave {
  float m[H];
  float l[H];
  float z[H][4];
  float o[H][TKV_D];
};

// ---- LDS plan (dynamic shared memory) ---------------------------------------------------
//   bk     per wave [hi/lo][H heads][68 words]: query-side operands of the next group
//   ring   per wave 3 K slots (codes, scalers) then 3 V slots (codes, scalers, zero-points);
//          the direct global->LDS loads put lane l's bytes at slot + 16*l (codes) or
//          slot + 4*l (fp16 rows), i.e. a slot is a copy of the group's packed block.  After
//          the main loop the start of a wave's ring holds its results for the workgroup merge.
//   cz     zero-point term of every group of the chunk, [group][H heads] float
// (a wave's bk area is its scratch for pieces of the fp16 tail before its first group, and for the
// merge weights after its last one)
// GS = quantization group / 32: the K scalers of a slot are those of the block's key group,
// the V scalers and zero-points [128 / (32 GS)][32 tokens] fp16 each.
template <int BITS, int GS, int W, int H>
struct Cfg {
  static constexpr int kThreads = 64 * W;
  static constexpr int kCode = 512 * BITS;  // bytes of K (or V) codes of one block
  static constexpr int kKPart = kCode + 256;
  static constexpr int kVPart = kCode + 512;
  static constexpr int oVs = kCode;                 // V scalers inside a V slot
  static constexpr int oVz = kCode + 256;           // V zero-points (GS = 2: 128 bytes each, and as many unused)
  static constexpr int kDepth = 3;
  static constexpr int kWaveRing = kDepth * (kKPart + kVPart);
  // direct-to-LDS load instructions per part: 1 bit = two 4-byte-per-lane loads of codes, else
  // 16-byte-per-lane loads; one load each for scalers and zero-points (GS = 2: V's by half of the lanes)
  static constexpr int kCodeLoads = BITS == 1 ? 2 : BITS / 2;
  static constexpr int kKLoads = kCodeLoads + 1;
  static constexpr int kVLoads = kCodeLoads + 2;
  static constexpr int kCodeWords = BITS == 1 ? 2 : 2 * BITS;  // code words per lane and part
  static constexpr int kBkWave = 2 * H * kBkStride * 4;
  static constexpr int kMaxGpc = max_gpc(H);
  static constexpr int oRing = W * kBkWave;
  static constexpr int oCz = oRing + W * kWaveRing;
  static constexpr int kLdsBytes = oCz + kMaxGpc * H * 4;
  static_assert(H * TKV_D * 4 <= kBkWave && (TKV_BLK + 1) * H * 4 <= kBkWave, "the tail's scratch fits in a wave's operand area");
  static_assert((W + 2) * H * 4 <= kBkWave, "so do the merge weights");
  static_assert(sizeof(MergeWave<H>) <= (size_t)kWaveRing, "a wave's results fit in its own ring");
  // chunk classes and loads in flight of the cross-chunk merge: one thread per item, 64 chunks in one round
  static constexpr int kMergeClasses = H == 4 ? 4 : W == 12 ? 3 : 2, kMergeLoads = H == 4 ? 16 : W == 12 ? 22 : 32;
  static_assert(tkv::merge_lds_floats(kMergeClasses, H, TKV_MAX_CHUNKS, kThreads) * 4 <= W * kWaveRing, "merge scratch must fit in the ring");
  static_assert(kLdsBytes + 64 <= 160 * 1024, "LDS budget of one compute unit");
};

// Column group whose column of acc_o[cb] counts: one that carries the weights of the block's
// channel group u = cb / (2 GS) (H = 8: u % 2; the other columns hold products with another u).
template <int GS, int H>
__device__ constexpr int owner_group(int cb) {
  return H == 4 ? cb / 2 : GS == 1 ? (cb / 2) % 2 : cb / 4;
}

// fp16 tail (the unquantized tokens): wave w of the last chunk takes the 32-token pieces w,
// w + W, ... and leaves its result as the state its block loop starts from: accumulators in the
// layout and units of the block loop (acc_o: channel rows of the column group that owns them, codes'
// 2^-24 and weights' 2^kEP included; acc_z: denominator) and their reference m_run, kTailRoomLog2
// under the largest logit.  The blocks' weights are fp16 and need a reference of their own: the first
// block sets it like any wave's first block does, kRefBelowMax under its largest logit, unless that
// is more than the room below the tail's.  With the tail's largest logit as the reference they lose
// their bits in fp16's subnormals wherever the recent tokens weigh most or the values are small (2 bit,
// 800 tokens, values of 1e-3: relative error 1.8e-3 to 3.7e-3, 3e-4 with their own).
//
// Everything runs on the matrix cores: the logits as K rows (A operand, straight from memory)
// against the exact fp16 query (the set-up's B operand), in the token order of a block's tiles;
// P.V in float32, on v_mfma_f32_4x4x1 for 4 heads (16 independent 4 heads x 4 channels products of
// one token each) and v_mfma_f32_16x16x4 for 8: either's B operand is one channel of one token per
// lane, so a lane's 16-byte piece of a V row feeds eight of them with no transpose, and the
// weights keep all their bits.  A wave is bound by
// the latency of its loads (16 in flight per lane) and then by some 300 instructions: 3.8 us from the
// set-up barrier at 2000 tokens, all pieces in parallel.  Plain float math with one token per lane
// pair and the weights broadcast lane by lane, on 4 waves, took 9 to 12.5 us, longer than
// everything else a workgroup had to do at up to 32768 tokens (2 bit, one sequence: 2000 tokens
// 18.0 -> 13.5 us per call, 8190 18.0 -> 14.4, 131060 30.3 -> 29.5; 64 sequences of 2000 62 -> 47).
//
// New tokens of the step are read from the caller's buffers: their ring rows are being written.
struct TailPiece {
  uintx4 kf[2][4];  // K rows as A operands of the two 16-token tiles
  uintx4 vf[8];     // V: channels 8 slot .. 8 slot + 7 of tokens 4 j + rb
};
struct TailRows {
  const char *k_ring, *v_ring, *k_new, *v_new;  // this head's rows
  uint32_t new_pitch;                           // bytes between a head's new rows
  int nq, n_old, n, s0, ring;
  __device__ TailRows(const MfmaParams& p, int b, int h, size_t bh, int nq_, int n_, int ring_) {
    nq = nq_, n = n_, ring = ring_;
    n_old = p.k_new != nullptr ? n - p.n_add.n[b] : n;
    s0 = nq % ring;  // ring slot of the tail's first token
    k_ring = reinterpret_cast<const char*>(p.k_resid + bh * ring * TKV_D);
    v_ring = reinterpret_cast<const char*>(p.v_resid + bh * ring * TKV_D);
    const size_t first = p.k_new != nullptr ? ((size_t)b * p.n_stride * p.hkv + h) * TKV_D : 0;
    k_new = reinterpret_cast<const char*>(p.k_new + first);
    v_new = reinterpret_cast<const char*>(p.v_new + first);
    new_pitch = (uint32_t)p.hkv * TKV_D * 2u;
  }
  __device__ const uintx4* row(const char* ring_rows, const char* new_rows, int tok, int lane_bytes) const {
    int s = s0 + (tok - nq);
    s = s >= ring ? s - ring : s;
    const bool old = tok < n_old;
    const uint32_t off = (old ? (uint32_t)s * (TKV_D * 2u) : (uint32_t)(tok - n_old) * new_pitch) + (uint32_t)lane_bytes;
    return reinterpret_cast<const uintx4*>((old ? ring_rows : new_rows) + off);
  }
  __device__ void load(TailPiece& t, int t0, int lane) const {
    const int slot = lane % 16, rb = lane / 16, cnt = min(32, n - t0);  // rows past the end re-read the last one with weight 0
#pragma unroll
    for (int tau = 0; tau < 2; ++tau) {
      const int y = 8 * (slot / 4) + 4 * tau + slot % 4;
      const uintx4* r = row(k_ring, k_new, t0 + min(y, cnt - 1), 16 * rb);
#pragma unroll
      for (int m = 0; m < 4; ++m) t.kf[tau][m] = r[4 * m];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) t.vf[j] = *row(v_ring, v_new, t0 + min(4 * j + rb, cnt - 1), 16 * slot);
  }
};

template <int BITS, int GS, int W, int H>
__device__ inline void tail_pieces(const TailRows& rows, float scale2, const uintx4 (&bq)[4], float* sc, int wave,
                                   int lane, floatx4 (&acc_o)[8], floatx4& acc_z, float& m_run) {
  const int slot = lane % 16, rb = lane / 16, hs = slot % H, us = slot / H;
  float L = 0.f;
  floatx4 acc[8];  // channel 8 slot + y; H = 4: tokens 4 j + rb, rows = heads; H = 8: rows = heads 4 (rb % 2) + x
#pragma unroll
  for (int y = 0; y < 8; ++y) acc[y] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int t0 = rows.nq + 32 * wave; t0 < rows.n; t0 += 32 * W) {
    const int cnt = min(32, rows.n - t0);
    TailPiece t;
    rows.load(t, t0, lane);
    __builtin_amdgcn_sched_barrier(0);  // all loads in flight before the first is used
    floatx4 s[2];
#pragma unroll
    for (int tau = 0; tau < 2; ++tau) {
      s[tau] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < 4; ++m) s[tau] = mfma(t.kf[tau][m], bq[m], s[tau]);
    }
    // this lane: head hs, tokens 8 rb + i (the same in all column groups)
    float x[8], mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[i] = 8 * rb + i < cnt ? s[i / 4][i % 4] * scale2 : -INFINITY;
      mx = fmaxf(mx, x[i]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // finite: the piece holds at least one token; a whole number, so that the room below is taken off exactly
    const float mn = ceilf(fmaxf(m_run, mx));
    const float alpha = __builtin_amdgcn_exp2f(m_run - mn);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[i] = __builtin_amdgcn_exp2f(x[i] - mn);
      sum += x[i];
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    L = __builtin_fmaf(L, alpha, sum);
    m_run = mn;
    // weights to [token][head]; a wave's LDS operations execute in order
    if (us == 0) {
#pragma unroll
      for (int i = 0; i < 8; ++i) sc[(8 * rb + i) * H + hs] = x[i];
      if (rb == 0) sc[TKV_BLK * H + hs] = alpha;
    }
    float w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = sc[(4 * j + rb) * H + lane % H];
    const floatx4 al = *reinterpret_cast<const floatx4*>(sc + TKV_BLK * H + (H == 4 ? 0 : 4 * (rb % 2)));
#pragma unroll
    for (int y = 0; y < 8; ++y) acc[y] *= al;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
#pragma unroll
      for (int y = 0; y < 8; ++y) {
        const uint32_t vw = t.vf[j][y / 2];
        const float vv = (float)as_half2(vw)[y % 2];
        acc[y] = H == 4 ? __builtin_amdgcn_mfma_f32_4x4x1f32(w[j], vv, acc[y], 0, 0, 0)
                        : __builtin_amdgcn_mfma_f32_16x16x4f32(w[j], vv, acc[y], 0, 0, 0);
      }
    }
  }
  if (H == 8) {
    if (rb < 2) {
#pragma unroll
      for (int y = 0; y < 8; ++y)
#pragma unroll
        for (int x = 0; x < 4; ++x) sc[(4 * rb + x) * TKV_D + 8 * slot + y] = acc[y][x];
    }
  } else {
  // sum over the four token classes rb: every exchange halves the values a lane keeps; in the end
  // it holds channels 8 slot + 2 rb', + 1 of the four heads (rb' = 2 (lane / 32) + (lane / 16) % 2)
  float v[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = acc[i / 4][i % 4];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v[i]), __builtin_bit_cast(uint32_t, v[i + 16]), false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    v[i] = __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, v[i]), __builtin_bit_cast(uint32_t, v[i + 8]), false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    v[i] = __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
  }
#pragma unroll
  for (int hh = 0; hh < 4; ++hh)
    *reinterpret_cast<float2_t*>(sc + hh * TKV_D + 8 * slot + 2 * rb) = float2_t{v[hh], v[4 + hh]};
  }
  constexpr float room = (float)(1ull << kTailRoomLog2);
#pragma unroll
  for (int cb = 0; cb < 8; ++cb) {
    const float scale = room / (float)(1 << (24 - kEP - (BITS == 1 && cb % 2 ? 4 : 0)));
    const floatx4 o = *reinterpret_cast<const floatx4*>(sc + hs * TKV_D + 16 * cb + 4 * rb) * scale;
    acc_o[cb] = owner_group<GS, H>(cb) == us ? o : floatx4{0.f, 0.f, 0.f, 0.f};
  }
  acc_z[0] = rb == 1 ? L * room : 0.f;
  m_run -= (float)kTailRoomLog2;
}

#ifdef TKV_PHASE
#define TKV_PH()                                \
  do {                                          \
    __builtin_amdgcn_sched_barrier(0);          \
    ph[ph_n++] = wall_clock64();                \
    __builtin_amdgcn_sched_barrier(0);          \
  } while (0)
#else
#define TKV_PH() \
  do {           \
  } while (0)
#endif

template <int BITS, int GS, int W, int H>
__global__ __launch_bounds__(64 * W) void quant_attn_mfma_kernel(MfmaParams p) {
  tkv::fetch_arguments<sizeof(MfmaParams)>();
  using C = Cfg<BITS, GS, W, H>;
  constexpr int KSH = GS - 1;          // key group of a block = block >> KSH
  constexpr int NU = 4 / GS;           // channel groups of a value row
  constexpr int GRP = TKV_BLK * GS;    // quantization group
  constexpr int NWORDS = TKV_D * BITS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_next;
  __shared__ uint32_t s_flag;
#ifdef TKV_PHASE
  long long ph[8];
  int ph_n = 0;
#endif
  TKV_PH();  // 0 kernel start

  // blockIdx.x counts the chunks of all sequences: which sequence, which of its chunks
  int b = 0, chunk = blockIdx.x, chunk_base = 0;
  while (b + 1 < p.batch && chunk >= p.chunks.n[b]) {
    chunk -= p.chunks.n[b];
    chunk_base += p.chunks.n[b];
    ++b;
  }
  const int n_chunks = p.chunks.n[b];
  const int part = (int)blockIdx.y & p.split;  // which four query heads of the group (only ever 1 where split is)
  const int h = (int)blockIdx.y >> p.split;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);  // wave-uniform: keeps group addresses scalar
  const int group = p.hq / p.hkv;
  const int G = p.split == 0 ? group : part == 0 ? 4 : group - 4;  // query heads of this workgroup, at most H
  const int qh0 = h * group + 4 * part;                            // the first of them
  const int n = p.lens.n[b];
  const int nq = tkv::n_quantized(n, p.residual, GRP);
  const int jq = nq / TKV_BLK;
  const size_t bh = (size_t)b * p.hkv + h;
  const size_t grp_base = bh * (size_t)(p.capacity / TKV_BLK);   // first packed block of this head
  const size_t kgrp_base = bh * (size_t)(p.capacity / GRP);      // first key group
  // Work split of this sequence: a 32-token piece of the tail counts as tail_blocks groups and the
  // tail belongs to the last chunk, which gets correspondingly fewer quantized groups.
  const bool has_tail = chunk == n_chunks - 1;
  // A group that the step's new tokens complete is quantized by the workgroup of the last chunk, which owns it.
  const int jq_old = p.complete == 0 ? jq : tkv::n_quantized(n - p.n_add.n[b], p.residual, GRP) / TKV_BLK;
  const int tail_equiv = p.tail_blocks * ((n - nq + 31) / 32) + (jq_old != jq ? kCompleteBlocks : 0);
  const uint32_t work = (uint32_t)(jq + tail_equiv);
  const int blk0 = min((int)(work * (uint32_t)chunk / (uint32_t)n_chunks), jq_old);
  const int blk1 = has_tail ? jq : min((int)(work * (uint32_t)(chunk + 1) / (uint32_t)n_chunks), jq_old);
  if (has_tail && jq_old != jq) {  // (GS blocks: the host sees to it that it is one group, of old tokens only)
    const int ring = p.residual + GRP;
    const size_t first = grp_base + jq_old, kgrp = kgrp_base + (jq_old >> KSH);
    const tkv::quantizer::GroupOut out = {
        const_cast<uint32_t*>(p.k_codes) + first * NWORDS,       const_cast<uint32_t*>(p.v_codes) + first * NWORDS,
        const_cast<__half*>(p.k_scale) + kgrp * TKV_D,           const_cast<__half*>(p.k_zero) + kgrp * TKV_D,
        const_cast<__half*>(p.v_scale) + first * (TKV_D / GS),   const_cast<__half*>(p.v_zero) + first * (TKV_D / GS)};
    static_assert(tkv::quantizer::group_lds(GRP) <= C::kLdsBytes, "LDS of the group");
    tkv::quantizer::quantize_group_block<BITS, GRP, 64 * W>(
        [&](int kv, int t) { return tkv::pick(kv != 0, p.k_resid, p.v_resid) + (bh * ring + (size_t)((jq_old * TKV_BLK + t) % ring)) * TKV_D; },
        out, smem, tid);
  }
  const int last = max(blk1 - 1, blk0);  // groups past the chunk are clamped (and ignored)

  const int slot = lane % 16, rb = lane / 16;
  const int hs = slot % H, us = slot / H;  // this lane's operand column: head, column group
  const __half* qrow = p.q + ((size_t)b * p.hq + (size_t)qh0) * TKV_D;
  typedef uint32_t BkArr[2][H][kBkStride];
  uint32_t(*bk_s)[H][kBkStride] = reinterpret_cast<BkArr*>(smem)[wave];
  float* cz_s = reinterpret_cast<float*>(smem + C::oCz);
  // Byte offsets (wave-uniform) of this wave's ring slots; the roles rotate every step.
  const uint32_t ring_off = C::oRing + wave * C::kWaveRing;
  const uint32_t lane16 = 16u * (uint32_t)lane, lane4 = 4u * (uint32_t)lane;  // unsigned: scalar base + 32-bit lane offset

  // ---- loads: asynchronous global -> LDS copies of a group's K part / V part ------------
  // Through descriptors of the head's arrays, block offsets scalar (as global loads, which the compiler takes for ones that may
  // return out of order, no load before them could be waited for without them).
  auto array_of = [&](const void* base, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000); };
  constexpr uint32_t kCodeBytes = NWORDS * 4, kVMetaBytes = TKV_D / GS * 2;  // of a block
  const auto k_codes = array_of(p.k_codes + grp_base * NWORDS, (uint32_t)jq * kCodeBytes);
  const auto v_codes = array_of(p.v_codes + grp_base * NWORDS, (uint32_t)jq * kCodeBytes);
  const auto k_scale = array_of(p.k_scale + kgrp_base * TKV_D, (uint32_t)(jq >> KSH) * (TKV_D * 2));
  const auto v_scale = array_of(p.v_scale + grp_base * (TKV_D / GS), (uint32_t)jq * kVMetaBytes);
  const auto v_zero = array_of(p.v_zero + grp_base * (TKV_D / GS), (uint32_t)jq * kVMetaBytes);
  const auto k_zero = array_of(p.k_zero + kgrp_base * TKV_D, (uint32_t)(jq >> KSH) * (TKV_D * 2));
  // the query rows of the workgroup's heads as MFMA B operand, exact (heads >= G re-read head G-1, in bounds; their results are not used)
  auto load_query_rows = [&](uintx4 (&to)[4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m)
      to[m] = *reinterpret_cast<const uintx4*>(qrow + (size_t)(hs < G ? hs : G - 1) * TKV_D + 32 * m + 8 * rb);
  };
  // GS = 2: 128 bytes each of V scalers and zero-points.  Lanes 32..63 read at kNone, past the end of any array (2^28 bytes at most,
  // 131072 blocks), where nothing is fetched; what they write to LDS is not used.  (With a lane mask around either load the compiler
  // counts them as loads that may not have been issued, and waits for others in their place.  us per call so / now, 2 bit, 32/8 heads,
  // 98413 tokens 22.6, 22.3; 64/8 27.4, 26.9; 32/8, 131071 25.5, 25.2; 2000 10.5, 10.4.)
  constexpr uint32_t kNone = 0x80000000u;
  const uint32_t lane4_meta = GS == 1 || lane < 32 ? lane4 : kNone;
  auto load_codes = [&](unsigned char* s, auto codes, uint32_t at) {
    if (BITS == 1) {
      buffer_to_lds<4>(codes, s, lane4, at);
      buffer_to_lds<4>(codes, s + 256, lane4, at + 256);
    } else {
#pragma unroll
      for (int x = 0; x < BITS / 2; ++x) buffer_to_lds<16>(codes, s + 1024 * x, lane16, at + 1024 * x);
    }
  };
  auto load_kpart = [&](uint32_t so, int g) {
    const uint32_t gi = (uint32_t)min(g, last);
    unsigned char* s = smem + so;
    load_codes(s, k_codes, gi * kCodeBytes);
    buffer_to_lds<4>(k_scale, s + C::kCode, lane4, (gi >> KSH) * (TKV_D * 2));
  };
  auto load_vpart = [&](uint32_t so, int g) {
    const uint32_t gi = (uint32_t)min(g, last);
    unsigned char* s = smem + so;
    load_codes(s, v_codes, gi * kCodeBytes);
    buffer_to_lds<4>(v_scale, s + C::oVs, lane4_meta, gi * kVMetaBytes);
    buffer_to_lds<4>(v_zero, s + C::oVz, lane4_meta, gi * kVMetaBytes);
  };

  // The first three groups of a wave are fixed (wave, wave + W, wave + 2W), the rest come
  // from the workgroup's counter: their loads can start before anything else is set up.
  // ring roles: kq = K part the next QK reads, kk = K part whose scalers are prepared next,
  // kl = K slot being loaded; vp = V part of the current group, vn = the one after, vl = V
  // slot being loaded
  uint32_t kl = ring_off, kq = ring_off + C::kKPart, kk = ring_off + 2 * C::kKPart;
  uint32_t vp = ring_off + 3 * C::kKPart, vn = vp + C::kVPart, vl = vp + 2 * C::kVPart;
  const int g0 = blk0 + wave;
  int g1 = g0 + W, g2 = g0 + 2 * W;
  const bool active = g0 < blk1;
  const int ng = blk1 - blk0;
  // Eq. 2 in this launch: the step's new rows go into the fp16 ring, into slots whose tokens were
  // quantized long ago.  Nothing in this launch reads those slots: the tail waves take the new
  // rows from the caller's buffers.
  const int n_copy = has_tail && p.k_new != nullptr ? 32 * p.n_add.n[b] : 0;  // 16-byte pieces
  auto new_piece = [&](int x) -> const uintx4* {
    return reinterpret_cast<const uintx4*>(tkv::pick(x % 32 >= 16, p.k_new, p.v_new) + (((size_t)b * p.n_stride + x / 32) * p.hkv + h) * TKV_D) + x % 16;
  };
  auto ring_piece = [&](int x) -> uintx4* {
    const int ring = p.residual + GRP, add = p.n_add.n[b];
    const __half* to = tkv::pick(x % 32 >= 16, p.k_resid, p.v_resid) + (bh * ring + (size_t)((n - add + x / 32) % ring)) * TKV_D;
    return reinterpret_cast<uintx4*>(const_cast<__half*>(to)) + x % 16;
  };
  if (tid == 0) s_next = blk0 + 3 * W;
  float scale2 = p.scale2;
  asm volatile("" : "+s"(scale2));  // (else it is fetched anew before each of zero_terms' products)
  // Set-up loads, then the ring prologue behind them: one memory round trip covers both.  Only waves that have blocks load, and of
  // them only those that work out zero-point terms wait in front of the barrier: wave 0, up to 16 blocks.  No set-up load is in flight
  // where a path without it joins (hence the tail's own load of the query rows): there the compiler would wait for loads behind
  // it too, and the block loop would begin when the whole ring is full, 28 MB for a launch of 256 workgroups.  us per call, first with
  // that, then with the set-up loads in every wave and a wait for them in front of the barrier, then so (a call of 2 bit, 2000
  // tokens passes the barrier 1.8, 2.5 and 1.5 us after its start; of 2 / 64, 131071 tokens 3.8, 4.2 and 3.3), 32/8 heads: 2 bit, 2000 tokens
  // 10.9, 11.2, 10.4; 131071 27.2, 26.1, 26.0; 4 bit, 2000 10.4, 10.5, 9.9; 2 / 64, 16 x 300 10.2, 10.6, 10.1; 2000 10.9, 11.2, 10.5;
  // 131071 26.3, 26.1, 25.6; 1 / 64, 32/4 heads, 98413 21.9, 21.9, 21.4.
  uint32_t q2[H];  // K-prep role: this lane owns channels 2*lane, 2*lane+1
  if (active) {
    uintx4 copied;
    if (tid < n_copy) copied = *new_piece(tid);
#pragma unroll
    for (int hh = 0; hh < H; ++hh)
      q2[hh] = reinterpret_cast<const uint32_t*>(qrow + (size_t)(hh < G ? hh : G - 1) * TKV_D)[lane];
    const bool zero_point_wave = 16 * wave < ng;  // (a wave without blocks has no groups either)
    uintx4 bq[4];  // exact fp16 query as MFMA B operand
    uintx4 az[4];  // zero-point rows of 16 groups as MFMA A operand
    auto load_az = [&](int t0) {
      const uint32_t at = (uint32_t)(min(blk0 + t0 + slot, last) >> KSH) * (TKV_D * 2) + 16u * (uint32_t)rb;
#pragma unroll
      for (int m = 0; m < 4; ++m) az[m] = __builtin_amdgcn_raw_buffer_load_b128(k_zero, at + 64u * m, 0, 0);
    };
    if (zero_point_wave) {
      load_query_rows(bq);
      load_az(16 * wave);
    }
    __builtin_amdgcn_sched_barrier(0);
    // issue order K0 V0 K1 K2 V1, then per step [K(i+3) V(i+2)]: the counter retires loads
    // in order, so "at most N outstanding" names exactly which parts have landed
    load_kpart(kl, g0);
    load_vpart(vp, g0);
    load_kpart(kq, g1);
    load_kpart(kk, g2);
    load_vpart(vn, g1);
    __builtin_amdgcn_sched_barrier(0);
    // ---- zero-point term of every group of the chunk: cz[g][head] = scale2 * sum_c q[c] z_g[c],
    // 16 groups per MFMA (A rows = groups, B = the exact fp16 query).  Column groups hold the same numbers, and there is room up
    // to the next multiple of 16 groups: written without a condition.
    static_assert(C::kMaxGpc % 16 == 0, "room of the last 16 groups");
    auto zero_terms = [&](int t0) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < 4; ++m) acc = mfma(az[m], bq[m], acc);
#pragma unroll
      for (int x = 0; x < 4; ++x) cz_s[(t0 + 4 * rb + x) * H + hs] = acc[x] * scale2;
    };
    if (zero_point_wave) {
      zero_terms(16 * wave);
      for (int t0 = 16 * (wave + W); t0 < ng; t0 += 16 * W) {
        load_az(t0);
        zero_terms(t0);
      }
    }
    if (tid < n_copy) *ring_piece(tid) = copied;
  } else if (tid < n_copy) {
    *ring_piece(tid) = *new_piece(tid);
  }
  for (int x = tid + 64 * W; x < n_copy; x += 64 * W) *ring_piece(x) = *new_piece(x);
  TKV_PH();  // 1 this wave's set-up work done
  // cz table and group counter are in place (a bare barrier: __syncthreads() would also wait for
  // every load in flight)
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  TKV_PH();  // 2 set-up done

  // Next group index from the workgroup's LDS counter.  Written as inline assembly: the
  // compiler orders every LDS atomic it knows of behind all outstanding direct-to-LDS
  // loads (vmcnt(0)), which would drain the prefetch ring at every step.
  const uint32_t next_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)&s_next;
  auto grab = [&]() -> int {
    int v = 0;
    if (lane == 0) {
      const int one = 1;
      asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(next_addr), "v"(one) : "memory");
    }
    return __builtin_amdgcn_readfirstlane(v);
  };

  // state of the block loop: accumulators and the head's softmax reference
  floatx4 acc_o[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc_o[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  floatx4 acc_z = {0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY;
  if (has_tail && wave * 32 < n - nq) {
    uintx4 bq[4];
    load_query_rows(bq);
    tail_pieces<BITS, GS, W, H>(TailRows(p, b, h, bh, nq, n, p.residual + GRP), p.scale2, bq,
                                reinterpret_cast<float*>(smem) + wave * (C::kBkWave / 4), wave, lane, acc_o, acc_z, m_run);
  }
  TKV_PH();  // 3 tail done

  // codes carry 2^-24, query side 2^kEK, so S = acc * 2^(24-kEK)
  const float K1 = p.scale2 * (float)(1 << (24 - kEK));

  // A operand of the z_v / denominator MFMA: rows 0..NU-1 hold z_v[u = row] (loaded per group)
  // times the constant that undoes the weight-side scaling, row 4 holds that constant
  // alone (denominator), the other rows are zero.  Built branch-free as load * zmul + zadd.
  const int zrow = slot;                          // as A operand this lane holds row `slot`
  const int zrow_ld = zrow < NU ? zrow : NU - 1;  // other rows load a valid row and multiply it by 0
  half2_t zmul[4], zadd[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    // element k = 2j + e of this lane carries 2^-kEP * (2^j | 4^j | 16^(j%2))
    const int fs = BITS == 1 ? j : BITS == 2 ? 2 * j : 4 * (j % 2);
    const float w = (float)(1 << fs) / (float)(1 << kEP);
    const _Float16 wm = (_Float16)(zrow < NU ? w : 0.f), wa = (_Float16)(zrow == 4 ? w : 0.f);
    zmul[j] = half2_t{wm, wm};
    zadd[j] = half2_t{wa, wa};
  }
  // exponent offsets that put 2^kEP / (2^j | 4^j | 16^(j%2)) into the weights; value i of the
  // lane (tile tau = i/4, row x = i%4) is element kappa = 4 tau + x, register j = kappa/2
  float off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int j = i / 2;
    off[i] = BITS == 1 ? (float)(kEP - j) : BITS == 2 ? (float)(kEP - 2 * j) : (float)(kEP - 4 * (j % 2));
  }

  float qf[H][2];  // query times the factor that undoes the field position of this lane's channels (set before the first group)

  // ---- pipeline stages of one group.  Every stage is split into its LDS reads and its
  // arithmetic, so that a step can issue the reads well ahead of their use (a wave issues in
  // order: a read that is waited for right away stalls it for the whole LDS latency).
  // K: scalers x query -> hi/lo operands in LDS
  auto read_ks = [&](uint32_t so) -> uint32_t {
    return *reinterpret_cast<const uint32_t*>(smem + so + C::kCode + lane4);
  };
  auto stage_k = [&](uint32_t ks2) {
#pragma unroll
    for (int hh = 0; hh < H; ++hh) {
      const uint32_t hi = mix_hi_pair(qf[hh][0], qf[hh][1], ks2);  // products are exact in float32
      bk_s[0][hh][lane] = hi;
      bk_s[1][hh][lane] = mix_lo_pair(qf[hh][0], qf[hh][1], ks2, hi);
    }
  };
  // QK: partial logits of the group's 32 tokens (two 16-token tiles); even column groups
  // read the hi rows of the query-side operand, odd ones the lo rows
  const uint32_t* bk_row = &bk_s[us & 1][hs][4 * rb];
  struct QkIn {
    uint32_t kw[C::kCodeWords];
    uintx4 bk[4];
  };
  auto read_codes = [&](const unsigned char* s, uint32_t (&cw)[C::kCodeWords]) {
    if (BITS == 1) {
      cw[0] = *reinterpret_cast<const uint32_t*>(s + lane4);
      cw[1] = *reinterpret_cast<const uint32_t*>(s + 256 + lane4);
    } else {
#pragma unroll
      for (int x = 0; x < BITS / 2; ++x) {
        const uintx4 t = *reinterpret_cast<const uintx4*>(s + 1024 * x + lane16);
#pragma unroll
        for (int y = 0; y < 4; ++y) cw[4 * x + y] = t[y];
      }
    }
  };
  auto read_qk = [&](uint32_t so, QkIn& in) {
    read_codes(smem + so, in.kw);
#pragma unroll
    for (int m = 0; m < 4; ++m) in.bk[m] = *reinterpret_cast<const uintx4*>(bk_row + 16 * m);
  };
  auto stage_qk = [&](const QkIn& in, floatx4 (&acc_s)[2]) {
    acc_s[0] = floatx4{0.f, 0.f, 0.f, 0.f};
    acc_s[1] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (BITS == 1) {
#pragma unroll
      for (int tau = 0; tau < 2; ++tau) {
        uintx4 a[4];
        extract1(in.kw[tau], a);
#pragma unroll
        for (int m = 0; m < 4; ++m) acc_s[tau] = mfma(a[m], in.bk[m], acc_s[tau]);
      }
      return;
    }
#pragma unroll
    for (int m2 = 0; m2 < 2; ++m2) {  // pairs of MFMA steps m = 2*m2, 2*m2+1
#pragma unroll
      for (int tau = 0; tau < 2; ++tau) {
        uintx4 a[2];
        if (BITS == 2) {
          extract2(in.kw[(2 * tau + m2) % C::kCodeWords], a[0], a[1]);
        } else {
          extract4(in.kw[(4 * tau + 2 * m2) % C::kCodeWords], a[0]);
          extract4(in.kw[(4 * tau + 2 * m2 + 1) % C::kCodeWords], a[1]);
        }
#pragma unroll
        for (int y = 0; y < 2; ++y) acc_s[tau] = mfma(a[y], in.bk[2 * m2 + y], acc_s[tau]);
      }
    }
  };
  // weights and weight-side operands
  constexpr bool kTwoSets = H == 8 && GS == 1;  // weights for u = 0, 1 and for u = 2, 3
  struct PvIn {
    uintx4 sv, sv2, zv;
    uint32_t vw[C::kCodeWords];
    float cz;
  };
  auto read_pv = [&](uint32_t so, int gc, PvIn& in) {
    const unsigned char* s = smem + so;
    in.sv = *reinterpret_cast<const uintx4*>(s + C::oVs + ((H == 4 ? us / GS : us) * TKV_BLK + 8 * rb) * 2);
    if (kTwoSets) in.sv2 = *reinterpret_cast<const uintx4*>(s + C::oVs + ((2 + us) * TKV_BLK + 8 * rb) * 2);
    in.zv = *reinterpret_cast<const uintx4*>(s + C::oVz + (zrow_ld * TKV_BLK + 8 * rb) * 2);
    read_codes(s, in.vw);
    in.cz = cz_s[(gc - blk0) * H + hs];
  };
  struct POps {
    uintx4 b2, bp, a_zv;
    uintx4 b3;  // kTwoSets: the weights for u = 2, 3
  };
  // The weights 2^(x - m_run) go to the matrix cores as fp16, so m_run (a per-head reference,
  // not necessarily the running maximum) only has to keep them below 2^kHeadroomLog2: that
  // is checked on the weights themselves (an integer maximum of their bit patterns), and
  // only a failed check (rare after the first groups) pays for the exact maximum, the
  // accumulator rescale and a second pass.
  auto stage_soft = [&](const PvIn& in, const floatx4 (&acc_s)[2], POps& o) {
    const float cz = in.cz;
    float xs[8];  // hi + lo partial sums: every lane of a head ends up with the full logit
#pragma unroll
    for (int x = 0; x < 8; ++x) xs[x] = ror_add<H>(acc_s[x / 4][x % 4]);
    float pw[8];
    auto weights = [&]() {
      const float czm = cz - m_run;
#pragma unroll
      for (int x = 0; x < 8; ++x) pw[x] = __builtin_amdgcn_exp2f(__builtin_fmaf(xs[x], K1, czm + off[x]));
    };
    weights();
    {
      // bit patterns of non-negative floats (and of inf / NaN) order like integers
      uint32_t mm = 0u;
#pragma unroll
      for (int x = 0; x < 8; ++x) mm = max(mm, __builtin_bit_cast(uint32_t, pw[x]));
      constexpr uint32_t kLimit = (uint32_t)(127 + kEP + kHeadroomLog2) << 23;  // 2^(kEP + headroom)
      if (__builtin_amdgcn_ballot_w64(mm >= kLimit) != 0ull) {
        const float mx = fmaxf(fmaxf(fmaxf(xs[0], xs[1]), fmaxf(xs[2], xs[3])), fmaxf(fmaxf(xs[4], xs[5]), fmaxf(xs[6], xs[7])));
        float mn = __builtin_fmaf(mx, K1, cz);  // largest logit among this lane's 8 tokens
        // over the lanes that hold other tokens of the same head (the column groups of a head hold the
        // same logits, and its neighbours in the row of 16 lanes are other heads)
        mn = fmaxf(mn, __shfl_xor(mn, 16, 64));
        mn = fmaxf(mn, __shfl_xor(mn, 32, 64));
        // New reference: kRefBelowMax under the head's largest logit (never lower than before).
        // The largest weight is then 2^kRefBelowMax and the many small ones, which carry most of
        // the mass in a long context, sit that much further inside fp16's normal range.
        mn = fmaxf(m_run, mn - (float)kRefBelowMax);
        const float alpha = exp2f(m_run - mn);  // 0 on the first group
#pragma unroll
        for (int i = 0; i < 8; ++i) acc_o[i] *= alpha;
        acc_z *= alpha;
        m_run = mn;
        weights();
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float2_t w2 = {pw[2 * j], pw[2 * j + 1]};
      o.bp[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(w2, half2_t));
      const uint32_t bpj = o.bp[j], svj = in.sv[j], zvj = in.zv[j];
      // weight x scaler: one rounding of the exact product of two fp16 numbers
      o.b2[j] = __builtin_bit_cast(uint32_t, as_half2(bpj) * as_half2(svj));
      if (kTwoSets) {
        const uint32_t sv2j = in.sv2[j];
        o.b3[j] = __builtin_bit_cast(uint32_t, as_half2(bpj) * as_half2(sv2j));
      }
      const half2_t t = __builtin_elementwise_fma(as_half2(zvj), zmul[j], zadd[j]);
      o.a_zv[j] = __builtin_bit_cast(uint32_t, t);
    }
  };
  // P.V: 8 blocks of 16 channels + the z_v / denominator MFMA
  auto stage_pv = [&](const PvIn& in, const POps& o) {
    acc_z = mfma(o.a_zv, o.bp, acc_z);
    auto block = [&](int cb, uintx4 a) {
      const bool second = kTwoSets && cb >= 4;
      acc_o[cb] = mfma(a, second ? o.b3 : o.b2, acc_o[cb]);
    };
    if (BITS == 1) {
#pragma unroll
      for (int wd = 0; wd < 2; ++wd) {
        uintx4 a[4];
        extract1(in.vw[wd], a);
#pragma unroll
        for (int y = 0; y < 4; ++y) block(4 * wd + y, a[y]);
      }
      return;
    }
#pragma unroll
    for (int wd = 0; wd < 4; ++wd) {
      uintx4 a[2];
      if (BITS == 2) {
        extract2(in.vw[wd % C::kCodeWords], a[0], a[1]);
      } else {
        extract4(in.vw[((wd / 2) * 4 + 2 * (wd % 2)) % C::kCodeWords], a[0]);
        extract4(in.vw[((wd / 2) * 4 + 2 * (wd % 2) + 1) % C::kCodeWords], a[1]);
      }
#pragma unroll
      for (int y = 0; y < 2; ++y) block(2 * wd + y, a[y]);
    }
  };
#define TKV_WAIT_VMCNT(N) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory")
  constexpr int L = C::kKLoads + C::kVLoads;  // load instructions issued per pipeline step

  // ---- software pipeline over this wave's groups g[0], g[1], ...  Step i computes the
  // logits of group i+1, the weights and P.V of group i and the query-side operand of
  // group i+2, while the K part of group i+3 and the V part of group i+2 are in flight.
  if (active) {
    floatx4 acc_a[2], acc_b[2];
    TKV_WAIT_VMCNT(2 * C::kKLoads + C::kVLoads);  // K0, V0 landed
    // (1 bit: 2^(lane%4), times 2^4 in odd 32-channel blocks; 2 bit: 4^(lane%4); 4 bit: 16^(lane%2))
    const int shift = BITS == 1 ? lane % 4 + 4 * ((lane / 16) % 2) : BITS == 2 ? 2 * (lane % 4) : 4 * (lane % 2);
    const float comp = (float)(1 << kEK) / (float)(1 << shift);
#pragma unroll
    for (int hh = 0; hh < H; ++hh) {
      const half2_t qq = as_half2(q2[hh]);
      qf[hh][0] = hh < G ? (float)qq[0] * comp : 0.f;
      qf[hh][1] = hh < G ? (float)qq[1] * comp : 0.f;
    }
    stage_k(read_ks(kl));
    {
      QkIn qi;
      read_qk(kl, qi);
      stage_qk(qi, acc_a);
    }
    TKV_WAIT_VMCNT(L);  // + K1
    stage_k(read_ks(kq));
    // One step is one straight-line block; groups past the chunk are clamped copies whose
    // results are dropped by leaving the loop.  gc = group i (valid), gn3 / gv2 = groups
    // whose K / V part is fetched now.  LDS reads go out one stage ahead of their use.
    auto step = [&](int gc, int gn3, int gv2, floatx4 (&acc_c)[2], floatx4 (&acc_n)[2]) {
      QkIn qi;
      read_qk(kq, qi);  // K(i+1) landed during the previous step
      __builtin_amdgcn_sched_barrier(0);
      load_kpart(kl, gn3);
      load_vpart(vl, gv2);
      TKV_WAIT_VMCNT(2 * L);  // K(i+1), V(i) landed
      PvIn pi;
      read_pv(vp, gc, pi);
      __builtin_amdgcn_sched_barrier(0);
      stage_qk(qi, acc_n);
      POps po;
      stage_soft(pi, acc_c, po);
      TKV_WAIT_VMCNT(L + C::kVLoads);  // + K(i+2)
      const uint32_t ks2 = read_ks(kk);
      __builtin_amdgcn_sched_barrier(0);
      stage_pv(pi, po);
      stage_k(ks2);
      uint32_t t = kq;
      kq = kk, kk = kl, kl = t;
      t = vp;
      vp = vn, vn = vl, vl = t;
    };
    int gc = g0;
    for (;;) {
      const int g3 = grab();
      step(gc, g3, g2, acc_a, acc_b);
      if (g1 >= blk1) break;
      const int g4 = grab();
      step(g1, g4, g3, acc_b, acc_a);
      if (g2 >= blk1) break;
      gc = g2;  // rotate: group i+2 becomes the current one
      g1 = g3;
      g2 = g4;
    }
  }
#undef TKV_WAIT_VMCNT
  TKV_PH();  // 4 this wave's groups done
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no direct-to-LDS load may land after the ring is reused

  // ---- per-wave results -> LDS, each wave into its own (now idle) ring, so no wave waits for
  // another before writing.  acc_z rows: lanes 0..15 (rb 0) hold rows 0..3 = z-terms for
  // u = row; lanes 16..31 register 0 hold row 4 = denominator.
  auto merge_of = [&](int w) -> MergeWave<H>& {
    return *reinterpret_cast<MergeWave<H>*>(smem + C::oRing + w * C::kWaveRing);
  };
  MergeWave<H>& mw = merge_of(wave);
  if (rb == 0 && us == 0) {
#pragma unroll
    for (int x = 0; x < NU; ++x) mw.z[hs][x] = acc_z[x];
    mw.m[hs] = m_run;
  }
  if (rb == 1 && us == 0) mw.l[hs] = acc_z[0];
#pragma unroll
  for (int cb = 0; cb < 8; ++cb) {
    // 1 bit: the codes of odd 16-channel blocks sit four mantissa bits higher
    const float unscale = (float)(1 << (24 - kEP - (BITS == 1 && cb % 2 ? 4 : 0)));
    if (owner_group<GS, H>(cb) == us) {
      // written by lanes of this same wave just above: a wave's LDS operations execute in order
      const float zt = mw.z[hs][cb / (2 * GS)];
      *reinterpret_cast<floatx4*>(&mw.o[hs][16 * cb + 4 * rb]) = acc_o[cb] * unscale + zt;
    }
  }
  __syncthreads();
  TKV_PH();  // 5 all waves done, results in LDS
  // merge weights of the W wave entries: every wave works them out for itself (lane = (entry,
  // head)) into scratch of its own, which spares the workgroup a barrier
  float(*s_w)[H] = reinterpret_cast<float(*)[H]>(smem + wave * C::kBkWave);  // [W]
  float(*s_ml)[H] = s_w + W;                                                  // [2]: maximum, sum
  {
    constexpr int EP = 64 / H, NP = (W + EP - 1) / EP;  // entries per pass, passes
    const int hh = lane % H;
    float me[NP], le[NP], M = -INFINITY, Lsum = 0.f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int e = lane / H + EP * i;
      me[i] = e < W ? merge_of(e).m[hh] : -INFINITY;
      le[i] = e < W ? merge_of(e).l[hh] : 0.f;
      M = fmaxf(M, me[i]);
    }
    M = tkv::over_stride<H>(M, tkv::MaxOf{});
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int e = lane / H + EP * i;
      const float wgt = me[i] == -INFINITY ? 0.f : exp2f(me[i] - M);
      Lsum = __builtin_fmaf(le[i], wgt, Lsum);
      if (e < W) s_w[e][hh] = wgt;
    }
    Lsum = tkv::over_stride<H>(Lsum, tkv::SumOf{});
    if (lane < H) {
      s_ml[0][hh] = M;
      s_ml[1][hh] = Lsum;
    }
  }
  static_assert(C::kThreads >= H * TKV_D / 2, "two channels per thread");
  if (tid < G * TKV_D / 2) {
    const int hh = tid / (TKV_D / 2), c = 2 * (tid % (TKV_D / 2));
    float2_t O = {0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) O += *reinterpret_cast<const float2_t*>(&merge_of(w).o[hh][c]) * s_w[w][hh];
    if (n_chunks == 1) {  // nothing to merge with
      const float Lsum = s_ml[1][hh];
      const float inv0 = Lsum > 0.f ? O[0] / Lsum : 0.f, inv1 = Lsum > 0.f ? O[1] / Lsum : 0.f;
      *reinterpret_cast<uint32_t*>(p.out + ((size_t)b * p.hq + (size_t)qh0 + hh) * TKV_D + c) = pack2((_Float16)inv0, (_Float16)inv1);
    } else {
      float* head = p.parts + ((size_t)chunk_base * p.hq + ((size_t)qh0 + hh) * n_chunks) * TKV_PART_STRIDE;
      // device-scope stores: visible to the merging workgroup without a cache write-back
      auto store2 = [](float* at, float2_t v) {
        __hip_atomic_store(reinterpret_cast<uint64_t*>(at), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      store2(tkv::part_o(head, chunk) + c, O);
      if (c == 0) store2(tkv::part_ml(head, n_chunks, chunk), float2_t{s_ml[0][hh], s_ml[1][hh]});
    }
  }

  if (n_chunks == 1) return;
  // ---- the last workgroup of this (sequence, KV head) to arrive merges all chunks.
  // Partials travel through device-scope (cache-bypassing) stores and loads, ordered by
  // waiting for the stores to complete before the arrival counter is bumped: a release /
  // acquire fence pair would write back and invalidate the whole L2 (tens of microseconds).
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  TKV_PH();  // 6 partial written
  __syncthreads();
  uint32_t* arrival = p.arrivals + (size_t)b * gridDim.y + blockIdx.y;
  if (tid == 0) s_flag = atomicAdd(arrival, 1u) == (uint32_t)(n_chunks - 1) ? 1u : 0u;
  __syncthreads();
  if (s_flag != 0u) {
    if (tid == 0) *arrival = 0u;
    const float* head0 = p.parts + ((size_t)chunk_base * p.hq + (size_t)qh0 * n_chunks) * TKV_PART_STRIDE;
    float* scratch = reinterpret_cast<float*>(smem + C::oRing);  // the waves' results have been consumed
    tkv::merge_chunks<C::kMergeClasses, C::kMergeLoads>(head0, G, n_chunks, p.out + ((size_t)b * p.hq + (size_t)qh0) * TKV_D, scratch, tid, C::kThreads);
  }
  TKV_PH();  // 7 end
#ifdef TKV_PHASE
  if (p.prof && lane == 0) {
    long long* dst = p.prof + ((size_t)(blockIdx.y * gridDim.x + blockIdx.x) * W + wave) * 8;
    for (int i = 0; i < 8; ++i) dst[i] = ph[i];
  }
#endif
}

template <int BITS, int GS, int W, int H>
int32_t launch_heads(const MfmaParams& p, dim3 grid, hipStream_t s) {
  using C = Cfg<BITS, GS, W, H>;
  // more than 64 KiB of dynamic LDS needs an opt-in, once per kernel
  static const bool lds_ok =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&quant_attn_mfma_kernel<BITS, GS, W, H>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes) == hipSuccess;
  if (!lds_ok) return TKV_E_HIP;
  TKV_LAUNCH((quant_attn_mfma_kernel<BITS, GS, W, H>), grid, C::kThreads, C::kLdsBytes, s, p);
  return TKV_OK;
}
template <int BITS, int GS, int W>
int32_t launch_variant(const MfmaParams& p, dim3 grid, hipStream_t s) {
  return p.hq / p.hkv <= 4 || p.split != 0 ? launch_heads<BITS, GS, W, 4>(p, grid, s) : launch_heads<BITS, GS, W, 8>(p, grid, s);
}

}  // namespace

namespace tkv {
#ifdef TKV_PHASE
void* g_mfma_prof = nullptr;
#endif

// Chunks per (sequence, KV head): about `target_blocks` workgroups in total (one per
// compute unit), at least one 32-token block per wave, and no more blocks per chunk than
// the zero-point table of a workgroup holds.
int32_t launch_quant_attn_mfma(const tkv_quant_desc* d, const tkv_quant_cache* c, const __half* q, __half* out,
                               float scale2, float* parts, size_t parts_floats, uint32_t* arrivals, int target_blocks,
                               const TkvSeqLens& lens, const QuantNewTokens* fresh, hipStream_t s) {
  if (d->head_dim != TKV_D) return TKV_E_UNSUPPORTED;
  const int variant = d->bits * 100 + d->group_size;
  const int waves = d->bits == 4 ? 8 : 12;
  auto most_chunks = [waves](int blocks) { return blocks <= kOneChunkRounds * waves ? 1 : (blocks + waves - 1) / waves; };
  // Chunks per KV head over the whole batch: about target_blocks workgroups in all, shared out
  // among the sequences in proportion to their work (32-token blocks, a 32-token piece of the
  // fp16 tail counting as kTailBlocks), so that every workgroup sweeps about the same number of blocks
  // whatever the mix of lengths.  Per sequence: at least one block per wave, at most 64 chunks
  // (unless the tuning hook asks for more workgroups than that gives), no more blocks per chunk
  // than the zero-point table of a workgroup holds.
  MfmaParams p;
  int heads = 0, total_chunks = 0;
  long long total_work = 0;
  auto plan = [&](int split, int tail_blocks) -> int32_t {
    const int kMaxGpc = max_gpc(split ? 4 : d->n_q_heads / d->n_kv_heads);
    p.split = split;
    p.tail_blocks = tail_blocks;
    heads = d->n_kv_heads << split;
    int per_head = (target_blocks + heads - 1) / heads;
    if (per_head < d->batch) per_head = d->batch;
    const int chunk_cap = target_blocks > 64 * d->batch * heads ? TKV_MAX_CHUNKS : 64;
    total_work = 0;
    int work[TKV_MAX_BATCH], extra[TKV_MAX_BATCH];  // extra: a group that this launch quantizes, for the tail's workgroup
    for (int b = 0; b < d->batch; ++b) {
      const int n = lens.n[b];
      const int g = tkv::n_quantized(n, d->residual, d->group_size) / TKV_BLK;
      extra[b] = fresh != nullptr && fresh->complete &&
                         g != tkv::n_quantized(n - fresh->n_add.n[b], d->residual, d->group_size) / TKV_BLK
                     ? kCompleteBlocks
                     : 0;
      work[b] = g + tail_blocks * ((n - g * TKV_BLK + 31) / 32) + extra[b];
      total_work += work[b];
    }
    total_chunks = 0;
    for (int b = 0; b < d->batch; ++b) {
      int nc = total_work > 0 ? (int)(((long long)per_head * work[b] + total_work / 2) / total_work) : 1;
      const int c_work = most_chunks(work[b] - extra[b]);
      if (nc > c_work) nc = c_work;
      if (nc > chunk_cap) nc = chunk_cap;
      if (nc < 1) nc = 1;
      if ((work[b] + nc - 1) / nc > kMaxGpc) nc = (work[b] + kMaxGpc - 1) / kMaxGpc;
      if (nc > TKV_MAX_CHUNKS) return TKV_E_UNSUPPORTED;
      p.chunks.n[b] = nc;
      total_chunks += nc;
    }
    // Rounding may leave a few chunks too many (a second round of workgroups for a handful of
    // them) or too few (idle compute units): take them from the sequences whose chunks are the
    // lightest, give them to those whose chunks are the heaviest.
    while (total_chunks > per_head) {
      int pick = -1;
      for (int b = 0; b < d->batch; ++b) {
        const int nc = p.chunks.n[b];
        if (nc <= 1 || (work[b] + nc - 2) / (nc - 1) > kMaxGpc) continue;
        if (pick < 0 || (long long)work[b] * (p.chunks.n[pick] - 1) < (long long)work[pick] * (nc - 1)) pick = b;
      }
      if (pick < 0) break;
      --p.chunks.n[pick];
      --total_chunks;
    }
    while (total_chunks < per_head) {
      int pick = -1;
      for (int b = 0; b < d->batch; ++b) {
        const int nc = p.chunks.n[b];
        if (nc >= chunk_cap || nc >= most_chunks(work[b] - extra[b])) continue;
        if (pick < 0 || (long long)work[b] * p.chunks.n[pick] > (long long)work[pick] * nc) pick = b;
      }
      if (pick < 0) break;
      ++p.chunks.n[pick];
      ++total_chunks;
    }
    if ((size_t)total_chunks * d->n_q_heads * TKV_PART_STRIDE > parts_floats) return TKV_E_WORKSPACE;
    return TKV_OK;
  };
  // Groups of 5 to 8 query heads go to one workgroup, or to two of up to 4 heads that each read the
  // codes (twice the unpacking, half the operand preparation, merge and chunks per workgroup).  Two
  // where one would leave a quarter of the compute units idle (at most 64 chunks per sequence) or
  // where two have few blocks each, so that the second reading costs less than the longer chain of 8
  // heads; but not where one per sequence and head is more than half a round already (64 sequences of
  // 900 tokens, 32 / 4 heads, 2 bit: 32.5 us per call in two, 19.4 in one).  us per call, two against
  // one, blocks per workgroup of two:
  //   64 / 8 heads, 2 bit: 3000 tokens (7) 13.0, 14.9; 20000 (41) 17.7, 18.6; 30000 (60) 19.7, 20.1;
  //     45000 (89) 23.1, 22.1; 131000 (257) 39.9, 33.3
  //   32 / 4 heads, 4 bit: 20000 (20) 14.5, 17.0; 65000 (64) 20.3, 21.2; 131000 (128) 28.6, 26.8
  //   8 / 1 heads, 4 bit (never more than 64 compute units busy in one): 65000 (16) 16.7, 27.6; 131000 18.9, 28.9
  //   1 bit / 64: 32 / 4 heads: 20000 (20) 15.8, 17.2; 45000 (44) 18.5, 19.6; 65000 (64) 20.7, 20.7; 80000 (78) 22.3, 21.8; 98413 (96)
  //     24.2, 22.7; 131000 (128) 27.1, 24.8; 64 / 8: 20000 (40) 18.2, 18.3; 30000 (59) 20.1, 19.7; 45000 (89) 23.3, 21.6; 8 / 1: 65000
  //     (16) 18.0, 23.9
  //   2 bit / 64: 32 / 4: 65000 (64) 20.4, 20.8; 131000 26.6, 24.8
  constexpr int kTwoWorkgroupsBlocks = 80;
  const bool large_group = d->n_q_heads / d->n_kv_heads > 4;
  int32_t st = plan(0, kTailBlocks);
  if (large_group &&
      (st != TKV_OK || (2 * d->n_kv_heads * d->batch <= target_blocks &&
                        (4ll * total_chunks * heads < 3ll * target_blocks ||
                         2 * total_work * d->n_kv_heads < (long long)kTwoWorkgroupsBlocks * target_blocks))))
    st = plan(1, kTailBlocks);
  // What else there is where that makes more chunks than may be or than the partials' room takes: a
  // smaller allowance for the tail (two workgroups never take more chunks than one: their zero-point
  // table holds twice the blocks).
  if (st != TKV_OK) st = plan(large_group ? 1 : 0, kTailBlocksLeast);
  if (st != TKV_OK) return st;
  // Quantizing a completed group in this launch keeps one workgroup per head busy for 2 to 3 us, a launch of its own takes 5
  // to 8 once: not where the workgroups come in several rounds, each of which would wait for that.
  if (fresh != nullptr && fresh->complete && total_chunks * heads > target_blocks) return TKV_E_UNSUPPORTED;
  p.k_codes = (const uint32_t*)c->k_codes;
  p.v_codes = (const uint32_t*)c->v_codes;
  p.k_scale = (const __half*)c->k_scale;
  p.k_zero = (const __half*)c->k_zero;
  p.v_scale = (const __half*)c->v_scale;
  p.v_zero = (const __half*)c->v_zero;
  p.k_resid = (const __half*)c->k_resid;
  p.v_resid = (const __half*)c->v_resid;
  p.q = q;
  p.parts = parts;
  p.arrivals = arrivals;
  p.out = out;
  p.scale2 = scale2;
  p.hq = d->n_q_heads;
  p.hkv = d->n_kv_heads;
  p.residual = d->residual;
  p.capacity = d->capacity;
  p.batch = d->batch;
#ifdef TKV_PHASE
  p.prof = (long long*)g_mfma_prof;
#endif
  p.lens = lens;
  p.k_new = nullptr;
  p.complete = fresh != nullptr && fresh->complete ? 1 : 0;
  if (fresh != nullptr) {
    p.k_new = fresh->k_new;
    p.v_new = fresh->v_new;
    p.n_stride = fresh->n_stride;
    p.n_add = fresh->n_add;
  }
  const dim3 grid(total_chunks, heads, 1);
  switch (variant) {
    case 232: return launch_variant<2, 1, 12>(p, grid, s);
    case 432: return launch_variant<4, 1, 8>(p, grid, s);
    case 164: return launch_variant<1, 2, 12>(p, grid, s);
    case 264: return launch_variant<2, 2, 12>(p, grid, s);
  }
  return TKV_E_UNSUPPORTED;
}

}  // namespace tkv

#ifdef TKV_PHASE
// profiling builds (-DTKV_PHASE): device buffer that receives [workgroup][wave][8] wall-clock stamps
extern "C" void tkv_debug_set_dump(void* ptr) { tkv::g_mfma_prof = ptr; }
#endif
