// tkv_quant_attn_decode: Eq. 3 (Sec. 2.1) over the dequantized cache of a
// quantization-friendly layer (Sec. 4.3), split over token chunks with a
// log-sum-exp merge.
#include <algorithm>
#include <atomic>
#include <mutex>

#include "tkv_common.h"

namespace tkv {
// matrix-core path (tkv_quant_attn_mfma.hip); returns TKV_E_UNSUPPORTED when the
// shape is not one it is built for.
int32_t launch_quant_attn_mfma(const tkv_quant_desc* d, const tkv_quant_cache* c, const __half* q, __half* out,
                               float scale2, float* parts, size_t parts_floats, uint32_t* arrivals, int target_blocks,
                               const TkvSeqLens& lens, const QuantNewTokens* fresh, hipStream_t s);
}  // namespace tkv

namespace {

std::atomic<int> g_kernel_choice{0};      // 0: the setting's own kernel, 1: shape-generic reference kernel
std::atomic<int> g_target_blocks{0};      // workgroups the split-K launch aims at; 0 = one per compute unit of the stream

struct QuantAttnParams {
  const uint32_t* k_codes;
  const uint32_t* v_codes;
  const __half* k_scale;
  const __half* k_zero;
  const __half* v_scale;
  const __half* v_zero;
  __half* k_resid;
  __half* v_resid;
  const __half* q;
  float* parts;  // [B][Hq][n_chunks + 1][D + 4]
  float scale2;  // sm_scale * log2(e)
  int32_t batch, hq, hkv, bits, group, residual, capacity;
  int32_t groups_per_chunk, n_chunks;  // chunk size in blocks of 32 tokens; chunk n_chunks is the fp16 tail
  TkvSeqLens lens;
  // float32 kernel: the step's new tokens when the call also appends them (Eq. 2), the last n_add[b] tokens of sequence b, rows
  // [B][n_stride][Hkv][D]; nullptr: none
  const __half* k_new;
  const __half* v_new;
  int32_t n_stride;
  TkvSeqLens n_add;
};

__device__ inline float wave_half_max(float v) {
  // max over the 32 lanes that share l / 32
  for (int m = 16; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m, 64));
  return v;
}

// Shape-generic reference kernel: plain float32 arithmetic, one wave per 32-token
// block, no matrix cores.  Correct for every supported descriptor and any alignment of the query;
// serves calls only on request and where quant_attn_f32_kernel's 32-bit query loads do not fit.
__global__ __launch_bounds__(256) void quant_attn_generic_kernel(QuantAttnParams p) {
  __shared__ float qs[4][TKV_D];            // query heads of this KV head, zero padded
  __shared__ float ksz[4][TKV_D][2];        // per wave: K scale, zero of the current group
  __shared__ float pw[4][4][TKV_BLK];       // per wave: weights p[h][t]
  __shared__ float alpha_s[4][4];           // per wave: rescale factors
  __shared__ uint32_t vblk[4][TKV_D * 4];   // per wave: packed V block (<= 512 words)
  __shared__ float red_m[4][4], red_l[4][4];
  __shared__ float red_o[4][4][TKV_D];

  // Groups of more than 4 query heads per KV head are served 4 heads at a time: blockIdx.y runs
  // over (KV head, quarter of its group).
  const int split = (p.hq / p.hkv + 3) / 4;
  const int b = blockIdx.z, h = blockIdx.y / split, chunk = blockIdx.x;
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  const int qh0 = h * (p.hq / p.hkv) + 4 * (blockIdx.y % split);  // first query head of this workgroup
  const int G = min(4, (h + 1) * (p.hq / p.hkv) - qh0);
  const int n = p.lens.n[b];
  const int nq = tkv::n_quantized(n, p.residual, p.group);
  const int jq = nq / TKV_BLK;  // packed blocks of 32 tokens
  const size_t bh = (size_t)b * p.hkv + h;
  const size_t n_blocks_cap = (size_t)(p.capacity / TKV_BLK);
  const size_t n_groups_cap = (size_t)(p.capacity / p.group);
  const int bpg = p.group / TKV_BLK;  // blocks per key group
  const int nu = TKV_D / p.group;     // channel groups of a value row
  const int nwords = TKV_D * p.bits;
  const int ring = p.residual + p.group;
  const bool tail = chunk == p.n_chunks;

  for (int i = tid; i < 4 * TKV_D; i += 256) {
    const int hh = i / TKV_D, c = i % TKV_D;
    qs[hh][c] = hh < G ? __half2float(p.q[((size_t)b * p.hq + (size_t)qh0 + hh) * TKV_D + c]) : 0.f;
  }
  __syncthreads();

  // blocks of 32 tokens this workgroup owns: [blk0, blk1)
  int blk0, blk1;
  if (!tail) {
    blk0 = chunk * p.groups_per_chunk;
    blk1 = min(blk0 + p.groups_per_chunk, jq);
  } else {
    blk0 = 0;
    blk1 = (n - nq + TKV_BLK - 1) / TKV_BLK;
  }

  const int t = lane % 32, hp = lane / 32;
  float m_run[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  float l_run[4] = {0.f, 0.f, 0.f, 0.f};
  float o_run[4][2] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
  const int c0 = 2 * lane, u = c0 / p.group;

  for (int blk = blk0 + wave; blk < blk1; blk += 4) {
    float acc0 = 0.f, acc1 = 0.f;
    bool valid = true;
    if (!tail) {
      const size_t grp = bh * n_blocks_cap + blk;            // packed block
      const size_t kgrp = bh * n_groups_cap + blk / bpg;     // its key group
      // K scale / zero of this group -> LDS
      for (int c = lane; c < TKV_D; c += 64) {
        ksz[wave][c][0] = __half2float(p.k_scale[kgrp * TKV_D + c]);
        ksz[wave][c][1] = __half2float(p.k_zero[kgrp * TKV_D + c]);
      }
      for (int w = lane; w < nwords; w += 64) vblk[wave][w] = p.v_codes[grp * nwords + w];
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_s_waitcnt(0);
      const uint32_t* kblk = p.k_codes + grp * nwords;
      const uint32_t cmask = (1u << p.bits) - 1u;
      for (int c = 0; c < TKV_D; ++c) {
        int w, f;
        tkv::k_code_pos(p.bits, t, c, w, f);
        const float code = (float)((kblk[w] >> (p.bits * f)) & cmask);
        const float kh = code * ksz[wave][c][0] + ksz[wave][c][1];
        acc0 += qs[2 * hp][c] * kh;
        acc1 += qs[2 * hp + 1][c] * kh;
      }
    } else {
      const int tok = nq + blk * TKV_BLK + t;
      valid = tok < n;
      if (valid) {
        const __half* krow = p.k_resid + (bh * ring + (size_t)(tok % ring)) * TKV_D;
        for (int c = 0; c < TKV_D; ++c) {
          const float kh = __half2float(krow[c]);
          acc0 += qs[2 * hp][c] * kh;
          acc1 += qs[2 * hp + 1][c] * kh;
        }
      }
    }
    const float x0 = valid ? acc0 * p.scale2 : -INFINITY;
    const float x1 = valid ? acc1 * p.scale2 : -INFINITY;
    const float g0 = wave_half_max(x0), g1 = wave_half_max(x1);
    // publish p and alpha for this wave
    {
      const float mo0 = m_run[2 * hp], mo1 = m_run[2 * hp + 1];
      const float mn0 = fmaxf(mo0, g0), mn1 = fmaxf(mo1, g1);
      pw[wave][2 * hp][t] = exp2f(x0 - mn0);
      pw[wave][2 * hp + 1][t] = exp2f(x1 - mn1);
      if (t == 0) {
        alpha_s[wave][2 * hp] = exp2f(mo0 - mn0);
        alpha_s[wave][2 * hp + 1] = exp2f(mo1 - mn1);
      }
      // every lane tracks all four maxima; fetch the other half's via LDS below
      red_m[wave][2 * hp] = mn0;
      red_m[wave][2 * hp + 1] = mn1;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0);
    float al[4];
    for (int hh = 0; hh < 4; ++hh) {
      al[hh] = alpha_s[wave][hh];
      m_run[hh] = red_m[wave][hh];
    }
    // P.V for channels c0, c0+1
    float s0[4] = {0.f, 0.f, 0.f, 0.f}, s1[4] = {0.f, 0.f, 0.f, 0.f}, ls[4] = {0.f, 0.f, 0.f, 0.f};
    for (int tt = 0; tt < TKV_BLK; ++tt) {
      float v0, v1;
      if (!tail) {
        const size_t grp = bh * n_blocks_cap + blk;
        const float sc = __half2float(p.v_scale[(grp * nu + u) * TKV_BLK + tt]);
        const float ze = __half2float(p.v_zero[(grp * nu + u) * TKV_BLK + tt]);
        const uint32_t cmask = (1u << p.bits) - 1u;
        int w, f;
        tkv::v_code_pos(p.bits, tt, c0, w, f);
        v0 = (float)((vblk[wave][w] >> (p.bits * f)) & cmask) * sc + ze;
        tkv::v_code_pos(p.bits, tt, c0 + 1, w, f);
        v1 = (float)((vblk[wave][w] >> (p.bits * f)) & cmask) * sc + ze;
      } else {
        const int tok = nq + blk * TKV_BLK + tt;
        if (tok < n) {
          const __half* vrow = p.v_resid + (bh * ring + (size_t)(tok % ring)) * TKV_D;
          v0 = __half2float(vrow[c0]);
          v1 = __half2float(vrow[c0 + 1]);
        } else {
          v0 = v1 = 0.f;
        }
      }
      for (int hh = 0; hh < 4; ++hh) {
        const float pp = pw[wave][hh][tt];
        s0[hh] += pp * v0;
        s1[hh] += pp * v1;
        ls[hh] += pp;
      }
    }
    for (int hh = 0; hh < 4; ++hh) {
      o_run[hh][0] = o_run[hh][0] * al[hh] + s0[hh];
      o_run[hh][1] = o_run[hh][1] * al[hh] + s1[hh];
      l_run[hh] = l_run[hh] * al[hh] + ls[hh];
    }
    __builtin_amdgcn_wave_barrier();
  }

  // merge the four waves
  __syncthreads();
  if (lane == 0)
    for (int hh = 0; hh < 4; ++hh) {
      red_m[wave][hh] = m_run[hh];
      red_l[wave][hh] = l_run[hh];
    }
  for (int hh = 0; hh < 4; ++hh) {
    red_o[wave][hh][c0] = o_run[hh][0];
    red_o[wave][hh][c0 + 1] = o_run[hh][1];
  }
  __syncthreads();
  const int n_parts = p.n_chunks + 1;
  for (int i = tid; i < G * TKV_D; i += 256) {
    const int hh = i / TKV_D, c = i % TKV_D;
    float M = -INFINITY;
    for (int w = 0; w < 4; ++w) M = fmaxf(M, red_m[w][hh]);
    float L = 0.f, O = 0.f;
    for (int w = 0; w < 4; ++w) {
      const float mw = red_m[w][hh];
      const float wgt = mw == -INFINITY ? 0.f : exp2f(mw - M);
      L += red_l[w][hh] * wgt;
      O += red_o[w][hh][c] * wgt;
    }
    float* dst = p.parts + (((size_t)b * p.hq + (size_t)qh0 + hh) * n_parts + chunk) * TKV_PART_STRIDE;
    dst[TKV_PART_O + c] = O;
    if (c == 0) {
      dst[0] = M;
      dst[1] = L;
    }
  }
}

// ---- quant_attn_f32_kernel -----------------------------------------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ inline half2_t as_half2(uint32_t w) { return __builtin_bit_cast(half2_t, w); }

// The eight codes of a field octet: field f = i / 2 + 4 (i % 2) (4 bits: nibbles of one word) or
// i / 2 + 16 (i % 2) + base (1 bit).  Code i is left where an fp16 number has its lowest mantissa bits, so one instruction
// yields two codes: half i % 2 of pair i / 2 is the subnormal code * 2^-code_exp(i), and a multiply-add that takes a scaler times
// 2^code_exp(i), both exact, rounds what code times scaler plus zero-point rounds.
template <int BITS>
__device__ constexpr int code_exp(int i) {
  return BITS == 4 ? 24 - 4 * (i / 2 % 2) : 24 - i / 2 % 4;
}
template <int BITS>
__device__ inline void codes_of(uint32_t w, int base, half2_t (&pair)[4]) {
  if (BITS == 4) {
    const uint32_t hi = w >> 8;
    pair[0] = as_half2(w & 0x000F000Fu), pair[1] = as_half2(w & 0x00F000F0u);
    pair[2] = as_half2(hi & 0x000F000Fu), pair[3] = as_half2(hi & 0x00F000F0u);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) pair[k] = as_half2((w >> base) & (0x00010001u << k));
  }
}

// Float32 kernel of the settings (4 bits, groups of 64) and (1 bit, groups of 32): every logit, weight
// and partial sum is the float32 number that quant_attn_generic_kernel computes, operation for
// operation (one fused multiply-add per element of q.K-hat in channel order, per element of p.V-hat in
// token order; 32-token blocks dealt to four accumulation streams per chunk, merged in the same order),
// so the results are the same bits on every call and the same as that kernel's.  What differs is who
// does the work.  The generic kernel gives each stream a wave whose halves hold two heads each, reads
// every code from memory where it is used and every operand from LDS.  Here a wave takes two streams,
// one per half, and a lane one token for all H heads (logits) or four channels of all heads (values): no
// lane works for a head that does not exist, packed words and scalers of the next block are
// loaded into registers while this one is worked on, two codes unpack with one instruction into fp16 subnormals that the
// multiply-adds take as they are, query elements are scalar operands.  Bound by vector instructions: 1.6 + H per element and contraction.
//
// 4 bits, 32 / 32 heads, 20479 + 16857 tokens: 44 us per call, 542 on the generic kernel; 32 / 8 heads, 65500
// tokens: 42 and 256; 1 bit, 39 and 252.  With a byte conversion (4 bits) or an extraction and a conversion (1 bit) per code and
// fp16 scalers 48, 48 and 46; 1 bit, 32 / 32, 20000 tokens 30.0, now 25.0.  The matrix cores serve the first three in 45, 26 and 25 us, but
// their operands are fp16: scalers above 1024 overflow, weights below 2^-14 lose bits, and the order of
// the blocks is decided at run time.
// Workgroups that a compute unit holds: 2 waves each, 2 to 4 of them per SIMD with the registers of each variant (its attribute
// says so, as the least and the most: the chunks are planned for that many.  Without a most (then a fourth wave for 4 bits and one head, a
// third for four) 16 x 900 tokens of 32/32 heads take 24.5 us, 23.6 with it; 44 x 4000 209, 182; 25 x 8000 of 32/8 121, 115, but 32 x 4000 of
// 32/32 127, 141, and 64 x 4000 of 32/8 119, 152).
constexpr int kF32TailsLast = 9;  // chunks of more blocks than this: tails behind them, else in front
constexpr int f32_waves(int bits, int heads) { return bits == 4 ? (heads == 4 ? 2 : 3) : heads == 1 ? 4 : 3; }
inline int f32_resident(int bits, int group) { return 2 * f32_waves(bits, group > 2 ? 4 : group); }
template <int BITS, int GRP, int H>
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(f32_waves(BITS, H), f32_waves(BITS, H))))
void quant_attn_f32_kernel(QuantAttnParams p) {
#pragma clang fp contract(off)
  constexpr int NU = TKV_D / GRP;        // channel groups of a value row
  constexpr int NWORDS = TKV_D * BITS;   // words of a packed block
  constexpr int BPG = GRP / TKV_BLK;     // blocks per key group
  // With 4 heads an octet's scalers and zero-points are fetched where they are used and the pieces of the values kept apart: all of them
  // hoisted above one another do not fit the registers.  With one head that costs, with two it makes no difference.  (The pieces of the keys,
  // 32 channels each, are apart for any number of heads.)  us per call without / with it: 4 bit, 32/8 heads, 65500 tokens 45.1, 42.4; 32 x 900 26.1,
  // 24.7; 16/8, 4 x 30000 44.1, 43.7; 1 bit, 32/32, 16 x 2500 40.5, 41.7.
  constexpr bool kApart = H == 4;
  constexpr int KW = BITS == 4 ? 4 : 1;  // words per lane and 8-channel (8-token) class
  // per wave, half: scalers times 2^code_exp in float32, zero-points in fp16
  __shared__ __attribute__((aligned(16))) float ksc[2][2][TKV_D], vsc[2][2][NU * TKV_BLK];
  __shared__ __attribute__((aligned(16))) uint32_t kze[2][2][TKV_D / 2], vze[2][2][NU * TKV_BLK / 2];
  __shared__ __attribute__((aligned(16))) float pws[2][2][H][TKV_BLK];          // per wave, half: weights
  __shared__ float red_m[4][H], red_l[4][H];
  __shared__ float red_o[4][H][TKV_D];

  const int group = p.hq / p.hkv, split = (group + H - 1) / H;
  // blockIdx.x runs over the chunks of all (sequence, KV head, H query heads of its group) units and over their tails
  // apart: the chunks, which are the work, fall evenly on the compute units (with a tail behind every head's chunks, some
  // dies can get the tails and others the chunks).  Tails, which are a chain of round trips, go first where the chunks
  // are short, else last: 4 bit, 32/8 heads, 5000 tokens (4 blocks per chunk, 4 heads) 18.5 us per call, 21.7 with the tails last; 32/32,
  // 16 x 2500 tokens (37 blocks) 53.4 with the tails last, 63.0 first.
  const int units = p.hkv * split, n_heavy = p.batch * units * p.n_chunks, n_tails = (int)gridDim.x - n_heavy;
  const bool tails_last = p.groups_per_chunk > kF32TailsLast;
  const int at = (int)blockIdx.x - (tails_last ? 0 : n_tails);  // place among the chunks
  const bool tail = at < 0 || at >= n_heavy;
  const int x = at < 0 ? at + n_tails : at - n_heavy;           // ... and among the tails
  const int unit = tail ? x : at / p.n_chunks, chunk = tail ? p.n_chunks : at % p.n_chunks;
  const int b = unit / units, y_unit = unit % units, h = y_unit / split;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int half = lane / 32, t = lane % 32;          // stream of this wave, token of its block
  const int vh = t / 16, l16 = t % 16;                // values: channels 64 vh + 16 j + l16
  const int stream = 2 * wave + half;
  const int qh0 = h * group + H * (y_unit % split);
  const int G = min(H, (h + 1) * group - qh0);
  const int n = p.lens.n[b];
  const int nq = tkv::n_quantized(n, p.residual, GRP);
  const int jq = nq / TKV_BLK;
  const size_t bh = (size_t)b * p.hkv + h;
  const int ring = p.residual + GRP;
  const int blk0 = tail ? 0 : chunk * p.groups_per_chunk;
  const int blk1 = tail ? (n - nq + TKV_BLK - 1) / TKV_BLK : min(blk0 + p.groups_per_chunk, jq);

  // query rows through the constant address space: uniform loads, scalar operands
  typedef const __attribute__((address_space(4))) uint32_t* ScalarWords;
  uint64_t qrow[H];
#pragma unroll
  for (int hh = 0; hh < H; ++hh)  // heads past the group re-read its last one; their results are not used
    qrow[hh] = (uint64_t)(uintptr_t)(p.q + ((size_t)b * p.hq + (size_t)qh0 + min(hh, G - 1)) * TKV_D);
  // (the loads stay inside the block loop: kept across it the elements would take 64 H registers)
  auto pin_query = [&]() {
#pragma unroll
    for (int hh = 0; hh < H; ++hh) asm volatile("" : "+s"(qrow[hh]));
  };

  float m_run[H], l_run[H], o_run[H][4];
#pragma unroll
  for (int hh = 0; hh < H; ++hh) {
    m_run[hh] = -INFINITY, l_run[hh] = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) o_run[hh][j] = 0.f;
  }

  // q . k of one token, eight channels at a time
  auto dot8 = [&](float (&acc)[H], int c, const float (&kh)[8]) {
#pragma unroll
    for (int hh = 0; hh < H; ++hh) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const half2_t q2 = as_half2(((ScalarWords)qrow[hh])[c / 2 + i / 2]);
        acc[hh] = __builtin_fmaf((float)q2[i % 2], kh[i], acc[hh]);
      }
    }
  };
  // logits -> weights (in LDS for the half's lanes) and the factor for what is accumulated so far
  auto soften = [&](const float (&acc)[H], bool valid, bool on, float (&al)[H]) {
#pragma unroll
    for (int hh = 0; hh < H; ++hh) {
      const float x = valid ? acc[hh] * p.scale2 : -INFINITY;
      const float mn = fmaxf(m_run[hh], wave_half_max(x));
      pws[wave][half][hh][t] = exp2f(x - mn);
      al[hh] = exp2f(m_run[hh] - mn);
      m_run[hh] = on ? mn : m_run[hh];
    }
    __builtin_amdgcn_wave_barrier();
  };
  // weights of eight tokens, then one token's share of p . V
  auto weights8 = [&](float (&pp)[H][8], int t0) {
#pragma unroll
    for (int hh = 0; hh < H; ++hh) {
#pragma unroll
      for (int i = 0; i < 8; i += 4) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(&pws[wave][half][hh][t0 + i]);
#pragma unroll
        for (int y = 0; y < 4; ++y) pp[hh][i + y] = w[y];
      }
    }
  };
  auto accumulate = [&](bool on, const float (&al)[H], const float (&s)[H][4], const float (&ls)[H]) {
    // (selects: behind a branch the compiler moves all of p . V there, its operands waiting in registers)
#pragma unroll
    for (int hh = 0; hh < H; ++hh) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float o = __builtin_fmaf(o_run[hh][j], al[hh], s[hh][j]);
        o_run[hh][j] = on ? o : o_run[hh][j];
      }
      const float l = __builtin_fmaf(l_run[hh], al[hh], ls[hh]);
      l_run[hh] = on ? l : l_run[hh];
    }
    __builtin_amdgcn_wave_barrier();
  };

  if (!tail) {
    const size_t blk_base = bh * (size_t)(p.capacity / TKV_BLK), grp_base = bh * (size_t)(p.capacity / GRP);
    const int r = 4 * (t / 8) + t % 4, tau = (t % 8) / 4;
    uint32_t kw[4][KW], vw[4][KW];  // packed words of the block: keys by 8-channel class, values by 8-token class
    u32x2 ks, kz;
    uint32_t vs[NU / 2], vz[NU / 2];
    auto load_k = [&](int blk) {
      const size_t g = blk_base + blk;
      const uint32_t* src = p.k_codes + g * NWORDS;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        if constexpr (BITS == 4) {
          const u32x4 w = *reinterpret_cast<const u32x4*>(src + 256 * tau + 4 * (r + 16 * kb));
#pragma unroll
          for (int y = 0; y < 4; ++y) kw[kb][y] = w[y];
        } else {
          kw[kb][0] = src[64 * tau + r + 16 * kb];
        }
      }
      const size_t o = (grp_base + blk / BPG) * TKV_D + 4 * t;
      ks = *reinterpret_cast<const u32x2*>(p.k_scale + o);
      kz = *reinterpret_cast<const u32x2*>(p.k_zero + o);
    };
    auto load_v = [&](int blk) {
      const size_t g = blk_base + blk;
      const uint32_t* src = p.v_codes + g * NWORDS;
#pragma unroll
      for (int tb = 0; tb < 4; ++tb) {
        if constexpr (BITS == 4) {
          const u32x4 w = *reinterpret_cast<const u32x4*>(src + 256 * vh + 4 * (l16 + 16 * tb));
#pragma unroll
          for (int y = 0; y < 4; ++y) vw[tb][y] = w[y];
        } else {
          vw[tb][0] = src[64 * vh + l16 + 16 * tb];
        }
      }
      const size_t o = g * (NU * TKV_BLK) + NU * t;
#pragma unroll
      for (int i = 0; i < NU / 2; ++i) {
        vs[i] = *reinterpret_cast<const uint32_t*>(p.v_scale + o + 2 * i);
        vz[i] = *reinterpret_cast<const uint32_t*>(p.v_zero + o + 2 * i);
      }
    };
    // scaler y of the pair w of neighbouring channels or tokens, the first of them at place i of an octet
    auto scaled = [](uint32_t w, int y, int i) { return (float)as_half2(w)[y] * (float)(1 << code_exp<BITS>(i)); };
    const int ki = 4 * (t % 2), vi = NU * t % 8;  // places of this lane's first key and value scaler in their octets
    const int first = blk0 + 2 * wave;  // first block of this wave's lower half
    auto mine = [&](int base) { return min(base + half, blk1 - 1); };  // (a half past the end repeats the last block and drops the result)
    if (first < blk1) {
      load_k(mine(first));
      load_v(mine(first));
    }
    for (int base = first; base < blk1; base += 4) {
      pin_query();
      const bool on = base + half < blk1;
      const int next = min(base + 4, blk1 - 1);
      *reinterpret_cast<f32x4*>(&ksc[wave][half][4 * t]) =
          f32x4{scaled(ks[0], 0, ki), scaled(ks[0], 1, ki), scaled(ks[1], 0, ki + 2), scaled(ks[1], 1, ki + 2)};
      *reinterpret_cast<u32x2*>(&kze[wave][half][2 * t]) = kz;
#pragma unroll
      for (int i = 0; i < NU / 2; ++i) {
        *reinterpret_cast<f32x2*>(&vsc[wave][half][NU * t + 2 * i]) = f32x2{scaled(vs[i], 0, vi + 2 * i), scaled(vs[i], 1, vi + 2 * i)};
        vze[wave][half][NU / 2 * t + i] = vz[i];
      }
      __builtin_amdgcn_wave_barrier();
      float acc[H];
#pragma unroll
      for (int hh = 0; hh < H; ++hh) acc[hh] = 0.f;
      // scalers and zero-points of an octet of channels, from LDS two octets ahead (kAhead octets' registers)
      constexpr int kAhead = kApart ? 1 : 3;
      f32x4 sc[kAhead][2];
      u32x4 ze[kAhead];
      auto request = [&](int c) {
        if (c >= TKV_D) return;
        const int o = c / 8 % kAhead;
        sc[o][0] = *reinterpret_cast<const f32x4*>(&ksc[wave][half][c]);
        sc[o][1] = *reinterpret_cast<const f32x4*>(&ksc[wave][half][c + 4]);
        ze[o] = *reinterpret_cast<const u32x4*>(&kze[wave][half][c / 2]);
      };
      if (!kApart) request(0), request(8);
#pragma unroll
      for (int c = 0; c < TKV_D; c += 8) {
        const int kb = (c / 8) % 4, o = c / 8 % kAhead;
        request(kApart ? c : c + 16);
        half2_t code[4];
        codes_of<BITS>(kw[kb][BITS == 4 ? c / 32 : 0], 4 * ((c / 32) % 2) + 8 * (c / 64), code);
        float kh[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t zi = ze[o][i / 2];
          kh[i] = __builtin_fmaf((float)code[i / 2][i % 2], sc[o][i / 4][i % 4], (float)as_half2(zi)[i % 2]);
        }
        dot8(acc, c, kh);
        if (c % 32 == 24) __builtin_amdgcn_sched_barrier(0);
      }
      load_k(mine(next));
      float al[H];
      soften(acc, true, on, al);
      float s[H][4], ls[H];
#pragma unroll
      for (int hh = 0; hh < H; ++hh) {
        ls[hh] = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) s[hh][j] = 0.f;
      }
#pragma unroll
      for (int tb = 0; tb < 4; ++tb) {
        float pp[H][8];
        weights8(pp, 8 * tb);
        float sc[NU / 2][8];  // scalers and zero-points of the eight tokens in this lane's channel groups
        u32x4 ze[NU / 2];
#pragma unroll
        for (int y = 0; y < NU / 2; ++y) {
          const int u = NU == 2 ? vh : 2 * vh + y;
          ze[y] = *reinterpret_cast<const u32x4*>(&vze[wave][half][(u * TKV_BLK + 8 * tb) / 2]);
#pragma unroll
          for (int i = 0; i < 8; i += 4) {
            const f32x4 w = *reinterpret_cast<const f32x4*>(&vsc[wave][half][u * TKV_BLK + 8 * tb + i]);
#pragma unroll
            for (int x = 0; x < 4; ++x) sc[y][i + x] = w[x];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          half2_t code[4];
          codes_of<BITS>(vw[tb][BITS == 4 ? j : 0], 4 * j, code);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t zi = ze[NU == 2 ? 0 : j / 2][i / 2];
            const float v = __builtin_fmaf((float)code[i / 2][i % 2], sc[NU == 2 ? 0 : j / 2][i], (float)as_half2(zi)[i % 2]);
#pragma unroll
            for (int hh = 0; hh < H; ++hh) s[hh][j] = __builtin_fmaf(pp[hh][i], v, s[hh][j]);
          }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
          for (int hh = 0; hh < H; ++hh) ls[hh] = ls[hh] + pp[hh][i];
        }
        if (kApart || tb == 3) __builtin_amdgcn_sched_barrier(0);
      }
      load_v(mine(next));
      accumulate(on, al, s, ls);
    }
  } else {
    // the fp16 tail: rows from the ring, the lane's four channels side by side (4 t ..) for the values.  Bound by
    // its chain of round trips: a block's key rows are requested at once, and the value rows as the keys' registers come
    // free.  (Loaded in eight pieces, each waited for before the next: 32/32 heads, 168 tokens 13.1 us per call, 11.1 now;
    // 316 tokens, 32 sequences 59.0, 52.6.)
    const int slot_n = (n - 1) % ring;
    for (int base = 2 * wave; base < blk1; base += 4) {
      pin_query();
      const bool on = base + half < blk1;
      const int tok0 = nq + TKV_BLK * min(base + half, blk1 - 1), tok = tok0 + t, slot0 = tok0 % ring;
      auto row = [&](const __half* rows, int y) {  // of token tok0 + y, or the last one
        const int slot = tok0 + y < n ? slot0 + y : slot_n;
        return rows + (bh * ring + (size_t)(slot < ring ? slot : slot - ring)) * TKV_D;
      };
      if (p.k_new != nullptr) {
        // The step's new tokens in this block join the ring first, a token per half-wave; every workgroup of the KV head
        // writes the same bytes and reads back its own.  On the chain of the wave with the newest tokens alone.  us per
        // decode step, the append in a launch of its own / here: 4 bit, 32/8 heads, 1500 tokens 15.3, 13.0; 65500 tokens 49.8,
        // 48.1; 32 x 900 28.2, 26.2; 1 bit, 64/8, 4 x 3000 25.7, 23.3.
        const int n_old = n - p.n_add.n[b];
        for (int i = max(tok0, n_old); i < min(tok0 + TKV_BLK, n); ++i) {
          const __half* src = tkv::pick(t >= 16, p.k_new, p.v_new) + (((size_t)b * p.n_stride + (i - n_old)) * p.hkv + h) * TKV_D;
          const u32x4 w = reinterpret_cast<const u32x4*>(src)[t % 16];
          reinterpret_cast<u32x4*>(tkv::pick(t >= 16, p.k_resid, p.v_resid) + (bh * ring + (size_t)(i % ring)) * TKV_D)[t % 16] = w;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      const u32x4* krow = reinterpret_cast<const u32x4*>(row(p.k_resid, t));
      u32x4 kr[TKV_D / 8];
      u32x2 vr[TKV_BLK];
#pragma unroll
      for (int y = 0; y < TKV_D / 8; ++y) kr[y] = krow[y];
      __builtin_amdgcn_sched_barrier(0);
      float acc[H];
#pragma unroll
      for (int hh = 0; hh < H; ++hh) acc[hh] = 0.f;
#pragma unroll
      for (int c = 0; c < TKV_D; c += 32) {
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          float kh[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t wi = kr[c / 8 + y][i / 2];
            kh[i] = (float)as_half2(wi)[i % 2];
          }
          dot8(acc, c + 8 * y, kh);
        }
        __builtin_amdgcn_sched_barrier(0);
        // eight value rows take the registers of 32 key channels
#pragma unroll
        for (int i = c / 4; i < c / 4 + 8; ++i) vr[i] = reinterpret_cast<const u32x2*>(row(p.v_resid, i))[t];
        __builtin_amdgcn_sched_barrier(0);
      }
      float al[H];
      soften(acc, tok < n, on, al);
      float s[H][4], ls[H];
#pragma unroll
      for (int hh = 0; hh < H; ++hh) {
        ls[hh] = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) s[hh][j] = 0.f;
      }
#pragma unroll
      for (int t0 = 0; t0 < TKV_BLK; t0 += 8) {
        float pp[H][8];
        weights8(pp, t0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const bool valid = tok0 + t0 + i < n;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t wj = vr[t0 + i][j / 2];
            const float v = valid ? (float)as_half2(wj)[j % 2] : 0.f;
#pragma unroll
            for (int hh = 0; hh < H; ++hh) s[hh][j] = __builtin_fmaf(pp[hh][i], v, s[hh][j]);
          }
#pragma unroll
          for (int hh = 0; hh < H; ++hh) ls[hh] = ls[hh] + pp[hh][i];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      accumulate(on, al, s, ls);
    }
  }

  // merge the four streams
#pragma unroll
  for (int hh = 0; hh < H; ++hh) {
    if (t == 0) {
      red_m[stream][hh] = m_run[hh];
      red_l[stream][hh] = l_run[hh];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) red_o[stream][hh][tail ? 4 * t + j : 64 * vh + 16 * j + l16] = o_run[hh][j];
  }
  __syncthreads();
  const int c = tid;
  for (int hh = 0; hh < G; ++hh) {
    float M = -INFINITY;
    for (int w = 0; w < 4; ++w) M = fmaxf(M, red_m[w][hh]);
    float L = 0.f, O = 0.f;
    for (int w = 0; w < 4; ++w) {
      const float mw = red_m[w][hh];
      const float wgt = mw == -INFINITY ? 0.f : exp2f(mw - M);
      L = __builtin_fmaf(red_l[w][hh], wgt, L);
      O = __builtin_fmaf(red_o[w][hh][c], wgt, O);
    }
    float* dst = p.parts + (((size_t)b * p.hq + (size_t)qh0 + hh) * (p.n_chunks + 1) + chunk) * TKV_PART_STRIDE;
    dst[TKV_PART_O + c] = O;
    if (c == 0) {
      dst[0] = M;
      dst[1] = L;
    }
  }
}

// Query heads that a workgroup takes: up to 4, which unpack a code once for all of them; fewer where that leaves compute
// units idle, up to four workgroups on each: with 4 heads a block costs 4.8 us, a chain of 2500 vector
// instructions.  4 bit, us per call, always 4 / by this: 32/8 heads, 891 tokens 17.5, 11.9; 1500 tokens 17.1, 12.0; 5000
// tokens 18.8, 14.7 (17.9 with at most two workgroups each); 64/8, 821 tokens 22.2, 14.2; 8/1, 60000 tokens 30.0, 27.2.
// Tails are workgroups too, and read their rows once more for every split: they count as one, and as two before the
// last split.  Without them counted / with them (always 4): 4 bit, 32/8, 32 x 300 tokens 26.8, 18.3 (17.6); 64 x 200 29.2, 22.5 (22.5), 16 x
// 300 16.0, 13.4 (16.4); 64/8, 32 x 430 37.5, 26.2 (26.0), 16 x 300 27.5, 18.5 (17.5); 1 bit, 32/8, 32 x 300 22.0, 17.5 (17.3).  (A few
// more than four for every compute unit, since the longest sequences have just that: 1 bit, 8/1, 98135 tokens, 1028 workgroups
// 34.1, 37.2 with 4 heads.)
constexpr int kF32Alone = 1024 + 32;
// any_group: some sequence has quantized tokens (the one chunk that there is otherwise has nothing to do).
template <int BITS, int GRP>
int32_t launch_f32(const QuantAttnParams& p, bool any_group, hipStream_t s) {
  const int group = p.hq / p.hkv;
  auto units = [&](int heads) { return p.batch * p.hkv * ((group + heads - 1) / heads); };
  int heads = group > 2 ? 4 : group;
  const int chunks = any_group ? p.n_chunks : 0;
  while (heads > 1 && (long long)units(heads / 2) * (chunks + (heads == 2 ? 2 : 1)) <= kF32Alone) heads /= 2;
  const int grid = units(heads) * (p.n_chunks + 1);
  if (heads == 1) TKV_LAUNCH((quant_attn_f32_kernel<BITS, GRP, 1>), grid, 128, 0, s, p);
  else if (heads == 2) TKV_LAUNCH((quant_attn_f32_kernel<BITS, GRP, 2>), grid, 128, 0, s, p);
  else TKV_LAUNCH((quant_attn_f32_kernel<BITS, GRP, 4>), grid, 128, 0, s, p);
  return TKV_OK;
}

// Log-sum-exp merge of the chunk partials of one query head; writes fp16.  One workgroup per query head; a thread takes one channel of
// kThreadClasses of the four classes of parts (every fourth part each).  Bound by latency: the maxima and sums and the first kMergeLoads parts
// of each of a thread's classes are requested at once (16 or 64 parts in one round trip).  us per call with one thread per channel, four parts
// requested at a time behind two round trips for the weights, and with four threads: 1 bit, 32/8 heads, 65500 tokens 40.6, 38.7; 4 bit, 32/8,
// 65500 44.7, 42.3; 5000 14.4, 12.9.  Up to 16 parts see launch_attn_merge.
constexpr int kMergeClasses = 4;
template <int kMergeLoads, int kThreadClasses>
__global__ __launch_bounds__(kMergeClasses / kThreadClasses * TKV_D) void attn_merge_kernel(const float* parts, __half* out, int n_parts) {
  constexpr int kOwn = (TKV_MAX_CHUNKS + TKV_D) / TKV_D;  // parts whose weights one of the first TKV_D threads works out
  __shared__ float wgt[TKV_MAX_CHUNKS + 1];
  __shared__ float red_m[2], red_l[2];
  __shared__ float red_o[kMergeClasses][TKV_D];
  const size_t head = blockIdx.x;  // b * Hq + i
  const int tid = threadIdx.x, c = tid % TKV_D, j = __builtin_amdgcn_readfirstlane(tid / TKV_D);
  const float* base = parts + head * n_parts * TKV_PART_STRIDE;
  const int n4 = n_parts / kMergeClasses * kMergeClasses;  // the parts past it join the first class
  float2 ml[kOwn];
  if (j == 0) {
#pragma unroll
    for (int y = 0; y < kOwn; ++y)
      ml[y] = *reinterpret_cast<const float2*>(base + (size_t)min(c + TKV_D * y, n_parts - 1) * TKV_PART_STRIDE);
  }
  float v[kMergeLoads][kThreadClasses];
  auto request = [&](int k0) {
#pragma unroll
    for (int y = 0; y < kMergeLoads; ++y)
#pragma unroll
      for (int x = 0; x < kThreadClasses; ++x)
        v[y][x] = base[(size_t)min(k0 + kMergeClasses * y + x, n_parts - 1) * TKV_PART_STRIDE + TKV_PART_O + c];
  };
  request(kThreadClasses * j);
  if (j == 0) {
    float m = -INFINITY;
#pragma unroll
    for (int y = 0; y < kOwn; ++y) m = fmaxf(m, ml[y].x);
    m = tkv::over_wave(m, tkv::MaxOf{});
    if (c % 64 == 0) red_m[c / 64] = m;
  }
  __syncthreads();
  if (j == 0) {
    const float M = fmaxf(red_m[0], red_m[1]);
    float lsum = 0.f;
#pragma unroll
    for (int y = 0; y < kOwn; ++y) {
      const int k = c + TKV_D * y;
      if (k < n_parts) {
        const float w = ml[y].x == -INFINITY ? 0.f : exp2f(ml[y].x - M);
        wgt[k] = w;
        lsum += w * ml[y].y;
      }
    }
    for (int m = 32; m >= 1; m >>= 1) lsum += __shfl_xor(lsum, m, 64);
    if (c % 64 == 0) red_l[c / 64] = lsum;
  }
  __syncthreads();
  float O[kThreadClasses] = {};
  for (int k0 = kThreadClasses * j;;) {
#pragma unroll
    for (int y = 0; y < kMergeLoads; ++y) {
      const int k = k0 + kMergeClasses * y;
      if (k < n4) {
#pragma unroll
        for (int x = 0; x < kThreadClasses; ++x) O[x] = __builtin_fmaf(v[y][x], wgt[k + x], O[x]);
      }
    }
    k0 += kMergeClasses * kMergeLoads;
    if (k0 >= n4) break;
    request(k0);
  }
  if (j == 0)
    for (int k = n4; k < n_parts; ++k) O[0] = __builtin_fmaf(base[(size_t)k * TKV_PART_STRIDE + TKV_PART_O + c], wgt[k], O[0]);
  if constexpr (kThreadClasses < kMergeClasses) {
#pragma unroll
    for (int x = 0; x < kThreadClasses; ++x) red_o[kThreadClasses * j + x][c] = O[x];
    __syncthreads();
    if (j != 0) return;
  }
  const auto class_sum = [&](int x) { return kThreadClasses < kMergeClasses ? red_o[x][c] : O[x]; };
  const float L = red_l[0] + red_l[1], sum = (class_sum(0) + class_sum(1)) + (class_sum(2) + class_sum(3));
  out[head * TKV_D + c] = __float2half_rn(L > 0.f ? sum / L : 0.f);
}

}  // namespace

namespace tkv {
int32_t launch_attn_merge(const float* parts, __half* out, int n_heads_total, int n_parts, hipStream_t s) {
  // Up to 16 parts are one thread's loads: a thread per channel, and of 4 parts or fewer no load that would repeat the last one's.
  // Four threads per channel are 16384 waves for 2048 heads, and behind them the next call's attention falls unevenly on the compute
  // units.  us per call with four / with one, 32/8 heads: 1 bit, 64 x 100 tokens (2 parts) 19.7, 16.8; 64 x 300 (3) 27.3, 25.1; 50 x 4000 (3; the
  // attention alone 158, 118) 156, 119; 4 bit, 50 x 4000 (6) 102.8, 100.1; one sequence of 900 to 1900 tokens (7 to 15) the same.
  const dim3 grid(n_heads_total);
  if (n_parts <= kMergeClasses) TKV_LAUNCH((attn_merge_kernel<1, kMergeClasses>), grid, TKV_D, 0, s, parts, out, n_parts);
  else if (n_parts <= 4 * kMergeClasses) TKV_LAUNCH((attn_merge_kernel<4, kMergeClasses>), grid, TKV_D, 0, s, parts, out, n_parts);
  else TKV_LAUNCH((attn_merge_kernel<16, 1>), grid, kMergeClasses * TKV_D, 0, s, parts, out, n_parts);
  return TKV_OK;
}
}  // namespace tkv

extern "C" int32_t tkv_debug_quant_attn_config(int32_t kernel_choice, int32_t target_blocks) {
  if (kernel_choice < 0 || kernel_choice > 1 || target_blocks < -1) return TKV_E_INVAL;
  g_kernel_choice = kernel_choice;
  if (target_blocks > 0) g_target_blocks = target_blocks;
  if (target_blocks == -1) g_target_blocks = 0;  // back to one workgroup per compute unit of the stream
  return TKV_OK;
}

namespace {

// Settings of the matrix-core kernel.  4 bits with groups of 64 and 1 bit with groups of 32 stay in
// float32 (quant_attn_f32_kernel).
bool on_matrix_cores(const tkv_quant_desc* d) {
  return d->bits == 2 || d->group_size == (d->bits == 4 ? 32 : 64);
}

bool f32_takes(const tkv_quant_desc* d, const void* q) {
  return (d->group_size == (d->bits == 4 ? 64 : 32)) && d->bits != 2 && (uintptr_t)q % 4 == 0;
}

// Body of both entry points.  parts: room for parts_floats floats of split-K partials; arrivals:
// one zero word per (sequence, KV head, four query heads of its group).  TKV_E_WORKSPACE if the launch's partials do not fit.
// fresh: the step's new tokens, already counted in seq_len_host but not yet in the fp16 ring, which the
// matrix-core and float32 kernels write them into; TKV_E_UNSUPPORTED otherwise, and for the float32 kernel where they
// complete a group, before anything is launched.
int32_t quant_attn_decode_impl(const tkv_quant_desc* d, const tkv_quant_cache* c, const void* q, void* out,
                               float sm_scale, float* parts, size_t parts_floats, uint32_t* arrivals,
                               hipStream_t s, const tkv::QuantNewTokens* fresh = nullptr) {
  QuantAttnParams p;
  int max_groups = 0;
  for (int b = 0; b < d->batch; ++b) {
    const int32_t n = c->seq_len_host[b];
    if (n < 0) return TKV_E_INVAL;
    if (n > d->capacity) return TKV_E_CAPACITY;
    p.lens.n[b] = n;
    const int g = tkv::n_quantized(n, d->residual, d->group_size) / TKV_BLK;  // in blocks of 32 tokens
    if (g > max_groups) max_groups = g;
  }
  // Chunking of the float32 kernels.  A compute unit holds 4 to 8 of their workgroups at once (registers), and the
  // launch ends with the fullest compute unit: the number of chunks is the one that makes its work least (its chunks' blocks
  // and about 6 more for the fixed part of each, its tails', and another workgroup's where not all are resident at
  // once), out of those that fill what is resident, tails included, and those with 4 to 8 chunks per compute unit.  (A matter
  // of the sizes alone, whatever the stream may use of the machine: the chunks decide the order of the sums.)  us per
  // call with about 1024 chunks, the tails in between and groups of 5 to 8 not counted twice, against this: 4 bit, 32/32 heads,
  // 2 x 20479 tokens 65.9, 51.4; 16 x 2500 64.1, 52.7; 20000 28.2, 28.2; 32/8, 65500 tokens 57.2, 48.0; 50 x 4000 162.7, 116.5; 32
  // x 900 36.3, 26.0; 64/8, 30000 47.1, 41.0; 1 bit, 32/32, 2 x 20000 69.6, 51.7.
  // Short chunks have the tails in front of them (kF32TailsLast) and are over soon: what counts there is that no SIMD gets a third wave, so
  // that four workgroups per compute unit, tails included, are all that counts as resident, however many the registers allow.  us per call
  // with as many as those allow / so: 4 bit, 16/8 heads, 24 x 900 tokens 19.9, 16.1 (17.4 with two waves per SIMD allowed for two heads);
  // 32 x 1300 26.2, 22.8; 6 x 6000 25.0, 20.8; 8/8, 32 x 750 18.1, 14.7; 1 bit, 32/8, 24 x 900 26.1, 19.9; 6 x 6000 32.6, 25.7.  Of 270 shapes of
  // which this changes the plan three are more than 0.8 % slower, all with four heads at 1 bit: 32/8, 48 x 500 27.9, 28.4.
  const int units = d->batch * d->n_kv_heads * ((d->n_q_heads / d->n_kv_heads + 3) / 4);
  int gpc = 4, n_chunks = 1;
  long long least = -1;
  const int resident = 256 * f32_resident(d->bits, d->n_q_heads / d->n_kv_heads);
  const int resident_short = std::min(resident, 4 * 256);
  for (int round = 2; round <= 8; ++round) {
    const int want = round == 2 ? resident_short / units - 1 : round == 3 ? resident / units - 1 : 256 * round / units;
    const int target = std::min(std::max(want, 1), TKV_MAX_CHUNKS);
    const int blocks = std::max((max_groups + target - 1) / target, 4);
    const int chunks = std::max((max_groups + blocks - 1) / blocks, 1);
    const long long per_cu = std::max(((long long)units * chunks + 255) / 256, 4ll);
    const long long cost = per_cu * (blocks + 6) + (units + 255) / 256 * 12 +
                           ((long long)units * (chunks + 1) > (blocks > kF32TailsLast ? resident : resident_short) ? blocks + 18 : 0);
    if (least < 0 || cost < least) least = cost, gpc = blocks, n_chunks = chunks;
  }

  p.k_codes = (const uint32_t*)c->k_codes;
  p.v_codes = (const uint32_t*)c->v_codes;
  p.k_scale = (const __half*)c->k_scale;
  p.k_zero = (const __half*)c->k_zero;
  p.v_scale = (const __half*)c->v_scale;
  p.v_zero = (const __half*)c->v_zero;
  p.k_resid = (__half*)c->k_resid;
  p.v_resid = (__half*)c->v_resid;
  p.q = (const __half*)q;
  p.parts = parts;
  p.scale2 = sm_scale * 1.44269504088896340736f;
  p.batch = d->batch;
  p.hq = d->n_q_heads;
  p.hkv = d->n_kv_heads;
  p.bits = d->bits;
  p.group = d->group_size;
  p.residual = d->residual;
  p.capacity = d->capacity;
  p.groups_per_chunk = gpc;
  p.n_chunks = n_chunks;

  const int choice = g_kernel_choice.load();
  if (choice == 0 && on_matrix_cores(d)) {
    // matrix-core kernel: one launch covers the quantized groups and the fp16 tail
    int target_blocks = g_target_blocks.load();
    // one workgroup per compute unit that the stream may use: on a stream with a compute-unit
    // mask a launch sized for the whole machine would leave a few workgroups for a second round
    if (target_blocks == 0) target_blocks = tkv::stream_compute_units(s);
    const int32_t st = tkv::launch_quant_attn_mfma(d, c, p.q, (__half*)out, p.scale2, p.parts, parts_floats, arrivals,
                                                   target_blocks, p.lens, fresh, s);
    if (st != TKV_E_UNSUPPORTED) return st;
  }
  // the float32 kernel of the two settings reads the query in 32-bit scalar words; the generic one
  // takes it at any fp16 address
  const bool f32 = choice == 0 && f32_takes(d, q);
  if (fresh != nullptr && (!f32 || fresh->complete)) return TKV_E_UNSUPPORTED;
  p.k_new = fresh != nullptr ? fresh->k_new : nullptr;
  p.v_new = fresh != nullptr ? fresh->v_new : nullptr;
  p.n_stride = fresh != nullptr ? fresh->n_stride : 0;
  p.n_add = fresh != nullptr ? fresh->n_add : TkvSeqLens{};
  // float32 kernels; fewer chunks where the partials' room is the fixed array and takes no more
  auto fits = [&]() { return (size_t)d->batch * d->n_q_heads * (n_chunks + 1) * TKV_PART_STRIDE <= parts_floats; };
  while (!fits() && n_chunks > 1) {
    p.groups_per_chunk = (max_groups + n_chunks - 2) / (n_chunks - 1);
    p.n_chunks = n_chunks = (max_groups + p.groups_per_chunk - 1) / p.groups_per_chunk;
  }
  if (!fits()) return TKV_E_WORKSPACE;
  const int split = (d->n_q_heads / d->n_kv_heads + 3) / 4;
  const dim3 grid(n_chunks + 1, d->n_kv_heads * split, d->batch);
  if (f32 && d->bits == 4) {
    if (const int32_t st = launch_f32<4, 64>(p, max_groups > 0, s); st != TKV_OK) return st;
  } else if (f32) {
    if (const int32_t st = launch_f32<1, 32>(p, max_groups > 0, s); st != TKV_OK) return st;
  } else {
    TKV_LAUNCH(quant_attn_generic_kernel, grid, 256, 0, s, p);
  }
  return tkv::launch_attn_merge(p.parts, (__half*)out, d->batch * d->n_q_heads, n_chunks + 1, s);
}

int32_t check_decode_args(const tkv_quant_desc* d, const tkv_quant_cache* c, const void* q, const void* out) {
  const int32_t st = tkv::check_quant_desc(d);
  if (st != TKV_OK) return st;
  if (!c || !c->seq_len_host || !q || !out) return TKV_E_INVAL;
  if (!c->k_codes || !c->k_scale || !c->k_zero || !c->v_codes || !c->v_scale || !c->v_zero || !c->k_resid ||
      !c->v_resid)
    return TKV_E_INVAL;
  return TKV_OK;
}

}  // namespace

extern "C" int32_t tkv_quant_attn_decode(const tkv_quant_desc* d, const tkv_quant_cache* c, const void* q,
                                         void* out, float sm_scale, void* workspace, size_t workspace_bytes,
                                         void* stream) {
  int32_t st = check_decode_args(d, c, q, out);
  if (st != TKV_OK) return st;
  if (!workspace) return TKV_E_INVAL;
  size_t need = 0;
  tkv_quant_cache_sizes(d, nullptr, &need);
  if (workspace_bytes < need) return TKV_E_WORKSPACE;
  // arrival counters sit behind the partials (zero before first use, left zero by every call)
  const size_t parts_floats = (size_t)d->batch * d->n_q_heads * (TKV_MAX_CHUNKS + 1) * TKV_PART_STRIDE;
  uint32_t* arrivals = (uint32_t*)((char*)workspace + ((parts_floats * sizeof(float) + 255) & ~(size_t)255));
  return quant_attn_decode_impl(d, c, q, out, sm_scale, (float*)workspace, parts_floats, arrivals, (hipStream_t)stream);
}

// ---- tkv_quant_decode: Eq. 2 and Eq. 3 of a quantized layer's decode step in one call ----------
extern "C" int32_t tkv_quant_decode(const tkv_quant_desc* d, tkv_quant_cache* c, const void* k_new,
                                    const void* v_new, int32_t n_new, const int32_t* n_valid_host, const void* q,
                                    void* out, float sm_scale, void* workspace, size_t workspace_bytes,
                                    void* stream) {
  int32_t st = check_decode_args(d, c, q, out);
  if (st != TKV_OK) return st;
  if (!workspace || n_new < 0 || (n_new > 0 && (!k_new || !v_new))) return TKV_E_INVAL;
  size_t need = 0;
  tkv_quant_cache_sizes(d, nullptr, &need);
  if (workspace_bytes < need) return TKV_E_WORKSPACE;
  if (n_new == 0) return tkv_quant_attn_decode(d, c, q, out, sm_scale, workspace, workspace_bytes, stream);
  // One launch of the matrix-core kernel, or the float32 kernel and its merge: the new rows join the fp16 ring there, and, on
  // the matrix cores, a group that they complete is quantized there as well if it is one, if all of its tokens are in the ring
  // already and if no slot that the new rows take is one of theirs (any step of up to residual tokens but
  // for some of several).  Else the append's launches, then the attention's.
  tkv::QuantNewTokens fresh;
  fresh.k_new = (const __half*)k_new;
  fresh.v_new = (const __half*)v_new;
  fresh.n_stride = n_new;
  fresh.complete = false;
  const bool mfma = on_matrix_cores(d);
  bool one_launch = g_kernel_choice.load() == 0 && (mfma || f32_takes(d, q));
  for (int b = 0; b < d->batch; ++b) {
    const int64_t n0 = c->seq_len_host[b];
    const int32_t add = n_valid_host ? n_valid_host[b] : n_new;
    if (n0 < 0 || add < 0 || add > n_new) return TKV_E_INVAL;
    if (n0 + add > d->capacity) return TKV_E_CAPACITY;
    fresh.n_add.n[b] = add;
    const int32_t g = d->group_size, n1 = (int32_t)n0 + add;
    const int32_t nq0 = tkv::n_quantized((int32_t)n0, d->residual, g), nq1 = tkv::n_quantized(n1, d->residual, g);
    if (nq1 != nq0) {
      fresh.complete = true;
      if (!mfma || nq1 - nq0 != g || add > d->residual || n1 - nq0 > d->residual + g) one_launch = false;
    }
  }
  auto two_calls = [&]() -> int32_t {
    st = tkv_quantize_append_ragged(d, c, k_new, v_new, n_new, n_valid_host, stream);
    if (st != TKV_OK) return st;
    return tkv_quant_attn_decode(d, c, q, out, sm_scale, workspace, workspace_bytes, stream);
  };
  if (!one_launch) return two_calls();
  const size_t parts_floats = (size_t)d->batch * d->n_q_heads * (TKV_MAX_CHUNKS + 1) * TKV_PART_STRIDE;
  uint32_t* arrivals = (uint32_t*)((char*)workspace + ((parts_floats * sizeof(float) + 255) & ~(size_t)255));
  for (int b = 0; b < d->batch; ++b) c->seq_len_host[b] += fresh.n_add.n[b];
  st = quant_attn_decode_impl(d, c, q, out, sm_scale, (float*)workspace, parts_floats, arrivals, (hipStream_t)stream,
                              &fresh);
  if (st != TKV_OK)  // nothing was launched: the cache is as it was
    for (int b = 0; b < d->batch; ++b) c->seq_len_host[b] -= fresh.n_add.n[b];
  // (a completing step with more workgroups than compute units, or a sequence of more chunks than the matrix-core kernel has)
  if (st == TKV_E_UNSUPPORTED) return two_calls();
  return st;
}

// ---- tkv_quant_attn_decode for callers that cannot hand over a workspace -----------------
// The split-K partials and arrival counters live in a fixed array in device memory that is part
// of the library image (every GPU the library runs on holds its own copy until the process
// ends).  In host code the array's name is only a stand-in for the symbol: the address that
// kernels may use is looked up once per device with that device current.
namespace {

constexpr size_t kStaticCounterWords = TKV_STATIC_MAX_HEADS;   // one per (sequence, KV head, four query heads)
constexpr size_t kStaticPartsBytes = TKV_STATIC_PARTS_BYTES;
constexpr size_t kStaticBytes = kStaticCounterWords * sizeof(uint32_t) + kStaticPartsBytes;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

constexpr int kMaxDevices = 64;
std::mutex g_static_mutex;
unsigned char* g_static_ptr[kMaxDevices] = {};  // device address of `scratch` on each device

int32_t static_scratch(unsigned char** ptr_out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TKV_E_HIP;
  std::lock_guard<std::mutex> lock(g_static_mutex);
  if (g_static_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return TKV_E_HIP;
    g_static_ptr[dev] = (unsigned char*)ptr;
  }
  *ptr_out = g_static_ptr[dev];
  return TKV_OK;
}

// Clears the arrival counters (a fill kernel, not a memset node: the call may be recorded
// into a graph by its caller).
__global__ __launch_bounds__(256) void clear_words_kernel(uint32_t* dst, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = 0u;
}

}  // namespace

extern "C" int32_t tkv_quant_attn_decode_static(const tkv_quant_desc* d, const tkv_quant_cache* c, const void* q,
                                                void* out, float sm_scale, void* stream) {
  int32_t st = check_decode_args(d, c, q, out);
  if (st != TKV_OK) return st;
  const int bh = d->batch * d->n_kv_heads * ((d->n_q_heads / d->n_kv_heads + 3) / 4);
  if ((size_t)bh > kStaticCounterWords) return TKV_E_WORKSPACE;
  unsigned char* base = nullptr;
  st = static_scratch(&base);
  if (st != TKV_OK) return st;
  uint32_t* arrivals = (uint32_t*)base;
  float* parts = (float*)(base + kStaticCounterWords * sizeof(uint32_t));
  hipStream_t s = (hipStream_t)stream;
  // the array keeps whatever the previous call left: the counters must start at zero
  TKV_LAUNCH(clear_words_kernel, dim3((bh + 255) / 256), 256, 0, s, arrivals, bh);
  return quant_attn_decode_impl(d, c, q, out, sm_scale, parts, kStaticPartsBytes / sizeof(float), arrivals, s);
}
