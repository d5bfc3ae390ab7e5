// Eq. 4's quantizer (Sec. 2.2): pieces shared by the append kernels and the attention's in-launch append.
// Its float32 operations are part of the contract, each a single rounded one: no function here lets the compiler
// fuse any of them.
#pragma once

#include "tkv_common.h"

namespace tkv {
namespace quantizer {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Eq. 4's code with the stored fp16 s and z: clamp(rint(RN32(d / s)), 0, 2^b - 1), d = RN32(x - z), without
// the division.  The decision points h = j - 1/2 make s h exact in float32 (11 + 5 bits), and two
// different float32 numbers d and s h are at least 2^-24 apart relatively, which is more than half
// an ulp of the quotient at every h, so RN32(d / s) lies on the same side of h as d of s h and
// equals h exactly when d = s h: rint then goes to the even neighbour.  The clamp is the number of
// decision points there are.  Where s is 0 or not finite every comparison is with NaN: code 0, which is
// what the division gives as well (0 or NaN, and the clamp takes NaN to 0); x = NaN has code 0 likewise.
template <int BITS>
struct CodeRule {
  float z, s, inv;
  float t1, t2, t3;
  __device__ CodeRule(_Float16 scale, _Float16 zero) {
#pragma clang fp contract(off)
    z = (float)zero;
    const bool usable = scale > (_Float16)0.f && scale < (_Float16)INFINITY;
    s = usable ? (float)scale : NAN;
    if (BITS == 4) {
      inv = usable ? __builtin_amdgcn_rcpf(s) : 0.f;
      t1 = 0.5f * s;
    } else {
      t1 = 0.5f * s, t2 = 1.5f * s, t3 = 2.5f * s;
    }
  }
  __device__ uint32_t code(_Float16 x) const {
#pragma clang fp contract(off)
    const float d = (float)x - z;
    if (BITS == 1) return d > t1 ? 1u : 0u;
    if (BITS == 2) return (d > t1 ? 1u : 0u) + (d >= t2 ? 1u : 0u) + (d > t3 ? 1u : 0u);
    // 4 bits: a lower neighbour c0 in {code - 1, code} from an approximate quotient (off by far less
    // than the quarter that it is shifted by), then the one decision point above it; a tie goes up
    // from an odd c0
    const float magic = 12582912.0f;  // 1.5 x 2^23: the sum holds the rounded integer in its low bits
    const float m = __builtin_amdgcn_fmed3f(__builtin_fmaf(d, inv, -0.25f), -0.25f, 14.0f) + magic;  // NaN: the lower end
    const float c0 = m - magic;
    const float T = __builtin_fmaf(s, c0, t1);  // exact; unordered with d where either is NaN: never passed
    const uint32_t mb = __builtin_bit_cast(uint32_t, m);
    const uint32_t db = __builtin_bit_cast(uint32_t, d) + (mb & 1u);  // d >= 0, T > 0: ordered like integers
    return (mb & 15u) + (!__builtin_isunordered(d, T) && db > __builtin_bit_cast(uint32_t, T) ? 1u : 0u);
  }
};

// x / (2^b - 1) correctly rounded: Markstein's correction of x RN(1/q) (q = 3 and 15 checked for every
// mantissa; x is a difference of fp16 numbers, far from both ends of the exponent range, or not finite
// and then left alone).
template <int BITS>
__device__ inline float over_qmax(float x) {
#pragma clang fp contract(off)
  if (BITS == 1) return x;
  constexpr float q = (float)((1 << BITS) - 1), y = 1.0f / q;
  const float a = x * y;
  return a < INFINITY ? __builtin_fmaf(__builtin_fmaf(-q, a, x), y, a) : a;
}

// packed fp16 minimum / maximum (as the instruction has them: the library functions quiet NaNs first)
__device__ inline uint32_t pk_min(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ inline uint32_t pk_max(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int CTRL>
__device__ inline uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
__device__ inline half2_t as_half2(uint32_t w) { return __builtin_bit_cast(half2_t, w); }
__device__ inline uint32_t pack2(_Float16 lo, _Float16 hi) {
  const half2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, v);
}

// One group of GRP tokens of one KV head quantized by a whole workgroup of NT >= 512 threads (row(kv, t): keys or values of its
// token t): codes, scalers and zero-points as quantize_append_kernel writes them.  smem: group_lds(GRP) bytes.  Contains
// barriers; every store has completed at the end, so that the workgroup may load the group like any other.  Bound by
// latency (one round trip for the rows, three barriers): about 2.5 us in front of the attention of the workgroup that owns the
// tail.  With unpadded rows and a scaler per element read on its own it was 5 to 8.
struct GroupOut {
  uint32_t *k_codes, *v_codes;                        // the group's first block
  __half *k_scale, *k_zero, *v_scale, *v_zero;        // of the group; of its first block
};
constexpr int kGroupPitch = TKV_D * 2 + 16;  // LDS bytes of a staged row (padded against bank conflicts)
constexpr int group_lds(int grp) { return 2 * grp * kGroupPitch + 2 * 4 * 64 * 4 + 2 * 64 * 4 + 2 * 128 * 4; }
template <int BITS, int GRP, int NT, typename Row>
__device__ inline void quantize_group_block(const Row& row, const GroupOut& out, unsigned char* smem, int tid) {
#pragma clang fp contract(off)
  constexpr int NU = TKV_D / GRP;   // channel groups of a value row
  constexpr int NB = GRP / TKV_BLK; // code blocks
  constexpr int kRow = kGroupPitch;
  static_assert(NT >= 512 && GRP * NU == TKV_D, "256 threads for the keys, two for each of 128 value groups");
  unsigned char* rows = smem;                                             // [2][GRP][128] fp16: keys, values
  uint32_t* part = reinterpret_cast<uint32_t*>(smem + 2 * GRP * kRow);    // [2][4][64] minima, maxima of channel pairs
  uint32_t* ksz = part + 2 * 4 * 64;                                      // [2][64] scalers, zero-points of channel pairs
  uint32_t* vsz = ksz + 2 * 64;                                           // [128] (scaler, zero-point) of token t, channel group u
  constexpr int kPieces = 2 * GRP * 16, kRounds = (kPieces + NT - 1) / NT;  // 16-byte pieces, all in one round trip
  u32x4 piece[kRounds];
#pragma unroll
  for (int y = 0; y < kRounds; ++y) {
    const int i = min(tid + NT * y, kPieces - 1);
    piece[y] = reinterpret_cast<const u32x4*>(row(i / (GRP * 16), i / 16 % GRP))[i % 16];
  }
#pragma unroll
  for (int y = 0; y < kRounds; ++y) {
    const int i = tid + NT * y;
    if (i < kPieces) reinterpret_cast<u32x4*>(rows + i / 16 * kRow)[i % 16] = piece[y];
  }
  __syncthreads();
  if (tid < 256) {  // keys: a wave takes a quarter of the tokens, a lane two channels
    const int pair = tid % 64, quarter = tid / 64;
    const uint32_t* col = reinterpret_cast<const uint32_t*>(rows + quarter * (GRP / 4) * kRow) + pair;
    uint32_t mn = col[0], mx = mn;
#pragma unroll
    for (int t = 1; t < GRP / 4; ++t) {
      const uint32_t w = col[t * (kRow / 4)];
      mn = pk_min(mn, w), mx = pk_max(mx, w);
    }
    part[quarter * 64 + pair] = mn;
    part[256 + quarter * 64 + pair] = mx;
  } else if (tid < 512) {  // values: two lanes per token and channel group, half of its channels each
    const int x = tid - 256, pr = x / 2, t = pr / NU, u = pr % NU;
    const u32x4* src = reinterpret_cast<const u32x4*>(rows + (GRP + t) * kRow + 2 * GRP * u) + (x % 2) * (GRP / 16);
    uint32_t mn = 0, mx = 0;
#pragma unroll
    for (int i = 0; i < GRP / 16; ++i) {
      const u32x4 w = src[i];
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        const uint32_t v = w[y];
        mn = i + y == 0 ? v : pk_min(mn, v);
        mx = i + y == 0 ? v : pk_max(mx, v);
      }
    }
    mn = pk_min(mn, dpp<0xB1 /* quad_perm 1 0 3 2 */>(mn));
    mx = pk_max(mx, dpp<0xB1>(mx));
    mn = pk_min(mn, (mn >> 16) | (mn << 16));
    mx = pk_max(mx, (mx >> 16) | (mx << 16));
    const _Float16 z = as_half2(mn)[0], s = (_Float16)over_qmax<BITS>((float)as_half2(mx)[0] - (float)z);
    if (x % 2 == 0) {
      vsz[pr] = pack2(s, z);
      const size_t o = (size_t)((t / TKV_BLK) * NU + u) * TKV_BLK + t % TKV_BLK;  // stored per block as [u][t]
      reinterpret_cast<_Float16*>(out.v_scale)[o] = s;
      reinterpret_cast<_Float16*>(out.v_zero)[o] = z;
    }
  }
  __syncthreads();
  if (tid < 64) {
    uint32_t mn = part[tid], mx = part[256 + tid];
#pragma unroll
    for (int y = 1; y < 4; ++y) mn = pk_min(mn, part[64 * y + tid]), mx = pk_max(mx, part[256 + 64 * y + tid]);
    const half2_t lo = as_half2(mn), hi = as_half2(mx);
    const uint32_t s = pack2((_Float16)over_qmax<BITS>((float)hi[0] - (float)lo[0]), (_Float16)over_qmax<BITS>((float)hi[1] - (float)lo[1]));
    ksz[tid] = s;
    ksz[64 + tid] = mn;
    reinterpret_cast<uint32_t*>(out.k_scale)[tid] = s;
    reinterpret_cast<uint32_t*>(out.k_zero)[tid] = mn;
  }
  __syncthreads();
  // codes: field f and field f + kFields / 2 of a word are two adjacent channels of a token (keys), one channel of
  // two adjacent tokens (values)
  constexpr int kWords = TKV_D * BITS, kHalf = 16 / BITS;  // words of one packed block, fields of half a word
  auto rule_pair = [](uint32_t x, uint32_t s, uint32_t z) -> uint32_t {
    const CodeRule<BITS> r0(as_half2(s)[0], as_half2(z)[0]), r1(as_half2(s)[1], as_half2(z)[1]);
    return r0.code(as_half2(x)[0]) | r1.code(as_half2(x)[1]) << 16;
  };
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  for (int w0 = 64 * wave; w0 < 2 * NB * kWords; w0 += NT) {  // (uniform: a wave's words are keys or values of one block)
    const bool is_v = w0 >= NB * kWords;
    const int word = (is_v ? w0 - NB * kWords : w0) + lane, blk = word / kWords, w = word % kWords;
    uint32_t acc = 0;
    if (!is_v) {
#pragma unroll
      for (int f = 0; f < kHalf; ++f) {
        int t, c;
        k_code_elem(BITS, w, f, t, c);
        const uint32_t x = *reinterpret_cast<const uint32_t*>(rows + (t + TKV_BLK * blk) * kRow + 2 * c);
        acc |= rule_pair(x, ksz[c / 2], ksz[64 + c / 2]) << (BITS * f);
      }
    } else {
#pragma unroll
      for (int f = 0; f < kHalf; ++f) {
        int t, c;
        v_code_elem(BITS, w, f, t, c);
        t += TKV_BLK * blk;
        const unsigned char* at = rows + (GRP + t) * kRow + 2 * c;
        const uint32_t x = *reinterpret_cast<const uint16_t*>(at) | (uint32_t)*reinterpret_cast<const uint16_t*>(at + kRow) << 16;
        const uint32_t a = vsz[t * NU + c / GRP], d = vsz[(t + 1) * NU + c / GRP];  // (scaler, zero-point) of the two tokens
        acc |= rule_pair(x, (a & 0xFFFFu) | d << 16, a >> 16 | (d & 0xFFFF0000u)) << (BITS * f);
      }
    }
    (is_v ? out.v_codes : out.k_codes)[word] = acc;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

}  // namespace quantizer
}  // namespace tkv
