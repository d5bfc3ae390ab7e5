// tkv_quantize_append: cache update (Sec. 2.1, Eq. 2) and static quantization of the
// groups that become complete (Sec. 2.2, Eq. 4; Sec. 4.3: keys per channel, values
// per token; fp16 zero-point and scaler, Sec. 4.4).
#include "tkv_common.h"

// The quantizer's float32 operations are part of the contract (each a single
// rounded operation); keep the compiler from fusing any of them.
#pragma clang fp contract(off)

namespace {

struct QuantAppendParams {
  uint32_t* k_codes;
  uint32_t* v_codes;
  __half* k_scale;
  __half* k_zero;
  __half* v_scale;
  __half* v_zero;
  __half* k_resid;
  __half* v_resid;
  const __half* k_new;
  const __half* v_new;
  int32_t hkv, bits, group, residual, capacity;
  int32_t n_stride;   // rows per sequence in k_new / v_new
  int32_t unit_blocks;  // workgroups in x that quantize (four units of 64 tokens each); those behind them copy to the ring
  TkvSeqLens n_old;
  TkvSeqLens n_add;   // valid new rows per sequence (<= n_stride)
};

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

// The append in one launch; blockIdx.y = 2 head + (0: keys, 1: values).  blockIdx.x < unit_blocks
// quantizes: a wave takes one unit, two code blocks of 32 tokens (two groups of 32 or one of 64).  Lane cp + 8 tb holds tokens
// 8 tb .. 8 tb + 7 of two 8-channel pieces in registers (16 loads of 16 bytes in flight), the pieces
// being those that share a word of packed codes; minima and maxima are packed fp16 operations over
// the lane's tokens or channels and a butterfly over the lanes that share a group.  The finished
// words take their places in a per-wave image of the two blocks in LDS, which goes out in 16-byte
// stores.  Bound by the memory traffic: 512 B read and 48 to 160 B written per token-head; 131072
// tokens of 8 KV heads take 127 us at 2 bit (5.0 TB/s; a plain copy of a GiB runs at 5.2 on this card),
// 138 at 4.  With the divisions of Eq. 4 taken literally, the elements staged in LDS and picked out one
// by one, and a second launch for the ring, it was bound by vector instructions: 187 and 189 us.
// blockIdx.x >= unit_blocks copies new tokens that stay unquantized into the fp16 ring, 16 tokens per
// workgroup.  In the same launch only where no slot that it writes is still read as a
// token to quantize (the host checks).
template <int BITS, int GRP>
__global__ __launch_bounds__(256, 4) void quantize_append_kernel(QuantAppendParams p) {
  constexpr int NU = TKV_D / GRP;     // channel groups of a value row
  constexpr int GPU = 64 / GRP;       // token groups per unit
  constexpr int kBlkBytes = 512 * BITS;
  __shared__ __attribute__((aligned(16))) unsigned char image[4][2 * kBlkBytes];

  const int b = blockIdx.z, h = blockIdx.y / 2, tid = threadIdx.x, lane = tid % 64;
  const bool is_v = blockIdx.y % 2 != 0;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int n0 = p.n_old.n[b], n1 = n0 + p.n_add.n[b];
  const int ring = p.residual + GRP;
  const size_t bh = (size_t)b * p.hkv + h;
  if ((int)blockIdx.x >= p.unit_blocks) {
    const int nq1 = tkv::n_quantized(n1, p.residual, GRP);
    const int tok = max(n0, nq1) + 16 * ((int)blockIdx.x - p.unit_blocks) + tid / 16, part = tid % 16;
    if (tok >= n1) return;
    const __half* src = (is_v ? p.v_new : p.k_new) + (((size_t)b * p.n_stride + (size_t)(tok - n0)) * p.hkv + h) * TKV_D;
    __half* dst = (is_v ? p.v_resid : p.k_resid) + (bh * ring + (size_t)(tok % ring)) * TKV_D;
    reinterpret_cast<uint4*>(dst)[part] = reinterpret_cast<const uint4*>(src)[part];
    return;
  }
  const int j0 = tkv::n_quantized(n0, p.residual, GRP) / GRP;
  const int j1 = tkv::n_quantized(n1, p.residual, GRP) / GRP;
  const int j = j0 + GPU * (4 * (int)blockIdx.x + wave);  // first group of this wave's unit
  if (j >= j1) return;
  const int cp = lane % 8, tb = lane / 8;
  const int tok0 = GRP * j + 8 * tb;               // this lane's tokens: tok0 .. tok0 + 7
  const bool live = tok0 < GRP * j1;               // (32: the second group of the last unit may not exist)
  // The lane's rows (x[token][piece]): channels ch .. ch + 7 and ch + second .. (Called in either branch
  // below, not in front of them: values alive across a branch that the compiler turns into predicated
  // straight-line code would need a second set of registers.)
  u32x4 x[8][2];
  auto load = [&](int ch, int second) {
    const __half* news = (is_v ? p.v_new : p.k_new) + ((size_t)b * p.n_stride * p.hkv + h) * TKV_D + ch;
    const size_t pitch = (size_t)p.hkv * TKV_D;
    if (GRP * j >= n0) {  // (uniform) all of the unit's tokens are new: past the end re-reads the lane's first valid row
      const __half* row = news + (size_t)(live ? tok0 - n0 : GRP * j - n0) * pitch;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[i][0] = *reinterpret_cast<const u32x4*>(row);
        x[i][1] = *reinterpret_cast<const u32x4*>(row + second);
        row += pitch;
      }
    } else {
      const __half* olds = (is_v ? p.v_resid : p.k_resid) + bh * ring * TKV_D + ch;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int tok = live ? tok0 + i : GRP * j + i;
        const __half* row = tok < n0 ? olds + (size_t)(tok % ring) * TKV_D : news + (size_t)(tok - n0) * pitch;
        x[i][0] = *reinterpret_cast<const u32x4*>(row);
        x[i][1] = *reinterpret_cast<const u32x4*>(row + second);
      }
    }
  };
  unsigned char* img = image[wave] + (tb / 4) * kBlkBytes;  // this lane's block
  const int tb4 = tb % 4;                                    // 8-token piece inside the block
  const size_t blk0 = bh * (size_t)(p.capacity / TKV_BLK) + (size_t)j * (GRP / TKV_BLK);

  // One channel (values: token) after the other: left to itself the compiler starts all of them at
  // once and spills 40 registers.
  auto pin = [](uint32_t (&w)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(w[i]));
  };
  if (!is_v) {
    // ---- keys: (s, z) per channel over the group's tokens
    const int ch = 64 * (cp / 4) + 8 * (cp % 4);
    load(ch, 32);
    uint32_t mn[8], mx[8];  // channel pairs of the two pieces
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      mn[y] = mx[y] = x[0][y / 4][y % 4];
#pragma unroll
      for (int i = 1; i < 8; ++i) {
        const uint32_t w = x[i][y / 4][y % 4];
        mn[y] = pk_min(mn[y], w);
        mx[y] = pk_max(mx[y], w);
      }
      mn[y] = pk_min(mn[y], dpp<0x128 /* row_ror:8 */>(mn[y]));
      mx[y] = pk_max(mx[y], dpp<0x128>(mx[y]));
      {
        const auto a = __builtin_amdgcn_permlane16_swap(mn[y], mn[y], false, false);
        const auto c = __builtin_amdgcn_permlane16_swap(mx[y], mx[y], false, false);
        mn[y] = pk_min(a[0], a[1]);
        mx[y] = pk_max(c[0], c[1]);
      }
      if (GRP == 64) {
        const auto a = __builtin_amdgcn_permlane32_swap(mn[y], mn[y], false, false);
        const auto c = __builtin_amdgcn_permlane32_swap(mx[y], mx[y], false, false);
        mn[y] = pk_min(a[0], a[1]);
        mx[y] = pk_max(c[0], c[1]);
      }
    }
    uint32_t sc[8];
    uint32_t w[8];  // code words of the lane's tokens (4 bits: one word per token and piece)
#pragma unroll
    for (int piece = 0; piece < 2; ++piece) {
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = BITS == 4 || piece == 0 ? 0u : w[i];
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        const half2_t lo = as_half2(mn[4 * piece + y]), hi = as_half2(mx[4 * piece + y]);
        const half2_t s = {(_Float16)over_qmax<BITS>((float)hi[0] - (float)lo[0]),
                           (_Float16)over_qmax<BITS>((float)hi[1] - (float)lo[1])};
        sc[4 * piece + y] = __builtin_bit_cast(uint32_t, s);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const CodeRule<BITS> rule(s[e], lo[e]);
          const int shift = BITS * y + (BITS == 4 ? 0 : 4 * BITS * piece) + 16 * e;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t xw = x[i][piece][y];
            w[i] |= rule.code(as_half2(xw)[e]) << shift;
          }
          pin(w);
        }
      }
      if (BITS != 4 && piece == 0) continue;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = 4 * tb4 + i % 4, tau = i / 4, kb = cp % 4, wd = cp / 4;
        if (BITS == 1) {  // a word is shared by two lanes: bytes 0 and 2, bytes 1 and 3
          unsigned char* at = img + 4 * (64 * tau + r + 16 * kb) + wd;
          at[0] = (unsigned char)w[i];
          at[2] = (unsigned char)(w[i] >> 16);
        } else if (BITS == 2) {
          reinterpret_cast<uint32_t*>(img)[4 * (r + 16 * kb) + 2 * tau + wd] = w[i];
        } else {
          reinterpret_cast<uint32_t*>(img)[256 * tau + 4 * (r + 16 * kb) + 2 * wd + piece] = w[i];
        }
      }
    }
    if (live && (GRP == 64 ? tb == 0 : tb4 == 0)) {
      const size_t o = (bh * (size_t)(p.capacity / GRP) + (size_t)(tok0 / GRP)) * TKV_D + ch;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        *reinterpret_cast<u32x4*>(p.k_scale + o + 32 * q) = u32x4{sc[4 * q], sc[4 * q + 1], sc[4 * q + 2], sc[4 * q + 3]};
        *reinterpret_cast<u32x4*>(p.k_zero + o + 32 * q) = u32x4{mn[4 * q], mn[4 * q + 1], mn[4 * q + 2], mn[4 * q + 3]};
      }
    }
  } else {
    // ---- values: (s, z) per token over each group of GRP channels
    load(32 * (cp / 2) + 8 * (cp % 2), 16);
    _Float16 sc[8], ze[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // tokens
      uint32_t mn = x[i][0][0], mx = mn;
#pragma unroll
      for (int y = 1; y < 8; ++y) {
        const uint32_t v = x[i][y / 4][y % 4];
        mn = pk_min(mn, v);
        mx = pk_max(mx, v);
      }
      mn = pk_min(mn, dpp<0xB1 /* quad_perm 1 0 3 2 */>(mn));
      mx = pk_max(mx, dpp<0xB1>(mx));
      if (GRP == 64) {
        mn = pk_min(mn, dpp<0x4E /* quad_perm 2 3 0 1 */>(mn));
        mx = pk_max(mx, dpp<0x4E>(mx));
      }
      mn = pk_min(mn, (mn >> 16) | (mn << 16));
      mx = pk_max(mx, (mx >> 16) | (mx << 16));
      ze[i] = as_half2(mn)[0];
      sc[i] = (_Float16)over_qmax<BITS>((float)as_half2(mx)[0] - (float)ze[i]);
    }
    const int wd = cp / 2, hf = cp % 2;
    uint32_t w[8];  // code words of the lane's channels (4 bits: one word per channel and piece)
#pragma unroll
    for (int piece = 0; piece < 2; ++piece) {
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = BITS == 4 || piece == 0 ? 0u : w[i];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint32_t sz = pack2(sc[i], ze[i]);
        asm volatile("" : "+v"(sz));  // (worked out per piece rather than kept for all tokens)
        const CodeRule<BITS> rule(as_half2(sz)[0], as_half2(sz)[1]);
        const int shift = BITS * (i / 2) + (BITS == 4 ? 0 : 4 * BITS * piece) + 16 * (i % 2);
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          const uint32_t xw = x[i][piece][y];
#pragma unroll
          for (int e = 0; e < 2; ++e) w[2 * y + e] |= rule.code(as_half2(xw)[e]) << shift;
        }
        pin(w);
      }
      if (BITS != 4 && piece == 0) continue;
#pragma unroll
      for (int i = 0; i < 8; ++i) {  // channels
        const int l = 8 * hf + i + 16 * tb4;
        if (BITS == 1) {
          unsigned char* at = img + 4 * (64 * (wd / 2) + l) + wd % 2;
          at[0] = (unsigned char)w[i];
          at[2] = (unsigned char)(w[i] >> 16);
        } else if (BITS == 2) {
          reinterpret_cast<uint32_t*>(img)[4 * l + wd] = w[i];
        } else {
          reinterpret_cast<uint32_t*>(img)[256 * (wd / 2) + 4 * l + 2 * (wd % 2) + piece] = w[i];
        }
      }
    }
    if (live && (GRP == 64 ? cp % 4 == 0 : hf == 0)) {  // stored per block as [u][t]
      const size_t o = ((blk0 + tb / 4) * NU + cp / (GRP == 64 ? 4 : 2)) * TKV_BLK + 8 * tb4;
      *reinterpret_cast<u32x4*>(p.v_scale + o) = u32x4{pack2(sc[0], sc[1]), pack2(sc[2], sc[3]), pack2(sc[4], sc[5]), pack2(sc[6], sc[7])};
      *reinterpret_cast<u32x4*>(p.v_zero + o) = u32x4{pack2(ze[0], ze[1]), pack2(ze[2], ze[3]), pack2(ze[4], ze[5]), pack2(ze[6], ze[7])};
    }
  }
  // the wave's image: its LDS operations execute in order, other waves have images of their own
  __builtin_amdgcn_wave_barrier();
  unsigned char* dst = reinterpret_cast<unsigned char*>(is_v ? p.v_codes : p.k_codes) + blk0 * kBlkBytes;
  const int valid = min(GPU, j1 - j) * GRP / TKV_BLK * kBlkBytes;
#pragma unroll
  for (int q = 0; q < BITS; ++q) {
    const int at = 16 * (64 * q + lane);
    // (non-temporal: the codes do not push the prompt's rows out of the caches: 134 -> 127 us at 131072
    // tokens; the same hint on the row loads makes it slower)
    if (at < valid) __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(image[wave] + at), reinterpret_cast<u32x4*>(dst + at));
  }
}

}  // namespace

extern "C" int32_t tkv_quantize_append_ragged(const tkv_quant_desc* d, tkv_quant_cache* c, const void* k_new,
                                              const void* v_new, int32_t n_new, const int32_t* n_valid_host,
                                              void* stream) {
  int32_t st = tkv::check_quant_desc(d);
  if (st != TKV_OK) return st;
  if (!c || !c->seq_len_host || n_new < 0) return TKV_E_INVAL;
  if (n_new == 0) return TKV_OK;
  if (!k_new || !v_new || !c->k_codes || !c->k_scale || !c->k_zero || !c->v_codes || !c->v_scale ||
      !c->v_zero || !c->k_resid || !c->v_resid)
    return TKV_E_INVAL;

  QuantAppendParams p;
  int max_groups = 0, max_copy = 0;
  bool together = true;  // no ring slot written is one that a token to quantize is still read from
  for (int b = 0; b < d->batch; ++b) {
    const int64_t n0 = c->seq_len_host[b];
    const int32_t add = n_valid_host ? n_valid_host[b] : n_new;
    if (n0 < 0 || add < 0 || add > n_new) return TKV_E_INVAL;
    if (n0 + add > d->capacity) return TKV_E_CAPACITY;
    p.n_old.n[b] = (int32_t)n0;
    p.n_add.n[b] = add;
    const int32_t n1 = (int32_t)n0 + add;
    const int32_t g = d->group_size;
    const int groups = (tkv::n_quantized(n1, d->residual, g) - tkv::n_quantized((int32_t)n0, d->residual, g)) / g;
    const int32_t nq1 = tkv::n_quantized(n1, d->residual, g);
    const int copy = n1 - (n0 > nq1 ? (int32_t)n0 : nq1);
    const int32_t nq0 = tkv::n_quantized((int32_t)n0, d->residual, g);
    if (groups > 0 && nq0 < n0 && n1 - (d->residual + g) > nq0) together = false;
    if (groups > max_groups) max_groups = groups;
    if (copy > max_copy) max_copy = copy;
  }
  p.k_codes = (uint32_t*)c->k_codes;
  p.v_codes = (uint32_t*)c->v_codes;
  p.k_scale = (__half*)c->k_scale;
  p.k_zero = (__half*)c->k_zero;
  p.v_scale = (__half*)c->v_scale;
  p.v_zero = (__half*)c->v_zero;
  p.k_resid = (__half*)c->k_resid;
  p.v_resid = (__half*)c->v_resid;
  p.k_new = (const __half*)k_new;
  p.v_new = (const __half*)v_new;
  p.hkv = d->n_kv_heads;
  p.bits = d->bits;
  p.group = d->group_size;
  p.residual = d->residual;
  p.capacity = d->capacity;
  p.n_stride = n_new;

  hipStream_t s = (hipStream_t)stream;
  const int units = (max_groups * d->group_size + 63) / 64, unit_blocks = (units + 3) / 4, ring_blocks = (max_copy + 15) / 16;
  auto run = [&](int x_units, int x_ring) -> int32_t {
    if (x_units + x_ring == 0) return TKV_OK;
    p.unit_blocks = x_units;
    const dim3 grid(x_units + x_ring, 2 * d->n_kv_heads, d->batch);
    switch (d->bits * 100 + d->group_size) {
      case 132: TKV_LAUNCH((quantize_append_kernel<1, 32>), grid, 256, 0, s, p); break;
      case 232: TKV_LAUNCH((quantize_append_kernel<2, 32>), grid, 256, 0, s, p); break;
      case 432: TKV_LAUNCH((quantize_append_kernel<4, 32>), grid, 256, 0, s, p); break;
      case 164: TKV_LAUNCH((quantize_append_kernel<1, 64>), grid, 256, 0, s, p); break;
      case 264: TKV_LAUNCH((quantize_append_kernel<2, 64>), grid, 256, 0, s, p); break;
      case 464: TKV_LAUNCH((quantize_append_kernel<4, 64>), grid, 256, 0, s, p); break;
      default: return TKV_E_UNSUPPORTED;
    }
    return TKV_OK;
  };
  if (together) {
    st = run(unit_blocks, ring_blocks);
  } else {  // long appends onto a cache that already holds a tail: quantize first, then reuse its slots
    st = run(unit_blocks, 0);
    if (st == TKV_OK) st = run(0, ring_blocks);
  }
  if (st != TKV_OK) return st;
  for (int b = 0; b < d->batch; ++b) c->seq_len_host[b] += p.n_add.n[b];
  return TKV_OK;
}

extern "C" int32_t tkv_quantize_append(const tkv_quant_desc* d, tkv_quant_cache* c, const void* k_new,
                                       const void* v_new, int32_t n_new, void* stream) {
  return tkv_quantize_append_ragged(d, c, k_new, v_new, n_new, nullptr, stream);
}
