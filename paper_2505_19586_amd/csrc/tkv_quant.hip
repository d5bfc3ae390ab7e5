// tkv_quantize_append: cache update (Sec. 2.1, Eq. 2) and static quantization of the
// groups that become complete (Sec. 2.2, Eq. 4; Sec. 4.3: keys per channel, values
// per token; fp16 zero-point and scaler, Sec. 4.4).
#include "tkv_common.h"
#include "tkv_quantizer.h"

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
  int32_t hkv, residual, capacity;
  int32_t n_stride;      // rows per sequence in k_new / v_new
  int32_t quant_blocks;  // workgroups in x that quantize; those behind them copy to the ring
  int32_t ring_tokens;   // tokens that each of those takes
  TkvSeqLens n_old;
  TkvSeqLens n_add;   // valid new rows per sequence (<= n_stride)
};

using namespace tkv::quantizer;

// New tokens that stay unquantized, from the caller's rows to the fp16 ring: p.ring_tokens of those of sequence
// b, keys or values of one head, 256 threads (a token is 16 of them).
__device__ inline void ring_rows(const QuantAppendParams& p, int b, int h, bool is_v, int group, int piece, int tid) {
  constexpr int kPass = 64, kLoads = kPass / 16;
  const int n0 = p.n_old.n[b], n1 = n0 + p.n_add.n[b], ring = p.residual + group, part = tid % 16;
  const int first = max(n0, tkv::n_quantized(n1, p.residual, group)) + p.ring_tokens * piece, end = min(n1, first + p.ring_tokens);
  const __half* news = tkv::pick(is_v, p.k_new, p.v_new) + ((size_t)b * p.n_stride * p.hkv + h) * TKV_D;
  __half* olds = tkv::pick(is_v, p.k_resid, p.v_resid) + ((size_t)b * p.hkv + h) * ring * TKV_D;
  if (p.ring_tokens == 16) {  // one each (the pass below would load this token four times)
    const int tok = first + tid / 16;
    if (tok < end)
      reinterpret_cast<u32x4*>(olds + (size_t)(tok % ring) * TKV_D)[part] =
          reinterpret_cast<const u32x4*>(news + (size_t)(tok - n0) * p.hkv * TKV_D)[part];
    return;
  }
  for (int t0 = first + tid / 16; t0 < end; t0 += kPass) {
    u32x4 w[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      w[i] = reinterpret_cast<const u32x4*>(news + (size_t)(min(t0 + 16 * i, end - 1) - n0) * p.hkv * TKV_D)[part];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int tok = t0 + 16 * i;
      if (tok < end) reinterpret_cast<u32x4*>(olds + (size_t)(tok % ring) * TKV_D)[part] = w[i];
    }
  }
}

// The same where nothing is quantized, or after quantize_group_kernel: blockIdx.y = 0: keys, 1: values.  A thread takes 16 bytes of one token and
// head, so that a decode step's token of 8 heads is one workgroup (64 sequences, 32 heads: 2.2 us per
// call; 3.7 with a workgroup per head).
__global__ __launch_bounds__(256) void ring_kernel(QuantAppendParams p, int group) {
  tkv::fetch_arguments<sizeof(QuantAppendParams)>();
  const int b = blockIdx.z, i = blockIdx.x * 256 + threadIdx.x;
  const bool is_v = blockIdx.y != 0;
  const int n0 = p.n_old.n[b], n1 = n0 + p.n_add.n[b], ring = p.residual + group;
  const int first = max(n0, tkv::n_quantized(n1, p.residual, group));
  const int row = i / 16, part = i % 16, tok = first + row / p.hkv, h = row % p.hkv;
  if (tok >= n1) return;
  const __half* src = tkv::pick(is_v, p.k_new, p.v_new) + (((size_t)b * p.n_stride + (size_t)(tok - n0)) * p.hkv + h) * TKV_D;
  __half* dst = tkv::pick(is_v, p.k_resid, p.v_resid) + (((size_t)b * p.hkv + h) * ring + (size_t)(tok % ring)) * TKV_D;
  reinterpret_cast<uint4*>(dst)[part] = reinterpret_cast<const uint4*>(src)[part];
}

// Eq. 4's code with the stored fp16 s and z, literally: one subtraction, one division, rint.
__device__ inline float quant_code(float x, float z, float s, float qmax) {
  const float d = x - z;
  const float t = d / s;
  float c = rintf(t);
  c = fminf(fmaxf(c, 0.0f), qmax);
  return s == 0.0f ? 0.0f : c;
}

// The append of a few groups of 32 in one launch: blockIdx.x < quant_blocks is one group of one KV head, keys and
// values, whose elements 256 threads stage in LDS and pick out 32 each.  Bound by latency: a lane of
// quantize_append_kernel has 128 elements, which is less work in all but a longer chain (a decode step
// that completes a group of 8 heads: 4.1 us per call at 2 bit, 6.3 with that kernel; 4.5 and 7.3 at 4; the
// host's rule for which of them has more).  blockIdx.x >= quant_blocks copies
// to the ring, keys and values of one head, under the same condition as there.
template <int BITS>
__global__ __launch_bounds__(256) void quantize_group_kernel(QuantAppendParams p) {
  tkv::fetch_arguments<sizeof(QuantAppendParams)>();
  constexpr int GRP = TKV_BLK;        // a token group is one code block
  constexpr int NU = TKV_D / GRP;     // channel groups of a value row
  __shared__ __half kt[GRP][TKV_D];
  __shared__ __half vt[GRP][TKV_D];
  __shared__ float ks[TKV_D], kz[TKV_D];
  __shared__ float vs[GRP][NU], vz[GRP][NU];

  const int b = blockIdx.z, h = blockIdx.y, tid = threadIdx.x;
  const int n0 = p.n_old.n[b], n1 = n0 + p.n_add.n[b];
  if ((int)blockIdx.x >= p.quant_blocks) {
    ring_rows(p, b, h, false, GRP, (int)blockIdx.x - p.quant_blocks, tid);
    ring_rows(p, b, h, true, GRP, (int)blockIdx.x - p.quant_blocks, tid);
    return;
  }
  const int j0 = tkv::n_quantized(n0, p.residual, GRP) / GRP;
  const int j1 = tkv::n_quantized(n1, p.residual, GRP) / GRP;
  const int j = j0 + (int)blockIdx.x;
  if (j >= j1) return;
  const int ring = p.residual + GRP;
  const size_t bh = (size_t)b * p.hkv + h;
  const size_t n_groups_cap = (size_t)(p.capacity / GRP), n_blocks_cap = n_groups_cap;

  // stage the group's K rows and V rows (16-byte chunks)
  for (int i = tid; i < GRP * 16; i += 256) {
    const int t = i / 16, part = i % 16;
    const int tok = GRP * j + t;
    const uint4 *ksrc, *vsrc;
    if (tok < n0) {
      const size_t row = (bh * ring + (size_t)(tok % ring)) * TKV_D;
      ksrc = reinterpret_cast<const uint4*>(p.k_resid + row);
      vsrc = reinterpret_cast<const uint4*>(p.v_resid + row);
    } else {
      const size_t row = (((size_t)b * p.n_stride + (size_t)(tok - n0)) * p.hkv + h) * TKV_D;
      ksrc = reinterpret_cast<const uint4*>(p.k_new + row);
      vsrc = reinterpret_cast<const uint4*>(p.v_new + row);
    }
    reinterpret_cast<uint4*>(&kt[t][0])[part] = ksrc[part];
    reinterpret_cast<uint4*>(&vt[t][0])[part] = vsrc[part];
  }
  __syncthreads();

  constexpr float qmax = (float)((1 << BITS) - 1);
  if (tid < TKV_D) {
    // keys: one (s, z) per channel over the group's tokens
    const int c = tid;
    float mn = __half2float(kt[0][c]), mx = mn;
    for (int t = 1; t < GRP; ++t) {
      const float x = __half2float(kt[t][c]);
      mn = fminf(mn, x);
      mx = fmaxf(mx, x);
    }
    const float range = mx - mn;
    const float s32 = range / qmax;
    const __half s16 = __float2half_rn(s32);
    const __half z16 = __float2half_rn(mn);  // exact: mn is an fp16 value
    const size_t o = (bh * n_groups_cap + j) * TKV_D + c;
    p.k_scale[o] = s16;
    p.k_zero[o] = z16;
    ks[c] = __half2float(s16);
    kz[c] = __half2float(z16);
  } else {
    // values: one (s, z) per token and channel group; 128 threads cover GRP * NU = 128 pairs
    const int pr = tid - TKV_D;
    const int t = pr / NU, u = pr % NU;
    float mn = 0.f, mx = 0.f;
    for (int i = 0; i < GRP; ++i) {
      const int c = GRP * u + ((i + pr) % GRP);  // rotated start: fewer LDS bank conflicts
      const float x = __half2float(vt[t][c]);
      mn = i == 0 ? x : fminf(mn, x);
      mx = i == 0 ? x : fmaxf(mx, x);
    }
    const float range = mx - mn;
    const float s32 = range / qmax;
    const __half s16 = __float2half_rn(s32);
    const __half z16 = __float2half_rn(mn);
    const size_t o = ((bh * n_blocks_cap + j) * NU + u) * TKV_BLK + t;  // stored per block as [u][t]
    p.v_scale[o] = s16;
    p.v_zero[o] = z16;
    vs[t][u] = __half2float(s16);
    vz[t][u] = __half2float(z16);
  }
  __syncthreads();

  constexpr int nwords = TKV_D * BITS;  // words of one packed block: 32*128*bits/32
  constexpr int nfields = 32 / BITS;
  uint32_t* kdst = p.k_codes + (bh * n_blocks_cap + j) * (size_t)nwords;
  uint32_t* vdst = p.v_codes + (bh * n_blocks_cap + j) * (size_t)nwords;
#pragma unroll
  for (int w0 = 0; w0 < nwords; w0 += 256) {
    const int w = w0 + tid;
    if (nwords % 256 != 0 && w >= nwords) break;
    uint32_t kw = 0, vw = 0;
#pragma unroll
    for (int f = 0; f < nfields; ++f) {
      int t, c;
      tkv::k_code_elem(BITS, w, f, t, c);
      const float kc = quant_code(__half2float(kt[t][c]), kz[c], ks[c], qmax);
      kw |= (uint32_t)kc << (BITS * f);
      tkv::v_code_elem(BITS, w, f, t, c);
      const float vc = quant_code(__half2float(vt[t][c]), vz[t][c / GRP], vs[t][c / GRP], qmax);
      vw |= (uint32_t)vc << (BITS * f);
    }
    kdst[w] = kw;
    vdst[w] = vw;
  }
}

// The append of a few groups of 64 in one launch: a group's keys and values per workgroup of 1024 threads, by the quantizer of
// the attention's launch.  Bound by latency as well; a lane of quantize_append_kernel has eight times the elements: one group of
// 32 heads, a decode step's, 4.9 us per call at 2 bit, 6.6 with that kernel; 5.9 and 7.6 at 4.
template <int BITS>
__global__ __launch_bounds__(1024) void quantize_group64_kernel(QuantAppendParams p) {
  tkv::fetch_arguments<sizeof(QuantAppendParams)>();
  constexpr int GRP = 64;
  __shared__ __attribute__((aligned(16))) unsigned char smem[group_lds(GRP)];
  const int b = blockIdx.z, h = blockIdx.y, tid = threadIdx.x;
  const int n0 = p.n_old.n[b], n1 = n0 + p.n_add.n[b], ring = p.residual + GRP;
  if ((int)blockIdx.x >= p.quant_blocks) {  // two pieces of p.ring_tokens, keys and values
    const int part = __builtin_amdgcn_readfirstlane(tid / 256);
    ring_rows(p, b, h, part % 2 != 0, GRP, 2 * ((int)blockIdx.x - p.quant_blocks) + part / 2, tid % 256);
    return;
  }
  const int j = tkv::n_quantized(n0, p.residual, GRP) / GRP + (int)blockIdx.x;
  if (j >= tkv::n_quantized(n1, p.residual, GRP) / GRP) return;
  const size_t bh = (size_t)b * p.hkv + h, grp = bh * (size_t)(p.capacity / GRP) + j, blk = grp * (GRP / TKV_BLK);
  const GroupOut out = {p.k_codes + blk * (TKV_D * BITS), p.v_codes + blk * (TKV_D * BITS), p.k_scale + grp * TKV_D,
                        p.k_zero + grp * TKV_D,           p.v_scale + blk * (TKV_D / 2),    p.v_zero + blk * (TKV_D / 2)};
  static_assert(TKV_D / GRP * TKV_BLK == TKV_D / 2, "value scalers of a block");
  quantize_group_block<BITS, GRP, 1024>(
      [&](int kv, int t) {
        const int tok = GRP * j + t;
        const __half* olds = tkv::pick(kv != 0, p.k_resid, p.v_resid) + (bh * ring + (size_t)(tok % ring)) * TKV_D;
        const __half* news = tkv::pick(kv != 0, p.k_new, p.v_new) + (((size_t)b * p.n_stride + (size_t)(tok - n0)) * p.hkv + h) * TKV_D;
        return tok < n0 ? olds : news;
      },
      out, smem, tid);
}


// The append in one launch; blockIdx.y = 2 head + (0: keys, 1: values).  blockIdx.x < quant_blocks
// quantizes: a wave takes one unit, two code blocks of 32 tokens (two groups of 32 or one of 64).  Lane cp + 8 tb holds tokens
// 8 tb .. 8 tb + 7 of two 8-channel pieces in registers (16 loads of 16 bytes in flight), the pieces
// being those that share a word of packed codes; minima and maxima are packed fp16 operations over
// the lane's tokens or channels and a butterfly over the lanes that share a group.  The finished
// words take their places in a per-wave image of the two blocks in LDS, which goes out in 16-byte
// stores.  Bound by the memory traffic: 512 B read and 48 to 160 B written per token-head; 131072
// tokens of 8 KV heads take 127 us at 2 bit (5.0 TB/s; a plain copy of a GiB runs at 5.2 on this card),
// 138 at 4.  With the divisions of Eq. 4 taken literally, the elements staged in LDS and picked out one
// by one, and a second launch for the ring, it was bound by vector instructions: 187 and 189 us.
// blockIdx.x >= quant_blocks copies new tokens that stay unquantized into the fp16 ring, p.ring_tokens per
// workgroup.  In the same launch only where no slot that it writes is still read as a
// token to quantize (the host checks).
template <int BITS, int GRP>
__global__ __launch_bounds__(256, 4) void quantize_append_kernel(QuantAppendParams p) {
  tkv::fetch_arguments<sizeof(QuantAppendParams)>();
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
  if ((int)blockIdx.x >= p.quant_blocks) {
    ring_rows(p, b, h, is_v, GRP, (int)blockIdx.x - p.quant_blocks, tid);
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
  p.residual = d->residual;
  p.capacity = d->capacity;
  p.n_stride = n_new;

  hipStream_t s = (hipStream_t)stream;
  const int g = d->group_size, hkv = d->n_kv_heads, variant = d->bits * 100 + g;
  auto copy = [&]() -> int32_t {
    if (max_copy > 0) TKV_LAUNCH(ring_kernel, dim3((max_copy * hkv + 15) / 16, 2, d->batch), 256, 0, s, p, g);
    return TKV_OK;
  };
  // Which kernel: quantize_group_kernel up to two groups of 32 per compute unit (2 bits), three (4 bits)
  // or four (4 bits and the ring in a launch of its own), quantize_append_kernel beyond and for 1 bit (its
  // codes are one comparison).  Groups of 64: quantize_group64_kernel up to one workgroup per compute unit, those that copy included.  us per
  // call, the group kernel against the other, 8 heads from an empty cache: 2 bit, 400 tokens (64 groups)
  // 4.3, 6.3; 2000 (464) 5.7, 6.5; 3000 (712) 7.1, 6.6; 8200 (2016) 15.2, 11.5; 4 bit, 400 4.6, 7.3; 2000 6.1,
  // 7.6; 3000 7.5, 7.7; 6000 (1464) 11.8, 10.7; 1 bit, 400 6.8, 4.2.  Groups of 64: 2 bit, 300 tokens (16 groups) 5.0, 6.1; 2000 (232) 5.5,
  // 6.7; 3000 (352) 7.7, 6.9; 16 x 300 (256, and 128 copying) 9.5, 8.3; 4 bit, 300 5.9, 7.0; 2000 6.5, 7.8; 3000 9.6, 8.0; 16 x 300 11.2,
  // 10.2; 1 bit, 300 4.6, 4.0; 2000 5.0, 4.6; onto a tail, the copy a launch of its own: 2 bit, 2048 tokens onto 150 (256) 7.3, 9.1; 2600
  // (320) 9.6, 9.1; 32 heads, 500 onto 170 (256) 8.6, 9.7; 600 (320) 10.1, 9.8; 4 bit, 2048 8.5, 10.1; 2600 11.3, 10.3; 24 x 100 tokens onto 190
  // (384, short copies) 16.4, 18.1 on the other side of the line.
  const int few_groups = d->bits == 1 ? 0 : g == 64 ? 256 : d->bits == 2 ? 512 : together ? 768 : 1024;
  const int few_copies = g == 64 && together ? (max_copy + 63) / 64 : 0;
  const bool few = (max_groups + few_copies) * hkv * d->batch <= few_groups;
  const int quant_blocks = few ? max_groups : ((max_groups * g + 63) / 64 + 3) / 4;
  // Tokens per workgroup that copies: many behind a few workgroups that quantize (the copy is over long before
  // those are; 32 sequences of 300 tokens, 8 heads: 13.7 us per call, 21.7 with 64, 19.9 with 16), a few where
  // it is what the launch ends with (8 x 8000 tokens, 1 bit / 64: 45 us, 48 with 256).
  p.ring_tokens = few ? 32 : together && quant_blocks <= 16 ? 256 : 16;
  const int per_block = few && g == 64 ? 2 * p.ring_tokens : p.ring_tokens;
  const int ring_blocks = (max_copy + per_block - 1) / per_block;
  auto run = [&](int x_quant, int x_ring) -> int32_t {
    if (x_quant + x_ring == 0) return TKV_OK;
    p.quant_blocks = x_quant;
    const dim3 grid(x_quant + x_ring, few ? hkv : 2 * hkv, d->batch);
    switch (variant + (few ? 1000 : 0)) {
      case 1232: TKV_LAUNCH((quantize_group_kernel<2>), grid, 256, 0, s, p); break;
      case 1432: TKV_LAUNCH((quantize_group_kernel<4>), grid, 256, 0, s, p); break;
      case 1264: TKV_LAUNCH((quantize_group64_kernel<2>), grid, 1024, 0, s, p); break;
      case 1464: TKV_LAUNCH((quantize_group64_kernel<4>), grid, 1024, 0, s, p); break;
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
  if (max_groups == 0) {
    st = copy();
  } else if (together) {
    st = run(quant_blocks, ring_blocks);
  } else {  // long appends onto a cache that already holds a tail: quantize first, then reuse its slots
    st = run(quant_blocks, 0);
    if (st == TKV_OK) st = few ? copy() : run(0, ring_blocks);
  }
  if (st != TKV_OK) return st;
  for (int b = 0; b < d->batch; ++b) c->seq_len_host[b] += p.n_add.n[b];
  return TKV_OK;
}

extern "C" int32_t tkv_quantize_append(const tkv_quant_desc* d, tkv_quant_cache* c, const void* k_new,
                                       const void* v_new, int32_t n_new, void* stream) {
  return tkv_quantize_append_ragged(d, c, k_new, v_new, n_new, nullptr, stream);
}
