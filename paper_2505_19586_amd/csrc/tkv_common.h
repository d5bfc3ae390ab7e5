// Internal helpers shared by the tkv HIP sources (gfx950 only).
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>
#include <utility>

#include "tkv.h"
#include "tkv_debug.h"

#define TKV_D 128      // head_dim
#define TKV_BLK 32     // tokens per block of packed codes (the quantization group is 32 or 64)
#define TKV_WAVE 64

// Room of the partial attention result of one chunk and one query head, in floats: max logit (in log2
// units after scaling), sum of weights, the weighted V sum, two unused words.  merge_chunks has the pairs of all chunks
// behind the sums of all chunks (part_o, part_ml); attn_merge_kernel has each pair, then two unused words, in front of its sum.
#define TKV_PART_O 4
#define TKV_PART_STRIDE (TKV_D + TKV_PART_O)

// Upper bound on split-K chunks per (sequence, KV head), tail chunk excluded.
#define TKV_MAX_CHUNKS 256

#define TKV_HIP_TRY(expr)                      \
  do {                                         \
    hipError_t _e = (expr);                    \
    if (_e != hipSuccess) return TKV_E_HIP;    \
  } while (0)

struct TkvSeqLens {
  int32_t n[TKV_MAX_BATCH];
};

namespace tkv {

// The new tokens of a step that a quantized layer's attention call also appends:
// k_new, v_new fp16 [B][n_stride][Hkv][D], the first n_add[b] rows of sequence b.
struct QuantNewTokens {
  const __half* k_new;
  const __half* v_new;
  int32_t n_stride;
  bool complete;  // some sequence completes a quantization group with them (one, of tokens that are in the ring already)
  TkvSeqLens n_add;
};

// Number of quantized tokens of a sequence of n tokens (residual w, group g).
__host__ __device__ inline int32_t n_quantized(int32_t n, int32_t w, int32_t g) {
  return n >= w ? ((n - w) / g) * g : 0;
}

// Kernel launch whose status is the launch's own return value: the process-wide "last error" of
// the HIP runtime is neither read nor cleared, so an earlier error of the calling program is
// never reported as the library's and never erased.
template <typename... KArgs, typename... Args>
inline int32_t launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t s,
                      Args&&... args) {
  static_assert(sizeof...(KArgs) == sizeof...(Args), "kernel argument count");
  std::tuple<KArgs...> vals{static_cast<KArgs>(std::forward<Args>(args))...};
  void* ptrs[sizeof...(KArgs)];
  std::apply([&](auto&... v) { int i = 0; ((ptrs[i++] = (void*)&v), ...); }, vals);
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds_bytes, s) == hipSuccess
             ? TKV_OK
             : TKV_E_HIP;
}
#define TKV_LAUNCH(kernel, grid, block, lds, stream, ...)                                                  \
  do {                                                                                                     \
    if (tkv::launch(kernel, grid, block, lds, stream, __VA_ARGS__) != TKV_OK) return TKV_E_HIP;            \
  } while (0)

// Compute units that kernels of this stream may use: those of its compute-unit mask
// (hipExtStreamCreateWithCUMask), all of the device's for an ordinary stream.  Launches that
// aim at one workgroup per compute unit size themselves with it.
inline int stream_compute_units(hipStream_t s) {
  static const int device_cus = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      v = 0;
    return v > 0 ? v : 256;
  }();
  uint32_t mask[16] = {0};
  if (hipExtStreamGetCUMask(s, 16, mask) != hipSuccess) {
    (void)hipGetLastError();
    return device_cus;
  }
  int cus = 0;
  for (uint32_t m : mask) cus += __builtin_popcount(m);
  return cus > 0 && cus <= device_cus ? cus : device_cus;
}

int32_t check_quant_desc(const tkv_quant_desc* d);
// Merges [n_heads_total][n_parts][TKV_PART_STRIDE] float partials (max in log2 units, sum,
// weighted V) into fp16 [n_heads_total][D].
int32_t launch_attn_merge(const float* parts, __half* out, int n_heads_total, int n_parts, hipStream_t s);
int32_t check_sparse_desc(const tkv_sparse_desc* d);

// Device-visible address of a caller's buffer.  kDevHostOnly: pinned host memory only
// (TKV_E_NOTPINNED otherwise); kDevAny: pinned host memory or device memory; kDevDeviceOnly:
// device memory only (TKV_E_INVAL otherwise).
enum DevView { kDevHostOnly, kDevAny, kDevDeviceOnly };
inline int32_t device_view(const void* ptr, DevView mode, const void** dev) {
  hipPointerAttribute_t attr;
  const hipError_t e = hipPointerGetAttributes(&attr, ptr);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    if (mode == kDevDeviceOnly) return TKV_E_INVAL;
    return e == hipErrorInvalidValue ? TKV_E_NOTPINNED : TKV_E_HIP;
  }
  if (attr.type == hipMemoryTypeDevice) {
    if (mode == kDevHostOnly) return TKV_E_NOTPINNED;
    *dev = ptr;
    return TKV_OK;
  }
  if (mode == kDevDeviceOnly) return TKV_E_INVAL;
  if (attr.type != hipMemoryTypeHost || attr.devicePointer == nullptr) return TKV_E_NOTPINNED;
  *dev = attr.devicePointer;
  return TKV_OK;
}

// ---- cross-chunk merge by the last workgroup of a (sequence, KV head) --------------------
// Partials cross workgroups through device-scope stores and loads (they bypass the caches
// that are not coherent between workgroups).  Such loads are served slowly, one load
// instruction after the other, so the merge uses as few and as wide ones as it can: all of
// them are issued before the first is used.

typedef float tkv_floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t tkv_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t tkv_u32x2 __attribute__((ext_vector_type(2)));

// Device-scope loads of 4, 8 or 16 bytes through a buffer descriptor over [base, base + bytes)
// (base must be uniform over the wave; byte offsets are 32 bit).  The "sc1" cache policy makes
// them device-scope like an agent-scope atomic load, but up to 16 bytes wide, and the compiler
// itself tracks when their results arrive.  An offset at or beyond `bytes` reads nothing and
// returns 0, which spares the callers a branch around loads they do not need (kNone).
struct AgentBuf {
  static constexpr uint32_t kNone = 0xFFFFFFF0u;
  __amdgpu_buffer_rsrc_t r;
  __device__ AgentBuf(const void* base, uint32_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000)) {}
  __device__ tkv_u32x4 x4(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 16); }
  __device__ tkv_u32x2 x2(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 16); }
  __device__ uint32_t x1(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 16); }
};

// Where chunk k of a query head lies in the head's n_chunks * TKV_PART_STRIDE floats: the weighted V
// sums of all chunks first, then their (maximum, sum) pairs side by side: 64 of them are four lines
// instead of 64, and such loads cost by the line.
__device__ inline float* part_o(float* head, int k) { return head + (size_t)k * TKV_D; }
__device__ inline float* part_ml(float* head, int n_chunks, int k) { return head + (size_t)n_chunks * TKV_D + 2 * k; }

// Fetches the BYTES of a kernel's arguments at its start, all lines in one round trip.  (The compiler loads an argument shortly before
// its use; every line that is touched for the first time there is a round trip of its own on the way to the first load of data.)
// us per pass without and with it, in turn: sparse decode step, 4095 tokens, 32/8 heads 23.6, 23.1; dynamic channels, 98101 tokens (three
// launches) 63.9, 63.3; quantized decode, 2 bit, 2000 tokens 10.45, 10.4; 4 bit, 32770 16.9, 16.7; 1 bit, 98413 21.4, 21.25.  No difference: dense
// preference score of 131072 keys (eight launches), 131072 tokens quantized (where a compute unit's later workgroups find the lines cached;
// 64 x 300 tokens, 2 bit, 32/32 heads 105.8, 107.4).  The float32 attention kernel does without: 0.1 slower with it.
template <int BYTES>
__device__ inline void fetch_arguments() {
  static_assert(BYTES <= 16 * 64, "lines");
  const auto* words = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
  uint32_t w[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) w[i] = words[16 * (64 * i < BYTES ? i : 0)];
  asm volatile("" ::"s"(w[0]), "s"(w[1]), "s"(w[2]), "s"(w[3]), "s"(w[4]), "s"(w[5]), "s"(w[6]), "s"(w[7]), "s"(w[8]), "s"(w[9]),
               "s"(w[10]), "s"(w[11]), "s"(w[12]), "s"(w[13]), "s"(w[14]), "s"(w[15]));
}

// One of two of a kernel's pointer arguments.  (Chosen per lane as they stand, the compiler chooses between their addresses among the
// arguments and loads the pointer from there: a round trip more.  In the append of a completed group and the float32 kernel's tails: 4 bit,
// 32/32 heads, 20480 + 16857 tokens 54.5 us per decode step, 53.1 now.)
template <typename T>
__device__ inline T* pick(bool second, T* a, T* b) {
  typedef __attribute__((address_space(1))) T Global;  // (named, so that loads and stores through it stay global ones)
  Global *ga = (Global*)a, *gb = (Global*)b;
  asm("" : "+s"(ga), "+s"(gb));
  return (T*)(second ? gb : ga);
}

// Cross-lane exchanges without LDS traffic: quads, halves of a row of 16 lanes and rows by data-parallel primitives, rows
// and half-waves against each other by register swaps.
template <int CTRL>
__device__ inline float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <typename F>
__device__ inline float over_rows(float v, F f) {  // every lane: f over the four lanes with its place in a row
  const auto a = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, v), false, false);
  const uint32_t a0 = a[0], a1 = a[1];
  v = f(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1));
  const auto c = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, v), false, false);
  const uint32_t c0 = c[0], c1 = c[1];
  return f(__builtin_bit_cast(float, c0), __builtin_bit_cast(float, c1));
}
template <typename F>
__device__ inline float over_wave(float v, F f) {
  v = f(v, dpp<0xB1>(v));   // quad_perm: lane ^ 1
  v = f(v, dpp<0x4E>(v));   // quad_perm: lane ^ 2
  v = f(v, dpp<0x141>(v));  // row_half_mirror: the other quad of eight lanes
  v = f(v, dpp<0x140>(v));  // row_mirror: the other eight of the row
  return over_rows(v, f);
}
// ... over the lanes whose number is the same modulo H (4 or 8)
template <int H, typename F>
__device__ inline float over_stride(float v, F f) {
  static_assert(H == 4 || H == 8, "lanes of a row in steps of H");
  v = f(v, dpp<0x128>(v));                  // row_ror:8
  if (H == 4) v = f(v, dpp<0x124>(v));      // row_ror:4
  return over_rows(v, f);
}
struct MaxOf { __device__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct SumOf { __device__ float operator()(float a, float b) const { return a + b; } };

// head0: partials of the G heads of this KV head, n_chunks * TKV_PART_STRIDE floats each (part_o, part_ml); out0: fp16
// [G][128].  lds: merge_lds_floats(KS, G, n_chunks, nthr) floats.  Called by every thread of the
// workgroup (nthr a multiple of 64).  KS: chunk classes summed side by side (2 to
// 4, so that the 32 G KS items are at most one per thread); kPer: loads in flight per thread.  64
// chunks come in one round of loads where KS kPer >= 64.
// Bound by its round trip and by what one compute unit can load (64 chunks of 8 heads: 264 KiB).  A wave fetches the
// maxima and sums of its own head (of two heads where 32 KS items are no whole number of waves) and its channels at once and
// works out the chunks' weights by itself: one round trip, one barrier.  us per call with the pairs fetched by the whole
// workgroup before everything else and the weights shared through LDS / so: quantized attention, 2 bit, 32/8 heads, 2000
// tokens (7 chunks) 12.1, 10.9; 8000 13.5, 12.5; 131000 (32 chunks) 29.3, 28.0; 4/1, 50000 (132 chunks) 17.2, 15.5; 1 bit, 32/4,
// 98413 (64 chunks of 8 heads) 23.0, 21.9.  (With the pairs in front of the chunks' sums, a line each: 16.6 and 23.7 for the last two.)
// More than 64 chunks, one sequence of one to three KV heads (4/1 from 25000 tokens on): their pairs come in a second and third
// round trip, which costs less than the workgroup's rounds did: 2 bit, 4/1, 131071 tokens (256 chunks) 22.5, 19.6; 8/2 (128) 19.7, 17.7; 8/1, 400000
// (256 chunks of 8 heads) 34.4, 31.8.
constexpr int merge_lds_floats(int KS, int G, int n_chunks, int nthr) {
  return nthr / 64 * (KS == 3 ? 2 : 1) * ((n_chunks + 63) / 64 * 64) + G * KS * TKV_D + G;
}
template <int KS = 4, int kPer = 16>
__device__ inline void merge_chunks(const float* head0, int G, int n_chunks, __half* out0, float* lds, int tid,
                                    int nthr) {
  constexpr int kItems = 32 * KS;          // item = (head, chunk class ks, channel quad c4): chunks ks, ks + KS, ...
  constexpr int kTwo = KS == 3 ? 2 : 1;    // heads that a wave's 64 items may belong to
  static_assert(KS == 3 || kItems % 64 == 0, "a wave's items are one head's");
  const int lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int cw_len = (n_chunks + 63) / 64 * 64;
  float* cw = lds + wave * kTwo * cw_len;                  // [kTwo][cw_len] this wave's chunk weights
  float* red = lds + nthr / 64 * kTwo * cw_len;            // [G][KS][128]
  float* Ls = red + G * KS * TKV_D;                        // [G]
  const uint32_t head_bytes = (uint32_t)n_chunks * TKV_PART_STRIDE * 4u;
  const AgentBuf pb(head0, (uint32_t)G * head_bytes);
  for (int first = 64 * wave; first < G * kItems; first += nthr) {
    const uint32_t item = (uint32_t)(first + lane);
    const bool on = item < (uint32_t)(G * kItems);
    const int h0 = (int)((uint32_t)first / kItems), h1 = kTwo == 1 ? h0 : min((int)((uint32_t)(first + 63) / kItems), G - 1);
    const int hh = on ? (int)(item / kItems) : h0, r = (int)(item % kItems);
    const int ks = r / 32, c4 = r % 32, mine = on ? n_chunks : 0;
    const uint32_t base = (uint32_t)hh * head_bytes + 16u * (uint32_t)c4;
    auto pair_of = [&](int z, int k) {  // (maximum, sum) of chunk k of the wave's head z
      return pb.x2(k < n_chunks ? (uint32_t)(z ? h1 : h0) * head_bytes + (uint32_t)n_chunks * (TKV_D * 4u) + 8u * (uint32_t)k : AgentBuf::kNone);
    };
    tkv_u32x2 ml[kTwo];
#pragma unroll
    for (int z = 0; z < kTwo; ++z) ml[z] = pair_of(z, lane);
    tkv_u32x4 ov[kPer];
    auto request = [&](int k0) {
#pragma unroll
      for (int y = 0; y < kPer; ++y) {
        const int k = k0 + KS * y + ks;
        // (one comparison: two make a branch per load, and the compiler waits for the loads before a branch to be done)
        ov[y] = pb.x4(k < mine ? base + (uint32_t)k * (TKV_D * 4u) : AgentBuf::kNone);
      }
    };
    request(0);
    __builtin_amdgcn_sched_barrier(0);  // everything is requested before the first result is waited for
#pragma unroll
    for (int z = 0; z < kTwo; ++z) {
      // (elements copied out before the cast: a bit cast applied directly to a vector element
      // reads element 0 with this compiler)
      const uint32_t v_max = ml[z].x, v_sum = ml[z].y;
      const float m0 = lane < n_chunks ? __uint_as_float(v_max) : -INFINITY;
      float M = m0;
      for (int k = 64 + lane; k < cw_len; k += 64) {  // (more than 64 chunks)
        const uint32_t v = pair_of(z, k).x;
        M = fmaxf(M, k < n_chunks ? __uint_as_float(v) : -INFINITY);
      }
      M = over_wave(M, MaxOf{});
      float L = 0.f;
      auto weigh = [&](int k, float m, float l) {
        const float w = m == -INFINITY ? 0.f : exp2f(m - M);
        cw[z * cw_len + k] = w;  // (read below by this wave alone, whose LDS operations execute in order)
        L = __builtin_fmaf(l, w, L);
      };
      weigh(lane, m0, __uint_as_float(v_sum));  // (an absent chunk's pair reads as zeros)
      for (int k = 64 + lane; k < cw_len; k += 64) {
        const tkv_u32x2 v = pair_of(z, k);
        const uint32_t v_m = v.x, v_l = v.y;
        weigh(k, k < n_chunks ? __uint_as_float(v_m) : -INFINITY, __uint_as_float(v_l));
      }
      L = over_wave(L, SumOf{});
      // (a head that two waves work on: the same number from both)
      if (lane == 0) Ls[z ? h1 : h0] = L;
    }
    const float* w_of = cw + (kTwo == 2 && hh != h0 ? cw_len : 0);
    tkv_floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0;;) {
#pragma unroll
      for (int y = 0; y < kPer; ++y) {
        const int k = k0 + KS * y + ks;
        const float w = w_of[k];  // (past the last chunk: whatever is there, not used)
        acc += __builtin_bit_cast(tkv_floatx4, ov[y]) * (k < n_chunks ? w : 0.f);
      }
      k0 += KS * kPer;
      if (k0 >= n_chunks) break;
      request(k0);
    }
    if (on) *reinterpret_cast<tkv_floatx4*>(red + (hh * KS + ks) * TKV_D + 4 * c4) = acc;
  }
  __syncthreads();
  for (int i = tid; i < G * TKV_D; i += nthr) {
    const int hh = i / TKV_D, c = i % TKV_D;
    float O = red[hh * KS * TKV_D + c] + red[(hh * KS + 1) * TKV_D + c];
    if (KS == 3) O += red[(hh * KS + 2) * TKV_D + c];
    if (KS == 4) O += red[(hh * KS + 2) * TKV_D + c] + red[(hh * KS + 3) * TKV_D + c];
    const float Lsum = Ls[hh];
    out0[(size_t)hh * TKV_D + c] = __float2half_rn(Lsum > 0.f ? O / Lsum : 0.f);
  }
}

// Eq. 10 (Sec. 4.2, Stage 1) for one (sequence, KV head), by a whole workgroup of NT = 128, 256, ... 1024
// threads (contains barriers):
//   s_c = (((|q_0,c| + |q_1,c|) + ...) over the G <= 8 query heads) * kmax[c],
// every operation one float32 operation; the ds channels with the largest s (ties: lower
// channel first) go to out[0..ds) in ascending order (and to out2 unless null).
// q0: the G query rows [G][TKV_D]; s_s, s_sel: TKV_D words of LDS scratch each.
// In the scoring launch everything waits for this: the query rows come in one round trip (not one per head),
// a channel's rank is counted by NT / 128 lanes side by side and its place taken from a ballot: the scoring launch of
// 32/4 heads, 98101 tokens 20.8 -> 17.2 us, of 32/32 heads, 2234 tokens 16.5 -> 13.3; on its own (in a graph) 6.2 -> 3.4.
template <int NT>
__device__ inline void select_channels_block(const __half* q0, int G, const float* kmax, int ds, float* s_s,
                                             uint32_t* s_sel, int32_t* out, int32_t* out2) {
#pragma clang fp contract(off)
  constexpr int P = NT / TKV_D;  // lanes per channel, a power of two of at most 8
  static_assert(P >= 1 && P <= 8 && (P & (P - 1)) == 0 && NT % TKV_D == 0, "lanes per channel");
  const int tid = threadIdx.x, lane = tid % 64;
  if (tid < TKV_D) {
    __half v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = q0[(size_t)min(j, G - 1) * TKV_D + tid];
    const float km = kmax[tid];
    float a = fabsf(__half2float(v[0]));
#pragma unroll
    for (int j = 1; j < 8; ++j) a = j < G ? a + fabsf(__half2float(v[j])) : a;
    s_s[tid] = a * km;
  }
  __syncthreads();
  {
    const int c = tid / P, part = tid % P;
    const float s = s_s[c];
    int rank = 0;  // channels that come before this one: larger s, or equal s and lower index
#pragma unroll 16
    for (int y = 0; y < TKV_D / P; ++y) {
      const int j = part * (TKV_D / P) + y;
      const float sj = s_s[j];
      rank += (sj > s || (sj == s && j < c)) ? 1 : 0;
    }
#pragma unroll
    for (int d = 1; d < P; d <<= 1) rank += __shfl_xor(rank, d, 64);
    if (part == 0) s_sel[c] = rank < ds ? 1u : 0u;
  }
  __syncthreads();
  if (tid < TKV_D) {  // ascending output: behind the selected channels below this one
    const unsigned long long m0 = __builtin_amdgcn_ballot_w64(s_sel[lane] != 0u), m1 = __builtin_amdgcn_ballot_w64(s_sel[64 + lane] != 0u);
    const unsigned long long mine = tid < 64 ? m0 : m1;
    if ((mine >> lane) & 1ull) {
      const int pos = (tid < 64 ? 0 : __builtin_popcountll(m0)) + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u));
      if (pos < ds) {  // (NaN products precede everything: more than ds of them must not leave the list)
        out[pos] = tid;
        if (out2) out2[pos] = tid;
      }
    }
  }
  __syncthreads();
}

// Carve-up of the sparse-layer workspace (per bh = (sequence, KV head)):
//   keys  uint32 [BH][capacity]   order-preserving image of the approximate scores
//   cand  uint2  [BH][capacity + 4096]  (key, token) pairs in or above the threshold bin; the
//                                 workgroup that owns tokens [T x, T x + T) lists them from entry T x
//                                 (T = tokens per workgroup of the launch, rounded up to 4)
//   hist  uint32 [BH][8192]       histogram of the 13-bit key prefix
//   ctrl  uint32 [BH][8]          1: arrival counter of the Top-K selection; 4: arrival counter of
//                                 the attention
//   blk   uint32 [BH][nblk_cap]   length of each workgroup's list
//   parts float  [B][Hq][64][D+4] split partials of the sparse attention
struct SparseWs {
  uint32_t* keys;
  uint2* cand;
  size_t cand_stride;  // entries per (sequence, KV head)
  uint32_t* hist;
  uint32_t* ctrl;
  uint32_t* blk;
  float* parts;
  int32_t nblk_cap;
};
inline size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }
inline size_t sparse_ws_layout(const tkv_sparse_desc* d, size_t off[6], int32_t* nblk_cap) {
  const size_t bh = (size_t)d->batch * d->n_kv_heads, cap = (size_t)d->capacity;
  const int32_t nb = (int32_t)((cap + 1023) / 1024 + 1);
  size_t o = 0;
  off[0] = o; o = align16(o + bh * cap * 4);
  off[1] = o; o = align16(o + bh * (cap + 4096) * 8);
  off[2] = o; o += bh * 8192 * 4;
  off[3] = o; o = align16(o + bh * 8 * 4);
  off[4] = o; o = align16(o + bh * (size_t)nb * 4);
  off[5] = o; o = align16(o + (size_t)d->batch * d->n_q_heads * 64 * TKV_PART_STRIDE * 4);
  if (nblk_cap) *nblk_cap = nb;
  return o;
}
inline SparseWs carve_sparse_ws(const tkv_sparse_desc* d, void* workspace) {
  size_t off[6];
  SparseWs ws;
  sparse_ws_layout(d, off, &ws.nblk_cap);
  char* base = (char*)workspace;
  ws.keys = (uint32_t*)(base + off[0]);
  ws.cand = (uint2*)(base + off[1]);
  ws.cand_stride = (size_t)d->capacity + 4096;
  ws.hist = (uint32_t*)(base + off[2]);
  ws.ctrl = (uint32_t*)(base + off[3]);
  ws.blk = (uint32_t*)(base + off[4]);
  ws.parts = (float*)(base + off[5]);
  return ws;
}

// Position of logical element (t, c) of a block of 32 tokens x 128 channels inside the
// packed block: word index and field index.  Mirrors the layout text of tkv.h.
__host__ __device__ inline void k_code_pos(int bits, int t, int c, int& word, int& field) {
  const int r = 4 * (t / 8) + t % 4, tau = (t % 8) / 4;
  const int lane = r + 16 * ((c % 32) / 8);
  if (bits == 1) {
    word = 64 * tau + lane;
    field = (c % 8) / 2 + 4 * ((c / 32) % 2) + 8 * (c / 64) + 16 * (c % 2);
  } else if (bits == 2) {
    word = 4 * lane + 2 * tau + c / 64;
    field = (c % 8) / 2 + 4 * ((c / 32) % 2) + 8 * (c % 2);
  } else {
    word = 256 * tau + 4 * lane + c / 32;
    field = (c % 8) / 2 + 4 * (c % 2);
  }
}

__host__ __device__ inline void v_code_pos(int bits, int t, int c, int& word, int& field) {
  const int lane = c % 16 + 16 * (t / 8);
  if (bits == 1) {
    word = 64 * (c / 64) + lane;
    field = (t % 8) / 2 + 4 * ((c / 16) % 2) + 8 * ((c / 32) % 2) + 16 * (t % 2);
  } else if (bits == 2) {
    word = 4 * lane + c / 32;
    field = (t % 8) / 2 + 4 * ((c / 16) % 2) + 8 * (t % 2);
  } else {
    word = 256 * (c / 64) + 4 * lane + (c / 16) % 4;
    field = (t % 8) / 2 + 4 * (t % 2);
  }
}

// Inverse maps: which (t, c) does field F of word w hold.
__host__ __device__ inline void k_code_elem(int bits, int w, int F, int& t, int& c) {
  int lane, tau, r, kb;
  if (bits == 1) {
    tau = w / 64;
    lane = w % 64;
    const int f = F % 16, e = F / 16;
    r = lane % 16;
    kb = lane / 16;
    c = 32 * ((f / 4) % 2) + 64 * (f / 8) + 8 * kb + 2 * (f % 4) + e;
  } else if (bits == 2) {
    lane = w / 4;
    tau = (w % 4) / 2;
    const int wd = w % 2, f = F % 8, e = F / 8;
    r = lane % 16;
    kb = lane / 16;
    c = 64 * wd + 32 * (f / 4) + 8 * kb + 2 * (f % 4) + e;
  } else {
    tau = w / 256;
    lane = (w % 256) / 4;
    const int m = w % 4, f = F % 4, e = F / 4;
    r = lane % 16;
    kb = lane / 16;
    c = 32 * m + 8 * kb + 2 * f + e;
  }
  t = 8 * (r / 4) + 4 * tau + r % 4;
}

__host__ __device__ inline void v_code_elem(int bits, int w, int F, int& t, int& c) {
  if (bits == 1) {
    const int lane = w % 64, f = F % 16, e = F / 16;
    const int r = lane % 16, kb = lane / 16;
    const int cb = 4 * (w / 64) + (f / 4) % 2 + 2 * (f / 8);
    t = 8 * kb + 2 * (f % 4) + e;
    c = 16 * cb + r;
  } else if (bits == 2) {
    const int lane = w / 4, wd = w % 4, f = F % 8, e = F / 8;
    const int r = lane % 16, kb = lane / 16;
    const int cb = 2 * wd + f / 4;
    t = 8 * kb + 2 * (f % 4) + e;
    c = 16 * cb + r;
  } else {
    const int lam = w / 256, lane = (w % 256) / 4, f = F % 4, e = F / 4;
    const int r = lane % 16, kb = lane / 16;
    const int cb = 4 * lam + w % 4;
    t = 8 * kb + 2 * f + e;
    c = 16 * cb + r;
  }
}

}  // namespace tkv
