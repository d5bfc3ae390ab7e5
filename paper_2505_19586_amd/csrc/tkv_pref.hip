// Offline identification (Sec. 4.1): dense preference score of a layer, Eq. 6-8, and the
// classification of Eq. 9.
//
// Per (sequence, KV head) the attention logits of the R = G * n_q most recent query rows
// against all n keys are a dense contraction (v_mfma_f32_16x16x32_f16); what Eq. 7 needs of a
// row is not the index set of its top_k entries but their softmax mass, which ties do not
// change.  Logits are never written to memory.
//
//   pass 0  logits of a sample, one key out of every 16, as block maxima of four keys.
//   bound   per row: L, chosen from the sample so that for keys that know nothing of its picks (they are fixed, not drawn)
//           about one row in 6 x 10^7 has less than top_k logits above it (about 1.8 top_k are; every row is checked), and a
//           reference m, the sample's maximum.
//   pass 2  all logits: softmax denominator against m, the logits above L to the row's candidates.
//   exact   the same once more for the slabs with a row that the sample misled (too few or too many
//           candidates, a denominator beyond float's range), with a bound that cannot fail; these three
//           launches return at once as a rule (short prompts take this form alone, without the sample):
//     pass 1  block maxima of all keys: every (row, lane slot of a wave) keeps the maximum of
//             the <= 32 logits it sees in a round of 8 key chunks.  The blocks of a row are
//             disjoint, so the top_k-th largest block maximum L is a lower bound of the row's
//             top_k-th largest logit T, and at most 32 (top_k - 1) logits lie above it.
//     bound   per row: L (radix select over the block maxima) and the row maximum m.
//     pass 2
//   final   per row: T = top_k-th largest candidate if there are top_k of them, else L (the
//           rest of the top_k entries are ties at L); mass of the top_k entries, summed in
//           64-bit fixed point so that the result does not depend on the order in which
//           candidates were appended; Eq. 8 per head in a fixed order.
//
// Two evaluations of all logits, the first only for the exact bound, were the rule before: 32/8 heads, n_q = 64,
// 131072 keys, k = 1024: 74 (pass 1) + 20 + 151 (pass 2) + 21 + 7 us of kernels; now 13 + 10 + 129 + 27 + 4 and three
// launches that return at once.  28618 keys, n_q = 16, k = 1024 (fewer blocks than k: every logit was a candidate)
// 1180 -> 56 us per call.
//
// Shape of the passes: a workgroup of 16 waves owns up to 256 rows and every P-th chunk
// of 128 keys; a chunk is staged once in LDS (direct global -> LDS loads, three or four buffers deep, one
// barrier per chunk) and read by all waves as A operands; each wave holds 32 (16) rows as MFMA B operands in
// registers, and waves of the same rows share a chunk's key tiles: few rows, many waves per row (64 rows on
// 2 of 8 groups of waves before: 32/32 heads, n_q = 16, 131000 keys 470 -> 239 us).  D layout: a lane holds 4
// keys x 1 query, so a row's constants (L, m) and its partial denominator are per-lane scalars.
// Bound by vector-instruction issue next to the matrix instructions: pass 2 takes 90 us without its hits.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "tkv_common.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 1024;
constexpr int kChunk = 128;          // keys per staged chunk
constexpr int kChunkBytes = kChunk * 256;
constexpr int kRing1 = 4;            // chunk buffers in LDS: passes 0 and 1
constexpr int kRing2 = 3;            // pass 2 (the waves' hit buffers need the room)
constexpr int kRound = 8;            // chunks per block-maximum round: blocks of at most 8 chunks x 4 tiles = 32 keys
constexpr int kStride = 16;          // the sample takes one key out of every 16
constexpr int kSampleBlocks = 2048;  // most block maxima of a row's sample: 32 per lane of the wave that searches them
constexpr int kSlotBlocks = 32;      // block maxima per row and chunk of the sample: four keys each
constexpr int kMaxRows = 256;        // rows of the widest workgroup
constexpr int kHitCap = 192;         // hits a wave buffers: fewer than 64 left over and 64 from each of two query tiles
constexpr int kHitBytes = kHitCap * 16 + kHitCap;  // a quadruple of logits and its row each
constexpr int kPass1Lds = kRing1 * kChunkBytes;
constexpr int kPass2Lds = kRing2 * kChunkBytes + 2 * kMaxRows * 4 + 16 * kHitBytes;
static_assert(kPass2Lds <= 160 * 1024 && kHitBytes % 16 == 0, "LDS of a pass");

// How the 16 waves of a workgroup share its work: `groups` query groups of 16 qt rows, SUB = 16 / groups waves per
// group that share the key tiles of a chunk.
template <int QT_, int GROUPS_>
struct Shape {
  static constexpr int QT = QT_;          // query tiles (16 rows each) per wave
  static constexpr int GROUPS = GROUPS_;  // query groups of a workgroup
  static constexpr int SUB = 16 / GROUPS;
  static constexpr int T = kChunk / 16 / SUB;  // key tiles of a chunk per wave
  static constexpr int ROWS = GROUPS * QT * 16;
  static_assert(T >= 1 && T <= 4 && ROWS <= kMaxRows, "tiles of a chunk, rows of a workgroup");
};

struct PrefParams {
  const __half* q_last;  // [B][n_q][Hq][128]
  const __half* k;       // [B][n][Hkv][128]
  float* blkmax;         // [Hkv][R][nblk]; the sample's [Hkv][R][s_nblk]
  float* bound;          // [Hkv][R][2]: L, the reference m of the denominators (raw dot products)
  float* den;            // [Hkv][R][P]: partial softmax denominators
  float* seg;            // [Hkv][R][P][seg_cap]: a workgroup's candidates (logits above L) of a row, in no particular order
  uint32_t* seg_cnt;     // [Hkv][R][P]
  float* cand;           // [Hkv][R][cand_cap]: further candidates, where a workgroup has more than seg_cap of a row
  uint32_t* cursor;      // [Hkv][R][4]: candidates found, those in cand, non-zero if a partial denominator is not finite;
                         //   zero between calls
  uint32_t* failed;      // [Hkv][slabs]: the sample's bound did not do for some row of the slab
  float* row_p;          // [Hkv][R]
  float* p_out;          // [B][Hq]
  float scale2;          // sm_scale * log2(e)
  int32_t hq, hkv, n_q, n, b, top_k;
  int32_t slabs;
  int32_t P;             // workgroups per (KV head, slab): workgroup r owns chunks r, r + P, ...
  int32_t rounds;        // block-maximum rounds of a workgroup
  int32_t nblk;          // P * rounds * 16 SUB
  int32_t seg_cap, cand_cap;
  int32_t s_P, s_rounds, s_per_round, s_nblk;  // the same of the sample; chunks per round
  int32_t s_rank;        // L: the s_rank-th largest block maximum of the sample or a little below it; 0: -inf
  int32_t exact;         // 1: the passes and the bound of the exact form, for failed slabs only; 2: for all, no sample before
};

__device__ inline uint32_t float_key(float s) {
  const uint32_t u = __float_as_uint(s);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// The i-th sampled key: one of the 16 keys from 16 i on, picked by mixing the bits of i, so that no
// structure of a prompt (periods, runs) meets the sample's.  The constants are the first 32 bits of the fractions of
// (sqrt 5 - 1) / 2, sqrt 5, sqrt 3 and sqrt 2; with this order and these shifts the picks are as even as random ones: over 2048 to
// 262144 of them chi-square of single picks, of pairs up to 2047 apart and of periods up to 1024 within 2.7 standard deviations.
__device__ inline int sample_key(int i) {
  uint32_t x = (uint32_t)i * 0x9E3779B9u + 0x3C6EF372u;
  x = (x ^ (x >> 16)) * 0xBB67AE85u;
  x = (x ^ (x >> 16)) * 0x6A09E667u;
  return kStride * i + (int)(x >> 28);
}

__device__ inline void lds_load16(const void* g, void* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
#define TKV_WAIT_VMCNT(N) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory")

// max(a, b) as the median of (a, b, +inf): one instruction, where fmaxf costs three (it quiets
// NaNs in both operands first; no NaN is expected here, and none could be selected)
__device__ inline float max_f32(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, INFINITY); }

// Does the sample's bound of a row have to be replaced: fewer than top_k candidates, more than fit, or a
// denominator that left float's range against the sample's reference.
__device__ inline bool row_failed(const PrefParams& p, size_t gr) {
  const uint4 c = *reinterpret_cast<const uint4*>(p.cursor + gr * 4);
  return c.x < (uint32_t)p.top_k || c.x > (uint32_t)p.cand_cap || c.z != 0u;
}

// PASS 0: block maxima of the sample.  PASS 1: block maxima of all keys.  PASS 2: denominators and candidates.
//
// Key chunks travel global -> LDS directly (no registers), into a ring of buffers: while chunk i
// is computed on, the next three are in flight.  A load instruction of a wave fills 1 KiB
// of LDS in lane order, i.e. 4 key rows of 256 bytes; the lanes pick their 16-byte pieces so
// that piece c of row r lands at slot (c + r) mod 16 of its row: the A-operand reads (16 rows,
// same piece) then touch 16 different slots and are free of bank conflicts.
template <int PASS, class S>
__global__ __launch_bounds__(kThreads) void pref_pass_kernel(PrefParams p) {
  tkv::fetch_arguments<sizeof(PrefParams)>();
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int QT = S::QT, T = S::T, SUB = S::SUB, kRing = PASS == 2 ? kRing2 : kRing1;
  uint32_t* lcnt = reinterpret_cast<uint32_t*>(smem + kRing2 * kChunkBytes);  // pass 2: candidates per row [kMaxRows]
  float* lrow = reinterpret_cast<float*>(lcnt + kMaxRows);                    // L per row [kMaxRows]
  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int g = wave % S::GROUPS, s = wave / S::GROUPS;
  const int col = lane % 16, kb = lane / 16;
  const int r_wg = blockIdx.x, h = blockIdx.y, slab = blockIdx.z;
  const int G = p.hq / p.hkv, R = G * p.n_q;
  const int rows_here = min(S::ROWS, R - slab * S::ROWS);
  const size_t row_first = (size_t)h * R + (size_t)slab * S::ROWS;
  if (PASS != 0 && p.exact == 1) {
    bool bad;
    if (PASS == 1) {
      bad = __syncthreads_or(tid < rows_here && row_failed(p, row_first + tid)) != 0;
      if (r_wg == 0 && tid == 0) p.failed[h * p.slabs + slab] = bad ? 1u : 0u;
    } else {
      bad = p.failed[h * p.slabs + slab] != 0u;
    }
    if (!bad) return;
  }
  const int row0 = slab * S::ROWS + g * (16 * QT);  // first row of this wave
  const int nqt = max(0, min(QT, (R - row0) / 16));  // query tiles of this wave (R is a multiple of 16)
  const int n_keys = PASS == 0 ? (p.n + kStride - 1) / kStride : p.n;
  const int P = PASS == 0 ? p.s_P : p.P;
  const int n_chunks = (n_keys + kChunk - 1) / kChunk;
  const int my_chunks = r_wg < n_chunks ? (n_chunks - r_wg + P - 1) / P : 0;
  // chunks below hold keys of the prompt only
  const int n_full = PASS == 0 ? p.n / (kStride * kChunk) : p.n / kChunk;

  // B operands: this wave's query rows (row = query head of the group * n_q + position)
  uintx4 bq[QT][4];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int r = min(row0 + 16 * qt + col, R - 1), j = r / p.n_q, i = r % p.n_q;
    const __half* qrow = p.q_last + (((size_t)p.b * p.n_q + i) * p.hq + (size_t)h * G + j) * TKV_D;
#pragma unroll
    for (int m = 0; m < 4; ++m) bq[qt][m] = *reinterpret_cast<const uintx4*>(qrow + 32 * m + 8 * kb);
  }
  float L[QT], mrow[QT], den[QT];
  // this wave's hits: quadruples of logits, one of them at least above its row's L, and the row in the workgroup
  unsigned char* hit_v = smem + kRing2 * kChunkBytes + 2 * kMaxRows * 4 + wave * kHitBytes;
  unsigned char* hit_r = hit_v + kHitCap * 16;
  uint32_t n_hit = 0;  // (uniform)
  if (PASS == 2) {
    if (tid < kMaxRows) {
      lcnt[tid] = 0;
      lrow[tid] = p.bound[((size_t)h * R + min(slab * S::ROWS + tid, R - 1)) * 2];
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      const int r = min(row0 + 16 * qt + col, R - 1);
      const float2 lm = *reinterpret_cast<const float2*>(p.bound + ((size_t)h * R + r) * 2);
      L[qt] = lm.x, mrow[qt] = -lm.y * p.scale2, den[qt] = 0.f;  // (minus the reference, log2 units)
    }
  }
  constexpr int NB = PASS == 0 ? T : 4;  // running maxima per query tile: per key tile of the sample, per key slot
  float bm[QT][NB];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt)
#pragma unroll
    for (int x = 0; x < NB; ++x) bm[qt][x] = -INFINITY;

  // this wave brings rows 8 wave .. 8 wave + 7 of every chunk: two load instructions
  const int crow = lane / 16, lslot = lane % 16;
  auto load_chunk = [&](int c, int buf) {
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int r = 8 * wave + 4 * y + crow;               // row of the chunk
      // (keys past the end re-read the last one and are masked below)
      const int key = min(PASS == 0 ? sample_key(c * kChunk + r) : c * kChunk + r, p.n - 1);
      const int piece = (lslot - r) & 15;
      const __half* src = p.k + (((size_t)p.b * p.n + key) * p.hkv + h) * TKV_D + 8 * piece;
      lds_load16(src, smem + buf * kChunkBytes + (8 * wave + 4 * y) * 256);
    }
  };

  // one key tile of the chunk in buffer `base` against this wave's rows
  auto tile_step = [&](const unsigned char* base, int c, int tt, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;  // all query tiles present, no key past the end
    const int tile = s + SUB * tt;
    const int key0 = c * kChunk + tile * 16;
    auto valid = [&](int x) {
      const int i = key0 + 4 * kb + x;
      return FULL || (PASS == 0 ? sample_key(i) : i) < p.n;
    };
    floatx4 acc[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) acc[qt] = floatx4{0.f, 0.f, 0.f, 0.f};
    const unsigned char* arow = base + (tile * 16 + col) * 256;
    __builtin_amdgcn_s_setprio(1);  // (matrix instructions before other waves' vector work: pass 2 131 -> 128 us)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uintx4 a = *reinterpret_cast<const uintx4*>(arow + ((4 * m + kb + col) & 15) * 16);
#pragma unroll
      for (int qt = 0; qt < QT; ++qt)
        if (FULL || qt < nqt)
          acc[qt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a),
                                                           __builtin_bit_cast(half8, bq[qt][m]), acc[qt], 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
    // this lane: keys key0 + 4 kb + x of the query row (row0 + 16 qt + col); logits stay in units
    // of the raw dot product (sm_scale > 0 keeps their order)
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      if (!FULL && qt >= nqt) continue;
      float mx = -INFINITY;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        if (!valid(x)) acc[qt][x] = -INFINITY;
        const float v = acc[qt][x];
        if (PASS == 1) bm[qt][x] = max_f32(bm[qt][x], v);
        else mx = x == 0 ? v : max_f32(mx, v);
        if (PASS == 2) {
          const float e = __builtin_amdgcn_exp2f(fmaf(v, p.scale2, mrow[qt]));
          den[qt] += FULL || valid(x) ? e : 0.f;
        }
      }
      if (PASS == 0) bm[qt][tt] = max_f32(bm[qt][tt], mx);
      // PASS 2.  One logit in fifty to a hundred lies above L: of a wave's 64 quadruples a few hold one.  They are
      // appended whole to the wave's buffer: no atomic, no loop, and drained 64 at a time (a loop over the hits of a tile with
      // an LDS counter per row: 151 us; whole quadruples to per-lane lists in memory: 195, a third of it their
      // collection at the end; this: 129).  (In assembly: without a branch around the
      // stores the compiler can interleave the query tiles.  The accumulators' hazards are over: the comparison has
      // read them.)
      if (PASS == 2) {
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(mx > L[qt]);
        const uint32_t at = n_hit + __builtin_amdgcn_mbcnt_hi((uint32_t)(hit >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hit, 0u));
        const uint32_t at_v = (uint32_t)(uintptr_t)hit_v + 16u * at, at_r = (uint32_t)(uintptr_t)hit_r + at;
        const uint32_t row = (uint32_t)(g * (16 * QT) + 16 * qt + col);
        const floatx4 v = acc[qt];
        unsigned long long exec_was;
        asm volatile("s_and_saveexec_b64 %0, %1\n\tds_write_b128 %2, %3\n\tds_write_b8 %4, %5\n\ts_mov_b64 exec, %0"
                     : "=&s"(exec_was) : "s"(hit), "v"(at_v), "v"(v), "v"(at_r), "v"(row) : "scc");
        n_hit += (uint32_t)__builtin_popcountll(hit);
      }
    }
  };
  // the last `count` <= 64 of the wave's hits to their rows' candidates, one hit per lane
  auto drain = [&](uint32_t count) {
    asm volatile("" ::: "memory");  // (the compiler does not know of the stores; a wave's LDS operations are executed in order)
    n_hit -= count;
    const bool on = (uint32_t)lane < count;
    const uint32_t at = n_hit + (on ? (uint32_t)lane : 0u);
    const floatx4 v = *reinterpret_cast<const floatx4*>(hit_v + 16 * at);
    const int row = hit_r[at];
    const float lr = lrow[row];
    uint32_t above[4], cnt = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) above[x] = cnt, cnt += on && v[x] > lr ? 1u : 0u;
    uint32_t first;
    asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=v"(first) : "v"((uint32_t)(uintptr_t)&lcnt[row]), "v"(cnt) : "memory");
    const size_t gr = row_first + row;
    float* seg = p.seg + (gr * P + r_wg) * p.seg_cap;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if (on && v[x] > lr) {
        const uint32_t to = first + above[x];
        if (to < (uint32_t)p.seg_cap) {
          seg[to] = v[x];
        } else {
          const uint32_t far = atomicAdd(&p.cursor[gr * 4 + 1], 1u);
          if (far < (uint32_t)p.cand_cap) p.cand[gr * p.cand_cap + far] = v[x];
        }
      }
    }
    asm volatile("" ::: "memory");
  };

#pragma unroll
  for (int a = 0; a < kRing - 1; ++a)
    if (a < my_chunks) load_chunk(r_wg + a * P, a);
  for (int i = 0; i < my_chunks; ++i) {
    const int c = r_wg + i * P;
    // this wave's rows of chunk i have landed: vector-memory operations retire in order, and those of the
    // chunks after it (two instructions each) may still be out
    const int ahead = min(kRing - 2, my_chunks - 1 - i);
    if (ahead >= 2) TKV_WAIT_VMCNT(4); else if (ahead == 1) TKV_WAIT_VMCNT(2); else TKV_WAIT_VMCNT(0);
    // everyone's rows of chunk i are there, and everyone is through with chunk i-1 (its operand
    // reads have returned).  A bare barrier: __syncthreads() would also wait for the loads in flight.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (i + kRing - 1 < my_chunks) load_chunk(c + (kRing - 1) * P, (i + kRing - 1) % kRing);
    const int buf = i % kRing;
    if (nqt > 0) {
      const unsigned char* base = smem + buf * kChunkBytes;
      if (nqt == QT && c < n_full) {
#pragma unroll
        for (int tt = 0; tt < T; ++tt) {
          tile_step(base, c, tt, std::true_type{});
          if (PASS == 2)
            while (n_hit >= 64) drain(64);
        }
      } else {
#pragma unroll
        for (int tt = 0; tt < T; ++tt)
          if (c * kChunk + (s + SUB * tt) * 16 < n_keys) {  // (wave-uniform)
            tile_step(base, c, tt, std::false_type{});
            if (PASS == 2)
              while (n_hit >= 64) drain(64);
          }
      }
    }
    if (PASS == 1 && (i % kRound == kRound - 1 || i == my_chunks - 1)) {
      const int f = i / kRound;
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        if (qt < nqt) {
          float* dst = p.blkmax + ((size_t)h * R + row0 + 16 * qt + col) * p.nblk +
                       ((size_t)(r_wg * p.rounds + f) * SUB + s) * 16 + 4 * kb;
          *reinterpret_cast<float4*>(dst) = make_float4(bm[qt][0], bm[qt][1 % NB], bm[qt][2 % NB], bm[qt][3 % NB]);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) bm[qt][x] = -INFINITY;
      }
    }
    if (PASS == 0 && (i % p.s_per_round == p.s_per_round - 1 || i == my_chunks - 1)) {
      const int f = i / p.s_per_round;
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        float* dst = p.blkmax + ((size_t)h * R + row0 + 16 * qt + col) * p.s_nblk +
                     ((size_t)(r_wg * p.s_rounds + f) * SUB + s) * (4 * T) + kb * T;
#pragma unroll
        for (int tt = 0; tt < T; ++tt) {
          if (qt < nqt) dst[tt] = bm[qt][tt % NB];
          bm[qt][tt % NB] = -INFINITY;
        }
      }
    }
  }
  if (PASS != 2) {
    // rounds this workgroup has no chunks for: nothing was seen
    const int per = PASS == 0 ? p.s_per_round : kRound, rounds = PASS == 0 ? p.s_rounds : p.rounds;
    constexpr int kPerWave = PASS == 0 ? 4 * T : 16;  // block maxima per row, round and wave
    for (int f = (my_chunks + per - 1) / per; f < rounds; ++f)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt)
        if (qt < nqt) {
          float* dst = p.blkmax + ((size_t)h * R + row0 + 16 * qt + col) * (PASS == 0 ? p.s_nblk : p.nblk) +
                       ((size_t)(r_wg * rounds + f) * SUB + s) * kPerWave + kb * (kPerWave / 4);
#pragma unroll
          for (int x = 0; x < kPerWave / 4; ++x) dst[x] = -INFINITY;
        }
    return;
  }
  // ---- pass 2 epilogue: the last hits, denominators (fixed order: key lanes, then waves)
  if (n_hit != 0) drain(n_hit);
  __syncthreads();  // every wave is through with the chunk buffers: they now hold the partial denominators
  float* dsum = reinterpret_cast<float*>(smem);  // [SUB][ROWS]
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    float d = den[qt];
    d += __shfl_xor(d, 16, 64);
    d += __shfl_xor(d, 32, 64);
    if (kb == 0 && qt < nqt) dsum[s * S::ROWS + g * (16 * QT) + 16 * qt + col] = d;
  }
  __syncthreads();
  if (tid < rows_here) {
    const size_t gr = row_first + tid;
    float d = dsum[tid];
#pragma unroll
    for (int x = 1; x < SUB; ++x) d += dsum[x * S::ROWS + tid];
    p.den[gr * P + r_wg] = d;
    if (!(d < INFINITY)) atomicOr(&p.cursor[gr * 4 + 2], 1u);
    const uint32_t cnt = lcnt[tid];
    p.seg_cnt[gr * P + r_wg] = min(cnt, (uint32_t)p.seg_cap);
    if (cnt != 0) atomicAdd(&p.cursor[gr * 4], cnt);
  }
}

// An interval of keys that closes in on the one with a given number of keys above it: above(lo) = c_lo >= target >
// above(hi) = c_hi.  Two probes of three are placed as if the counts fell exponentially (a row's largest logits do,
// nearly), the third halves the interval, whatever the data.
struct Bracket {
  uint32_t lo, hi, c_lo, c_hi;
  __device__ uint32_t probe(uint32_t aim, int step) const {
    uint32_t d = (hi - lo) / 2;
    if (step % 3 != 2) {
      const float f = __builtin_amdgcn_logf((float)c_lo / (float)aim) / __builtin_amdgcn_logf((float)c_lo / ((float)c_hi + 0.5f));
      d = (uint32_t)(fminf(fmaxf(f, 0.f), 1.f) * (float)(hi - lo));
    }
    return lo + min(max(d, 1u), hi - lo - 1u);
  }
  __device__ void set(uint32_t mid, uint32_t c, uint32_t target) {
    if (c >= target) lo = mid, c_lo = c; else hi = mid, c_hi = c;
  }
};

// One wave per row: L and m from the sample.  L is chosen by bisection over the block maxima (kRegs per lane, counted
// by ballots: no LDS, no barrier): at least s_rank of them, and seldom more than an eighth more, lie above it.  Where
// many are equal there, L is their value and they are not candidates (the exact form takes over if the
// row then has too few).
template <int kRegs>
__global__ __launch_bounds__(256) void pref_sample_bound_kernel(PrefParams p) {
  tkv::fetch_arguments<sizeof(PrefParams)>();
  const int lane = threadIdx.x % 64;
  const size_t gr = (size_t)blockIdx.x * 4 + threadIdx.x / 64;
  if (gr >= (size_t)p.hq * p.n_q) return;
  const uint32_t kNone = float_key(-INFINITY);
  uint32_t key[kRegs], kmax = kNone;
#pragma unroll
  for (int j = 0; j < kRegs; ++j) {
    const int e = j * 64 + lane;
    key[j] = e < p.s_nblk ? float_key(p.blkmax[gr * p.s_nblk + e]) : kNone;
  }
#pragma unroll
  for (int j = 0; j < kRegs; ++j) kmax = max(kmax, key[j]);
  uint32_t kmin = kmax;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, d, 64));
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, d, 64));
  }
  kmax = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmax);
  kmin = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmin);
  auto above = [&](uint32_t t) {
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < kRegs; ++j) c += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(key[j] > t));
    return c;
  };
  const uint32_t rank = (uint32_t)p.s_rank;
  float L = -INFINITY;
  if (rank != 0) {
    Bracket br = {kNone, kmax, 0u, 0u};
    const uint32_t c_min = above(kmin);  // (as a rule the smallest of the lanes' maxima is a close start)
    if (c_min >= rank) br.lo = kmin, br.c_lo = c_min; else br.c_lo = above(kNone);
    if (br.c_lo >= rank) {
      for (int step = 0; br.hi - br.lo > 1 && br.c_lo > rank + rank / 8; ++step) {
        const uint32_t mid = br.probe(rank + rank / 16, step);
        br.set(mid, above(mid), rank);
      }
      L = key_float(br.c_lo > 4 * rank + 64 ? br.hi : br.lo);
    }
  }
  if (lane == 0) {
    p.bound[gr * 2] = L;
    p.bound[gr * 2 + 1] = key_float(kmax);
  }
}

constexpr int kSelRegs = 16;  // values per thread that the selection kernels keep in registers

// The values of a row, as order-preserving keys: held in registers when there are at most
// 256 * kSelRegs of them (value e at thread e % 256), else streamed from memory every time.
struct RowKeys {
  const float* src;
  uint32_t count;
  bool cached;
  uint32_t reg[kSelRegs];
  __device__ void load(const float* s, uint32_t n) {
    src = s, count = n, cached = n <= 256u * kSelRegs;
    if (cached) {
#pragma unroll
      for (int j = 0; j < kSelRegs; ++j) {
        const uint32_t e = threadIdx.x + 256u * j;
        reg[j] = e < n ? float_key(s[e]) : 0u;
      }
    }
  }
  template <typename F>
  __device__ void for_each(F f) const {
    if (cached) {
#pragma unroll
      for (int j = 0; j < kSelRegs; ++j)
        if (threadIdx.x + 256u * j < count) f(reg[j]);
    } else {
      for (uint32_t e = threadIdx.x; e < count; e += 256) f(float_key(src[e]));
    }
  }
};

// the rank-th largest (1 <= rank <= count) of a row's keys, by a workgroup of 256 threads:
// radix select, 8 bits per pass, over the bits below the keys' common prefix only (a row's
// keys lie close together: with digits taken from the top of the key, every LDS atomic of
// the first passes would hit the same few counters and be serialized).
// hist: 256 words of LDS, s_pick: 4 words.
__device__ inline uint32_t kth_largest_key(const RowKeys& keys, uint32_t rank, uint32_t* hist, uint32_t* s_pick) {
  const int tid = threadIdx.x;
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  keys.for_each([&](uint32_t key) { kmin = min(kmin, key), kmax = max(kmax, key); });
  for (int d = 32; d >= 1; d >>= 1) {
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, d, 64));
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, d, 64));
  }
  if (tid == 0) s_pick[2] = 0xFFFFFFFFu, s_pick[3] = 0u;
  __syncthreads();
  if (tid % 64 == 0) atomicMin(&s_pick[2], kmin), atomicMax(&s_pick[3], kmax);
  __syncthreads();
  kmin = s_pick[2], kmax = s_pick[3];
  int bits_left = 32 - __builtin_clz((kmin ^ kmax) | 1u);  // bits that differ between some keys (at least 1)
  uint32_t prefix = bits_left == 32 ? 0u : (kmax >> bits_left) << bits_left;
  uint32_t remaining = rank;
  while (bits_left > 0) {
    const int w = min(8, bits_left), shift = bits_left - w;
    hist[tid] = 0;
    __syncthreads();
    const uint32_t hi_mask = bits_left == 32 ? 0u : (0xFFFFFFFFu << bits_left);
    const uint32_t dmask = (1u << w) - 1u;
    keys.for_each([&](uint32_t key) {
      if ((key & hi_mask) == prefix) atomicAdd(&hist[(key >> shift) & dmask], 1u);
    });
    __syncthreads();
    if (tid < 64) {
      // wave 0: suffix sums over the 256 bins, 4 bins per lane, highest digit first
      const int l = tid;
      uint32_t c[4], tot = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = hist[255 - (4 * l + j)], tot += c[j];
      uint32_t incl = tot;
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (l >= d) incl += o;
      }
      uint32_t run = incl - tot;  // entries in higher digits than this lane's
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (run < remaining && remaining <= run + c[j]) {
          s_pick[0] = 255 - (4 * l + j);
          s_pick[1] = remaining - run;
        }
        run += c[j];
      }
    }
    __syncthreads();
    prefix |= s_pick[0] << shift;
    remaining = s_pick[1];
    bits_left = shift;
    __syncthreads();
  }
  return prefix;
}

// The exact form, one workgroup per row of a failed slab: L = the top_k-th largest block maximum (-inf if the row
// has fewer blocks than that), m = the row maximum.
template <int ROWS>
__global__ __launch_bounds__(256) void pref_bound_kernel(PrefParams p) {
  tkv::fetch_arguments<sizeof(PrefParams)>();
  __shared__ uint32_t hist[256];
  __shared__ uint32_t s_pick[4];
  __shared__ float s_max[4];
  const int tid = threadIdx.x;
  const size_t gr = blockIdx.x;
  const int R = p.hq / p.hkv * p.n_q;
  if (p.exact == 1 && p.failed[(int)(gr / R) * p.slabs + (int)(gr % R) / ROWS] == 0u) return;
  RowKeys keys;
  keys.load(p.blkmax + gr * p.nblk, (uint32_t)p.nblk);
  uint32_t mk = 0;
  keys.for_each([&](uint32_t key) { mk = max(mk, key); });
  float m = mk != 0 ? key_float(mk) : -INFINITY;
  for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  if (tid % 64 == 0) s_max[tid / 64] = m;
  __syncthreads();
  m = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
  float L = -INFINITY;
  if (p.nblk >= p.top_k) L = key_float(kth_largest_key(keys, (uint32_t)p.top_k, hist, s_pick));
  if (tid == 0) {
    p.bound[gr * 2] = L;
    p.bound[gr * 2 + 1] = m;
    *reinterpret_cast<uint4*>(p.cursor + gr * 4) = make_uint4(0, 0, 0, 0);
  }
}

__device__ inline unsigned long long block_sum_u64(unsigned long long v, unsigned long long* scratch) {
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  __syncthreads();
  if (threadIdx.x % 64 == 0) scratch[threadIdx.x / 64] = v;
  __syncthreads();
  return scratch[0] + scratch[1] + scratch[2] + scratch[3];
}

// 2^(x scale2 - m - e) <= 1 as 40-bit fixed point (exact but for bits below 2^-40: a float has 24 significant
// ones); the exponent x scale2 - m is formed as in pass 2, whose reference m can lie below the row's maximum
__device__ inline unsigned long long fixed_mass(float x, float scale2, float minus_m, int e) {
  return (unsigned long long)ldexpf(__builtin_amdgcn_exp2f(fmaf(x, scale2, minus_m)), 40 - e);
}

// A row's share of Eq. 8, 1 - (mass of its top_k largest entries), by a workgroup of 256 threads.  The candidates are
// gathered from the workgroups' segments into `list` (LDS, cap floats), or behind those in cand where they are too
// many for it.
__device__ inline void final_big_row(const PrefParams& p, size_t gr, float* list, uint32_t cap) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t s_pick[4];
  __shared__ unsigned long long scratch[4];
  __shared__ uint32_t s_kmax;
  __shared__ uint32_t s_at[257];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const float L = p.bound[gr * 2], minus_m = -p.bound[gr * 2 + 1] * p.scale2;
  float* cand = p.cand + gr * p.cand_cap;
  const uint32_t k = (uint32_t)p.top_k;
  if ((uint32_t)p.n <= k) {  // nothing lies outside a row of at most top_k entries
    if (tid == 0) p.row_p[gr] = 0.f;
    return;
  }
  // where each segment goes: exclusive prefix sums of the counts (P <= 256), the candidates in cand before them
  const uint32_t far = min(p.cursor[gr * 4 + 1], (uint32_t)p.cand_cap);
  const uint32_t mine = tid < p.P ? p.seg_cnt[gr * p.P + tid] : 0u;
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) s_pick[wave] = incl;
  __syncthreads();
  uint32_t base = far;
  for (int w = 0; w < wave; ++w) base += s_pick[w];
  s_at[tid] = base + incl - mine;
  if (tid == 255) s_at[256] = base + incl;
  if (tid == 0) s_kmax = float_key(L);
  __syncthreads();
  const uint32_t stored = min(s_at[256], (uint32_t)p.cand_cap);
  float* to = stored <= cap ? list : cand;
  if (to == list)
    for (uint32_t e = tid; e < far; e += 256) list[e] = cand[e];
  for (int r = wave; r < p.P; r += 4) {
    const uint32_t at = s_at[r], cnt = s_at[r + 1] - at;
    const float* seg = p.seg + (gr * p.P + r) * p.seg_cap;
    for (uint32_t e = lane; e < cnt; e += 64)
      if (at + e < stored) to[at + e] = seg[e];
  }
  __syncthreads();
  RowKeys keys;
  keys.load(to, stored);
  float T = L;
  if (stored >= k) T = key_float(kth_largest_key(keys, k, hist, s_pick));
  uint32_t kmax = 0;
  keys.for_each([&](uint32_t key) { kmax = max(kmax, key); });
  for (int d = 32; d >= 1; d >>= 1) kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, d, 64));
  if (lane == 0) atomicMax(&s_kmax, kmax);
  __syncthreads();
  const float top = fmaf(key_float(s_kmax), p.scale2, minus_m);
  const int e = top > 0.f ? (int)ceilf(fminf(top, 200.f)) : 0;
  const uint32_t tkey = float_key(T);
  unsigned long long mass = 0, above = 0;
  keys.for_each([&](uint32_t key) {
    if (key > tkey) mass += fixed_mass(key_float(key), p.scale2, minus_m, e), above += 1;
  });
  mass = block_sum_u64(mass, scratch);
  above = block_sum_u64(above, scratch);
  mass += (k - above) * fixed_mass(T, p.scale2, minus_m, e);  // the rest of the top_k entries equal T
  float den = 0.f;
  for (int r = 0; r < p.P; ++r) den += p.den[gr * p.P + r];
  const float result = den > 0.f ? 1.0f - (float)((double)mass * (1.0 / 1099511627776.0)) / ldexpf(den, -e) : 0.f;
  if (tid == 0) {
    p.row_p[gr] = result;
    *reinterpret_cast<uint4*>(p.cursor + gr * 4) = make_uint4(0, 0, 0, 0);
  }
}

// The same for the usual row: candidates gathered in one round of loads, held in registers (kRegs per thread), the
// top_k-th found by narrowing a bracket with counts from ballots.
template <int kRegs>
__global__ __launch_bounds__(256) void pref_final_kernel(PrefParams p) {
  tkv::fetch_arguments<sizeof(PrefParams)>();
  __shared__ float list[kRegs * 256];
  __shared__ uint32_t s_w[2][4], s_few[64], s_n, s_T;
  __shared__ float s_den[4];
  __shared__ unsigned long long s_mass[4];
  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const size_t gr = blockIdx.x;
  const uint32_t k = (uint32_t)p.top_k;
  if ((uint32_t)p.n <= k) {
    if (tid == 0) p.row_p[gr] = 0.f;
    return;
  }
  // a power of two of threads per segment
  int per_seg = 64;
  while (per_seg * p.P > 256) per_seg >>= 1;
  const int r = tid / per_seg, sub = tid % per_seg;
  const uint32_t cnt = r < p.P ? p.seg_cnt[gr * p.P + r] : 0u;
  float den = r < p.P && sub == 0 ? p.den[gr * p.P + r] : 0.f;
  const float L = p.bound[gr * 2], minus_m = -p.bound[gr * 2 + 1] * p.scale2;
  const uint32_t far = p.cursor[gr * 4 + 1];
  uint32_t incl = sub == 0 ? cnt : 0u;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)incl, d, 64);
    if (lane >= d) incl += o;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) den += __shfl_xor(den, d, 64);
  if (lane == 63) s_w[0][wave] = incl;
  if (lane == 0) s_den[wave] = den;
  if (tid == 0) s_n = 0u;
  __syncthreads();
  uint32_t at = incl - cnt, stored = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    at += w < wave ? s_w[0][w] : 0u;
    stored += s_w[0][w];
  }
  den = (s_den[0] + s_den[1]) + (s_den[2] + s_den[3]);
  if (far != 0 || stored > (uint32_t)kRegs * 256u) {  // (not expected by the host)
    __syncthreads();
    final_big_row(p, gr, list, kRegs * 256);
    return;
  }
  const float* seg = p.seg + (gr * p.P + r) * p.seg_cap;
  for (uint32_t i = sub; i < cnt; i += 8 * per_seg) {
    float v[8];
#pragma unroll
    for (int y = 0; y < 8; ++y) v[y] = seg[min(i + y * per_seg, cnt - 1)];
#pragma unroll
    for (int y = 0; y < 8; ++y)
      if (i + y * per_seg < cnt) list[at + i + y * per_seg] = v[y];
  }
  __syncthreads();
  uint32_t key[kRegs], kmax = 0u;  // 0: none (below every float's key)
#pragma unroll
  for (int j = 0; j < kRegs; ++j) {
    const uint32_t e = (uint32_t)(j * 256 + tid);
    key[j] = e < stored ? float_key(list[e]) : 0u;
    kmax = max(kmax, key[j]);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, d, 64));
  if (lane == 0) s_w[1][wave] = kmax;
  __syncthreads();
  kmax = max(max(s_w[1][0], s_w[1][1]), max(s_w[1][2], s_w[1][3]));
  uint32_t T = float_key(L);
  if (stored >= k) {
    Bracket br = {float_key(L), kmax, stored, 0u};  // above(lo) >= k > above(hi)
    int step = 0;
    while (br.hi - br.lo > 1 && br.c_lo - br.c_hi > 64) {
      // aimed a little to either side of k, so that both ends close in on it
      const uint32_t mid = br.probe(br.c_lo - k > 24 ? k + 12 : k > 24 ? k - 12 : k, step);
      uint32_t c = 0;
#pragma unroll
      for (int j = 0; j < kRegs; ++j) c += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(key[j] > mid));
      if (lane == 0) s_w[step & 1][wave] = c;
      __syncthreads();
      const uint32_t* w = s_w[step & 1];
      br.set(mid, w[0] + w[1] + w[2] + w[3], k);
      ++step;
    }
    T = br.hi;  // (more than 64 equal ones)
    if (br.hi - br.lo > 1) {
#pragma unroll
      for (int j = 0; j < kRegs; ++j)
        if (key[j] > br.lo && key[j] <= br.hi) s_few[atomicAdd(&s_n, 1u)] = key[j];
      __syncthreads();
      if (wave == 0) {
        const uint32_t n_few = s_n, own = (uint32_t)lane < n_few ? s_few[lane] : 0u, rem = k - br.c_hi;  // the rem-th largest of them
        uint32_t gt = 0, ge = 0;
        for (uint32_t y = 0; y < n_few; ++y) {
          const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)own, (int)y);
          gt += o > own ? 1u : 0u;
          ge += o >= own ? 1u : 0u;
        }
        if ((uint32_t)lane < n_few && gt < rem && rem <= ge) s_T = own;
      }
      __syncthreads();
      T = s_T;
    }
  }
  // a power of two takes the largest entry to at most 1: mass and denominator keep every bit
  const float top = fmaf(key_float(max(kmax, float_key(L))), p.scale2, minus_m);
  const int e = top > 0.f ? (int)ceilf(fminf(top, 200.f)) : 0;
  // fixed_mass in two limbs of 20 bits (the same integer)
  uint32_t m_hi = 0, m_lo = 0, above = 0;
#pragma unroll
  for (int j = 0; j < kRegs; ++j) {
    const bool on = key[j] > T;
    const float x = on ? ldexpf(__builtin_amdgcn_exp2f(fmaf(key_float(key[j]), p.scale2, minus_m)), 20 - e) : 0.f;
    const uint32_t h = (uint32_t)x;
    m_hi += h;
    m_lo += (uint32_t)((x - (float)h) * 1048576.0f);
    above += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(on));
  }
  unsigned long long mass = ((unsigned long long)m_hi << 20) + m_lo;
  for (int d = 32; d >= 1; d >>= 1) mass += __shfl_xor(mass, d, 64);
  __syncthreads();
  if (lane == 0) s_mass[wave] = mass, s_w[0][wave] = above;
  __syncthreads();
  if (tid == 0) {
    mass = s_mass[0] + s_mass[1] + s_mass[2] + s_mass[3];
    above = s_w[0][0] + s_w[0][1] + s_w[0][2] + s_w[0][3];
    mass += (unsigned long long)(k - above) * fixed_mass(key_float(T), p.scale2, minus_m, e);  // the rest of the top_k entries equal T
    p.row_p[gr] = den > 0.f ? 1.0f - (float)((double)mass * (1.0 / 1099511627776.0)) / ldexpf(den, -e) : 0.f;
    *reinterpret_cast<uint4*>(p.cursor + gr * 4) = make_uint4(0, 0, 0, 0);
  }
}

// ... and where many candidates are expected.
constexpr int kFinalCap = 8192;
__global__ __launch_bounds__(256) void pref_final_big_kernel(PrefParams p) {
  __shared__ float list[kFinalCap];
  final_big_row(p, blockIdx.x, list, kFinalCap);
}

// Eq. 8 per query head: the sum of its rows' shares, one wave per head in a fixed order.  (A
// launch of its own: an arrival counter per head in the kernel above, 64 atomics on one
// address each, cost three times what the launch does.)
__global__ __launch_bounds__(64) void pref_sum_kernel(PrefParams p) {
  const int jh = blockIdx.x, lane = threadIdx.x;  // query head
  float total = 0.f;
  for (int i = lane; i < p.n_q; i += 64) total += p.row_p[(size_t)jh * p.n_q + i];  // rows of a KV head: (head of the group, position)
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) total += __shfl_xor(total, d, 64);
  if (lane == 0) p.p_out[(size_t)p.b * p.hq + jh] = total;
}

int32_t check_pref_desc(const tkv_pref_desc* d) {
  if (!d || d->struct_size != sizeof(tkv_pref_desc)) return TKV_E_INVAL;
  if (d->n_q_heads <= 0 || d->n_kv_heads <= 0 || d->batch <= 0 || d->n_q <= 0 || d->top_k <= 0 || d->capacity <= 0)
    return TKV_E_INVAL;
  if (d->n_q_heads % d->n_kv_heads != 0) return TKV_E_INVAL;
  if (d->head_dim != TKV_D || d->batch > TKV_MAX_BATCH) return TKV_E_UNSUPPORTED;
  if (d->n_q % 16 != 0 || d->n_q > 256 || d->top_k > 4096) return TKV_E_UNSUPPORTED;
  return TKV_OK;
}

// Rows per workgroup: the fewest that hold a KV head's rows (its waves then share the keys instead of idling), 256
// at most; more rows are several slabs.
int pref_rows(const tkv_pref_desc* d) { return d->n_q_heads / d->n_kv_heads * d->n_q; }
int pref_slab_rows(const tkv_pref_desc* d) {
  const int R = pref_rows(d);
  return R <= 32 ? 32 : R <= 64 ? 64 : R <= 128 ? 128 : 256;
}
int pref_sub(int slab_rows) { return slab_rows <= 64 ? 8 : slab_rows == 128 ? 4 : 2; }  // Shape::SUB

// How the keys of a prompt of n tokens are shared out (see the kernel's header).
struct PrefSplit {
  int32_t P, rounds, nblk, s_P, s_rounds, s_per_round, s_nblk, s_rank;
};
// Candidates of a row that there is room for at least.  32 top_k hold what the exact bound lets through; of the sample's
// the least top_k need more: a rank of 13 to 21 stands for 16 times as many logits on average, and seven times that hardly
// ever (10^-18).  With 32 top_k alone nearly every slab of a prompt took the exact form as well: 32/8 heads, n_q = 64, 131072
// keys, us per call with 32 top_k / now: top_k = 1 369, 166; 8 376, 169; 16 326, 164 (two evaluations of all logits as a
// rule: 205, 220, 224).
constexpr size_t kCandLeast = 1536;
int pref_slabs(const tkv_pref_desc* d) { return (pref_rows(d) + pref_slab_rows(d) - 1) / pref_slab_rows(d); }
// most workgroups per (KV head, slab): the machine filled once
int pref_p_cap(const tkv_pref_desc* d) { return std::max(1, 256 / (d->n_kv_heads * pref_slabs(d))); }
int pref_rounds(int n_chunks, int P) { return ((n_chunks + P - 1) / P + kRound - 1) / kRound; }
PrefSplit pref_split(const tkv_pref_desc* d, int32_t n, int32_t n_cus) {
  PrefSplit sp;
  const int n_chunks = (n + kChunk - 1) / kChunk;
  const int fill = std::min(pref_p_cap(d), std::max(1, n_cus / (d->n_kv_heads * pref_slabs(d))));
  sp.P = std::min(fill, n_chunks);
  sp.rounds = pref_rounds(n_chunks, sp.P);
  sp.nblk = sp.P * sp.rounds * pref_sub(pref_slab_rows(d)) * 16;
  const int n_s = (n + kStride - 1) / kStride, s_chunks = (n_s + kChunk - 1) / kChunk;
  // chunk slots of a row's sample: one per workgroup; longer prompts put several chunks into one (larger blocks)
  const int slots = fill > 32 ? kSampleBlocks / kSlotBlocks : 32;
  sp.s_P = std::min({fill, s_chunks, slots});
  const int mine = (s_chunks + sp.s_P - 1) / sp.s_P;
  sp.s_rounds = std::min(mine, slots / sp.s_P);
  sp.s_per_round = (mine + sp.s_rounds - 1) / sp.s_rounds;
  sp.s_nblk = sp.s_P * sp.s_rounds * kSlotBlocks;
  // Rank in the sample that lies at or below the row's top_k-th logit but for one row in 6 x 10^7 (exp(-18) = 1.5e-8): were the picks
  // drawn, the number of the top_k largest that are among them, each with probability 1/16, would exceed its mean by t
  // with probability at most exp(-t^2 / (2 (variance + t / 3))) (Bernstein's bound).  The picks are fixed, and keys
  // made against them can defeat any rank: what counts is that the candidates of every row are counted, and the exact form.  Too
  // large a part of the sample: every logit is a candidate.
  const double mean = (double)d->top_k / kStride, var = mean * (1.0 - 1.0 / kStride), lambda = 18.0;
  const int rank = (int)std::ceil(mean + lambda / 3 + std::sqrt(lambda * lambda / 9 + 2 * lambda * var));
  sp.s_rank = 10 * rank > 9 * (n_s / 4) ? 0 : rank;
  return sp;
}

// Candidates that hardly a row of a prompt exceeds (a row with more than its final kernel keeps in registers takes the general
// form there: the kernel 10 to 40 us longer, were it one row of thousands).  Up to 9/8 s_rank of the sample's blocks of 4 s_per_round
// keys have a key above L; as many keys as make that part of the blocks, and three and a half standard deviations.
int pref_expect(const PrefSplit& sp, int32_t n) {
  if (sp.s_rank == 0) return n;
  const double above = sp.s_rank * 1.125, m = 4.0 * sp.s_per_round, blocks = std::max(above, (double)n / kStride / m);
  const double part = 1.0 - std::pow(1.0 - above / blocks, 1.0 / m);
  return (int)std::min<double>(n, n * part * (1.0 + 3.5 / std::sqrt(above)));
}

// Workspace of one sequence (sequences are processed one after the other); the counters come
// first: they must be zero before the first call.
struct PrefWs {
  uint32_t* cursor;
  uint32_t* failed;
  float* blkmax;
  float* bound;
  float* den;
  float* seg;
  uint32_t* seg_cnt;
  float* cand;
  float* row_p;
  int32_t seg_cap, cand_cap;
};
size_t pref_ws_layout(const tkv_pref_desc* d, char* base, PrefWs* out) {
  const size_t rows = (size_t)d->n_q_heads * d->n_q;  // Hkv * R
  const int slab_rows = pref_slab_rows(d), sub = pref_sub(slab_rows);
  // the split depends on n and on the stream (its compute units): size for the largest it can be;
  // for a given P the number of blocks grows with n
  const int n_chunks = (d->capacity + kChunk - 1) / kChunk;
  const int p_max = pref_p_cap(d);
  size_t nblk_max = kSampleBlocks;
  for (int P = 1; P <= p_max; ++P)
    nblk_max = std::max(nblk_max, (size_t)P * pref_rounds(n_chunks, P) * sub * 16);
  const size_t cand_cap = std::min<size_t>((size_t)d->capacity, std::max((size_t)32 * d->top_k, kCandLeast));
  // a segment's expected length: the row's candidates (about 1.8 top_k) over the workgroups that share them, and
  // room for what chance adds (a full segment is only slower); at least three whole chunks for short prompts, of which
  // most is a candidate
  const double mean = 1.8 * d->top_k / p_max;
  const int seg_cap = std::min(std::max((int)(mean + 5 * std::sqrt(mean)) + 8, 3 * kChunk), kChunk * ((n_chunks + p_max - 1) / p_max + 1));
  size_t o = 0;
  const size_t o_cur = o;    o = tkv::align16(o + rows * 4 * 4);
  const size_t o_fail = o;   o = tkv::align16(o + (size_t)d->n_kv_heads * pref_slabs(d) * 4);
  const size_t o_blk = o;    o = tkv::align16(o + rows * nblk_max * 4);
  const size_t o_bound = o;  o = tkv::align16(o + rows * 2 * 4);
  const size_t o_den = o;    o = tkv::align16(o + rows * p_max * 4);
  const size_t o_cand = o;   o = tkv::align16(o + rows * cand_cap * 4);
  const size_t o_rowp = o;   o = tkv::align16(o + rows * 4);
  const size_t o_seg = o;    o = tkv::align16(o + rows * p_max * seg_cap * 4);
  const size_t o_cnt = o;    o = tkv::align16(o + rows * p_max * 4);
  if (out) {
    out->cursor = (uint32_t*)(base + o_cur);
    out->failed = (uint32_t*)(base + o_fail);
    out->blkmax = (float*)(base + o_blk);
    out->bound = (float*)(base + o_bound);
    out->den = (float*)(base + o_den);
    out->cand = (float*)(base + o_cand);
    out->row_p = (float*)(base + o_rowp);
    out->seg = (float*)(base + o_seg);
    out->seg_cnt = (uint32_t*)(base + o_cnt);
    out->seg_cap = seg_cap;
    out->cand_cap = (int32_t)cand_cap;
  }
  return o;
}

// Prompts up to this long take the exact form at once, all slabs of it: five launches instead of eight.  Us per call, sample and
// three launches that return / this: 32/8 heads, n_q = 64: 150 keys, top_k = 1 61.5, 39.3; 1030, 6 66.8, 45.6; 1100, 16 72.1, 46.8;
// 2000, 256 84.7, 62.1; 2000, 1024 80.2, 75.5; 3072, 16 54.9, 49.5; 3072, 160 71.5, 56.1; 32/4, n_q = 16: 150, 1 43.2, 29.2; 2000,
// 1024 51.9, 52.5; 3072, 40 44.0, 37.1.  In longer ones the block maxima are many to find and to search: 4000, 1024 99.5,
// 109.4.
constexpr int kDirectKeys = 3072;

template <class S>
int32_t launch_pref(PrefParams p, const PrefSplit& sp, hipStream_t s) {
  static const bool lds_ok =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&pref_pass_kernel<0, S>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          kPass1Lds) == hipSuccess &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(&pref_pass_kernel<1, S>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          kPass1Lds) == hipSuccess &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(&pref_pass_kernel<2, S>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          kPass2Lds) == hipSuccess;
  if (!lds_ok) return TKV_E_HIP;
  const int rows = p.hq * p.n_q;
  const dim3 grid(sp.P, p.hkv, p.slabs);
  if (p.n > p.top_k && p.n <= kDirectKeys) {
    p.exact = 2;
    TKV_LAUNCH((pref_pass_kernel<1, S>), grid, kThreads, kPass1Lds, s, p);
    TKV_LAUNCH(pref_bound_kernel<S::ROWS>, dim3(rows), 256, 0, s, p);
    TKV_LAUNCH((pref_pass_kernel<2, S>), grid, kThreads, kPass2Lds, s, p);
  } else if (p.n > p.top_k) {
    p.exact = 0;
    TKV_LAUNCH((pref_pass_kernel<0, S>), dim3(sp.s_P, p.hkv, p.slabs), kThreads, kPass1Lds, s, p);
    if (p.s_nblk <= 1024) TKV_LAUNCH(pref_sample_bound_kernel<16>, dim3((rows + 3) / 4), 256, 0, s, p);
    else TKV_LAUNCH(pref_sample_bound_kernel<kSampleBlocks / 64>, dim3((rows + 3) / 4), 256, 0, s, p);
    TKV_LAUNCH((pref_pass_kernel<2, S>), grid, kThreads, kPass2Lds, s, p);
    // rows whose sample misled: their slabs again, with the bound that cannot fail (nothing to do, as a rule)
    p.exact = 1;
    TKV_LAUNCH((pref_pass_kernel<1, S>), grid, kThreads, kPass1Lds, s, p);
    TKV_LAUNCH(pref_bound_kernel<S::ROWS>, dim3(rows), 256, 0, s, p);
    TKV_LAUNCH((pref_pass_kernel<2, S>), grid, kThreads, kPass2Lds, s, p);
  }
  const int expect = pref_expect(sp, p.n);
  // Registers for more candidates than there are cost little, a row that does not fit much.  Us per call with 4 / 6 / 12 / 16 / 24 /
  // many: 28/4 heads, n_q = 32, 46361 keys, top_k = 185 73.6, 64.9, 66.7, 67.5, 70.3, 75.6; 32/8, n_q = 64, 131072 keys, 1024 191.9,
  // 192.1, 170.2, 172.1, 178.4, 188.0; 11552 keys, 28/4, 911 88.7, 88.4, 86.7, 84.0, 93.1, 97.3; 94961, 2000 200.4, 200.4, 201.1,
  // 184.4, 165.3, 188.6; 4/1, 94961, 1400 106, 107, 108, 69.4, 70.7, 105.5.
  if (expect <= 4 * 256) TKV_LAUNCH(pref_final_kernel<4>, dim3(rows), 256, 0, s, p);
  else if (expect <= 6 * 256) TKV_LAUNCH(pref_final_kernel<6>, dim3(rows), 256, 0, s, p);
  else if (expect <= 12 * 256) TKV_LAUNCH(pref_final_kernel<12>, dim3(rows), 256, 0, s, p);
  else if (expect <= 16 * 256) TKV_LAUNCH(pref_final_kernel<16>, dim3(rows), 256, 0, s, p);
  else if (expect <= 24 * 256) TKV_LAUNCH(pref_final_kernel<24>, dim3(rows), 256, 0, s, p);
  else TKV_LAUNCH(pref_final_big_kernel, dim3(rows), 256, 0, s, p);
  TKV_LAUNCH(pref_sum_kernel, dim3(p.hq), 64, 0, s, p);
  return TKV_OK;
}

}  // namespace

extern "C" int32_t tkv_dense_preference_sizes(const tkv_pref_desc* d, size_t* workspace_bytes) {
  int32_t st = check_pref_desc(d);
  if (st != TKV_OK) return st;
  if (!workspace_bytes) return TKV_E_INVAL;
  *workspace_bytes = pref_ws_layout(d, nullptr, nullptr) + 256;
  return TKV_OK;
}

extern "C" int32_t tkv_dense_preference(const tkv_pref_desc* d, const void* q_last, const void* k, int32_t n,
                                        float sm_scale, float* p_out, void* workspace, size_t workspace_bytes,
                                        void* stream) {
  int32_t st = check_pref_desc(d);
  if (st != TKV_OK) return st;
  if (!q_last || !k || !p_out || !workspace || n < 1) return TKV_E_INVAL;
  if (!(sm_scale > 0.f)) return TKV_E_INVAL;
  if (n > d->capacity) return TKV_E_CAPACITY;
  PrefWs ws;
  if (workspace_bytes < pref_ws_layout(d, (char*)workspace, &ws)) return TKV_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  int n_cus = tkv::stream_compute_units(s);
  if (n_cus > 256) n_cus = 256;
  const PrefSplit sp = pref_split(d, n, n_cus);
  PrefParams p;
  p.q_last = (const __half*)q_last;
  p.k = (const __half*)k;
  p.blkmax = ws.blkmax;
  p.bound = ws.bound;
  p.den = ws.den;
  p.cand = ws.cand;
  p.cursor = ws.cursor;
  p.failed = ws.failed;
  p.seg = ws.seg;
  p.seg_cnt = ws.seg_cnt;
  p.row_p = ws.row_p;
  p.p_out = p_out;
  p.scale2 = sm_scale * 1.44269504088896340736f;
  p.hq = d->n_q_heads;
  p.hkv = d->n_kv_heads;
  p.n_q = d->n_q;
  p.n = n;
  p.top_k = d->top_k;
  p.slabs = pref_slabs(d);
  p.P = sp.P;
  p.rounds = sp.rounds;
  p.nblk = sp.nblk;
  p.seg_cap = ws.seg_cap;
  p.cand_cap = ws.cand_cap;
  p.s_P = sp.s_P;
  p.s_rounds = sp.s_rounds;
  p.s_per_round = sp.s_per_round;
  p.s_nblk = sp.s_nblk;
  p.s_rank = sp.s_rank;
  p.exact = 0;
  for (int b = 0; b < d->batch; ++b) {
    p.b = b;
    switch (pref_slab_rows(d)) {
      case 32: st = launch_pref<Shape<1, 2>>(p, sp, s); break;
      case 64: st = launch_pref<Shape<2, 2>>(p, sp, s); break;
      case 128: st = launch_pref<Shape<2, 4>>(p, sp, s); break;
      default: st = launch_pref<Shape<2, 8>>(p, sp, s);
    }
    if (st != TKV_OK) return st;
  }
  return TKV_OK;
}

extern "C" int32_t tkv_classify_layer(const float* p_heads_host, int32_t n_heads, int32_t n_q, float tau,
                                      float* layer_score_out) {
  if (!p_heads_host || n_heads <= 0 || n_q <= 0) return TKV_E_INVAL;
  double sum = 0.0;
  for (int i = 0; i < n_heads; ++i) sum += (double)p_heads_host[i];
  const double score = sum / n_heads / n_q;
  if (layer_score_out) *layer_score_out = (float)score;
  return score > (double)tau ? 1 : 0;
}
