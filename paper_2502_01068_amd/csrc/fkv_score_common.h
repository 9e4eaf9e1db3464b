// Device helpers shared by the score kernels: MFMA operand loads and the K streaming loop.
#pragma once

#include <type_traits>

#include "fkv_dpp.h"
#include "fkv_internal.h"

namespace fkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float floatx16;

constexpr int kWaves = 8;            // one wave per KV head
constexpr int kThreads = kWaves * 64;
constexpr int kScoresSubShort = 4;   // k_scores: sub-tiles per block (incl. pooling halo), short inputs
constexpr int kScoresSubLong = 18;   // ... and the most for long inputs (LDS bound)
constexpr int kScoresSubWide = 9;    // ... when more than 8 virtual groups keep their window sums in LDS
constexpr int kSub = 32;             // tokens per MFMA sub-tile
constexpr int kStageBytes = kSub * kHeadDim * 2;  // 8 KiB per wave
constexpr float kNegBig = -1.0e30f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// The sequence a block works on.  Eight entries a step: one by one each costs a trip through the scalar cache (0.15 us).
__device__ __forceinline__ int find_seq(const SeqMap &map, int block) {
  int b = 0;
  for (int i = 1; i < map.n_seq && b == i - 1; i += 8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) b += (i + j < map.n_seq) & (block >= map.blk[i + j]);
  }
  return b;
}

// Orders this wave's LDS traffic (writes of one layout, reads of another) without a block barrier.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// `bytes` bytes from p on as a raw buffer: a lane's access past them reads zeros and touches no memory, so ranges need
// neither clamps nor branches, and addresses are 32-bit offsets.  p is the same in every lane.
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ __forceinline__ buffer_t buffer_of(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}

// MFMA A operand for virtual group g: lane (m = lane%32, hi = lane/32) holds, for step s, the 8
// values d = hi*64 + s*8 .. +7 of query row m (head vg_head0(g) + m/8, window row m%8), zeros for rows that the shape
// does not have.  The contraction index may be permuted freely as long as K uses the same permutation.  g is uniform.
template <typename A>
__device__ __forceinline__ void load_q(const A &a, int b, int g, int lane, bf16x8 (&qa)[8]) {
  const int m = lane & 31, hi = lane >> 5;
  const int hl = m >> 3, w = m & 7;
  const uint32_t seq_bytes = (uint32_t)(a.W * a.Hq) * (kHeadDim * 2);
  const buffer_t q = buffer_of(a.q_win + (size_t)b * a.W * a.Hq * kHeadDim, seq_bytes);
  const bool ok = hl < vg_heads(a, g) && w < a.W;
  const uint32_t at = ok ? (uint32_t)((w * a.Hq + vg_head0(a, g) + hl) * (kHeadDim * 2) + hi * 128) : seq_bytes;
#pragma unroll
  for (int s = 0; s < 8; ++s) qa[s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(q, (int)at, s * 16, 0));
}

// K rows of a wave's KV head, tokens `first` to `end` of a sequence, as 32-token tiles that go straight from global memory
// into the wave's LDS tile (gfx950's 128-bit LDS-direct loads: lane l of a load lands at tile offset 16 l, i.e. 4 tokens
// per load, 16 lanes a row), so no registers hold a tile in flight.  The XOR swizzle lies on the global side: the lane
// that owns LDS column c of token slot t fetches the row's column c ^ (t & 15).  Slots whose token lies outside [0, end)
// are not loaded; the caller ignores their logits.  What used to bound the resident score kernels at short inputs were the
// instructions around these loads (64-bit address products, clamps and a branch per load): the first tile's requests left
// 2.3 us after a wave's start and the next tile's 0.8 us after its operands were read.
struct KTiles {
  buffer_t rows;
  uint32_t at[4];       // byte offsets of this lane's part of token slots tq, 4 + tq, 8 + tq and 12 + tq of tile 0
  uint32_t half_bytes;  // 16 tokens
  uint8_t *stage;

  template <typename A>
  __device__ __forceinline__ KTiles(const A &a, int tok_base, int kv_head, int first, int end, uint8_t *stage_, int lane)
      : stage(stage_) {
    const uint32_t row = (uint32_t)a.Hkv * (kHeadDim * 2);  // a block's tokens span less than 2^31 bytes
    const int from = max(first, 0);
    rows = buffer_of(a.k + ((size_t)(tok_base + from) * a.Hkv + kv_head) * kHeadDim, (uint32_t)(end - 1 - from) * row + kHeadDim * 2);
    half_bytes = 16 * row;
    const int c = lane & 15, tq = lane >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int slot = i * 4 + tq;
      at[i] = (uint32_t)(first - from + slot) * row + ((c ^ slot) << 4);  // a token before the sequence wraps past the buffer's end
    }
  }
  template <int kAux>
  __device__ __forceinline__ void issue(int st) const {
    typedef __attribute__((address_space(3))) void *lptr_t;
    uint32_t lo = 2 * st * half_bytes, hi = lo + half_bytes;
    asm("" : "+s"(lo), "+s"(hi));  // else every load of a loop gets an induction variable of its own, in a register per lane
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (lptr_t)(stage + i * 1024), 16, (int)(at[i & 3] + (i < 4 ? lo : hi)), 0, 0, kAux);
  }
};

// LDS addresses of the 8 operands that lane (token n, half hi) reads of such a tile.
__device__ __forceinline__ void operand_addresses(const uint8_t *stage, int lane, uint32_t (&addr)[8]) {
  typedef __attribute__((address_space(3))) const void *lptr_t;
  const int n = lane & 31, hi = lane >> 5;
#pragma unroll
  for (int s = 0; s < 8; ++s) addr[s] = (uint32_t)(uintptr_t)(lptr_t)(stage + n * 256 + (((hi * 8 + s) ^ (n & 15)) << 4));
}

// The operands of a tile whose loads have been waited for; they have left the tile when this returns, so it can be
// requested anew before the contraction.  An asm block: ahead of an ordinary LDS read the compiler waits for every outstanding
// LDS-direct load (window output, 32768 tokens 33.0 -> 31.8 us per call, 22 sequences of 1600 104 -> 101).
template <int kN>
__device__ __forceinline__ void read_operands(u32x4 (&r)[kN], const uint32_t *addr) {
  static_assert(kN == 8 || kN == 4, "");
  if constexpr (kN == 8)
    asm volatile(
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %9\n\t"
        "ds_read_b128 %2, %10\n\t"
        "ds_read_b128 %3, %11\n\t"
        "ds_read_b128 %4, %12\n\t"
        "ds_read_b128 %5, %13\n\t"
        "ds_read_b128 %6, %14\n\t"
        "ds_read_b128 %7, %15\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
        : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]), "v"(addr[5]), "v"(addr[6]), "v"(addr[7])
        : "memory");
  else
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %5\n\t"
        "ds_read_b128 %2, %6\n\t"
        "ds_read_b128 %3, %7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
        : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3])
        : "memory");
}

// Raw logits of the tile that was requested last: acc[v][r] = q_row(m) . k(token lane % 32 of the tile) with m = (r/4)*8 +
// (lane/32)*4 + r%4, i.e. head r/4 of virtual group v and window row (lane/32)*4 + r%4.  `next` requests another tile as soon
// as this one's operands have left the LDS tile.  kHalf: operands held in registers at a time (8 or 4).
// kVg = 2: two virtual groups of one KV head take their logits from the same tile.
template <int kVg, int kHalf, typename Next>
__device__ __forceinline__ void tile_logits(const bf16x8 (&qa)[kVg][8], const uint32_t (&addr)[8], floatx16 (&acc)[kVg], Next next) {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the tile has landed
#pragma unroll
  for (int v = 0; v < kVg; ++v)
    acc[v] = (floatx16){0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s0 = 0; s0 < 8; s0 += kHalf) {
    u32x4 kb[kHalf];
    read_operands<kHalf>(kb, addr + s0);
    if (s0 + kHalf == 8) next();
#pragma unroll
    for (int s = 0; s < kHalf; ++s)
#pragma unroll
      for (int v = 0; v < kVg; ++v)
        acc[v] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa[v][s0 + s], __builtin_bit_cast(bf16x8, kb[s]), acc[v], 0, 0, 0);
  }
}

// The logits of n_sub consecutive tiles, the first of which has been requested: fn(st, acc) for tile st.  kAux: cache policy.
// At 131072 tokens the stream runs at the rate of the same loads without any work between them.
template <int kAux, int kVg, typename F>
__device__ __forceinline__ void stream_tiles(const KTiles &tiles, const bf16x8 (&qa)[kVg][8], int n_sub, int lane, F fn) {
  uint32_t addr[8];
  operand_addresses(tiles.stage, lane, addr);
#pragma unroll 1
  for (int st = 0; st < n_sub; ++st) {
    floatx16 acc[kVg];
    tile_logits<kVg, 8>(qa, addr, acc, [&] {
      if (st + 1 < n_sub) tiles.issue<kAux>(st + 1);
    });
    fn(st, acc);
  }
}

constexpr int kPlain = 0, kOnce = 2;  // cache policies of a tile's loads: as usual, non-temporal

// One element of the running (max, sum) of a softmax row: `one` is 1 if the logit is counted, else 0.  One exponential.
__device__ __forceinline__ void count_logit(float z, float one, float &mx, float &sm) {
  const float d = z - mx;
  const float e = fast_exp2(-fabsf(d));
  sm = d > 0.f ? __builtin_fmaf(sm, e, one) : __builtin_fmaf(one, e, sm);
  mx = d > 0.f ? z : mx;
}

// Block barrier that orders LDS accesses only.  __syncthreads also waits for the acknowledgement of every
// outstanding global store (about 1 us to device memory); where none of those has to be visible behind the
// barrier that wait is pure latency.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The first element of a row, whose (max, sum) is (kNegBig, 0) before it, makes it (z, one) where z is an ordinary number: what
// count_logit gives, without its exponential.  True if that holds for every live lane's 16 logits of a tile (an infinite or
// NaN one: false).  Wave-uniform.
__device__ __forceinline__ bool ordinary_tile(const floatx16 &z, bool live) {
  float s = 0.f;
#pragma unroll
  for (int q = 0; q < 16; ++q) s += fabsf(z[q]);
  return !__any(live && !(s < -kNegBig));
}

// Folds the per-lane running (max, sum) pairs of a wave's 32 softmax rows over the 32 token
// lanes, through a wave-private LDS transpose (`scratch` >= 4480 bytes, 4-byte aligned).
// In: mx[r], sm[r] of row m = (r/4)*8 + (lane/32)*4 + r%4 for token lane%32.
// Out (every lane; lanes l and l+32 agree): (M, S) of row lane%32, S relative to M.
// On return scratch[32*33 + m] still holds M of row m (kFoldMaxOffset floats into scratch).
// The summation order is fixed, so results are reproducible.
constexpr int kFoldMaxOffset = 32 * 33;
__device__ __forceinline__ float2 fold_rows(const float (&mx)[16], const float (&sm)[16], float *scratch, int lane) {
  const int n = lane & 31, hi = lane >> 5;
  float *T = scratch;             // [32 rows][33]
  float *Mrow = scratch + 32 * 33;
  wave_lds_sync();
#pragma unroll
  for (int r = 0; r < 16; ++r) T[((r >> 2) * 8 + hi * 4 + (r & 3)) * 33 + n] = mx[r];
  wave_lds_sync();
  const int row = lane & 31, half = lane >> 5;
  float M = kNegBig;
#pragma unroll
  for (int j = 0; j < 16; ++j) M = fmaxf(M, T[row * 33 + half * 16 + j]);
  M = fmaxf(M, __shfl_xor(M, 32));
  if (lane < 32) Mrow[row] = M;
  wave_lds_sync();
  float scaled[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) scaled[r] = sm[r] * fast_exp2(mx[r] - Mrow[(r >> 2) * 8 + hi * 4 + (r & 3)]);
#pragma unroll
  for (int r = 0; r < 16; ++r) T[((r >> 2) * 8 + hi * 4 + (r & 3)) * 33 + n] = scaled[r];
  wave_lds_sync();
  float S = 0.f;
#pragma unroll
  for (int j = 0; j < 16; ++j) S += T[row * 33 + half * 16 + j];
  S += __shfl_xor(S, 32);
  return make_float2(M, S);
}

// x(lane) + x(lane ^ 32) in every lane, low half first (one VALU lane swap, no LDS round trip).
__device__ __forceinline__ float add_across_halves(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The window sums of a token for the 4 heads of virtual group g, which both wave halves hold, into the group's rows[i][slot]: each
// half stores two of them.  A token that is not scored counts as 0 (see pool_and_write).
template <int kStride>
__device__ __forceinline__ void store_sums(const ScoreArgs &a, float (*rows)[kStride], int g, int slot, int hi, bool scored,
                                           const float (&sum)[4]) {
  const int heads = vg_heads(a, g);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float x = lane_pick(hi != 0, sum[2 * j], sum[2 * j + 1]);
    if (2 * j + hi < heads) rows[2 * j + hi][slot] = scored ? x : 0.f;
  }
}

// max(x, y, z) without the quietening of every operand that fmaxf on values from memory costs.
__device__ __forceinline__ float max3(float x, float y, float z) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
  return r;
}

// Pooling kernel 7 (the paper's) for the owned tokens of one virtual group, kPer neighbouring tokens per lane, whose kPer + 6
// taps are 8-byte LDS reads per head (the first tap of owned token jj is slot jj).  See pool_and_write.  Reads up to kPer - 1 slots past
// the last tap of an owned token (kPoolPad floats behind the last row); what they give is not used.
constexpr int kPoolPad = 4;
template <int kStride, bool kMax, int kPer, bool kPart>
__device__ __forceinline__ void pool7_group(const ScoreArgs &a, const float (*rows)[kStride], float *g_row, int g, int own, size_t col,
                                            int lane) {
#pragma clang fp contract(off)  // a pooled value is rounded before it enters a mean
  typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
  const int n_h = vg_heads(a, g), h0 = vg_head0(a, g);
#pragma unroll 1
  for (int jj = kPer * lane; jj < own; jj += 64 * kPer) {
    float p[kMaxGroup][kPer];
#pragma unroll
    for (int hl = 0; hl < kMaxGroup; ++hl) {
      const float2 *row = reinterpret_cast<const float2 *>(rows[hl < n_h ? hl : 0] + jj);
      float v[kPer + 6];
#pragma unroll
      for (int i = 0; i < kPer + 6; i += 2) {
        const float2 x = row[i / 2];
        v[i] = x.x;
        v[i + 1] = x.y;
      }
#pragma unroll
      for (int i = 0; i < kPer; i += 2) {
        if constexpr (kMax) {
          const float mid = max3(v[i + 1], v[i + 2], max3(v[i + 3], v[i + 4], max3(v[i + 5], v[i + 6], v[i + 6])));  // the taps both tokens have
          p[hl][i] = max3(mid, v[i], v[i]);
          p[hl][i + 1] = max3(mid, v[i + 7], v[i + 7]);
        } else {
#pragma unroll
          for (int e = i; e < i + 2; ++e)
            p[hl][e] = ((((((v[e] + v[e + 1]) + v[e + 2]) + v[e + 3]) + v[e + 4]) + v[e + 5]) + v[e + 6]) * a.inv_k;
        }
      }
    }
    auto put = [&](float *dst, const float (&x)[kPer], float f) {
#pragma unroll
      for (int i = 0; i < kPer; i += 2) {
        if (jj + i + 1 < own) *reinterpret_cast<f32x2u *>(dst + i) = f32x2u{x[i] * f, x[i + 1] * f};
        else if (jj + i < own) dst[i] = x[i] * f;
      }
    };
    float gs[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) gs[i] = 0.f;
#pragma unroll
    for (int hl = 0; hl < kMaxGroup; ++hl)
      if (hl < n_h) {
        if (a.scores_head) put(a.scores_head + (size_t)(h0 + hl) * a.sum_p + col + jj, p[hl], 1.f);
#pragma unroll
        for (int i = 0; i < kPer; ++i) gs[i] += p[hl][i];
      }
#pragma unroll
    for (int i = 0; i < kPer; i += 2)
      *reinterpret_cast<float2 *>(g_row + jj + i) = make_float2(gs[i], gs[i + 1]);  // past the last owned token: not read
    if (a.scores_group && a.vsh == 0) put(a.scores_group + (size_t)g * a.sum_p + col + jj, gs, a.inv_g);
    if (kPart && a.group_sums && g >= kSplitWaves) put(a.group_sums + (size_t)(g - kSplitWaves + 1) * a.sums_stride + col + jj, gs, 1.f);
  }
}

// Pools the per-head window sums along tokens (Eq. 1), averages the heads of each KV group
// (App. B.1) and all heads (Eq. 2) and writes the scores of the owned tokens [o0, o1).
// s_head[4 (v - g0) + i][slot] holds the window-summed probability of head i of virtual group v at token j0 + slot, 0 outside the
// prefix: neutral for max pooling (scores are >= 0) and the zero padding of avg pooling.
// Slots o0 - r - j0 .. o1 + r - 1 - j0 must be filled.  Contains block barriers.
// kPart: the block has the groups g0 .. g1 - 1 (all of a KV head's); where it does not have every group it leaves, instead of the mean
// over all heads, what that is added up from in order: the sum of the first kSplitWaves groups, then each later group's.
template <int kStride, bool kPart = false>
__device__ __forceinline__ void pool_and_write(const ScoreArgs &a, const float (*s_head)[kStride],
                                               float (*g_sum)[kStride], int j0, int o0, int o1, int col0, int g0 = 0, int g1 = 0) {
#pragma clang fp contract(off)
  const int r = a.pool_r;
  const int own = o1 - o0;
  const bool is_max = a.pool_mode == FKV_POOL_MAX;
  const int lane = threadIdx.x & 63, n_waves = blockDim.x >> 6;
  if (!kPart) g1 = a.V;
  const bool split = a.vsh != 0;  // a KV group spans two virtual groups: its mean is formed after the barrier
  for (int lg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); g0 + lg < g1; lg += n_waves) {  // one wave per virtual group
    const int g = g0 + lg;
    const float(*rows)[kStride] = s_head + lg * kMaxGroup;
    if (r == 3) {
      // two tokens per lane as long as that is one step of the loop; four then, for half the steps: each exposes its LDS reads
      // (32768 tokens: compress with 154 per block 56.2 -> 55.7 us per call, scores and window output 41.7 -> 41.4).  Kernels
      // whose rows cannot hold more, with six slots of halo, have no code for four (4 KB of 20).
      auto pool = [&](auto max_t, auto per, int n) {
        pool7_group<kStride, decltype(max_t)::value, decltype(per)::value, kPart>(a, rows, g_sum[lg], g, n, (size_t)col0 + o0, lane);
      };
      typedef std::integral_constant<int, 2> two_t;
      typedef std::integral_constant<int, 4> four_t;
      constexpr int kOneStep = 128;
      if (kStride - 6 <= kOneStep || own <= kOneStep) {
        const int n = min(own, kOneStep);  // says that it is one step: as a loop, 2048 tokens take 0.15 us more
        is_max ? pool(std::true_type{}, two_t{}, n) : pool(std::false_type{}, two_t{}, n);
      } else if constexpr (kStride - 6 > kOneStep) {
        is_max ? pool(std::true_type{}, four_t{}, own) : pool(std::false_type{}, four_t{}, own);
      }
      continue;
    }
    const int n_h = vg_heads(a, g), h0 = vg_head0(a, g);
#pragma unroll 1
    for (int jj = lane; jj < own; jj += 64) {
      const int c = o0 + jj - j0;  // slot of the pooled token
      float gs = 0.f;
#pragma unroll 1
      for (int hl = 0; hl < n_h; ++hl) {
        const float *row = rows[hl] + c;
        float p;
        if (is_max) {
          p = row[0];
          for (int t = -r; t <= r; ++t) p = fmaxf(p, row[t]);
        } else {
          p = 0.f;
          for (int t = -r; t <= r; ++t) p += row[t];
          p *= a.inv_k;
        }
        if (a.scores_head) a.scores_head[(size_t)(h0 + hl) * a.sum_p + col0 + o0 + jj] = p;
        gs += p;
      }
      g_sum[lg][jj] = gs;
      if (kPart && a.group_sums && g >= kSplitWaves) a.group_sums[(size_t)(g - kSplitWaves + 1) * a.sums_stride + col0 + o0 + jj] = gs;
      if (a.scores_group && !split) a.scores_group[(size_t)g * a.sum_p + col0 + o0 + jj] = gs * a.inv_g;
    }
  }
  const bool first_sums = kPart && a.group_sums != nullptr && g0 == 0;
  if (a.scores_tsp == nullptr && !first_sums && !(split && a.scores_group)) return;
  lds_barrier();
  if (split && a.scores_group) {
    for (int i = threadIdx.x; i < own * ((g1 - g0) >> 1); i += blockDim.x) {
      const int kv = i / own, jj = i - kv * own;
      a.scores_group[(size_t)((g0 >> 1) + kv) * a.sum_p + col0 + o0 + jj] = (g_sum[2 * kv][jj] + g_sum[2 * kv + 1][jj]) * a.inv_g;
    }
  }
  if (first_sums)
    for (int jj = threadIdx.x; jj < own; jj += blockDim.x) {
      float tot = 0.f;
#pragma unroll
      for (int i = 0; i < kSplitWaves; ++i) tot += g_sum[i][jj];
      a.group_sums[col0 + o0 + jj] = tot;
    }
  if (a.scores_tsp == nullptr) return;
  for (int jj = threadIdx.x; jj < own; jj += blockDim.x) {
    float tot = 0.f;
    for (int v0 = 0; v0 < a.V; v0 += kMaxKvHeads) {  // the reads of 8 groups at a time (there are rows for as many), added in order
      float x[kMaxKvHeads];
#pragma unroll
      for (int i = 0; i < kMaxKvHeads; ++i) x[i] = g_sum[v0 + i][jj];
#pragma unroll
      for (int i = 0; i < kMaxKvHeads; ++i) tot = v0 + i < a.V ? tot + x[i] : tot;
    }
    a.scores_tsp[col0 + o0 + jj] = tot * a.inv_h;
  }
}

}  // namespace fkv
