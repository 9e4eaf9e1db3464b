// Attention output of the observation-window rows: out[w][h] = sum_j Att[h, P+w, j] * V[j, g(h)], with
// the probabilities Att of Eq. 1 (Sec. 4.2).  The layer's fused attention kernel does not hand these
// probabilities out (Sec. 5.1), so the estimation step forms them itself; forming the window rows'
// output from them here lets the layer skip those rows.
//
// One wave works on 32-token tiles of one (sequence, virtual group): both contractions run on the
// matrix cores with the 32 softmax rows (4 heads x 8 window rows) of the group on the N side.
//   S^T = K . Q^T : A operand = K rows of the tile (token on the lane), B operand = Q rows.  The
//     result leaves softmax row n = lane % 32 on the lane and 16 tokens of the tile in its
//     registers, so the running maximum, the exponentials and the rescale factor are per-lane
//     scalars (two lanes share a row and meet once per tile).
//   O^T += V^T . P : B operand = the probabilities exactly as the first contraction left them
//     (the token order inside the contraction may be permuted freely as long as V uses the same
//     order); A operand = V transposed through the LDS tile: the lane reads the 8 bytes
//     d = 4m .. 4m+3 of each of its 8 tokens and feeds one 16-bit piece to each of the four
//     32-row output tiles, whose row m therefore stands for d = 4m + tile.
// The probabilities enter the second contraction as a bf16 pair (rounded value + remainder), which
// keeps 16 bits of them; fp32 accumulation throughout.
// K and V tiles go straight from global memory into the wave's two 8 KiB LDS tiles (128-bit
// LDS-direct loads); a tile's next load is issued as soon as its operands sit in registers.
// Tokens are split over blocks (8 waves each); a block merges its waves' running states through
// LDS and leaves one partial (max, sum, 32 x 128 accumulator) per (sequence, group, split); a second
// launch folds the splits in a fixed order.
#include "fkv_wout_merge.h"

namespace fkv {

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
constexpr int kWoWaves = 8;
constexpr int kWoThreads = kWoWaves * 64;
constexpr int kWoTileBytes = 2 * kStageBytes;       // K tile + V tile per wave
constexpr float kWoEmpty = -5.0e29f;                // running maximum before any visible key (> masked logits)

int wout_tiles_per_block_min(void) { return kWoWaves; }

__device__ __forceinline__ float max_across_halves(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ void read_v_half(u32x2 (&r)[8], uint32_t addr) {  // tokens (i & 3) + 8 (i / 4) from addr on
  asm volatile(
      "ds_read_b64 %0, %8\n\t"
      "ds_read_b64 %1, %8 offset:256\n\t"
      "ds_read_b64 %2, %8 offset:512\n\t"
      "ds_read_b64 %3, %8 offset:768\n\t"
      "ds_read_b64 %4, %8 offset:2048\n\t"
      "ds_read_b64 %5, %8 offset:2304\n\t"
      "ds_read_b64 %6, %8 offset:2560\n\t"
      "ds_read_b64 %7, %8 offset:2816\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(addr)
      : "memory");
}

// The window sums of a block's tokens from its kept probabilities: per head, over the window rows, relative to the row's whole sum.
// Every block of a group posts its rows' (max, sum) and reads the other splits', 32 blocks at most: one hop (an owner's fold and a
// second hop, as in fkv_score_exchange.h, serve grids where everybody's partials are too much to read for everybody).  The
// words are emptied by the scores' launch.  All blocks of the launch are resident at once where nothing else holds CUs (the host
// plans for that), and nothing depends on it: a block that does not get its words within kWoWaitTicks, or finds the context's error flag
// set, says so in its sums (kNoSum) and ends, and blocks that start after one has given up do not wait.  Contains block barriers.
__device__ __forceinline__ void leave_sums(const WoutArgs &a, uint8_t *lds, int b, int g, int t0, int t1, int tok_base, int P, unsigned poisoned,
                                           const float (&kept)[kWoKeepTiles][16], const float (&kept_m)[kWoKeepTiles]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hi = lane >> 5;
  constexpr int kPolls = kWoKeepSplits * kRowsPerGroup / kWoThreads;
  float2 *ms = reinterpret_cast<float2 *>(lds);  // [split][row]
  unsigned *late = reinterpret_cast<unsigned *>(lds + kWoKeepSplits * kRowsPerGroup * sizeof(float2));
  const float2 *box = a.boxes + ((size_t)b * a.V + g) * a.n_split * kRowsPerGroup;
  const int n_words = a.n_split * kRowsPerGroup;
  lds_barrier();  // the waves' states have been read
  unsigned long long w[kPolls];
#pragma unroll
  for (int j = 0; j < kPolls; ++j) w[j] = kEmpty64;
  bool ok = poisoned == 0u;
  if (ok) {
    const unsigned late_before = request_flag(a.counters + kCtrWoLate);  // travels beside the first poll
    BoundedWait<16> wait(a.timeout_ticks, kWoWaitTicks);
    while (true) {
      bool missing = false;
#pragma unroll
      for (int j = 0; j < kPolls; ++j)
        if (tid + j * kWoThreads < n_words && w[j] == kEmpty64) w[j] = box_peek(box + tid + j * kWoThreads);
#pragma unroll
      for (int j = 0; j < kPolls; ++j) missing |= tid + j * kWoThreads < n_words && w[j] == kEmpty64;
      if (!__any(missing)) break;
      if (__builtin_amdgcn_readfirstlane(late_before) != 0u || wait.expired()) { ok = false; break; }
    }
    if (!ok && lane == 0) __hip_atomic_store(a.counters + kCtrWoLate, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
#pragma unroll
  for (int j = 0; j < kPolls; ++j)
    if (tid + j * kWoThreads < n_words) __builtin_memcpy(&ms[tid + j * kWoThreads], &w[j], sizeof w[j]);
  if (lane == 0) late[wave] = ok ? 0u : 1u;
  lds_barrier();
#pragma unroll
  for (int i = 0; i < kWoWaves; ++i) ok = ok && late[i] == 0u;
  // row n's normaliser: each half of the wave takes every other split
  float2 st[kWoKeepSplits / 2];
  float M = kNegBig, S = 0.f;
#pragma unroll
  for (int i = 0; i < kWoKeepSplits / 2; ++i) {
    st[i] = ms[min(2 * i + hi, a.n_split - 1) * kRowsPerGroup + n];
    M = fmaxf(M, st[i].x);
  }
  M = max_across_halves(M);
#pragma unroll
  for (int i = 0; i < kWoKeepSplits / 2; ++i) S += 2 * i + hi < a.n_split ? st[i].y * fast_exp2(st[i].x - M) : 0.f;
  const float inv = 1.f / add_across_halves(S);
  const int head = n >> 3, sub = n & 7;
  const bool live = sub < a.W;
  const bool writes = sub < 4 && head < vg_heads(a, g);
  float *dst = a.sums + (size_t)(vg_head0(a, g) + (writes ? head : 0)) * a.sums_stride + (tok_base - b * a.W);
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
  for (int t = 0; t < kWoKeepTiles; ++t) {
    const int tile = t0 + wave + t * kWoWaves;
    if (tile < t1) {
      const float shrink = fast_exp2(kept_m[t] - M) * inv;  // against 2^(logit - log-sum-exp) no rounding of a large exponent
      float x[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        x[q] = live ? kept[t][q] * shrink : 0.f;
        x[q] += dpp_f32<kDppQuadXor1>(0.f, x[q]);
        x[q] += dpp_f32<kDppQuadXor2>(0.f, x[q]);
        x[q] += dpp_f32<kDppHalfMirror>(0.f, x[q]);
      }
      // lane (head, sub < 4) stores tokens 8 sub + 4 hi .. + 3 of the tile
      f32x4u v;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = lane_pick((sub & 2) != 0, lane_pick((sub & 1) != 0, x[i], x[4 + i]), lane_pick((sub & 1) != 0, x[8 + i], x[12 + i]));
        if (!ok) v[i] = __uint_as_float(kNoSum);
      }
      const int tok = tile * kSub + 8 * sub + 4 * hi;
      if (writes) {
        if (tok + 3 < P) *reinterpret_cast<f32x4u *>(dst + tok) = v;
        else
          for (int i = 0; i < 4; ++i)
            if (tok + i < P) dst[tok + i] = v[i];
      }
    }
  }
}

// kSums: the block also keeps its probabilities (at most kWoKeepTiles tiles a wave; relative to the running maximum of their tile,
// which is kept with them) and, once it has its rows' partials of every split, leaves the window-summed probabilities of its tokens, so
// that the scores need no second pass over K: 32768 tokens, K and V 24.8 + K again and scores 16.8 -> 28.7 + 6.7 us.  The stream
// is the other form's with operands in two halves and addresses formed anew per tile (with those in registers 18 went to scratch, 33.4
// us); the sums (exchange, 4 MB written) take 4 us.  A block posts its partials ahead of its output's merge, which the exchange hides
// behind.  Logits instead of probabilities kept: an exponential per value more, and larger errors (a log-sum-exp's rounding).
template <bool kKeepK, bool kSums>
__global__ __launch_bounds__(kWoThreads) void k_wout_partial(WoutArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds_all[kWoWaves * kWoTileBytes];
  __shared__ float2 ms_lds[kWoWaves][kRowsPerGroup];
  typedef __attribute__((address_space(1))) const void *gptr_t;
  typedef __attribute__((address_space(3))) void *lptr_t;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, hi = lane >> 5;
  const int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int tok_base = a.cu[b];
  const int Lb = a.cu[b + 1] - tok_base;
  const int P = Lb - a.W;
  const int n_tiles = (Lb + kSub - 1) / kSub;
  const int per = (n_tiles + a.n_split - 1) / a.n_split;
  const int t0 = split * per, t1 = min(n_tiles, t0 + per);
  uint8_t *ktile = lds_all + wave * kWoTileBytes, *vtile = ktile + kStageBytes;

  const int blk_id = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;  // timing builds only
  (void)blk_id;
  FKV_BTICK_AT(blk_id, 0);
  // direct-to-LDS tile loads: lane l of load i lands at tile offset i*1024 + 16 l, i.e. token slot
  // 4 i + l/16, 16-byte column l%16.  The K tile is XOR-swizzled (from the global side), V is plain.
  // Both streams are read once: the loads are marked non-temporal (measured 34.3 instead of 38.6 us per call at
  // 32768 tokens), except K when the caller reads it again right after this launch (kKeepK).
  // Addresses are a tile's own plus 32-bit offsets of its rows, kept within the sequence.
  const int c = lane & 15, tq = lane >> 4;
  const uint32_t row = (uint32_t)a.Hkv * (kHeadDim * 2);
  uint32_t row_at[8], col_k[4];
#pragma unroll
  for (int i = 0; i < 8; ++i) row_at[i] = (i * 4 + tq) * row;
#pragma unroll
  for (int i = 0; i < 4; ++i) col_k[i] = (c ^ (i * 4 + tq)) << 4;
  auto tile_of = [&](const uint16_t *x, int tile) {
    return reinterpret_cast<const uint8_t *>(x + ((size_t)(tok_base + tile * kSub) * a.Hkv + vg_kv_head(a, g)) * kHeadDim);
  };
  // The kept logits leave no registers for addresses of every load: they are formed anew per tile.
  auto form_addresses = [&] {
    if constexpr (kSums) {
      uint32_t base = tq * row;
      asm("" : "+v"(base));
#pragma unroll
      for (int i = 0; i < 8; ++i) row_at[i] = base + i * 4 * row;
    }
  };
  const KTiles k_tiles(a, tok_base, vg_kv_head(a, g), (t0 + wave) * kSub, Lb, ktile, lane);
  auto issue_k = [&](int tile) {
    if constexpr (kSums) {
      k_tiles.issue<kPlain>(tile - t0 - wave);
      return;
    }
    const uint8_t *rows = tile_of(a.k, tile);
    const uint32_t last = (uint32_t)min(kSub - 1, Lb - 1 - tile * kSub) * row;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(rows + (min(row_at[i], last) + col_k[i & 3])), (lptr_t)(ktile + i * 1024), 16, 0, kKeepK ? 0 : 2);
  };
  auto issue_v = [&](int tile) {
    keep_access_order();  // the wait for a K tile leaves the 8 youngest loads in flight: these
    form_addresses();
    const uint8_t *rows = tile_of(a.v, tile);
    const uint32_t last = (uint32_t)min(kSub - 1, Lb - 1 - tile * kSub) * row;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(rows + (min(row_at[i], last) + (c << 4))), (lptr_t)(vtile + i * 1024), 16, 0, 2);
  };

  floatx16 o[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int q = 0; q < 16; ++q) o[t][q] = 0.f;
  float m = kWoEmpty, s = 0.f;
  const int vis_last = a.causal ? P + (n & 7) : Lb - 1;  // last key softmax row n may see

  uint32_t kaddr[8];
  operand_addresses(ktile, lane, kaddr);
  const uint32_t vaddr = (uint32_t)(uintptr_t)(lptr_t)(vtile + hi * 1024 + n * 8);
  int tile = t0 + wave;
  bf16x8 qa[8];
  load_q(a, b, g, lane, qa);
  float kept[kSums ? kWoKeepTiles : 1][16], kept_m[kSums ? kWoKeepTiles : 1];  // 2^(logit - kept_m), laid out as acc below
  int step = 0;
  const unsigned flag = kSums ? request_flag(a.counters + kCtrError) : 0u;
  if (tile < t1) {
    issue_k(tile);
    issue_v(tile);
  }
#pragma unroll 1
  for (; tile < t1; tile += kWoWaves) {
    const bool more = tile + kWoWaves < t1;
    __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt(8): the K tile has landed (V may still be on its way)
    floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    constexpr int kHalf = kSums ? 4 : 8;  // operands in registers at a time
#pragma unroll
    for (int s0 = 0; s0 < 8; s0 += kHalf) {
      u32x4 kb[kHalf];
      if constexpr (kSums) {
        uint32_t at = kaddr[0], col = ((hi * 8) ^ (n & 15)) << 4;
        asm("" : "+v"(at), "+v"(col));
        at -= col;
#pragma unroll
        for (int s = 0; s < kHalf; ++s) kaddr[1 + s] = at + (col ^ ((s0 + s) << 4));
        read_operands<kHalf>(kb, kaddr + 1);
      } else {
        read_operands<kHalf>(kb, kaddr + s0);
      }
      if (s0 + kHalf == 8 && more) issue_k(tile + kWoWaves);
#pragma unroll
      for (int s8 = 0; s8 < kHalf; ++s8)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kb[s8]), qa[s0 + s8], acc, 0, 0, 0);
    }

    // acc[q] = logit of softmax row n and token slot 8*(q/4) + 4*hi + q%4 of the tile
    const int tok0 = tile * kSub;
    const bool edge = tok0 + kSub - 1 > (a.causal ? P : Lb - 1);  // some (row, token) pair of the tile is masked
    float z[16];
    float tmax = kNegBig;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int tok = tok0 + 8 * (q >> 2) + 4 * hi + (q & 3);
      z[q] = acc[q] * a.scale_log2e;
      if (edge && tok > vis_last) z[q] = kNegBig;
      tmax = fmaxf(tmax, z[q]);
    }
    tmax = max_across_halves(tmax);
    const float m_new = fmaxf(m, tmax);
    const float alpha = fast_exp2(m - m_new);
    m = m_new;
    float psum = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      z[q] = fast_exp2(z[q] - m_new);  // masked: 2^(-1e30 - m_new) = 0 because m_new >= kWoEmpty
      psum += z[q];
    }
    s = s * alpha + psum;
    if constexpr (kSums) {
#pragma unroll
      for (int t = 0; t < kWoKeepTiles; ++t)
        if (t == step) {
          asm volatile("");  // a branch, not a choice per register for every t
#pragma unroll
          for (int q = 0; q < 16; ++q) kept[t][q] = z[q];
          kept_m[t] = m_new;
        }
      ++step;
    }
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0ull) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) o[t][q] *= alpha;
    }
    bf16x8 ph[2], pl[2];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const __bf16 h = (__bf16)z[q];
      ph[q >> 3][q & 7] = h;
      pl[q >> 3][q & 7] = (__bf16)(z[q] - (float)h);
    }

    if (more) __builtin_amdgcn_s_waitcnt(0x0F78);  // the V tile has landed (the next K tile may be in flight)
    else __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      u32x2 r[8];  // r[i]: token slot 16*s2 + 8*(i/4) + 4*hi + i%4, the one acc register 8*s2 + i stands for
      read_v_half(r, vaddr + s2 * 4096);
      u32x4 va[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x2 e = r[2 * j], f = r[2 * j + 1];
        va[0][j] = (e.x & 0xffffu) | (f.x << 16);
        va[1][j] = (e.x >> 16) | (f.x & 0xffff0000u);
        va[2][j] = (e.y & 0xffffu) | (f.y << 16);
        va[3][j] = (e.y >> 16) | (f.y & 0xffff0000u);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[t]), ph[s2], o[t], 0, 0, 0);
        o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[t]), pl[s2], o[t], 0, 0, 0);
      }
    }
    if (more) issue_v(tile + kWoWaves);
  }

  FKV_BTICK_AT(blk_id, 1);
  // ---- the wave's state into its own (now idle) LDS tiles: O[row n][d], 16-byte chunks XOR-swizzled by row
  s = add_across_halves(s);
  float *ow = reinterpret_cast<float *>(ktile);
  int at_hi = 4 * hi;
  if constexpr (kSums) asm("" : "+v"(at_hi));  // else a row's number is kept through the loop, one register too many
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int mrow = 8 * (q >> 2) + at_hi + (q & 3);  // output row of the tiles; d = 4*mrow + tile
    *reinterpret_cast<float4 *>(ow + n * kHeadDim + ((mrow ^ n) << 2)) = make_float4(o[0][q], o[1][q], o[2][q], o[3][q]);
  }
  if (hi == 0) ms_lds[wave][n] = make_float2(m, s);
  __syncthreads();
  FKV_BTICK_AT(blk_id, 2);

  // ---- merge the waves in a fixed order and write the block's partial
  const unsigned poisoned = kSums ? __builtin_amdgcn_readfirstlane(flag) : 0u;
  const size_t slot = ((size_t)b * a.V + g) * a.n_split + split;
  float *po = a.part_o + slot * kWoRowFloats;
  auto leave_partials = [&] {
    if (threadIdx.x >= kRowsPerGroup) return;
    const int row = threadIdx.x;
    float M = ms_lds[0][row].x;
#pragma unroll
    for (int w = 1; w < kWoWaves; ++w) M = fmaxf(M, ms_lds[w][row].x);
    float S = 0.f;
#pragma unroll
    for (int w = 0; w < kWoWaves; ++w) S += ms_lds[w][row].y * fast_exp2(ms_lds[w][row].x - M);
    a.part_ms[slot * kRowsPerGroup + row] = make_float2(M, S);
    if (kSums && poisoned == 0u) box_post(a.boxes + slot * kRowsPerGroup + row, make_float2(M, S));
  };
  if (kSums) leave_partials();  // the exchange is waited for
#pragma unroll
  for (int j = 0; j < kWoRowFloats / 4 / kWoThreads; ++j) {
    const int idx = threadIdx.x + j * kWoThreads;
    const int row = idx >> 5, chunk = idx & 31;
    float M = ms_lds[0][row].x;
#pragma unroll
    for (int w = 1; w < kWoWaves; ++w) M = fmaxf(M, ms_lds[w][row].x);
    float4 accv = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < kWoWaves; ++w) {
      const float f = fast_exp2(ms_lds[w][row].x - M);
      const float4 x = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(lds_all + w * kWoTileBytes) +
                                                         row * kHeadDim + ((chunk ^ row) << 2));
      accv.x += f * x.x; accv.y += f * x.y; accv.z += f * x.z; accv.w += f * x.w;
    }
    *reinterpret_cast<float4 *>(po + row * kHeadDim + chunk * 4) = accv;
  }
  if (!kSums) leave_partials();
  if constexpr (kSums) leave_sums(a, lds_all, b, g, t0, t1, tok_base, P, poisoned, kept, kept_m);
  FKV_BTICK_AT(blk_id, 3);
}

constexpr int kWoMergeThreads = 256;
__global__ __launch_bounds__(kWoMergeThreads) void k_wout_merge(WoutArgs a) {
  merge_output(a, blockIdx.x, blockIdx.y * (kWoMergeThreads / 4) + (threadIdx.x >> 2), threadIdx.x & 3);
}

hipError_t launch_wout(const WoutArgs &a, hipStream_t s) {
  const dim3 grid(a.n_split, a.V, a.n_seq), block(kWoThreads);
  if (a.sums != nullptr)
    hipLaunchKernelGGL((k_wout_partial<true, true>), grid, block, 0, s, a);
  else if (a.keep_k)
    hipLaunchKernelGGL((k_wout_partial<true, false>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((k_wout_partial<false, false>), grid, block, 0, s, a);
  return hipGetLastError();
}
int wout_sums_max_blocks_per_cu(void) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_wout_partial<true, true>, kWoThreads, 0) != hipSuccess) return 0;
  return n;
}
hipError_t launch_wout_merge(const WoutArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_wout_merge, dim3(a.n_seq * a.V, kWoOutputs / (kWoMergeThreads / 4)), dim3(kWoMergeThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace fkv
