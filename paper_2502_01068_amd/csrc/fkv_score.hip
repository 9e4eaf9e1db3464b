// Window-attention saliency scores (Sec. 4.2 Eq. 1-2, App. B.1) for gfx950.
//
// Three launches, K streamed twice (the softmax normaliser of each of the Hq*W window rows
// depends on every key, so the rows' log-sum-exp must exist before any score does):
//   k_stats    one pass over K: per block, running (max, sum) of every softmax row
//   k_combine  folds the per-block partials into one log2-domain normaliser per row
//   k_scores   second pass over K: probabilities, window sum, per-head pooling in LDS,
//              group mean and all-head mean, written once
//
// The logits of one KV group are a [32 x 128] x [128 x 32 tokens] product: the 32 rows are
// the G<=4 heads of the group times the W<=8 window queries, exactly one 32x32x16 bf16 MFMA
// tile in M.  Tokens sit on the MFMA N axis, i.e. on lanes, so the per-row softmax statistics
// stay in registers per lane and are only reduced across lanes once per block.
//
// K path: one wave per KV head, its 32-token tiles straight into the wave's LDS tile (KTiles), the next one requested as soon
// as the operands have left it.
#include <type_traits>

#include "fkv_wout_merge.h"

namespace fkv {

int stats_chunk_tokens(void) { return kStatsChunk; }
int scores_sub_short(void) { return kScoresSubShort; }
int scores_sub_long(void) { return kScoresSubLong; }
int scores_sub_wide(void) { return kScoresSubWide; }

template <int kVg>
__global__ __launch_bounds__(kThreads) void k_stats(ScoreArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t stage_all[kWaves * kStageBytes];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, hi = lane >> 5;
  const int b = find_seq(a.map, blockIdx.x);
  const int tok_base = a.map.cu[b];
  const int Lb = a.map.cu[b + 1] - tok_base;
  const int P = Lb - a.W;
  const int t0 = ((int)blockIdx.x - a.map.blk[b]) * a.chunk;
  const int t1 = min(Lb, t0 + a.chunk);
  uint8_t *stage = stage_all + wave * kStageBytes;
  const int g = wave * kVg;
  if (g >= a.V) return;

  FKV_TICK(16);
  const KTiles tiles(a, tok_base, vg_kv_head(a, g), t0, t1, stage, lane);
  tiles.issue<kOnce>(0);
  bf16x8 qa[kVg][8];
  float mx[kVg][16], sm[kVg][16];
#pragma unroll
  for (int v = 0; v < kVg; ++v) {
    load_q(a, b, g + v, lane, qa[v]);
#pragma unroll
    for (int r = 0; r < 16; ++r) { mx[v][r] = kNegBig; sm[v][r] = 0.f; }
  }

  stream_tiles<kOnce>(tiles, qa, (t1 - t0 + kSub - 1) / kSub, lane, [&](int st, const floatx16 (&acc)[kVg]) {
    const int tok = t0 + st * kSub + n;
    const bool valid = tok < t1;
    bool ok[4];
    float one[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ok[i] = valid & ((a.causal == 0) | (tok <= P + hi * 4 + i));
      one[i] = ok[i] ? 1.f : 0.f;
    }
#pragma unroll
    for (int v = 0; v < kVg; ++v)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        count_logit(ok[r & 3] ? acc[v][r] * a.scale_log2e : kNegBig, one[r & 3], mx[v][r], sm[v][r]);
  });
  FKV_TICK(17);
#pragma unroll
  for (int v = 0; v < kVg; ++v) {
    const float2 ms = fold_rows(mx[v], sm[v], reinterpret_cast<float *>(stage), lane);
    if (lane < 32)
      a.partial[(size_t)((g + v) * kRowsPerGroup + lane) * a.partial_stride + blockIdx.x] = ms;
  }
  FKV_TICK(18);
}

// One wave per softmax row: grid.x = ceil(B*Hkv*32 / 4), 256 threads.  Lane l folds partials
// l, l+64, ... in order, then the 64 lanes are folded by a fixed butterfly.
__global__ __launch_bounds__(256) void k_combine(ScoreArgs a) {
  const int lane = threadIdx.x & 63;
  const int rid = blockIdx.x * 4 + (threadIdx.x >> 6);  // (b, g, m)
  const int rows_per_seq = a.V * kRowsPerGroup;
  if (rid >= a.map.n_seq * rows_per_seq) return;
  const int b = rid / rows_per_seq, gm = rid - b * rows_per_seq;
  const int p0 = a.map.blk[b], p1 = a.map.blk[b + 1];
  const float2 *src = a.partial + (size_t)gm * a.partial_stride;
  float M = kNegBig, S = 0.f;
  for (int p = p0 + lane; p < p1; p += 64) {
    const float2 v = src[p];
    const float mn = fmaxf(M, v.x);
    S = S * fast_exp2(M - mn) + v.y * fast_exp2(v.x - mn);
    M = mn;
  }
  float Mx = M;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) Mx = fmaxf(Mx, __shfl_xor(Mx, off));
  S *= fast_exp2(M - Mx);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) S += __shfl_xor(S, off);
  if (lane == 0) {
    const int row = gm & 31;
    const bool ok = (row >> 3) < vg_heads(a, gm >> 5) && (row & 7) < a.W;
    // probability = exp2(z*scale*log2e - (Mx + log2 S))
    a.rowstat[(size_t)b * rows_per_seq + gm] = ok ? (Mx + __log2f(S)) : 0.f;
  }
}

struct NoWout {};
struct WoutSums : WoutArgs {};  // with window sums; a type of its own: one kernel for both costs the others 0.4 us at 40000 tokens and more

// The window sums that k_wout_partial left for kVg groups of a block's tokens j0 .. j0 + n - 1, into its rows of s_head, 0 outside
// the prefix.  False (wave-uniform) if some are missing.
template <int kSlots, int kVg>
__device__ __forceinline__ bool take_sums(const ScoreArgs &a, const WoutArgs &wo, float (*s_head)[kSlots], int g, int col0, int j0, int n, int P,
                                          int lane) {
  bool missing = false;
  constexpr int kStep = 4;  // loads of a head's row in flight, of four heads
  for (int v = 0; v < kVg; ++v) {
    const int heads = vg_heads(a, g + v);
    const float *src = wo.sums + (size_t)vg_head0(a, g + v) * wo.sums_stride + col0;
    for (int s0 = lane; s0 < n; s0 += 64 * kStep) {
      float x[kMaxGroup][kStep];
#pragma unroll
      for (int h = 0; h < kMaxGroup; ++h)
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
          const int tok = j0 + s0 + 64 * i;
          x[h][i] = h < heads && s0 + 64 * i < n && tok >= 0 && tok < P ? src[(size_t)h * wo.sums_stride + tok] : 0.f;
        }
#pragma unroll
      for (int h = 0; h < kMaxGroup; ++h)
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
          missing |= __float_as_uint(x[h][i]) == kNoSum;
          if (h < heads && s0 + 64 * i < n) s_head[(g + v) * kMaxGroup + h][s0 + 64 * i] = x[h][i];
        }
    }
  }
  return !__any(missing);
}

// O = WoutSums: the window sums are pooled and averaged, K is read by blocks only that miss some of theirs.
// kMaxSub 32-token sub-tiles per block at most.  A block owns a.tile_own tokens (host-chosen so that the
// launch is one block per CU) and computes them and the pooling halo.  The window sums go straight into their own LDS array,
// next to the waves' staging tiles.  O = WoutArgs: the row normalisers come from the splits of k_wout_partial, folded by
// every block for itself while its first tile is on its way, and blocks 0 .. n_merge - 1 write the window rows' output:
// they run on CUs that the scores leave idle, and there is no launch between the two passes over K: scores and output of
// 32768 tokens, a merge launch of 4.9 us and scores of 15.2 before, 16.8 us for both now.
template <int kMaxSub, int kVg, int kAux, typename O>
__global__ __launch_bounds__(kThreads) void k_scores(ScoreArgs a, O wo, int n_merge) {
  constexpr int kSlots = kMaxSub * kSub, kGroups = kWaves * kVg;
  constexpr bool kSums = std::is_same<O, WoutSums>::value, kWout = kSums || std::is_same<O, WoutArgs>::value;
  __shared__ __attribute__((aligned(16))) uint8_t stage_all[kWaves * kStageBytes];
  __shared__ __attribute__((aligned(16))) float s_head_all[kGroups * kMaxGroup * kSlots + kPoolPad];  // window-summed probabilities per head
  float(*s_head)[kSlots] = reinterpret_cast<float(*)[kSlots]>(s_head_all);
  __shared__ __attribute__((aligned(16))) float g_sum[kGroups][kSlots];  // per virtual group sums of pooled head scores
  static_assert(__alignof__(g_sum) >= alignof(float2), "the pooling writes pairs of sums");
  if constexpr (kWout) {
    if ((int)blockIdx.x < n_merge) {
      constexpr int kUnits = kWoOutputs / (kThreads / 4);
      const int units = wo.n_seq * wo.V * kUnits;
      for (int u = blockIdx.x; u < units; u += n_merge)
        merge_output(wo, u / kUnits, (u % kUnits) * (kThreads / 4) + (threadIdx.x >> 2), threadIdx.x & 3);
      return;
    }
    if constexpr (kSums) {  // the mailboxes of k_wout_partial and its mark, for the next call
      if ((int)blockIdx.x == n_merge && threadIdx.x == 0)
        __hip_atomic_store(wo.counters + kCtrWoLate, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int n_words = wo.n_seq * wo.V * wo.n_split * kRowsPerGroup;
      for (int i = ((int)blockIdx.x - n_merge) * kThreads + threadIdx.x; i < n_words; i += ((int)gridDim.x - n_merge) * kThreads)
        box_clear(wo.boxes + i);
    }
  }

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, hi = lane >> 5;
  const int block = (int)blockIdx.x - n_merge;
  const int b = find_seq(a.map, block);
  const int tok_base = a.map.cu[b];
  const int Lb = a.map.cu[b + 1] - tok_base;
  const int P = Lb - a.W;
  const int r = a.pool_r;
  const int o0 = (block - a.map.blk[b]) * a.tile_own, o1 = min(P, o0 + a.tile_own);  // owned tokens
  const int j0 = o0 - r;  // first computed token (may be < 0)
  uint8_t *stage = stage_all + wave * kStageBytes;

  FKV_TICK(24);
  const int g = wave * kVg;
  bool have = false;
  if constexpr (kSums) have = g < a.V && take_sums<kSlots, kVg>(a, wo, s_head, g, tok_base - b * a.W, j0, o1 + r - j0, P, lane);
  if (g < a.V && !have) {
    const KTiles tiles(a, tok_base, vg_kv_head(a, g), j0, min(Lb, o1 + r), stage, lane);
    tiles.issue<kAux>(0);
    bf16x8 qa[kVg][8];
    float cst[kVg][16];
#pragma unroll
    for (int v = 0; v < kVg; ++v) {
      load_q(a, b, g + v, lane, qa[v]);
      const float *rs;
      if constexpr (kWout) {
        float *mine = g_sum[g + v];  // idle until the pooling
        merge_normalisers(wo, b * wo.V + g + v, g + v, lane, mine);
        wave_lds_sync();
        rs = mine;
      } else {
        rs = a.rowstat + ((size_t)b * a.V + g + v) * kRowsPerGroup;
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) cst[v][q] = rs[(q >> 2) * 8 + hi * 4 + (q & 3)];
    }

    stream_tiles<kAux>(tiles, qa, (o1 + r - j0 + kSub - 1) / kSub, lane, [&](int st, const floatx16 (&acc)[kVg]) {
      const int tok = j0 + st * kSub + n;
      const bool inb = (tok >= 0) & (tok < P);  // only prefix tokens are scored
#pragma unroll
      for (int v = 0; v < kVg; ++v) {
        float sum[4];
#pragma unroll
        for (int hl = 0; hl < 4; ++hl) {
          sum[hl] = 0.f;
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            const float e = fast_exp2(__builtin_fmaf(acc[v][hl * 4 + rr], a.scale_log2e, -cst[v][hl * 4 + rr]));
            sum[hl] += (hi * 4 + rr < a.W) ? e : 0.f;
          }
          sum[hl] = add_across_halves(sum[hl]);  // other half of the window rows
        }
        store_sums<kSlots>(a, s_head + (g + v) * kMaxGroup, g + v, st * kSub + n, hi, inb, sum);
      }
    });
  }
  FKV_TICK(25);
  __syncthreads();
  FKV_TICK(26);

  const int col0 = tok_base - b * a.W;  // column of this sequence's token 0 in the score rows
  pool_and_write<kSlots>(a, s_head, g_sum, j0, o0, o1, col0);
  FKV_TICK(27);
}

// One wave per virtual group of up to 4 heads; with more than 8 of those (5 to 8 heads per KV head, more than 4
// KV heads) a wave takes both groups of its KV head, so that K is read once per pass: 64 / 8 heads at 20001 tokens
// 69 -> 61 us per compress call, at 60000 tokens 101 -> 88 us.
hipError_t launch_stats(const ScoreArgs &a, int n_blocks, hipStream_t s) {
  if (a.V > kMaxKvHeads)
    hipLaunchKernelGGL(k_stats<2>, dim3(n_blocks), dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL(k_stats<1>, dim3(n_blocks), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_combine(const ScoreArgs &a, hipStream_t s) {
  const int rows = a.map.n_seq * a.V * kRowsPerGroup;
  hipLaunchKernelGGL(k_combine, dim3((rows + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}
// k_cached: K was just read by the launch before; plain loads then, so that what the caches still hold is used.
hipError_t launch_scores(const ScoreArgs &a, int n_blocks, bool k_cached, hipStream_t s) {
  const dim3 grid(n_blocks), block(kThreads);
  if (a.V > kMaxKvHeads)  // twice the heads in LDS: half the tile
    hipLaunchKernelGGL((k_scores<kScoresSubWide, 2, kOnce, NoWout>), grid, block, 0, s, a, NoWout{}, 0);
  else if (k_cached)
    hipLaunchKernelGGL((k_scores<kScoresSubLong, 1, kPlain, NoWout>), grid, block, 0, s, a, NoWout{}, 0);
  else if (a.tile_sub <= kScoresSubShort)
    hipLaunchKernelGGL((k_scores<kScoresSubShort, 1, kOnce, NoWout>), grid, block, 0, s, a, NoWout{}, 0);
  else
    hipLaunchKernelGGL((k_scores<kScoresSubLong, 1, kOnce, NoWout>), grid, block, 0, s, a, NoWout{}, 0);
  return hipGetLastError();
}

int wout_merge_units(const WoutArgs &a) { return a.n_seq * a.V * (kWoOutputs / (kThreads / 4)); }

hipError_t launch_wout_scores(const ScoreArgs &a, const WoutArgs &o, int n_blocks, int n_merge, hipStream_t s) {
  const dim3 grid(n_blocks + n_merge);
  if (o.sums != nullptr) {
    const WoutSums sums{o};
    if (a.V > kMaxKvHeads)
      hipLaunchKernelGGL((k_scores<kScoresSubWide, 2, kOnce, WoutSums>), grid, dim3(kThreads), 0, s, a, sums, n_merge);
    else
      hipLaunchKernelGGL((k_scores<kScoresSubLong, 1, kPlain, WoutSums>), grid, dim3(kThreads), 0, s, a, sums, n_merge);
  } else if (a.V > kMaxKvHeads)
    hipLaunchKernelGGL((k_scores<kScoresSubWide, 2, kOnce, WoutArgs>), grid, dim3(kThreads), 0, s, a, o, n_merge);
  else
    hipLaunchKernelGGL((k_scores<kScoresSubLong, 1, kPlain, WoutArgs>), grid, dim3(kThreads), 0, s, a, o, n_merge);
  return hipGetLastError();
}

}  // namespace fkv
