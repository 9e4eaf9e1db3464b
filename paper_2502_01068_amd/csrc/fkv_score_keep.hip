// Window-attention scores (Sec. 4.2 Eq. 1-2, App. B.1) of inputs whose logits do not all fit on the chip: the grid is
// resident like that of fkv_score_fused.hip, but a block keeps only the logits of its last tiles, in registers and LDS, while the
// grid agrees on the softmax normalisers, and streams its first tiles of K a second time afterwards.
//
//   phase 1  stream the block's tiles (owned tokens plus pooling halo): running (max, sum) of the owned tokens per
//            softmax row; raw logits of the last kLds + kKeep tiles stay on the chip
//   phase 2  grid exchange of the row statistics (fkv_score_exchange.h); the first tile of phase 3 is on its way
//   phase 3  probabilities of the tiles streamed again and, between their loads, of the kept ones; window sums to LDS
//   phase 4  pooling, head means, scores
//
// Against the two-pass kernels (fkv_score.hip), which read K twice and need three launches, K's second read shrinks
// by the kept part and a launch boundary (the statistics' way through memory and back) becomes the exchange:
// 131072 tokens (17 tiles per block, 10 kept) 97.6 -> 66.4 us in the kernel trace, 8 sequences of 8192-16384 tokens 82.4 ->
// 55.6 us.  With more than 4 query heads per KV head a wave takes both virtual groups of its KV head from one tile and
// keeps 3 tiles of each: 64 / 8 heads at 20001 tokens 40.0 -> 24.6 us.  The tiles go through loops whose code is 23.6 KB (27.7 KB for
// wide groups); written out tile by tile it was 63 KB (46 KB), fetched once each, with 64-bit addresses per load: 131072 tokens
// 68.5, 20001 tokens 28.0 us.
// A probability is 2^(logit * scale - log-sum-exp), the two-pass kernels' formula, whether its logit was kept or not; the
// normaliser is added up over other block shares in another order, so the scores are theirs up to its last bits.
#include "fkv_score_exchange.h"

namespace fkv {

typedef __attribute__((ext_vector_type(4))) float floatx4;
constexpr int kKeepSub = 17, kKeepSubWide = 9;  // tiles per block: the window sums of all heads wait for the pooling in LDS

int keep_sub_max(int v_groups) { return v_groups > kMaxKvHeads ? kKeepSubWide : kKeepSub; }

// kKeep tiles of logits stay in registers; the kLds tiles before those in the part of the window sums' array that
// the wave fills itself, which is idle until phase 3 (8 kept -> 10: 131072 tokens 3.5 us less, 100000 tokens 2.8).
template <int kVg, int kKeep, int kLds, int kMaxSub>
__global__ __launch_bounds__(kThreads) void k_score_keep(ScoreArgs a, FusedArgs f) {
  constexpr int kSlots = kMaxSub * kSub, kGroups = kWaves * kVg;
  __shared__ __attribute__((aligned(16))) uint8_t stage_all[kWaves * kStageBytes];
  __shared__ __attribute__((aligned(16))) float s_head_all[kGroups * kMaxGroup * kSlots + kPoolPad];  // window-summed probabilities per head
  float(*s_head)[kSlots] = reinterpret_cast<float(*)[kSlots]>(s_head_all);
  __shared__ __attribute__((aligned(16))) float g_sum[kGroups][kSlots];
  __shared__ float cst_lds[kGroups][kRowsPerGroup];
  __shared__ unsigned late_lds[kWaves];
  typedef ExchangeLds<kWaves, kMaxFusedBlocks> xch_t;
  static_assert(sizeof(xch_t) <= sizeof(g_sum), "the exchange's tables lie where the group sums go later");
  static_assert(__alignof__(g_sum) >= alignof(float2) && __alignof__(g_sum) >= alignof(xch_t), "the pooling writes pairs of sums");
  xch_t &xch = *reinterpret_cast<xch_t *>(g_sum);
  constexpr int kWaveSums = kVg * kMaxGroup * kSlots;  // floats of s_head that one wave fills
  static_assert(kLds * kVg * kRowsPerGroup * kSub <= kWaveSums && kWaveSums % 4 == 0, "logits kept in LDS");

  request_args(a, f);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, hi = lane >> 5;
  const int b = find_seq(a.map, blockIdx.x);
  const int tok_base = a.map.cu[b];
  const int Lb = a.map.cu[b + 1] - tok_base;
  const int P = Lb - a.W;
  const int r = a.pool_r;
  const int local = (int)blockIdx.x - a.map.blk[b];
  const int o0 = local * f.own[b], o1 = min(P, o0 + f.own[b]);            // owned prefix tokens
  const bool last = local == a.map.blk[b + 1] - a.map.blk[b] - 1;         // also owns the window columns
  const int c0 = o0 - r, c1 = last ? max(Lb, o1 + r) : o1 + r;            // computed tokens
  const int n_sub = (c1 - c0 + kSub - 1) / kSub;                          // <= kMaxSub (host guarantees)
  const int n_keep = min(n_sub, kKeep), n_lds = min(n_sub - n_keep, kLds), n_re = n_sub - n_keep - n_lds;
  const int col0 = tok_base - b * a.W;
  const int g = wave * kVg;
  const bool has_group = g < a.V;
  uint8_t *stage = stage_all + wave * kStageBytes;
  floatx4 *kept = reinterpret_cast<floatx4 *>(&s_head[0][0] + wave * kWaveSums) + lane;  // [tile][group][4][lane]
  const unsigned flag = request_flag(f.err);

  const KTiles tiles(a, tok_base, vg_kv_head(a, has_group ? g : 0), c0, min(Lb, c1), stage, lane);
  uint32_t addr[8];
  operand_addresses(stage, lane, addr);
  bf16x8 qa[kVg][8];
  // Two groups per wave leave no registers for eight operand addresses: they are formed anew per tile (held, two registers were
  // spilled: 20001 tokens of 64 / 8 heads 39.8 us per call instead of 39.3, 3000 tokens 24.6 instead of 23.8).
  typedef __attribute__((address_space(3))) const void *lptr_t;
  const uint32_t operand_row = (uint32_t)(uintptr_t)(lptr_t)(stage + n * 256), operand_column = ((hi * 8) ^ (n & 15)) << 4;
  auto logits = [&](floatx16 (&acc)[kVg], auto next) {
    if constexpr (kVg > 1) {
      uint32_t at[8], column = operand_column;
      asm("" : "+v"(column));
#pragma unroll
      for (int s = 0; s < 8; ++s) at[s] = operand_row + (column ^ (s << 4));
      tile_logits<kVg, 4>(qa, at, acc, next);
    } else {
      tile_logits<kVg, 4>(qa, addr, acc, next);
    }
  };

  // ---- phase 1
  float z[kKeep][kVg][16];
  float mx[kVg][16], sm[kVg][16];
  if (has_group) {
    // Tiles that will be read again are loaded plainly, all others non-temporal: 131072 tokens 2 us less than with every
    // load non-temporal, 4 us less than with none.
    if (n_re > 0) tiles.issue<kPlain>(0);
    else tiles.issue<kOnce>(0);
#pragma unroll
    for (int v = 0; v < kVg; ++v) {
      load_q(a, b, g + v, lane, qa[v]);
#pragma unroll
      for (int q = 0; q < 16; ++q) { mx[v][q] = kNegBig; sm[v][q] = 0.f; }
    }
    auto count = [&](int st, const floatx16 (&acc)[kVg]) {
      const int tok = c0 + st * kSub + n;
      const bool counted = ((tok >= o0) & (tok < o1)) | (last & (tok >= P) & (tok < Lb));
      bool ok[4];
      float one[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ok[i] = counted & ((a.causal == 0) | (tok <= P + hi * 4 + i));
        one[i] = ok[i] ? 1.f : 0.f;
      }
#pragma unroll
      for (int v = 0; v < kVg; ++v)
#pragma unroll
        for (int q = 0; q < 16; ++q)
          count_logit(ok[q & 3] ? acc[v][q] * a.scale_log2e : kNegBig, one[q & 3], mx[v][q], sm[v][q]);
    };
#pragma unroll 1
    for (int st = 0; st < n_re + n_lds; ++st) {  // there are kept tiles behind these
      floatx16 acc[kVg];
      logits(acc, [&] {
        if (st + 1 < n_re) tiles.issue<kPlain>(st + 1);
        else tiles.issue<kOnce>(st + 1);
      });
      if (st >= n_re) {
#pragma unroll
        for (int v = 0; v < kVg; ++v)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            kept[(((st - n_re) * kVg + v) * 4 + q) * 64] = floatx4{acc[v][4 * q], acc[v][4 * q + 1], acc[v][4 * q + 2], acc[v][4 * q + 3]};
      }
      count(st, acc);
    }
    const int st0 = n_re + n_lds;
#pragma unroll 1
    for (int k = 0; k < n_keep; ++k) {
      floatx16 acc[kVg];
      logits(acc, [&] {
        const bool more = k + 1 < n_keep;
        if (more || n_re > 0) tiles.issue<kOnce>(more ? st0 + k + 1 : 0);  // 0: the first tile of phase 3
      });
#pragma unroll
      for (int t = 0; t < kKeep; ++t)
        if (t == k) {
          asm volatile("");  // a branch, not a choice per register for every t
#pragma unroll
          for (int v = 0; v < kVg; ++v)
#pragma unroll
            for (int q = 0; q < 16; ++q) z[t][v][q] = acc[v][q];
        }
      count(st0 + k, acc);
    }
  }
  const unsigned poisoned = __builtin_amdgcn_readfirstlane(flag);  // ahead of the posts, see k_score_fused
  if (has_group) {
#pragma unroll
    for (int v = 0; v < kVg; ++v) {
      float mloc[16];
      fold_and_post(f, blockIdx.x, mx[v], sm[v], mloc, g + v, lane, poisoned);
    }
  }
  // A failed exchange leaves mailboxes in an unknown state: until the host has reset them
  // (fkv_clear_error) every launch only marks its scores invalid.
  if (poisoned != 0u) {
    __builtin_amdgcn_s_waitcnt(0x0F70);
    poison_scores(a, col0, o0, o1);
    return;
  }

  // ---- phase 2
  bool wave_ok = owner_duty(a, f, xch, wave, lane);
  if (has_group) wave_ok = wave_ok && collect_lse<kVg>(f, blockIdx.x, g, lane, cst_lds[g]);

  // ---- phase 3
  if (has_group && wave_ok) {
    wave_lds_sync();
    float cst[kVg][16];
#pragma unroll
    for (int v = 0; v < kVg; ++v)
#pragma unroll
      for (int q = 0; q < 16; ++q) cst[v][q] = cst_lds[g + v][(q >> 2) * 8 + hi * 4 + (q & 3)];
    auto finish = [&](int st, const auto &acc) {
      const int tok = c0 + st * kSub + n;
      const bool inb = (tok >= 0) & (tok < min(P, c1));  // only prefix tokens are scored; slots past c1 were never loaded
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
    };
    {
      float zl[kLds][kVg][16];
#pragma unroll
      for (int t = 0; t < kLds; ++t)
        if (t < n_lds)
#pragma unroll
          for (int v = 0; v < kVg; ++v)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const floatx4 x = kept[((t * kVg + v) * 4 + q) * 64];
#pragma unroll
              for (int i = 0; i < 4; ++i) zl[t][v][4 * q + i] = x[i];
            }
      wave_lds_sync();  // the sums may overwrite them
#pragma unroll
      for (int t = 0; t < kLds; ++t)
        if (t < n_lds) finish(n_re + t, zl[t]);
    }
    // A tile streamed again and one kept in registers in turn, whose probabilities are formed while the next tile is on its
    // way.  A loop, so that its code is fetched once.
    int re = 0, kp = 0;
#pragma unroll 1
    while (re < n_re || kp < n_keep) {
      float x[kVg][16];
      int st;
      if (re < n_re && (re <= kp || kp == n_keep)) {
        st = re++;
        floatx16 acc[kVg];
        logits(acc, [&] { if (re < n_re) tiles.issue<kOnce>(re); });
#pragma unroll
        for (int v = 0; v < kVg; ++v)
#pragma unroll
          for (int q = 0; q < 16; ++q) x[v][q] = acc[v][q];
      } else {
        st = n_re + n_lds + kp;
#pragma unroll
        for (int t = 0; t < kKeep; ++t)
          if (t == kp) {
            asm volatile("");
#pragma unroll
            for (int v = 0; v < kVg; ++v)
#pragma unroll
              for (int q = 0; q < 16; ++q) x[v][q] = z[t][v][q];
          }
        ++kp;
      }
      finish(st, x);
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // nothing may land in LDS after this point
  if (lane == 0) late_lds[wave] = wave_ok ? 0u : 1u;
  lds_barrier();
  bool grid_ok = true;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) grid_ok = grid_ok && late_lds[w] == 0u;

  // ---- phase 4
  if (grid_ok) {
    pool_and_write<kSlots>(a, s_head, g_sum, c0, o0, o1, col0);
  } else {
    poison_scores(a, col0, o0, o1);
    if (threadIdx.x == 0) __hip_atomic_store(f.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

hipError_t launch_score_keep(const ScoreArgs &a, const FusedArgs &f, hipStream_t s) {
  if (a.V > kMaxKvHeads)
    hipLaunchKernelGGL((k_score_keep<2, 2, 1, kKeepSubWide>), dim3(f.n_wg), dim3(kThreads), 0, s, a, f);
  else
    hipLaunchKernelGGL((k_score_keep<1, 8, 2, kKeepSub>), dim3(f.n_wg), dim3(kThreads), 0, s, a, f);
  return hipGetLastError();
}

int score_keep_max_blocks_per_cu(void) {  // they take nearly all of a CU's LDS, twice what k_score_fused does
  int n = 0, wide = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_score_keep<1, 8, 2, kKeepSub>, kThreads, 0) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&wide, k_score_keep<2, 2, 1, kKeepSubWide>, kThreads, 0) != hipSuccess) return 0;
  return n < wide ? n : wide;
}

}  // namespace fkv
