// Single-pass window-attention scores (Sec. 4.2 Eq. 1-2, App. B.1): K is read from HBM once.
//
// The softmax normaliser of every window row depends on all keys, so a block cannot turn its
// logits into probabilities until every block has seen its share of K.  Here the logits wait in
// registers: each block owns a contiguous token range small enough that its logits (up to 8 MFMA
// sub-tiles x 16 accumulator registers per lane) stay on chip, all blocks are resident at once
// (one per CU), and a grid-wide exchange of the per-row (max, sum) pairs sits between the K
// stream and the probability / pooling / averaging phase:
//
//   phase 1  stream the block's K rows (owned range plus pooling halo), keep raw logits in
//            registers, fold running (max, sum) of the owned tokens per softmax row
//   phase 2  every block posts its 256 row partials, a line of memory per 8 rows; each group of 8 rows has one owner
//            block somewhere in the grid that collects the group's partials from all blocks of the
//            sequence, folds them in a fixed order (bit-reproducible) and posts the rows' log-sum-exps to
//            every block of the sequence.  What the exchange costs is transactions: with one owner wave per
//            row every partial and every result was one of its own (109 000 at 213 blocks; with groups 14 000),
//            6.6 us from the last post to the last result instead of 3.5.  Groups of 16 rows (two folds per
//            wave) were 1.2 us slower, of 4 or 2 rows no faster.
//   phase 3  probabilities from the kept logits, window sum, LDS pooling, head means, write
//
// What bounds it at short inputs is instruction issue (two waves share a SIMD's vector issue, 4 cycles an instruction) and the
// two trips of the exchange; from about 30000 tokens on the K stream.  So a tile's requests are one addition each (KTiles),
// a tile is requested anew before its contraction, the row maxima take 100 instructions instead of 450, a kept tile goes to its
// registers by a branch, and the flag is looked at before the posts, whose acknowledgement it was waited for with.
// Kernel trace, before -> after: 2048 tokens 14.5 -> 11.5 us, 6554 17.6 -> 13.8, 12289 18.1 -> 14.7, 16384 (head-wise) 20.2 ->
// 16.5, 32768 25.4 -> 21.1.
//
// Short inputs leave CUs idle, and two waves a SIMD in those they use: their ranges go to two blocks of four waves each (fused_split;
// the same work per wave, so the same bits).  The mean over all heads, for which a block needs every group, is then left to the
// select, as sums.  us per call, before -> after: 1759 tokens 16.8 -> 15.0, 2048 with the mean 18.1 -> 17.5, 6554 22.9 ->
// 21.2, 3 sequences of 1700 20.7 -> 17.9, head-wise 3000 19.8 -> 18.6.
//
// Used when the batch fits the resident grid (about 61K tokens on 256 CUs); longer inputs take
// the kernel of fkv_score_keep.hip or the two-pass kernels.  Every wait in phase 2 is bounded: a wave that does not get what it waits
// for within the time limit raises the context's error flag, and its block writes NaN scores.
#include "fkv_score_exchange.h"

namespace fkv {

// Sub-tiles (of 32 tokens) a block keeps in registers.  The variants for inputs with fewer per block carry less code and
// registers for them.
constexpr int kFusedSubFew = 2;
constexpr int kFusedSubShort = 5;
constexpr int kFusedSubLong = 8;
constexpr int kFusedSlotsMax = kFusedSubLong * kSub;

int fused_slots(void) { return kFusedSlotsMax; }

// The split of a launch's ranges (see FusedArgs), or -1: a range is one block's work.  Only where every block still has a CU to
// itself, and ranges are of one or two sub-tiles then.  Blocks of four waves fold two softmax rows a wave for each group of rows they
// own: up to four virtual groups, for which a range stays one block, that is slower where blocks own several (us per call, blocks of
// eight waves and of four: 20 tokens of 16 / 4 heads 27.1, 28.6, 8 sequences of 40 16.8, 17.7, 24 of 900 13.0, 12.9).
int fused_split(int v_groups, int n_seq, int n_ranges, int n_sub, int max_blocks) {
  const int shift = v_groups > kSplitWaves ? 1 : 0;
  if (shift == 0 && n_seq * v_groups * (kRowsPerGroup / kOwnRows) > n_ranges) return -1;
  return v_groups <= kMaxKvHeads && n_sub <= kFusedSubFew && n_ranges <= kSplitRanges && (n_ranges << shift) <= max_blocks ? shift : -1;
}
// Block count up to which a layout of n_sub full sub-tiles per block is preferred over one more
// sub-tile per block (fewer, longer blocks): the exchange gets slower with the number of blocks, a sub-tile costs a trip to memory.
// Launches in a row, us (blocks: sub-tiles per block):
//    3000 tokens  79: 2 11.9, 116: 1 10.5, 158: 1 10.8, 250: 1 11.4     4096  71: 2 11.8, 128: 2 12.3, 158: 1 11.0, 256: 1 11.6
//    6554  80: 3 13.7, 113: 2 12.2, 160: 2 12.7, 252: 1 12.1             9001  112: 3 15.0, 156: 2 13.3, 205: 2 13.6, 250: 2 14.1
//   12289  160: 3 15.6, 212: 2 14.3, 224: 2 14.4, 256: 2 14.8           24000  160: 5 20.3, 197: 4 19.0, 223: 4 19.4, 256: 4 19.8
//   32768  192: 6 24.0, 213: 5 22.5, 256: 5 22.7                        49152  197: 8 29.7, 208: 8 29.4, 240: 7 28.7, 256: 7 30.0
// 224 fits these.  128 for one sub-tile comes from a sweep with the former exchange of one owner wave per row and is
// too low by now: 4096 tokens would be 0.8 us shorter on 158 blocks.  The shares decide the order of a row's sum and with it the
// last bits of the scores.  The kernel of fkv_score_keep.hip follows the rule too and takes every block for more
// sub-tiles than this one holds (64 / 8 heads: 3000 tokens 111: 2 18.7, 125: 1 15.6, 250: 1 16.3; 8000 127: 3 22.1, 160: 2 19.4,
// 250: 2 20.2; 20001 191: 4 25.8, 223: 3 23.9, 254: 3 24.3; 40000 208: 7 36.1, 224: 6 34.0, 255: 6 35.1).
int fused_preferred_blocks(int n_sub) { return n_sub == 1 ? 128 : n_sub * kSub <= kFusedSlotsMax ? 224 : kMaxFusedBlocks; }

// kW = kWaves: a block has all virtual groups of its range.  kW = 4: up to four of them, and a range 1 << f.split blocks.
template <int kFusedSub, int kW>
__global__ __launch_bounds__(kW * 64, 2) void k_score_fused(ScoreArgs a, FusedArgs f) {
  constexpr int kFusedSlots = kFusedSub * kSub;
  constexpr bool kSplit = kW < kWaves;
  __shared__ __attribute__((aligned(16))) uint8_t lds_all[kW * kStageBytes];
  __shared__ float cst_lds[kW][kRowsPerGroup];
  __shared__ ExchangeLds<kW, kSplit ? kSplitRanges : kMaxFusedBlocks> xch;
  __shared__ unsigned flag_lds[1];
  float(*s_head)[kFusedSlots] = reinterpret_cast<float(*)[kFusedSlots]>(lds_all);  // [kW*4][slots]
  float(*g_sum)[kFusedSlots] = reinterpret_cast<float(*)[kFusedSlots]>(lds_all + kW * kMaxGroup * kFusedSlots * 4);
  static_assert((kW * kMaxGroup + kW) * kFusedSlots * 4 <= kW * kStageBytes, "LDS reuse");

  request_args(a, f);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, hi = lane >> 5;
  const int range = kSplit ? (int)blockIdx.x >> f.split : (int)blockIdx.x;
  const int b = find_seq(a.map, range);
  const int tok_base = a.map.cu[b];
  const int Lb = a.map.cu[b + 1] - tok_base;
  const int P = Lb - a.W;
  const int r = a.pool_r;
  const int local = range - a.map.blk[b];
  const int n_ranges = a.map.blk[b + 1] - a.map.blk[b];
  const int o0 = local * f.own[b], o1 = min(P, o0 + f.own[b]);  // owned prefix tokens
  const bool last = local == n_ranges - 1;                      // also owns the window columns
  const int c0 = o0 - r;                                        // first computed token (may be < 0)
  const int c1 = last ? max(Lb, o1 + r) : o1 + r;               // the pooling halo may reach past the window (r > W)
  const int n_sub = (c1 - c0 + kSub - 1) / kSub;                // <= kFusedSub (host guarantees)
  const int col0 = tok_base - b * a.W;
  uint8_t *stage = lds_all + wave * kStageBytes;
  const int g0 = kSplit ? ((int)blockIdx.x & ((1 << f.split) - 1)) * kW : 0, g = g0 + wave;
  const bool has_group = g < a.V;  // the host takes this kernel only for V <= 8 (one wave per virtual group)

  const unsigned flag = request_flag(f.err);
  if (threadIdx.x == 0) flag_lds[0] = 1u;

  FKV_TICK(32);
  FKV_BTICK(0);
  // ---- phase 1: logits into registers, running statistics of the owned tokens
  float z[kFusedSub][16], mloc[16], mx[16], sm[16];
  if (has_group) {
    const KTiles tiles(a, tok_base, vg_kv_head(a, g), c0, min(Lb, c1), stage, lane);
    tiles.issue<kPlain>(0);
    FKV_WTICK(0);
    bf16x8 qa[1][8];
    load_q(a, b, g, lane, qa[0]);
    uint32_t addr[8];
    operand_addresses(stage, lane, addr);
#pragma unroll
    for (int q = 0; q < 16; ++q) { mx[q] = kNegBig; sm[q] = 0.f; }
#pragma unroll 1
    for (int st = 0; st < n_sub; ++st) {
      floatx16 logit[1];
      tile_logits<1, kFusedSub == kFusedSubLong ? 4 : 8>(qa, addr, logit, [&] {
        if (st + 1 < n_sub) tiles.issue<kPlain>(st + 1);
      });
      floatx16 &acc = logit[0];
      const int tok = c0 + st * kSub + n;
      const bool counted = ((tok >= o0) & (tok < o1)) | (last & (tok >= P) & (tok < Lb));
      const bool scored = (tok >= 0) & (tok < min(P, c1));  // a prefix token (owned or halo): its probability is formed in phase 3
      bool take[4];
      float one[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ok = counted & ((a.causal == 0) | (tok <= P + hi * 4 + i));
        take[i] = ok | scored;
        one[i] = ok ? 1.f : 0.f;
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[q] *= a.scale_log2e;
#pragma unroll
      for (int t = 0; t < kFusedSub; ++t)
        if (t == st) {
          asm volatile("");  // a branch, not 16 choices for every t
#pragma unroll
          for (int q = 0; q < 16; ++q) z[t][q] = acc[q];
        }
      // running reference = max over every logit that is counted or later scored, so that
      // 2^(z - reference) <= 1 for all of them; only counted keys enter the sum.  Masked window
      // keys and slots outside the sequence are neither: they must not move the reference.
      // A row's first tile: with at most two tiles their instructions are what the stream takes (2048 tokens 17.66 -> 17.46 us per
      // call, 6554 21.3 -> 21.1, 12289 24.9 -> 24.6); with more it is the memory, and the choice costs (16384 head-wise 31.9 -> 32.1).
      if (kFusedSub <= kFusedSubFew && st == 0 && ordinary_tile(acc, counted | scored)) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          mx[q] = take[q & 3] ? acc[q] : kNegBig;
          sm[q] = one[q & 3];
        }
      } else {
#pragma unroll
        for (int q = 0; q < 16; ++q) count_logit(take[q & 3] ? acc[q] : kNegBig, one[q & 3], mx[q], sm[q]);
      }
    }
    FKV_TICK(33);
  }
  // Looked at before the mailbox posts go out: a load is waited for together with them otherwise.
  const unsigned poisoned = __builtin_amdgcn_readfirstlane(flag);
  if (has_group) fold_and_post(f, range, mx, sm, mloc, g, lane, poisoned);
  // A failed exchange leaves mailboxes in an unknown state: until the host has reset them
  // (fkv_clear_error) every launch only marks its scores invalid.
  if (poisoned != 0u) {
    poison_scores(a, col0, o0, o1);
    return;
  }
  FKV_TICK(34);
  FKV_BTICK(1);
  FKV_WTICK(3);

  bool wave_ok = owner_duty(a, f, xch, wave, lane);
  FKV_TICK(35);

  // While the exchange is in flight: turn the kept logits into 2^(z - block reference).  The
  // global normaliser then costs one multiply per value instead of an exponential.
  if (has_group) {
#pragma unroll
    for (int st = 0; st < kFusedSub; ++st)
      if (st < n_sub) {
#pragma unroll
        for (int q = 0; q < 16; ++q) z[st][q] = fast_exp2(z[st][q] - mloc[q]);
      }
    if (a.W < kMaxWindow) {  // rows the window does not have: their logits may be NaN (0 times an infinite K)
#pragma unroll
      for (int st = 0; st < kFusedSub; ++st)
#pragma unroll
        for (int q = 0; q < 16; ++q)
          if (hi * 4 + (q & 3) >= a.W) z[st][q] = 0.f;
    }
  }
  FKV_TICK(36);

  // ---- phase 2b: collect the log-sum-exp of this wave's 32 rows from the block's result box
  if (has_group && wave_ok) {
    wave_ok = collect_lse<1>(f, range, g, lane, cst_lds[wave]);
  }
  FKV_BTICK(2);
  lds_barrier();  // every wave has left its staging tile (phase 3 reuses them); flag_lds is initialised
  if (!wave_ok && lane == 0) flag_lds[0] = 0u;
  FKV_TICK(37);

  // ---- phase 3: probabilities from the kept logits, window sums into LDS
  if (has_group && wave_ok) {
    float fac[16];  // 2^(block reference - global log-sum-exp) per row
#pragma unroll
    for (int q = 0; q < 16; ++q) fac[q] = fast_exp2(mloc[q] - cst_lds[wave][(q >> 2) * 8 + hi * 4 + (q & 3)]);
#pragma unroll
    for (int st = 0; st < kFusedSub; ++st) {
      if (st < n_sub) {
        const int tok = c0 + st * kSub + n;
        const bool inb = tok >= 0 && tok < min(P, c1);  // only prefix tokens are scored; slots past c1 were never loaded
        float sum[4];
#pragma unroll
        for (int hl = 0; hl < 4; ++hl) {
          sum[hl] = 0.f;
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            // Each probability is rounded before it is added: as one multiply-add the scores move by an ulp, and with
            // them which of two nearly equal tokens is kept.
#pragma clang fp contract(off)
            sum[hl] += z[st][hl * 4 + rr] * fac[hl * 4 + rr];
          }
          sum[hl] = add_across_halves(sum[hl]);  // other half of the window rows
        }
        store_sums<kFusedSlots>(a, s_head + wave * kMaxGroup, g, st * kSub + n, hi, inb, sum);
      }
    }
  }
  lds_barrier();
  FKV_TICK(40);
  const bool grid_ok = flag_lds[0] != 0u;
  if (grid_ok) {
    pool_and_write<kFusedSlots, kSplit>(a, s_head, g_sum, c0, o0, o1, col0, g0, min(a.V, g0 + kW));
  } else {
    poison_scores(a, col0, o0, o1);
    if (threadIdx.x == 0) __hip_atomic_store(f.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  FKV_TICK(41);
  FKV_BTICK(3);
}

hipError_t launch_score_fused(const ScoreArgs &a, const FusedArgs &f, hipStream_t s) {
  if (f.split >= 0)
    hipLaunchKernelGGL((k_score_fused<kFusedSubFew, kSplitWaves>), dim3(f.n_wg), dim3(kSplitWaves * 64), 0, s, a, f);
  else if (f.n_sub_max <= kFusedSubFew)
    hipLaunchKernelGGL((k_score_fused<kFusedSubFew, kWaves>), dim3(f.n_wg), dim3(kThreads), 0, s, a, f);
  else if (f.n_sub_max <= kFusedSubShort)
    hipLaunchKernelGGL((k_score_fused<kFusedSubShort, kWaves>), dim3(f.n_wg), dim3(kThreads), 0, s, a, f);
  else
    hipLaunchKernelGGL((k_score_fused<kFusedSubLong, kWaves>), dim3(f.n_wg), dim3(kThreads), 0, s, a, f);
  return hipGetLastError();
}

int score_fused_max_blocks_per_cu(void) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_score_fused<kFusedSubLong, kWaves>, kThreads, 0) != hipSuccess) return 0;
  return n;
}

}  // namespace fkv
