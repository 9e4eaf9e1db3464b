// The grid exchange of the resident score kernels: every block posts the (max, sum) of each softmax row over its
// tokens, owner blocks fold the rows and post their log-sum-exps back to every block of the sequence.
#pragma once

#include "fkv_dpp.h"
#include "fkv_mailbox.h"
#include "fkv_score_common.h"

namespace fkv {

constexpr int kOwnRows = 8;  // softmax rows per owner block

// kW waves per block, at most kRanges token ranges in a launch (a range has one block, or one for each half of its groups).
template <int kW, int kRanges>
struct ExchangeLds {
  static_assert(kOwnRows % kW == 0, "rows per wave");
  float2 part[kOwnRows][kRanges];  // owner blocks: partials of their rows, by range
  float lse[kOwnRows];
  unsigned late[kW];
};

// Writes NaN into every score this block owns: a call whose exchange failed must not leave
// plausible numbers behind.
__device__ __forceinline__ void poison_scores(const ScoreArgs &a, int col0, int o0, int o1) {
  const float nan = __uint_as_float(0x7FC00000u);
  const int own = o1 - o0;
  for (int i = threadIdx.x; i < own; i += blockDim.x) {
    const size_t col = (size_t)col0 + o0 + i;
    if (a.scores_group)
      for (int g = 0; g < a.Hkv; ++g) a.scores_group[(size_t)g * a.sum_p + col] = nan;
    if (a.scores_head)
      for (int h = 0; h < a.Hq; ++h) a.scores_head[(size_t)h * a.sum_p + col] = nan;
    if (a.scores_tsp) a.scores_tsp[col] = nan;
  }
}

// The error flag, on its way while K is streamed: waited for where it is first looked at.  The address is made to look
// different per lane, since the compiler waits on the spot for a load of a uniform value (0.7 us before the first K load).
__device__ __forceinline__ unsigned request_flag(const unsigned *err) {
  unsigned zero = 0;
  asm("" : "+v"(zero));
  return __hip_atomic_load(err + zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The arguments a block needs before its first load of K, requested together: left to itself the compiler loads each where
// it is first used, four trips one after the other.
__device__ __forceinline__ void request_args(const ScoreArgs &a, const FusedArgs &f) {
  asm volatile("" ::"s"(a.k), "s"(a.q_win), "s"(a.Hq), "s"(a.Hkv), "s"(a.G), "s"(a.W), "s"(a.V), "s"(a.vsh), "s"(a.pool_r), "s"(f.err),
               "s"(a.map.n_seq), "s"(a.scale_log2e), "s"(a.causal), "s"(f.part));
}

// Folds a wave's per-lane (max, sum) pairs of a virtual group's 32 rows over the token lanes and posts them.  mloc[q]:
// the block's maximum of row (q / 4) * 8 + hi * 4 + q % 4, in every lane.
__device__ __forceinline__ void fold_and_post(const FusedArgs &f, int range, const float (&mx)[16], const float (&sm)[16], float (&mloc)[16],
                                              int g, int lane, unsigned poisoned) {
  half_max16(mx, mloc);
  // lane q of each 16 ends up with row q's sum (and picks row q's maximum)
  float shrink[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) shrink[q] = fast_exp2(mx[q] - mloc[q]);
  const float ps = half_sums_of_products(sm, shrink, lane), pm = pick16(mloc, lane);
  // lanes 0-15 post the 16 rows of the low half, lanes 32-47 those of the high half
  if ((lane & 31) < 16 && poisoned == 0u) {
    const int q = lane & 15;
    const int row = g * kRowsPerGroup + (q >> 2) * 8 + (lane >> 5) * 4 + (q & 3);
    box_post(f.part + (size_t)range * kLseRowsPerBlock + row, make_float2(pm, ps));
  }
}

// Owner duty of a block.  A group of kOwnRows softmax rows of a sequence belongs to one block, group t to block
// t mod n_wg.  That block's waves collect the rows' partials from every range of the sequence, fold a row at a time
// each and post the log-sum-exps into those ranges' result boxes.  Contains block barriers in blocks that own a group.
// False if a wait ran out (block-uniform).
template <int kW, int kRanges>
__device__ __forceinline__ bool owner_duty(const ScoreArgs &a, const FusedArgs &f, ExchangeLds<kW, kRanges> &x, int wave, int lane) {
  bool wave_ok = true;
  const int groups_per_seq = a.V * (kRowsPerGroup / kOwnRows);
  const int n_groups = a.map.n_seq * groups_per_seq;
  for (int t = (int)blockIdx.x; t < n_groups; t += f.n_wg) {  // block-uniform
    const int tb = t / groups_per_seq, row0 = (t - tb * groups_per_seq) * kOwnRows;
    const int blk0 = a.map.blk[tb], nb = a.map.blk[tb + 1] - blk0;
    constexpr int kPerPass = kW * (64 / kOwnRows);  // ranges the block's lanes cover at a time
    constexpr int kPasses = kRanges / kPerPass;
    const int i0 = wave * (64 / kOwnRows) + lane / kOwnRows, rl = lane % kOwnRows;
    float2 *src = f.part + (size_t)blk0 * kLseRowsPerBlock + row0 + rl;
    unsigned long long v[kPasses];
#pragma unroll
    for (int i = 0; i < kPasses; ++i) v[i] = kEmpty64;
    BoundedWait<> wait(f.timeout_ticks);
    while (true) {
      bool missing = false;
#pragma unroll
      for (int i = 0; i < kPasses; ++i)
        if (i * kPerPass + i0 < nb && v[i] == kEmpty64) v[i] = box_peek(src + (size_t)(i * kPerPass + i0) * kLseRowsPerBlock);
#pragma unroll
      for (int i = 0; i < kPasses; ++i)
        if (i * kPerPass + i0 < nb && v[i] == kEmpty64) missing = true;
      if (!__any(missing)) break;
      if (wait.expired()) { wave_ok = false; break; }
    }
    if (wave_ok) {
#pragma unroll
      for (int i = 0; i < kPasses; ++i)
        if (i * kPerPass + i0 < nb) {
          box_clear(src + (size_t)(i * kPerPass + i0) * kLseRowsPerBlock);
          __builtin_memcpy(&x.part[rl][i * kPerPass + i0], &v[i], sizeof v[i]);
        }
    }
    if (lane == 0) x.late[wave] = wave_ok ? 0u : 1u;
    lds_barrier();
    bool late = false;
#pragma unroll
    for (int w = 0; w < kW; ++w) late = late || x.late[w] != 0u;
    if (late) { wave_ok = false; break; }  // the whole block
#pragma unroll
    for (int j = 0; j < kOwnRows / kW; ++j) {
      const int own = j * kW + wave;
      // Never (kW divides kOwnRows).  Without it the partial-keep kernel for wide groups spills a register (test_kernel_build_host.py
      // sees that); as a loop up to kOwnRows, which spills none either, 2048 tokens take 17.45 us per call for 17.37.
      if (own >= kOwnRows) break;
      float m = kNegBig, s = 0.f;
#pragma unroll
      for (int i = 0; i < kRanges / 64; ++i)
        if (i * 64 + lane < nb) {
          const float2 pv = x.part[own][i * 64 + lane];
          const float mn = fmaxf(m, pv.x);
          s = s * fast_exp2(m - mn) + pv.y * fast_exp2(pv.x - mn);
          m = mn;
        }
      const float mw = wave_fmax(m);
      const float sw = wave_fsum(s * fast_exp2(m - mw));
      const int row = row0 + own, in_group = row & (kRowsPerGroup - 1);
      const bool row_ok = (in_group >> 3) < vg_heads(a, row / kRowsPerGroup) && (in_group & 7) < a.W;
      if (lane == 0) x.lse[own] = row_ok ? mw + __log2f(sw) : 0.f;
    }
    lds_barrier();
    const float lse = x.lse[rl];
#pragma unroll
    for (int i = 0; i < kPasses; ++i)
      if (i * kPerPass + i0 < nb) box_post(f.lse + (size_t)(blk0 + i * kPerPass + i0) * kLseRowsPerBlock + row0 + rl, lse);
  }
  return wave_ok;
}

// The log-sum-exps of the 32 rows of virtual groups g .. g + kVg - 1 from the range's result boxes, a lane each, into dst
// (LDS, 32 kVg floats).  Wave-uniform result: false if the wait ran out.
template <int kVg>
__device__ __forceinline__ bool collect_lse(const FusedArgs &f, int range, int g, int lane, float *dst) {
  const bool mine = lane < kVg * kRowsPerGroup;
  float *box = f.lse + (size_t)range * kLseRowsPerBlock + g * kRowsPerGroup + (lane & (kVg * kRowsPerGroup - 1));
  unsigned bits = kEmpty32;
  BoundedWait<> wait(f.timeout_ticks);
  while (true) {
    if (mine && bits == kEmpty32) bits = box_peek(box);
    if (!__any(mine && bits == kEmpty32)) break;
    if (wait.expired()) return false;
  }
  if (mine) {
    box_clear(box);
    dst[lane] = __uint_as_float(bits);
  }
  return true;
}

}  // namespace fkv
