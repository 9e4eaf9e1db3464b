// The search of a row whose keys one block holds in registers (fkv_select.hip says how it goes and what bounds it), shared by
// the kernels that write its indices and that gather its rows as well.
#pragma once

#include "fkv_select_common.h"

namespace fkv {

constexpr int kListCap = 256;
constexpr int kShortKpt = 8;  // keys per thread of rows that are much shorter than their launch's longest, see k_select

struct SearchLds {
  uint32_t hist[kBins + 64];               // first: 16-byte aligned; + one spare word per lane for slots that are not counted
  uint32_t list[kListCap];                 // keys of the threshold's interval, relative to its smallest,
  uint32_t list_wave[kListCap];            // and the waves that hold them
  uint32_t tot[kSelWaves], cnt[kSelWaves]; // wave totals: histogram scan, keys kept for sure
  uint32_t low[kSelWaves];                 // smallest keys of an interval (the largest ones go to tot)
  uint32_t kmax, not_kmin, n_list, pick[3];
};

// Ahead of a block barrier and the search.
__device__ __forceinline__ void clear_search(SearchLds &s, int tid) {
  for (int i = tid; i < kBins / 4; i += kSelThreads) *reinterpret_cast<u32x4 *>(&s.hist[4 * i]) = u32x4{0u, 0u, 0u, 0u};
  if (tid < kListCap / 4) *reinterpret_cast<u32x4 *>(&s.list[4 * tid]) = u32x4{0u, 0u, 0u, 0u};
  if (tid < 3) (&s.kmax)[tid] = 0u;  // kmax, not_kmin, n_list
}

// What a row keeps: keys > T and the first need_eq keys == T.  before_gt, before_eq: keys > T and == T in the waves before this one.
struct RowCut { uint32_t T, need_eq, before_gt, before_eq; };

// The cut that keeps the kp largest of a row's P keys (0 < kp <= P), `key` as load_keys left it.  Contains block barriers.
template <int kKpt>
__device__ __forceinline__ RowCut find_cut(const uint32_t (&key)[kKpt], int P, int kp, int mis, int wave, int lane, SearchLds &s) {
  const int tid = wave * 64 + lane;
  {
    uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
    const int v_wave = wave * (64 * kKpt);
    if (v_wave >= mis && v_wave + 64 * kKpt <= mis + P) {
#pragma unroll
      for (int e = 0; e < kKpt; ++e) {
        kmax = max(kmax, key[e]);
        kmin = min(kmin, key[e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < kKpt; ++e) {
        kmax = max(kmax, key[e]);
        kmin = min(kmin, key[e] != 0u ? key[e] : 0xFFFFFFFFu);  // 0: no element
      }
    }
    kmax = wave_max_to_last(kmax);
    kmin = wave_min_to_last(kmin);
    if (lane == 63) {
      atomicMax(&s.kmax, kmax);
      atomicMax(&s.not_kmin, ~kmin);
    }
  }
  __syncthreads();
  // the interval [base, base + span] holds n_in keys, among them the `remaining`-th largest one of it: the threshold
  uint32_t base = uniform(~s.not_kmin), span = uniform(s.kmax) - base;
  uint32_t n_in = (uint32_t)P, remaining = (uint32_t)kp;
  RowCut cut{0u, 0u, 0u, 0u};

  // What the other waves hold of a key class: one word per wave through LDS.
  auto exchange = [&](uint32_t mine) {
    if (lane == 0) s.cnt[wave] = mine;
    __syncthreads();
    return wave_prefix(s.cnt, lane, wave).before;
  };
  auto settle = [&](uint32_t t, uint32_t eq) {  // the threshold is known without the list
    cut.T = t;
    cut.need_eq = eq;
    uint32_t mine = count_keys<kKpt>(key, [&](uint32_t k) { return k > t; });
    if (eq != 0u) mine |= count_keys<kKpt>(key, [&](uint32_t k) { return k == t; }) << 16;
    const uint32_t b = exchange(mine);
    cut.before_gt = b & 0xFFFFu;
    cut.before_eq = b >> 16;
  };

  while (true) {
    if (n_in == remaining) { settle(base - 1u, 0u); break; }  // the whole interval
    if (span == 0u) { settle(base, remaining); break; }
    if (n_in <= (uint32_t)kListCap) {
      uint64_t in[kKpt];
      uint32_t mine = 0, above = 0;
#pragma unroll
      for (int e = 0; e < kKpt; ++e) {
        in[e] = __builtin_amdgcn_ballot_w64(key[e] - base <= span);
        mine += __popcll(in[e]);
        above += key[e] > base + span ? 1u : 0u;
      }
      if (mine != 0u) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s.n_list, mine);
        at = uniform(at);
#pragma unroll
        for (int q = 0; q < kKpt / 4; ++q)
          if ((in[4 * q] | in[4 * q + 1] | in[4 * q + 2] | in[4 * q + 3]) != 0ull) {
#pragma unroll
            for (int e = 4 * q; e < 4 * q + 4; ++e) {
              if (key[e] - base <= span) {
                const uint32_t to = lanes_before(in[e], at);
                s.list[to] = key[e] - base + 1u;
                s.list_wave[to] = wave;
              }
              at += __popcll(in[e]);
            }
          }
      }
      cut.before_gt = exchange(wave_last(wave_sum_to_last(above)));
      // one list key per thread: its rank from a sweep over the list, four keys per read (unused entries are 0)
      if ((uint32_t)tid < n_in) {
        const uint32_t x = s.list[tid];
        uint32_t gt = 0, ge = 0;
        for (uint32_t j = 0; j < n_in; j += 4) {
          const u32x4 y = *reinterpret_cast<const u32x4 *>(&s.list[j]);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            gt += y[i] > x ? 1u : 0u;
            ge += y[i] >= x ? 1u : 0u;
          }
        }
        if (gt < remaining && remaining <= ge) {  // x is the threshold (equal keys write the same words)
          s.pick[0] = ge == remaining ? x - 1u : x;
          s.pick[1] = ge == remaining ? 0u : remaining - gt;
        }
      }
      __syncthreads();
      const uint32_t t = uniform(s.pick[0]);
      cut.need_eq = uniform(s.pick[1]);
      cut.T = base + t - 1u;
      for (uint32_t j = 0; j < n_in; j += 64) {  // kept and tied list keys of the waves before this one
        const bool live = j + lane < n_in && s.list_wave[j + lane] < (uint32_t)wave;
        const uint32_t x = live ? s.list[j + lane] : 0u;
        cut.before_gt += __popcll(__builtin_amdgcn_ballot_w64(live && x > t));
        if (cut.need_eq != 0u) cut.before_eq += __popcll(__builtin_amdgcn_ballot_w64(live && x == t));
      }
      break;
    }
    const int shift = max(21 - __clz((span - 1u) | 1u), 0);  // 2048 bins for keys base + 1 .. base + span
    const uint32_t spare = (uint32_t)kBins + lane;
#pragma unroll
    for (int e = 0; e < kKpt; ++e) {
      // empty slots and what lies below the interval or on its smallest key wrap above span
      const uint32_t rel = key[e] - (base + 1u);
      atomicAdd(&s.hist[rel < span ? rel >> shift : spare], 1u);
    }
    __syncthreads();
    // thread t owns bins 2 (1023 - t), + 1: thread order runs from the top bin down
    const int pair = kSelThreads - 1 - tid;
    const uint2 h = *reinterpret_cast<const uint2 *>(&s.hist[2 * pair]);
    *reinterpret_cast<uint2 *>(&s.hist[2 * pair]) = make_uint2(0u, 0u);
    const uint32_t mine = h.x + h.y;
    const uint32_t run = wave_scan_add(mine);
    if (lane == 63) s.tot[wave] = run;
    __syncthreads();
    const WavePrefix wp = wave_prefix(s.tot, lane, wave);
    if (remaining > wp.total) {  // the threshold is the interval's smallest key
      settle(base, remaining - wp.total);
      break;
    }
    const uint32_t above = wp.before + run - mine;
    if (above < remaining && remaining <= above + mine) {
      const bool top = remaining <= above + h.y;
      s.pick[0] = 2 * pair + (top ? 1 : 0);
      s.pick[1] = remaining - above - (top ? 0u : h.y);
      s.pick[2] = top ? h.y : h.x;
    }
    __syncthreads();
    const uint32_t at = uniform(s.pick[0]) << shift;
    base += 1u + at;
    span = min((1u << shift) - 1u, span - 1u - at);
    remaining = uniform(s.pick[1]);
    n_in = uniform(s.pick[2]);
    if (n_in > (uint32_t)kListCap && n_in != remaining) {
      // Too many for the list: ties, as a rule.  The interval shrinks to the keys it holds, so equal ones are seen as
      // such and do not queue up at one bin in another pass (9 rows of 20000 keys, two values: 36 -> 19 us).
      uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
#pragma unroll
      for (int e = 0; e < kKpt; ++e) {
        const bool in = key[e] - base <= span;
        kmax = max(kmax, in ? key[e] : 0u);
        kmin = min(kmin, in ? key[e] : 0xFFFFFFFFu);
      }
      kmax = wave_max_to_last(kmax);
      kmin = wave_min_to_last(kmin);
      if (lane == 63) {
        s.tot[wave] = kmax;
        s.low[wave] = kmin;
      }
      __syncthreads();
      kmax = wave_max_to_last(s.tot[lane & (kSelWaves - 1)]);
      kmin = wave_min_to_last(s.low[lane & (kSelWaves - 1)]);
      base = wave_last(kmin);
      span = wave_last(kmax) - base;
    }
  }
  return cut;
}

}  // namespace fkv
