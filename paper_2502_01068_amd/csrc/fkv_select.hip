// Top-k of one score row with the window merged in (Sec. 4.2): exact radix select on the
// order-preserving integer image of the fp32 scores, then an ordered compaction, so the
// output is ascending, has exactly k entries and equal scores go to the lower index.
//
// Rows of up to 32768 keys take one 1024-thread block each with the keys in registers (k_select below); longer
// ones the kernels of fkv_select_coop.hip / fkv_select_long.hip, or, where those do not take the call, one
// block that goes through the row in 32768-key chunks re-read from L2 per pass (select_row).  That one:
//   1. the row's smallest and largest key bound the search interval [lo, lo + 2^s); histogram
//      passes of up to 11 bits of (key - lo), most significant first, narrow it down to the key
//      T of the (k-W)-th largest prefix score.  Taking digits relative to the row's own range
//      spreads the keys over the 2048 LDS bins (fp32 exponents would crowd them into a few
//      dozen) and makes a constant row cost no pass at all.  After the first pass the few keys
//      left in the interval are collected into LDS, one per thread, and the remaining passes
//      run on that list.  Keys equal to the interval's lower end are never histogrammed (a row
//      may hold thousands of them: probabilities that underflowed to zero); their count is the
//      difference between the interval's key count and the histogram's total;
//   2. a scan of the per-item keep counts gives every kept key its output offset in index order: all
//      keys > T and the first `need_eq` keys == T by index.
#include "fkv_select_search.h"

namespace fkv {

__device__ __forceinline__ void select_row(const float *sc, int P, int kp, int32_t *out, uint32_t *hist,
                                           uint32_t *wsum, uint32_t *bcast, uint32_t *scan_tbl) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int mis = (int)((reinterpret_cast<uintptr_t>(sc) >> 2) & 3);
  const float *base = sc - mis;
  constexpr int kKpt = kMaxKpt, kChunk = kSelThreads * kKpt;
  const int n_chunks = (P + mis + kChunk - 1) / kChunk;
  uint32_t key[kKpt];
  FKV_TICK(0);
  FKV_BTICK(0);

  // ---- key range of the row: the radix digits are taken relative to the smallest key, so
  // the bins spread over the values the row really holds instead of over fp32's exponent
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  for (int ch = 0; ch < n_chunks; ++ch) {
    load_keys<kKpt>(base, mis, P, ch * kChunk, wave, lane, key);
#pragma unroll
    for (int e = 0; e < kKpt; ++e) {
      kmax = max(kmax, key[e]);
      kmin = min(kmin, key[e] - 1u);  // key 0 (no element) wraps to the largest value
    }
  }
  kmax = wave_max_to_last(kmax);
  kmin = wave_min_to_last(kmin);
  if (lane == 63) { wsum[wave] = kmin; wsum[kSelWaves + wave] = kmax; }
  __syncthreads();
  for (int w = 0; w < kSelWaves; ++w) {
    kmin = min(kmin, wsum[w]);
    kmax = max(kmax, wsum[kSelWaves + w]);
  }
  kmin += 1u;

  FKV_TICK(1);
  FKV_BTICK(1);
  // ---- narrow [lo, lo + 2^s) down to the key T of the kp-th largest score
  uint32_t lo = kmin, remaining = (uint32_t)kp, need_eq = remaining;
  uint32_t n_in = (uint32_t)P;  // keys in the current interval [lo, lo + 2^s)
  int s = (kmax == kmin) ? 0 : 32 - __clz(kmax - kmin);  // kmax - kmin < 2^s
  bool whole_bin = false;

  // Picks the histogram bin that holds the `remaining`-th largest candidate and narrows the
  // interval to it.  Expects hist filled and a barrier passed; leaves a barrier behind.
  auto narrow = [&](int shift) {
    const BinPick p = pick_bin(hist, wsum, bcast, remaining, n_in);
    n_in = p.in_bin;
    lo += p.digit << shift;
    remaining = p.remaining;
    need_eq = remaining;
    s = shift;
    whole_bin = p.in_bin == p.remaining;  // the whole bin is kept: no need to refine further
    return p.in_bin;                      // candidates left
  };
  auto clear_hist = [&]() {
    __syncthreads();  // wsum / hist / bcast readers of the previous round are done
    for (int i = tid; i < kBins; i += kSelThreads) hist[i] = 0;
    if (tid == 0) bcast[4] = 0;  // candidate-list length
    __syncthreads();
  };

  uint32_t n_cand = 0xFFFFFFFFu;
  if (s > 0) {
    // first pass: every key of the row
    const int shift = s - min(11, s);
    clear_hist();
    for (int ch = 0; ch < n_chunks; ++ch) {
      load_keys<kKpt>(base, mis, P, ch * kChunk, wave, lane, key);
      const uint32_t span = s >= 32 ? 0xFFFFFFFFu : ((1u << s) - 1u);
#pragma unroll
      for (int e = 0; e < kKpt; ++e) {
        // branch-free: what is not counted goes to a spare word per bank.  Not counted: empty slots (key 0)
        // and the keys equal to lo, whose number pick_bin recovers from the histogram's total
        const uint32_t rel = key[e] - lo;
        atomicAdd(&hist[(key[e] > lo && rel <= span) ? rel >> shift : (uint32_t)kBins + (lane & 31)], 1u);
      }
    }
    __syncthreads();
    FKV_TICK(8);
    n_cand = narrow(shift);
    FKV_TICK(9);
  }
  if (s > 0 && !whole_bin && n_cand <= (uint32_t)kSelThreads) {
    // Few keys are left in the interval (typically ~1 %): collect them into LDS, one per thread, and
    // finish the search on that list instead of sweeping all register keys again.
    uint32_t *cand = scan_tbl;  // free until the compaction
    const uint32_t span = (1u << s) - 1u;  // s <= 21 here
    for (int ch = 0; ch < n_chunks; ++ch) {
      load_keys<kKpt>(base, mis, P, ch * kChunk, wave, lane, key);
      // Valid keys lie in [0x007FFFFF, 0xFF800000] and span < 2^21, so a key below lo (or an empty
      // slot) wraps above span: one unsigned compare per key.  A wave reserves list space for all its
      // candidates with one LDS atomic (a scan over the lanes' counts gives each lane its place).
      uint32_t mine = 0;
#pragma unroll
      for (int e = 0; e < kKpt; ++e) mine += (key[e] - lo <= span) ? 1u : 0u;
      const uint32_t inc = wave_scan_add(mine);
      const uint32_t wave_n = wave_last(inc);
      if (wave_n == 0) continue;
      uint32_t wave_base = 0;
      if (lane == 63) wave_base = atomicAdd(&bcast[4], wave_n);
      wave_base = wave_last(wave_base);
      if (mine != 0) {
        uint32_t at = wave_base + inc - mine;
#pragma unroll
        for (int e = 0; e < kKpt; ++e) {
          const uint32_t rel = key[e] - lo;
          if (rel <= span) cand[at++] = rel;
        }
      }
    }
    __syncthreads();
    FKV_TICK(10);
    const uint32_t my_rel = (uint32_t)tid < n_cand ? cand[tid] : 0xFFFFFFFFu;
    uint32_t base_rel = 0;  // lo advanced since the list was built
    while (s > 0 && !whole_bin) {
      const int shift = s - min(11, s);
      const uint32_t span2 = (1u << s) - 1u;
      clear_hist();
      const uint32_t rel = my_rel - base_rel;
      if (my_rel >= base_rel && rel <= span2) atomicAdd(&hist[rel >> shift], 1u);
      __syncthreads();
      const uint32_t lo_before = lo;
      narrow(shift);
      base_rel += lo - lo_before;
    }
  } else {
    while (s > 0 && !whole_bin) {
      const int shift = s - min(11, s);
      const uint32_t span = (s >= 32) ? 0xFFFFFFFFu : ((1u << s) - 1u);  // candidates: key - lo <= span
      clear_hist();
      for (int ch = 0; ch < n_chunks; ++ch) {
        load_keys<kKpt>(base, mis, P, ch * kChunk, wave, lane, key);
#pragma unroll
        for (int e = 0; e < kKpt; ++e) {  // keys equal to lo are left to pick_bin's total, as in the first pass
          const uint32_t rel = key[e] - lo;
          atomicAdd(&hist[(key[e] > lo && rel <= span) ? rel >> shift : (uint32_t)kBins + (lane & 31)], 1u);
        }
      }
      __syncthreads();
      narrow(shift);
    }
  }
  if (whole_bin) need_eq = 0xFFFFFFFFu;
  __syncthreads();  // the candidate list (scan table) is free again
  // keep key > T, and key == T while fewer than need_eq equal keys came before it.  When a whole
  // bin is kept, T is the smallest key the bin could hold and every key == T is kept.
  const uint32_t T = lo;
  FKV_TICK(2);
  FKV_BTICK(2);

  // ---- ordered compaction.  Index order inside a wave is (q, lane, e).
  uint32_t run_gt = 0, run_eq = 0;
  for (int ch = 0; ch < n_chunks; ++ch) {
    load_keys<kKpt>(base, mis, P, ch * kChunk, wave, lane, key);
    compact_chunk<kKpt>(key, T, need_eq, run_gt, run_eq, ch * kChunk - mis, out, scan_tbl, wsum, bcast + 8);
  }
  FKV_TICK(3);
  FKV_BTICK(3);
}

struct SelectRow {
  const float *sc;
  int32_t *out;
  int P, k, kp;
  unsigned failed;  // the context's error flag, in flight: waited for where it is looked at
};
__device__ __forceinline__ SelectRow locate_row(const SelectArgs &a) {
  // All arguments that the row can need, requested together (left to itself the compiler loads each where it is first used, four
  // trips one after the other), both sets' among them.
  const int b = blockIdx.y;
  const int at0 = a.cu[b], at1 = a.cu[b + 1], n_rows0 = a.set[0].n_rows;
  const float *scores[2] = {a.set[0].scores, a.set[1].scores};
  int32_t *idx[2] = {a.set[0].idx_out, a.set[1].idx_out};
  const int64_t stride[2] = {a.set[0].row_stride, a.set[1].row_stride};
  const int total[2] = {a.set[0].total, a.set[1].total};
  const int c0[2] = {a.set[0].cnt_off[b], a.set[1].cnt_off[b]}, c1[2] = {a.set[0].cnt_off[b + 1], a.set[1].cnt_off[b + 1]};
  asm volatile("" ::"s"(at0), "s"(at1), "s"(n_rows0), "s"(a.n_sets), "s"(a.W), "s"(a.err), "s"(scores[0]), "s"(scores[1]), "s"(idx[0]),
               "s"(idx[1]), "s"(stride[0]), "s"(stride[1]), "s"(total[0]), "s"(total[1]), "s"(c0[0]), "s"(c0[1]), "s"(c1[0]), "s"(c1[1]));
  int zero = 0;
  asm("" : "+v"(zero));  // else the flag, a uniform value, is waited for on the spot
  SelectRow r;
  r.failed = a.err != nullptr ? a.err[zero] : 0u;
  const bool second = a.n_sets > 1 && (int)blockIdx.x >= n_rows0;
  const int row = (int)blockIdx.x - (second ? n_rows0 : 0);
  r.P = at1 - at0 - a.W;
  r.k = second ? c1[1] - c0[1] : c1[0] - c0[0];
  r.kp = r.k - a.W;  // prefix tokens to keep
  r.sc = (second ? scores[1] : scores[0]) + (size_t)row * (second ? stride[1] : stride[0]) + (at0 - b * a.W);
  r.out = (second ? idx[1] : idx[0]) + (size_t)row * (second ? total[1] : total[0]) + (second ? c0[1] : c0[0]);
  return r;
}
// The window's indices, which are always kept; while the flag is up, -1 in every index (the scores are invalid, none may look
// usable) and false.  Block-uniform.
__device__ __forceinline__ bool window_or_failed(const SelectArgs &a, const SelectRow &r) {
  if (uniform(r.failed) != 0u) {
    for (int i = threadIdx.x; i < r.k; i += kSelThreads) r.out[i] = -1;
    return false;
  }
  if ((int)threadIdx.x < a.W) r.out[r.kp + threadIdx.x] = r.P + threadIdx.x;
  return true;
}

// ---- rows of up to 32768 keys: everything in registers -----------------------------------------
// One 1024-thread block per row, kKpt keys per thread.  Bound by instruction issue and by the latency of the
// steps between block barriers (one block per row leaves most of the chip idle whatever is done), so per key
// there are: the order-preserving image (4), min / max (2), histogram address and LDS atomic (5), two tests
// against the threshold's bin (5) and the compaction (7: masks stay scalar, lane prefixes from v_mbcnt), and seven
// barriers in the usual case.
//   1. the row's smallest and largest key; 2048 bins over that range, one LDS atomic per key.  Keys equal to
//      the interval's smallest are not counted (a row may hold thousands of probabilities that underflowed to
//      zero): they are what the total lacks.
//   2. the threshold's bin; while it holds more than kListCap keys (ties, very long tails) it is binned again
//   3. its keys are listed in LDS, a thread each ranks them by a sweep over the list
//   4. ordered compaction, staged per wave in LDS.
// Per launch (kernel trace; another run gives up to 0.3 us more or less), before -> after the wave that a row ends in requests all
// its words at once, the arguments come in one batch and the flag travels beside the keys: 2040 keys 5.2 -> 4.7 us, 6546 7.3 ->
// 6.7, 12281 (max pooling) 10.6 -> 8.7, 20000 12.1 -> 10.2, 32 rows of 16376 9.3 -> 8.1, 72 rows of 8184-16376 10.5 -> 8.9.
// 24 and 32 keys per thread keep 7 and 31 scalars in vector lanes: 32 rows of 22000 keys 10.5 -> 9.6 us per call, of 30000 12.6 -> 11.4.
template <int kKpt>
struct SelectLds {
  SearchLds search;  // first: 16-byte aligned
  int32_t stage[kSelWaves][64 * kKpt + 64];  // kept indices of each wave, then a word per lane for dropped ones
};

template <int kKpt>
__device__ __forceinline__ void select_resident(const SelectArgs &a, const SelectRow &r, SelectLds<kKpt> &s) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mis = (int)((reinterpret_cast<uintptr_t>(r.sc) >> 2) & 3);
  uint32_t key[kKpt];
  load_keys<kKpt>(r.sc - mis, mis, r.P, 0, wave, lane, key);
  clear_search(s.search, tid);
  if (!window_or_failed(a, r)) return;
  __syncthreads();
  const RowCut cut = find_cut<kKpt>(key, r.P, r.kp, mis, wave, lane, s.search);
  compact_wave<kKpt>(key, cut.T, cut.need_eq, cut.before_gt, cut.before_eq, wave, -mis, r.out, s.stage[wave]);
}

// Rows of at most 1024 kKpt - 3 keys; longer ones of the call are left to another launch.  kKpt follows the longest row:
// rows much shorter than that take fewer keys per thread, since empty slots cost what full ones do and a batch of many
// short rows is several rounds of blocks (24000 and 62 times 1500 keys, 9 rows each: 27.0 -> 16.1 us per call).
template <int kKpt>
__global__ __launch_bounds__(kSelThreads) void k_select(SelectArgs a) {
  __shared__ __attribute__((aligned(16))) SelectLds<kKpt> lds;
  const SelectRow r = locate_row(a);
  if (r.P + 3 > kSelThreads * kKpt) return;
  if (r.kp <= 0) {
    window_or_failed(a, r);
    return;
  }
  if constexpr (kKpt > kShortKpt) {
    static_assert(sizeof(SelectLds<kShortKpt>) <= sizeof lds, "the short row's tables lie where the long one's would");
    if (r.P + 3 <= kSelThreads * kShortKpt) {
      select_resident<kShortKpt>(a, r, reinterpret_cast<SelectLds<kShortKpt> &>(lds));
      return;
    }
  }
  select_resident<kKpt>(a, r, lds);
}

// Longer rows on one block each, re-read from the caches pass by pass: only for calls with more such rows than the
// launch chain has state for.
__global__ __launch_bounds__(kSelThreads) void k_select_chunks(SelectArgs a) {
  __shared__ uint32_t hist[kBins + 32];  // + spare words for key slots that are not counted (never read; one
                                         // per bank, so they do not pile onto one address)
  __shared__ __attribute__((aligned(16))) uint32_t scan_tbl[kSelWaves * 64 * kMaxKpt];  // 128 KiB: scan tables / output staging
  __shared__ uint32_t wsum[2 * kSelWaves];
  __shared__ uint32_t bcast[8 + 64];  // broadcast slots, then one sink word per lane
  const SelectRow r = locate_row(a);
  if (r.P + 3 <= kSelThreads * kMaxKpt) return;
  if (!window_or_failed(a, r)) return;
  if (r.kp > 0) select_row(r.sc, r.P, r.kp, r.out, hist, wsum, bcast, scan_tbl);
}

hipError_t launch_select(SelectArgs a, uint32_t *long_state, const SelectCoop *coop, hipStream_t s) {
  int rows = 0;
  for (int i = 0; i < a.n_sets; ++i) rows += a.set[i].n_rows;
  {
    hipError_t e = hipSuccess;
    a.long_state = nullptr;
    if (coop != nullptr && try_launch_select_coop(a, rows, *coop, s, &e)) return e;
  }
  // Rows over one block's registers go to the multi-block chain when the call's row instances fit its state.
  int max_slices = 0, max_short = 0;
  for (int b = 0; b < a.n_seq; ++b) {
    const int P = a.cu[b + 1] - a.cu[b] - a.W;
    if (P + 3 > select_long_threshold())
      max_slices = max(max_slices, (P + 3 + select_long_chunk() - 1) / select_long_chunk());
    else
      max_short = max(max_short, P + 3);
  }
  const bool use_long = max_slices > 0 && long_state != nullptr && max_slices <= kLongMaxSlices &&
                        (int64_t)rows * a.n_seq <= kLongMaxInst;
  a.long_state = use_long ? long_state : nullptr;
  const dim3 grid(rows, a.n_seq), block(kSelThreads);
  hipError_t e = hipSuccess;
  if (max_short > 0) {  // keys per thread by the longest of these rows
    if (max_short <= kSelThreads * 4)
      hipLaunchKernelGGL(k_select<4>, grid, block, 0, s, a);
    else if (max_short <= kSelThreads * 8)
      hipLaunchKernelGGL(k_select<8>, grid, block, 0, s, a);
    else if (max_short <= kSelThreads * 16)
      hipLaunchKernelGGL(k_select<16>, grid, block, 0, s, a);
    else if (max_short <= kSelThreads * 24)
      hipLaunchKernelGGL(k_select<24>, grid, block, 0, s, a);
    else
      hipLaunchKernelGGL(k_select<32>, grid, block, 0, s, a);
    e = hipGetLastError();
  }
  if (e == hipSuccess && use_long) e = launch_select_long(a, rows, max_slices, s);
  if (e == hipSuccess && max_slices > 0 && !use_long) {
    hipLaunchKernelGGL(k_select_chunks, grid, block, 0, s, a);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace fkv
