// Select and gather in one launch (Sec. 4.2, App. B.1): every block finds a score row's cut for itself (the search of
// fkv_select.hip), has the row's kept indices in LDS then, writes its part of them and copies the part's K / V rows (a KV
// head's score row) or hidden rows (the TSP row).  Nothing is exchanged between blocks.
//
// Short calls are bound by the chain of launches (an empty one behind another costs 2.4 us), and a gather begins with its
// arguments and an index from memory.  The blocks of a row repeat its search, on CUs that the one-block select leaves idle; keys
// come from the caches.  Of 6.9 us at 2048 tokens with hidden rows, the launch, its arguments and the keys take 2.5, the search 2.1,
// the copy 2.3 (3.4 of 16.8 MB at 6554 tokens).  us per call, two launches -> one: 2048 tokens 19.4 -> 18.1, 6554 24.6 -> 23.0, 12289 paged
// 26.4 -> 24.5 (with 12 keys per thread; 16 take 0.5 more), 20001 of 64 / 8 heads 38.8 -> 36.7.  512 blocks of a share half as large: 1.4
// to 8 us more.  Chunks of hidden rows in flight per thread 2, 4, 8: 24000 tokens 46.6, 47.0, 45.8 us.  Up to which size: kSelGatherMaxShare.
#include "fkv_select_search.h"

namespace fkv {

struct GatherPart {  // what a block works on
  const float *sc;
  int32_t *out;       // the row's indices
  int b, row;         // sequence; KV head, or -1: the TSP row
  int P, k, i0, i1;   // prefix tokens, kept tokens, the block's part of them
  unsigned failed;
  bool summed;        // sc is the first of the groups' rows of sums
};

// load_keys for a row that is the sum of a.n_sums rows of the workspace, times inv_h: what the score kernels make the mean over
// all heads of where a block has every group, bit for bit.  Their stride is a multiple of four: whole groups of four are read.
template <int kKpt>
__device__ __forceinline__ void load_summed_keys(const SelectGatherArgs &a, const float *base, int mis, int P, int wave, int lane,
                                                 uint32_t (&key)[kKpt]) {
#pragma clang fp contract(off)
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < kKpt / 4; ++q) {
    const int at = slot_pos<kKpt>(wave, lane, q);
    f32x4 x[kMaxSums], tot = zero;
#pragma unroll
    for (int g = 0; g < kMaxSums; ++g)
      x[g] = g < a.n_sums && at < mis + P ? *reinterpret_cast<const f32x4 *>(base + g * a.sums_stride + at) : zero;
#pragma unroll
    for (int g = 0; g < kMaxSums; ++g) tot = g < a.n_sums ? tot + x[g] : tot;
#pragma unroll
    for (int e = 0; e < 4; ++e) key[4 * q + e] = at + e >= mis && at + e < mis + P ? order_key(tot[e] * a.inv_h) : 0u;
  }
}

__device__ __forceinline__ GatherPart locate_part(const SelectGatherArgs &a) {
  const SelectArgs &s = a.sel;
  // The sequence: up to nine in one batch of scalar loads, more with a lane each.  Eight a step until it is found, as before, is a chain
  // of up to eight trips through the scalar cache: 64 sequences of 200 tokens 46.3 us per paged call, 43.5 in two launches, 41.0 now.
  int b = 0;
  if (s.n_seq > 9) {
    static_assert(FKV_MAX_SEQS <= 64, "a lane per sequence");
    const int lane = threadIdx.x & 63;
    const int first = lane < s.n_seq ? a.blk[lane] : INT32_MAX;
    b = __popcll(__builtin_amdgcn_ballot_w64(first <= (int)blockIdx.x)) - 1;
  } else if (s.n_seq > 1) {
#pragma unroll
    for (int j = 1; j < 9; ++j) b += (j < s.n_seq) & ((int)blockIdx.x >= a.blk[j]);
  }
  // all arguments that the part can need, requested together
  const int at0 = s.cu[b], at1 = s.cu[b + 1], blk0 = a.blk[b], n_rows0 = s.set[0].n_rows;
  const int n_part[2] = {a.parts[0][b], a.parts[1][b]};
  const float *scores[2] = {s.set[0].scores, s.set[1].scores};
  int32_t *idx[2] = {s.set[0].idx_out, s.set[1].idx_out};
  const int64_t stride0 = s.set[0].row_stride;
  const float *sums = a.sums;
  const int total0 = s.set[0].total;
  const int c0[2] = {s.set[0].cnt_off[b], s.set[1].cnt_off[b]}, c1[2] = {s.set[0].cnt_off[b + 1], s.set[1].cnt_off[b + 1]};
  asm volatile("" ::"s"(at0), "s"(at1), "s"(blk0), "s"(n_rows0), "s"(s.W), "s"(s.err), "s"(scores[0]), "s"(scores[1]), "s"(idx[0]), "s"(idx[1]),
               "s"(stride0), "s"(sums), "s"(total0), "s"(c0[0]), "s"(c0[1]), "s"(c1[0]), "s"(c1[1]), "s"(n_part[0]), "s"(n_part[1]));
  int zero = 0;
  asm("" : "+v"(zero));  // else the flag, a uniform value, is waited for on the spot
  GatherPart p;
  p.failed = s.err != nullptr ? s.err[zero] : 0u;
  p.b = b;
  const int local = (int)blockIdx.x - blk0;
  const int row = (int)((uint32_t)local / (uint32_t)n_part[0]);
  const bool tsp = row >= n_rows0;
  p.row = tsp ? -1 : row;
  const int part = tsp ? local - n_rows0 * n_part[0] : local - row * n_part[0], parts = tsp ? n_part[1] : n_part[0];
  p.P = at1 - at0 - s.W;
  p.k = tsp ? c1[1] - c0[1] : c1[0] - c0[0];
  p.i0 = (int)((uint32_t)p.k * (uint32_t)part / (uint32_t)parts);  // parts <= the CUs (plan_select_gather), k <= 24581: below 2^31
  p.i1 = (int)((uint32_t)p.k * (uint32_t)(part + 1) / (uint32_t)parts);
  const int col = at0 - b * s.W;
  p.summed = tsp && sums != nullptr;
  p.sc = tsp ? (sums != nullptr ? sums : scores[1]) + col : scores[0] + (size_t)row * stride0 + col;
  p.out = tsp ? idx[1] + c0[1] : idx[0] + (size_t)row * total0 + c0[0];
  return p;
}

template <int kKpt>
struct SelectGatherLds {
  SearchLds search;  // first: 16-byte aligned
  int32_t kept[kSelThreads * kKpt + 64];  // the row's kept indices; a word per lane for dropped ones behind all of them
};

template <int kKpt>
__device__ __forceinline__ bool keep_row(const SelectGatherArgs &a, const GatherPart &p, SelectGatherLds<kKpt> &s) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mis = (int)((reinterpret_cast<uintptr_t>(p.sc) >> 2) & 3), kp = p.k - a.sel.W;
  uint32_t key[kKpt];
  if constexpr (kKpt <= kSplitMaxTokens / kSelThreads + 4) {
    if (p.summed) load_summed_keys<kKpt>(a, p.sc - mis, mis, p.P, wave, lane, key);
    else load_keys<kKpt>(p.sc - mis, mis, p.P, 0, wave, lane, key);
  } else {
    load_keys<kKpt>(p.sc - mis, mis, p.P, 0, wave, lane, key);
  }
  clear_search(s.search, tid);
  if (uniform(p.failed) != 0u) return false;
  __syncthreads();
  if (kp > 0) {
    const RowCut cut = find_cut<kKpt>(key, p.P, kp, mis, wave, lane, s.search);
    const uint32_t first = cut.before_gt + min(cut.before_eq, cut.need_eq);
    // a wave whose kept tokens all lie outside the part has nothing to place
    if ((int)first < p.i1 && (int)first + 64 * kKpt > p.i0)
      place_wave<kKpt>(key, cut.T, cut.need_eq, cut.before_eq, wave, -mis, s.kept + first, (uint32_t)(kSelThreads * kKpt) - first);
  }
  return true;
}

constexpr int kRowsInFlight = 2, kChunksInFlight = 8;  // per thread: rows of K and of V; 16-byte chunks of hidden rows

template <int kKpt>
__global__ __launch_bounds__(kSelThreads) void k_select_gather(SelectGatherArgs a) {
  __shared__ __attribute__((aligned(16))) SelectGatherLds<kKpt> lds;
  const GatherPart p = locate_part(a);
  const int tid = threadIdx.x;
  bool ok;
  if constexpr (kKpt > kShortKpt) {
    static_assert(sizeof(SelectGatherLds<kShortKpt>) <= sizeof lds, "the short row's tables lie where the long one's would");
    if (p.P + 3 <= kSelThreads * kShortKpt) ok = keep_row<kShortKpt>(a, p, reinterpret_cast<SelectGatherLds<kShortKpt> &>(lds));
    else ok = keep_row<kKpt>(a, p, lds);
  } else {
    ok = keep_row<kKpt>(a, p, lds);
  }
  const int i0 = p.i0, i1 = p.i1, kp = p.k - a.sel.W;
  if (!ok) {  // the scores are invalid: no index may look usable, and no row is copied
    for (int i = i0 + tid; i < i1; i += kSelThreads) p.out[i] = -1;
    return;
  }
  __syncthreads();
  const int32_t *kept = lds.kept;
  // The window is always kept.  Inside the sequence whatever the table holds: of a row with NaN scores places can be left open.
  auto token = [&](int i) { return i < kp ? min(max(kept[i], 0), p.P - 1) : p.P + i - kp; };
  for (int i = i0 + tid; i < i1; i += kSelThreads) p.out[i] = token(i);
  const int tok0 = a.sel.cu[p.b];
  if (p.row >= 0) {
    // 16 lanes a row of K and the same of V, 64 rows a step
    constexpr uint32_t kRow = kHeadDim * 2;
    const uint32_t col = (tid & 15) * 16, tok_row = (uint32_t)a.Hkv * kRow;
    const uint8_t *k = a.k + (size_t)tok0 * tok_row + p.row * kRow, *v = a.v + (size_t)tok0 * tok_row + p.row * kRow;
    const int off = a.sel.set[0].cnt_off[p.b];
    const size_t out0 = ((size_t)p.row * a.sel.set[0].total + off) * kRow;
    constexpr int kU = kRowsInFlight, kStep = kSelThreads / 16;
    for (int i = i0 + (tid >> 4); i < i1; i += kU * kStep) {
      u32x4 kv[kU], vv[kU];
      int page[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int t = i + u * kStep;
        if (t < i1) {
          page[u] = a.block_table != nullptr ? a.block_table[(size_t)p.b * a.max_pages + (t >> a.page_shift)] : 0;
          const size_t at = (size_t)token(t) * tok_row + col;
          kv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(k + at));
          vv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(v + at));
        }
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int t = i + u * kStep;
        if (t < i1) {
          size_t at = out0 + (size_t)t * kRow;
          if (a.block_table != nullptr) {
            if (page[u] < 0 || page[u] >= a.n_pages) continue;  // a table entry outside the pool writes nothing
            at = ((((size_t)page[u] << a.page_shift) + (t & ((1 << a.page_shift) - 1))) * a.Hkv + p.row) * kRow;
          }
          __builtin_nontemporal_store(kv[u], reinterpret_cast<u32x4 *>(a.k_out + at + col));
          __builtin_nontemporal_store(vv[u], reinterpret_cast<u32x4 *>(a.v_out + at + col));
        }
      }
    }
  } else {
    const uint32_t cpr = (uint32_t)a.x_row_bytes >> 4, n = (uint32_t)(i1 - i0) * cpr;  // chunks of 16 bytes; the host keeps them below 2^31
    const uint8_t *x = a.x + (size_t)tok0 * a.x_row_bytes;
    u32x4 *out = reinterpret_cast<u32x4 *>(a.x_out + ((size_t)a.sel.set[1].cnt_off[p.b] + i0) * a.x_row_bytes);
    for (uint32_t c = tid; c < n; c += kChunksInFlight * kSelThreads) {
      u32x4 val[kChunksInFlight];
#pragma unroll
      for (int u = 0; u < kChunksInFlight; ++u) {
        const uint32_t at = c + u * kSelThreads;
        if (at < n) {
          const uint32_t row = a.x_cpr_shift >= 0 ? at >> a.x_cpr_shift : at / cpr;
          val[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(x + (size_t)token(i0 + row) * a.x_row_bytes) + (at - row * cpr));
        }
      }
#pragma unroll
      for (int u = 0; u < kChunksInFlight; ++u)
        if (c + u * kSelThreads < n) __builtin_nontemporal_store(val[u], out + (c + u * kSelThreads));
    }
  }
}

hipError_t launch_select_gather(const SelectGatherArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)a.blk[a.sel.n_seq]), block(kSelThreads);
  switch ((a.longest + 4 * kSelThreads - 1) / (4 * kSelThreads)) {  // keys per thread by the longest row
    case 0:
    case 1: hipLaunchKernelGGL(k_select_gather<4>, grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL(k_select_gather<8>, grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL(k_select_gather<12>, grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL(k_select_gather<16>, grid, block, 0, s, a); break;
    case 5: hipLaunchKernelGGL(k_select_gather<20>, grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL(k_select_gather<24>, grid, block, 0, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace fkv
