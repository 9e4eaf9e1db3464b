// Index-driven row gathers (HiddenCompress / KVCompress, App. B.1): bit-exact copies of the
// kept rows into compacted buffers.  Up to three jobs (hidden rows, K rows, V rows) share one
// launch so the small K/V jobs fill the machine alongside the large hidden-row job.
//
// The unit of work is one 16-byte chunk; consecutive lanes take consecutive chunks of a row,
// so a 256-byte K/V head row is one 16-lane segment and an 8 KiB hidden row is 512 lanes.
// Each (job, head) owns a contiguous range of blocks, so the head and job lookups are scalar.
//
// Large calls are bound by HBM (6.2 TB/s read and written), small ones by the chain arguments - index - row - store.  A chunk's
// index used to be waited for before the next one's was requested, and the sequences were searched one by one per lane:
// kernel trace, before -> after: 2048 tokens 5.7 -> 4.6 us, 32768 23.1 -> 22.2, 16384 head-wise 9.1 -> 8.2, 8 ragged
// sequences 72.1 -> 67.9, 131072 87.6 -> 87.0.  With non-temporal stores: plain ones make this launch 10 % shorter at
// 131072 tokens and the whole call 11 % longer.  4 and 8 chunks per thread or all rows of a thread in flight before the first store: up to
// 4 us more at 131072 tokens; 64, 128 or 512 threads: the same.
#include "fkv_internal.h"

namespace fkv {

constexpr int kGatherThreads = 256;
constexpr int kGatherUnroll = 2;  // 16-byte chunks in flight per thread

int gather_blocks_per_head(const GatherJob &j) {
  const int64_t chunks = (int64_t)j.total_rows * (j.row_bytes / 16);
  const int64_t per_block = (int64_t)kGatherThreads * kGatherUnroll;
  return (int)((chunks + per_block - 1) / per_block);
}

// The sequence of kept row `first`, eight prefix sums a step (one by one each costs a trip through the scalar cache).  Uniform.
__device__ __forceinline__ int seq_of_row(const int *cnt_off, int n_seq, int first) {
  int b = 0;
  for (int i = 1; i < n_seq && b == i - 1; i += 8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) b += (i + j < n_seq) & (first >= cnt_off[i + j]);
  }
  return b;
}

// Calls fn(u, b, first row of b, first token of b, tokens of b) for the sequence b of every kept row t[u] (ascending with u), all
// between the block's first and last row.  As a rule these lie in one sequence: then b and its bounds are scalars.
template <typename F>
__device__ __forceinline__ void for_each_row(const int *cnt_off, const int *cu, int n_seq, int first, int last,
                                             const uint32_t (&t)[kGatherUnroll], F fn) {
  int b = seq_of_row(cnt_off, n_seq, first);
  if (last < cnt_off[b + 1]) {
    const int row0 = cnt_off[b], base = cu[b], n = cu[b + 1] - base;
#pragma unroll
    for (int u = 0; u < kGatherUnroll; ++u) fn(u, b, row0, base, n);
    return;
  }
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) {
    while ((int)t[u] >= cnt_off[b + 1]) ++b;
    fn(u, b, cnt_off[b], cu[b], cu[b + 1] - cu[b]);
  }
}
// The token of a kept index: one beyond its sequence is clamped into it (a wrong row, never an out-of-bounds read); a negative
// one is the mark of an invalid selection, its row is not copied.
__device__ __forceinline__ uint32_t kept_token(int base, int n, int raw) { return (uint32_t)(base + min(max(raw, 0), n - 1)); }

__global__ __launch_bounds__(kGatherThreads) void k_gather(GatherArgs a) {
  const int block = blockIdx.x;
  const int ji = ((a.n_jobs > 1) & (block >= a.job[1].blk0)) + ((a.n_jobs > 2) & (block >= a.job[2].blk0));
  const GatherJob &job = a.job[ji];
  const uint32_t rel = block - job.blk0;
  uint32_t h = 0, hb = rel;
  if (job.n_heads > 1) {
    h = rel / (uint32_t)job.blocks_per_head;  // uniform: scalar division
    hb = rel - h * job.blocks_per_head;
  }
  const uint32_t cpr = (uint32_t)job.row_bytes >> 4;       // chunks per row
  const uint32_t n_chunks = (uint32_t)job.total_rows * cpr; // per head; host guarantees < 2^31
  const uint32_t first = hb * (kGatherUnroll * kGatherThreads), c0 = first + threadIdx.x;
  const uint32_t end = min(first + kGatherUnroll * kGatherThreads, n_chunks) - 1u;  // the block's last chunk
  const int32_t *idx = job.idx + (size_t)h * job.total_rows;
  const uint8_t *src_h = job.src + (size_t)(job.head_div == 1 ? h : h / (uint32_t)job.head_div) * job.row_bytes;
  u32x4 *dst_h = reinterpret_cast<u32x4 *>(job.dst + (size_t)h * job.total_rows * job.row_bytes);
  auto row_of = [&](uint32_t c) { return job.cpr_shift >= 0 ? c >> job.cpr_shift : c / cpr; };

  uint32_t t[kGatherUnroll], tok[kGatherUnroll];
  int raw[kGatherUnroll];
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) t[u] = row_of(min(c0 + u * kGatherThreads, end));
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) raw[u] = idx[t[u]];  // on their way together
  for_each_row(job.cnt_off, a.cu, a.n_seq, (int)row_of(first), (int)row_of(end), t,
               [&](int u, int, int, int base, int n) { tok[u] = kept_token(base, n, raw[u]); });
  // rows are read once and written once: non-temporal both ways (plain stores leave the L2 dirty and
  // measurably slow the next score launch)
  u32x4 val[kGatherUnroll];
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) {
    const uint32_t col = min(c0 + u * kGatherThreads, end) - t[u] * cpr;
    val[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src_h + (uint64_t)tok[u] * job.src_row_stride) + col);
  }
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u)
    if (c0 + u * kGatherThreads <= end && raw[u] >= 0) __builtin_nontemporal_store(val[u], dst_h + (c0 + u * kGatherThreads));
}

// Paged destination: chunk c of the launch is 16 bytes of (kept slot t, KV head g), heads fastest,
// so the 16*Hkv lanes of one slot write one contiguous [Hkv][d] page entry.  blockIdx.y picks K or V.
// A block-table entry outside [0, n_pages) writes nothing.
__global__ __launch_bounds__(kGatherThreads) void k_gather_paged(PagedGatherArgs a) {
  const int which = blockIdx.y;
  const uint8_t *src = a.src[which];
  uint8_t *pages = a.pages[which];
  constexpr uint32_t kCpr = kHeadDim * 2 / 16;  // 16 chunks per head row
  const uint32_t n_chunks = (uint32_t)a.total_rows * a.Hkv * kCpr;
  const uint32_t first = blockIdx.x * (kGatherUnroll * kGatherThreads), c0 = first + threadIdx.x;
  const uint32_t end = min(first + kGatherUnroll * kGatherThreads, n_chunks) - 1u;  // the block's last chunk
  uint32_t t[kGatherUnroll], g[kGatherUnroll], tok[kGatherUnroll], tl[kGatherUnroll];
  int raw[kGatherUnroll], page[kGatherUnroll];
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) {
    const uint32_t r = min(c0 + u * kGatherThreads, end) / kCpr;
    t[u] = r / (uint32_t)a.Hkv;
    g[u] = r - t[u] * a.Hkv;
    raw[u] = a.idx[(size_t)g[u] * a.total_rows + t[u]];
  }
  for_each_row(a.cnt_off, a.cu, a.n_seq, (int)(first / kCpr / (uint32_t)a.Hkv), (int)(end / kCpr / (uint32_t)a.Hkv), t,
               [&](int u, int b, int row0, int base, int n) {
                 tl[u] = t[u] - row0;
                 page[u] = a.block_table[(size_t)b * a.max_pages + (tl[u] >> a.page_shift)];
                 tok[u] = kept_token(base, n, raw[u]);
               });
  const uint32_t col = threadIdx.x & (kCpr - 1u);
  static_assert(kGatherThreads % kCpr == 0, "a thread's chunks lie in the same column");
  u32x4 val[kGatherUnroll];
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u)
    val[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + ((uint64_t)tok[u] * a.Hkv + g[u]) * (kHeadDim * 2)) + col);
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u)
    if (c0 + u * kGatherThreads <= end && raw[u] >= 0 && page[u] >= 0 && page[u] < a.n_pages) {
      const size_t slot = ((size_t)page[u] << a.page_shift) + (tl[u] & ((1u << a.page_shift) - 1u));
      __builtin_nontemporal_store(val[u], reinterpret_cast<u32x4 *>(pages + (slot * a.Hkv + g[u]) * (kHeadDim * 2)) + col);
    }
}

hipError_t launch_gather_paged(const PagedGatherArgs &a, hipStream_t s) {
  const int64_t chunks = (int64_t)a.total_rows * a.Hkv * (kHeadDim * 2 / 16);
  const int64_t per_block = (int64_t)kGatherThreads * kGatherUnroll;
  const int n_blocks = (int)((chunks + per_block - 1) / per_block);
  if (n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_paged, dim3(n_blocks, a.src[1] ? 2 : 1), dim3(kGatherThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gather(const GatherArgs &a, int n_blocks, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather, dim3(n_blocks), dim3(kGatherThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace fkv
