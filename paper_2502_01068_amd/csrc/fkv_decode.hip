// Decode-step attention of one new query token per sequence over a KV cache, in particular the
// compacted cache KVCompress leaves behind (Algorithm 1 returns it; Sec. 5.3 measures decoding over
// it).  out[h] = sum_t softmax_t(scale * q[h].k[g(h),t]) * v[g(h),t], every cached token visible.
//
// Bound: the bytes of K and V (512 B per cached token and KV head).  Both contractions run on the matrix
// cores (16x16x32 tiles, the G <= 8 query heads of a KV head on the N side), where they take a few per
// cent of the time the bytes take; as vector dot products they were what the kernel waited for.
//   S = K . Q^T  A operand = 16 tokens x 32 of the 128 columns, read from a wave-private 8 KiB LDS tile that
//                128-bit LDS-direct loads fill with whole rows (16 lanes per row, XOR swizzle on the
//                global side; loading the operand layout itself touches 64 bytes of 16 rows per
//                instruction and cost 10 % on token-major caches).  The result leaves head n = lane % 16
//                on the lane and 8 tokens of the tile in its registers: the softmax is per lane, only the
//                running maximum is shared between the 4 lanes of a head.
//   O^T += V^T . P  B operand = the probabilities as the first contraction left them (the token order inside
//                a contraction is free as long as both operands agree).  A operand: lane (c, q) loads
//                column chunk c (8 values) of those same 8 tokens into registers, whole rows per
//                instruction; the 8x8 block is transposed inside the lane (32 byte permutes), so operand j
//                holds d = 8 c + j.
// Probabilities enter as three bf16 pieces that add up to the fp32 value.  A wave requests its next tile of 32
// tokens (16 KiB of K and V) while it works on the present one, as registers and LDS become free (what is waited for
// when: see step); one block of 4 waves per CU is enough (more resident waves were slower: 256 / 512 / 1024 blocks
// took 57 / 61 / 68 us for 304 MB).
//
// A row (KV head of a sequence) is one block's work, or is cut into equal pieces, one per block; or the tiles of
// all rows form one line that is cut into equal shares (see launch_decode).  Rows in pieces are folded by the last
// block that finishes one, in piece order (reproducible).  One launch per call, nothing waits.  The fold (4 us for 32
// pieces) is bound by what one CU reads past its caches: wider loads, more of them in flight and folding after all
// pieces of a block were each no faster.
//
// Measured (us per call, with vector dot products -> now): 218 tokens, 1 sequence 10.2 -> 4.9; 2048 tokens 11.0 -> 7.1;
// 32768 tokens 35.5 -> 25.6 (5.2 TB/s); 32 sequences of 2048-2560 tokens, paged, 119 -> 51.0 (5.9 TB/s).  Equal shares (34 to 46
// scalars kept in vector lanes, for the walk through the rows): 10 sequences of 12000-12800 tokens 87.7, 40 of 2400-3000, paged,
// 79.6, 48 of 500-1000 31.1, no slower than with 64-bit bounds in registers (87.9, 79.9, 33.3).
#include <algorithm>
#include <type_traits>

#include "fkv_dpp.h"
#include "fkv_internal.h"


namespace fkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;

constexpr int kDecTile = 32;                  // tokens a wave works on at a time
constexpr float kDecNegBig = -1.0e30f;

__device__ __forceinline__ float dec_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// The K tile's operands: waits until at most the 8 youngest loads (the V tile's) are outstanding, reads and waits for
// the reads, so that the tile may be overwritten.  One asm block: for an ordinary LDS read the compiler would
// wait for every outstanding load, the V tile's too (paged, it does so already, see step).
__device__ __forceinline__ void read_k_tile(u32x4 (&r)[8], const uint32_t (&addr)[4]) {
  asm volatile(
      "s_waitcnt vmcnt(8)\n\t"
      "ds_read_b128 %0, %8\n\t"
      "ds_read_b128 %1, %9\n\t"
      "ds_read_b128 %2, %10\n\t"
      "ds_read_b128 %3, %11\n\t"
      "ds_read_b128 %4, %8 offset:4096\n\t"
      "ds_read_b128 %5, %9 offset:4096\n\t"
      "ds_read_b128 %6, %10 offset:4096\n\t"
      "ds_read_b128 %7, %11 offset:4096\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3])
      : "memory");
}

// A lane's four operands from the queries in LDS, whose loads lie ahead of a tile of K and one of V (16 loads).
__device__ __forceinline__ void read_queries(bf16x8 (&qb)[4], uint32_t addr, bool live) {
  u32x4 r[4];
  asm volatile(
      "s_waitcnt vmcnt(16)\n\t"
      "ds_read_b128 %0, %4\n\t"
      "ds_read_b128 %1, %4 offset:64\n\t"
      "ds_read_b128 %2, %4 offset:128\n\t"
      "ds_read_b128 %3, %4 offset:192\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
      : "v"(addr)
      : "memory");
#pragma unroll
  for (int s = 0; s < 4; ++s) qb[s] = __builtin_bit_cast(bf16x8, live ? r[s] : u32x4{0u, 0u, 0u, 0u});
}

// The sum a row is divided by.  Zero: no token has a finite logit and the softmax no value; NaN then, and not what the
// kept-up pieces of the probabilities (see k_decode) divided by zero would give.
__device__ __forceinline__ float row_sum(float l) { return l > 0.f ? l : __uint_as_float(0x7FC00000u); }

__device__ __forceinline__ void agent_store2(float *p, float x, float y) {
  const float2 v = make_float2(x, y);
  unsigned long long bits;
  __builtin_memcpy(&bits, &v, sizeof bits);
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 agent_load2(const float *p) {
  const unsigned long long bits =
      __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  float2 v;
  __builtin_memcpy(&v, &bits, sizeof v);
  return v;
}

// The work of a launch is a line of 32-token tiles, row after row (a row = one KV head of one sequence); block i
// of N takes tiles [i T / N, (i + 1) T / N).  A row that lies inside one block is finished there; the pieces of a row
// that is cut go to partial slots, at most two per block (2 i: a piece that does not begin its row, 2 i + 1: one that does).
// T < 2^30; the products of these bounds are not, so they are formed from quotient and remainder.
__device__ __forceinline__ uint32_t share_at(uint32_t len, uint32_t part, uint32_t parts) {  // len * part / parts
  const uint32_t per = len / parts, rem = len - per * parts;
  return part * per + part * rem / parts;
}
__device__ __forceinline__ int dec_block_of(uint64_t tile, uint64_t tiles, uint64_t n_blocks) {
  return (int)(((tile + 1) * n_blocks - 1) / tiles);
}

// kAligned: every row of sequence b is cut into a.piece0[b + 1] - a.piece0[b] equal pieces, one per block (KV heads
// fastest), instead of equal shares of the line of tiles.  kPauses: the K requests of a tile go out in pairs, see launch_decode.
template <bool kPaged, bool kAligned, bool kPauses, int kWaves>
__global__ __launch_bounds__(kWaves * 64, 2) void k_decode(DecodeArgs a) {
  constexpr int kThr = kWaves * 64;
  constexpr int kTileBytes = kDecTile * kHeadDim * 2;
  __shared__ __attribute__((aligned(16))) uint8_t k_lds[kWaves][kTileBytes];
  __shared__ __attribute__((aligned(16))) float o_lds[kWaves][kMaxReal][kHeadDim];
  __shared__ float m_lds[kWaves][16], l_lds[kWaves][16];
  __shared__ unsigned last_lds;
  typedef __attribute__((address_space(1))) const void *gptr_t;
  typedef __attribute__((address_space(3))) void *lptr_t;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, q = lane >> 4;
  const int G = a.G;
  // 64-bit divisions in front of the first load took 400 instructions, and a search of the sequence entry by entry 0.15 us a step.
  int b = 0, at, at_end;
  int n_piece = 1, piece_blk0 = 0, kvh0 = 0;  // kAligned: pieces of the row, the block of its first one, its KV head
  if (kAligned) {
    const int unit = (int)((uint32_t)blockIdx.x / (uint32_t)a.Hkv);  // pieces before this one, KV heads left aside
    for (int i = 1; i < a.n_seq && b == i - 1; i += 8) {
#pragma unroll
      for (int j = 0; j < 8; ++j) b += (i + j < a.n_seq) & (unit >= a.piece0[i + j]);
    }
    n_piece = a.piece0[b + 1] - a.piece0[b];
    const int p = unit - a.piece0[b];
    kvh0 = (int)blockIdx.x - unit * a.Hkv;
    piece_blk0 = (int)blockIdx.x - p * a.Hkv;
    const int len = a.tile0[b + 1] - a.tile0[b];
    at = 0;
    at_end = len;
    if (n_piece > 1) {
      at = (int)share_at(len, p, n_piece);
      at_end = (int)share_at(len, p + 1, n_piece);
    }
  } else {
    at = (int)share_at(a.tiles, blockIdx.x, gridDim.x);
    at_end = (int)share_at(a.tiles, blockIdx.x + 1, gridDim.x);
  }
  uint8_t *stage = k_lds[wave];
  // Row c of the first contraction's A operand is token 4 (c % 4) + c / 4 of a half tile, so that row 4 q + r of
  // its result is token 4 r + q: the tokens whose V rows one load instruction brings to lane group q in turn.
  const int kt = 4 * (c & 3) + (c >> 2);
  uint32_t k_addr[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) k_addr[s] = (uint32_t)(uintptr_t)(lptr_t)stage + kt * 256 + (((4 * s + q) ^ kt) << 4);

  while (at < at_end) {
    // ---- the piece [tile0, tile1) of row (b, kvh)
    int row_at = 0, kvh = kvh0;  // kAligned: `at` counts from the row's first tile
    if (!kAligned) {
      while (at >= a.tile0[b + 1] * a.Hkv) ++b;
    }
    const int row_tiles = a.tile0[b + 1] - a.tile0[b];
    if (!kAligned) {
      const int seq_at = a.tile0[b] * a.Hkv;
      kvh = (int)((uint32_t)(at - seq_at) / (uint32_t)row_tiles);
      row_at = seq_at + kvh * row_tiles;
    }
    const int tile0 = at - row_at, tile1 = min(row_tiles, at_end - row_at);
    const int n = a.off[b + 1] - a.off[b];

    // The row's queries (8 rows of 256 B, those the group does not have are not read) go to the wave's part of o_lds, idle until
    // the end, ahead of the loads of K and V and in the same order: loaded into registers, the compiler would wait for them
    // together with everything requested.
    uint8_t *q_lds = reinterpret_cast<uint8_t *>(&o_lds[wave][0][0]);
    {
      const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.q + ((size_t)b * a.Hq + (size_t)kvh * G) * kHeadDim), 0,
                                                          G * kHeadDim * 2, 0x00027000);
#pragma unroll
      for (int i = 0; i < 2; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (lptr_t)(q_lds + i * 1024), 16, i * 1024 + lane * 16, 0, 0, 0);
      keep_access_order();  // read_queries waits for all but the 16 youngest loads: a tile of K and one of V
    }
    const size_t first = kPaged ? 0 : (size_t)a.off[b];  // a paged sequence is addressed through its block table
    typedef __attribute__((address_space(1))) const uint8_t *rows_t;
    const rows_t kb = (rows_t)(a.k + (size_t)kvh * a.head_stride + first * a.tok_stride);
    const rows_t vb = (rows_t)(a.v + (size_t)kvh * a.head_stride + first * a.tok_stride);
    const uint32_t row = (uint32_t)a.tok_stride * 2;  // bytes of a token's row, at most 2 KiB
    const int32_t *table = kPaged ? a.block_table + (size_t)b * a.max_pages : nullptr;

    // Page of this lane's token (lane % 32) of a tile; an entry outside the pool is clamped into it.
    auto page_of = [&](int tile) { return table[min(tile * kDecTile + (lane & 31), n - 1) >> a.page_shift]; };
    auto slot_of = [&](int tile, int page) {
      const int t = min(tile * kDecTile + (lane & 31), n - 1);
      return (min(max(page, 0), a.n_pages - 1) << a.page_shift) + (t & ((1 << a.page_shift) - 1));
    };
    u32x4 vr[8];
    uint32_t slots[8];  // paged: page slots of the rows that this lane's loads touch
    // Load i of a tile covers its tokens 4 i .. 4 i + 3, one per 16 lanes.  `slot`: page slots of the tile's tokens, one per lane
    // (paged cache only).  Unpaged, an address is the tile's own plus a 32-bit offset within the row's end.
    auto row_of = [&](rows_t base, int i, int tile, uint32_t column) {
      if constexpr (kPaged) return base + (uint64_t)slots[i] * row + column;
      const uint32_t last = (uint32_t)min(kDecTile - 1, n - 1 - tile * kDecTile) * row;
      return base + (min((4 * i + q) * row, last) + column);
    };
    auto rows_of = [&](rows_t base, int tile) {
      if constexpr (!kPaged) {
        base += (size_t)tile * kDecTile * row;
        asm("" : "+s"(base));  // else every load of the loop gets an address of its own, in two registers per lane
      }
      return base;
    };
    auto load_k = [&](int tile, int slot, auto pauses_t) {
      const rows_t rows = rows_of(kb, tile);
      if constexpr (kPaged) {
#pragma unroll
        for (int i = 0; i < 8; ++i) slots[i] = (uint32_t)__shfl(slot, 4 * i + q);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        __builtin_amdgcn_global_load_lds((gptr_t)row_of(rows, i, tile, (c ^ ((4 * i + q) & 15)) << 4), (lptr_t)(stage + i * 1024), 16, 0, 2);
        if constexpr (decltype(pauses_t)::value) {
          if (i & 1) __builtin_amdgcn_s_sleep(2);  // 128 cycles
        }
      }
    };
    auto load_v = [&](int tile) {  // of the tile that load_k was called for last
      keep_access_order();  // read_k_tile waits for all but the 8 youngest loads: these
      const rows_t rows = rows_of(vb, tile);
#pragma unroll
      for (int i = 0; i < 8; ++i) vr[i] = __builtin_nontemporal_load((__attribute__((address_space(1))) const u32x4 *)row_of(rows, i, tile, c << 4));
    };

    // B operand of the first contraction: head n = c, columns 8 (4 s + q) .. + 7 in step s; zeros past the last head
    bf16x8 qb[4];

    floatx4 o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = (floatx4){0.f, 0.f, 0.f, 0.f};
    float m = kDecNegBig, l = 0.f;

    int tile = tile0 + wave;
    int slot = 0, page_next = 0;
    {
      const int t = min(tile, tile1 - 1);  // a wave without a tile of its own loads one all the same: no branch around the loads
      if (kPaged) {
        const int page = page_of(t);
        page_next = page_of(t + kWaves);
        slot = slot_of(t, page);
      }
      load_k(t, slot, std::false_type{});
      load_v(t);
      read_queries(qb, (uint32_t)(uintptr_t)(lptr_t)(q_lds + (c & 7) * 256 + q * 16), c < G);
    }
    // One tile; kMore: the loads of the wave's next one go out as their registers and LDS become free (a
    // compile-time flag: no branch around loads).  The compiler's own waits are longer than need be.  Ordinary loads
    // behind LDS-direct ones are waited for together with everything requested: the V tile with the next K tile,
    // requested a contraction earlier; a paged cache's page entry, before the K tile is read, with the V tile.  Exact waits inside
    // the loop (V through LDS-direct loads, read in asm blocks like K) were no faster: 2048 tokens 7.77 against 7.65 us, 32
    // paged sequences 52.5 against 51.6 (with q in registers, see read_queries).
    auto step = [&](auto more_t) {
      constexpr bool kMore = decltype(more_t)::value;
      u32x4 kr[8];
      read_k_tile(kr, k_addr);
      if constexpr (kPaged && kMore) {
        slot = slot_of(tile + kWaves, page_next);
        page_next = page_of(tile + 2 * kWaves);
      }
      if constexpr (kMore) load_k(tile + kWaves, slot, std::bool_constant<kPauses>{});
      floatx4 acc[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        acc[h] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[4 * h + s]), qb[s], acc[h], 0, 0, 0);
      }

      // acc[h][r] = logit of head c and token 16 h + 4 r + q of the tile
      float z[8];
      float tmax = kDecNegBig;
      const bool edge = (tile + 1) * kDecTile > n;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        z[i] = acc[i >> 2][i & 3] * a.scale_log2e;
        if (edge && tile * kDecTile + 4 * i + q >= n) z[i] = -INFINITY;  // weight 0 below whatever the maximum: it is at least kDecNegBig
        tmax = fmaxf(tmax, z[i]);
      }
      tmax = quarters_max(tmax);
      const float m_new = fmaxf(m, tmax);
      const float alpha = dec_exp2(m - m_new);
      m = m_new;
      float psum = 0.f;
      // p = p0 + p1 + p2, 8 bits each, cut off and not rounded; the lower two are kept above 0, which adds less than
      // 2^-125 of V: an infinite V stays infinite in the sum (0 times it, or a negative piece, would make it NaN).
      constexpr float kTiny = 0x1p-126f;
      u32x4 p0, p1, p2;
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        uint32_t w0[2], w1[2], w2[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float p = dec_exp2(z[i + e] - m_new);
          psum += p;
          w0[e] = __float_as_uint(p);
          const float r1 = fmaxf(p - __uint_as_float(w0[e] & 0xffff0000u), kTiny);
          w1[e] = __float_as_uint(r1);
          w2[e] = __float_as_uint(fmaxf(r1 - __uint_as_float(w1[e] & 0xffff0000u), kTiny));
        }
        p0[i / 2] = __builtin_amdgcn_perm(w0[1], w0[0], 0x07060302u);
        p1[i / 2] = __builtin_amdgcn_perm(w1[1], w1[0], 0x07060302u);
        p2[i / 2] = __builtin_amdgcn_perm(w2[1], w2[0], 0x07060302u);
      }
      l = l * alpha + psum;
      if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0ull) {
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] *= alpha;
      }

      u32x4 va[8];  // va[j]: the 8 tokens' values of column 8 c + j
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          va[2 * w][i] = __builtin_amdgcn_perm(vr[2 * i + 1][w], vr[2 * i][w], 0x05040100u);
          va[2 * w + 1][i] = __builtin_amdgcn_perm(vr[2 * i + 1][w], vr[2 * i][w], 0x07060302u);
        }
      if constexpr (kMore) load_v(tile + kWaves);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bf16x8 vj = __builtin_bit_cast(bf16x8, va[j]);
        o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vj, __builtin_bit_cast(bf16x8, p2), o[j], 0, 0, 0);
        o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vj, __builtin_bit_cast(bf16x8, p1), o[j], 0, 0, 0);
        o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vj, __builtin_bit_cast(bf16x8, p0), o[j], 0, 0, 0);
      }
    };
    for (; tile + kWaves < tile1; tile += kWaves) step(std::true_type{});  // uniform per wave
    if (tile < tile1) step(std::false_type{});

    // ---- the waves' states into LDS: lane (head c, q) holds d = 32 q + 8 r + j in o[j][r]
    l = quarters_sum(l);
    if (c < G) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j4 = 0; j4 < 2; ++j4)
          *reinterpret_cast<float4 *>(&o_lds[wave][c][32 * q + 8 * r + 4 * j4]) =
              make_float4(o[4 * j4][r], o[4 * j4 + 1][r], o[4 * j4 + 2][r], o[4 * j4 + 3][r]);
      if (q == 0) { m_lds[wave][c] = m; l_lds[wave][c] = l; }
    }
    __syncthreads();
    const bool whole = tile0 == 0 && tile1 == row_tiles;  // this block has the entire row
    float *part = a.part + (2 * (size_t)blockIdx.x + (!kAligned && tile0 == 0 ? 1 : 0)) * kDecodeSlotFloats;
    float *out = a.out + ((size_t)b * a.Hq + (size_t)kvh * G) * kHeadDim;
    for (int e = tid; e < G * (kHeadDim / 2); e += kThr) {
      const int h = e >> 6, d = (e & 63) * 2;
      float M = m_lds[0][h];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) M = fmaxf(M, m_lds[w][h]);
      float L = 0.f, x = 0.f, y = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float f = dec_exp2(m_lds[w][h] - M);
        const float2 ov = *reinterpret_cast<const float2 *>(&o_lds[w][h][d]);
        L += f * l_lds[w][h];
        x += f * ov.x;
        y += f * ov.y;
      }
      if (whole) {
        const float sum = row_sum(L);
        *reinterpret_cast<float2 *>(out + h * kHeadDim + d) = make_float2(x / sum, y / sum);
      } else {
        agent_store2(part + h * kHeadDim + d, x, y);
        if (d == 0) agent_store2(part + kMaxReal * kHeadDim + 2 * h, M, L);
      }
    }
    at = row_at + tile1;
    if (whole) {
      if (kAligned) return;
      __syncthreads();  // the next piece reuses the tables
      continue;
    }

    // ---- count this piece; the last one of the row folds them
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int blk0 = kAligned ? piece_blk0 : dec_block_of(row_at, a.tiles, gridDim.x);
    const int n_split = kAligned ? n_piece : dec_block_of(row_at + row_tiles - 1, a.tiles, gridDim.x) - blk0 + 1;
    unsigned *count = a.count + b * kMaxKvHeads + kvh;
    if (tid == 0) {
      const unsigned old = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_lds = old + 1u == (unsigned)n_split ? 1u : 0u;
    }
    __syncthreads();
    if (last_lds != 0u) {
      if (tid == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
      // equal shares: piece p of the row lies in block blk0 + p; only the first one begins the row
      const float *src = a.part + 2 * (size_t)blk0 * kDecodeSlotFloats;
      auto piece = [&](int p) { return src + (size_t)(kAligned ? 2 * p * a.Hkv : p == 0 ? 1 : 2 * p) * kDecodeSlotFloats; };
      constexpr int kBatch = 16;  // partial rows in flight per lane
      for (int h = wave; h < G; h += kWaves) {  // one wave per head, two columns per lane
        const float2 ml = agent_load2(piece(min(lane, n_split - 1)) + kMaxReal * kHeadDim + 2 * h);
        float2 v[kBatch];
        auto request = [&](int s0) {
#pragma unroll
          for (int i = 0; i < kBatch; ++i) v[i] = agent_load2(piece(min(s0 + i, n_split - 1)) + h * kHeadDim + 2 * lane);
        };
        request(0);
        // the pieces' weights, a lane each
        const float mp = lane < n_split ? ml.x : kDecNegBig;
        const float f = dec_exp2(mp - wave_fmax(mp));
        const float L = row_sum(wave_fsum(lane < n_split ? ml.y * f : 0.f));
        const int weight = __float_as_int(lane < n_split ? f / L : 0.f);
        float x = 0.f, y = 0.f;
        for (int s0 = 0; s0 < n_split; s0 += kBatch) {
          if (s0 > 0) request(s0);
#pragma unroll
          for (int i = 0; i < kBatch; ++i) {  // past the last piece nothing is added: 0 times an infinite sum would be NaN
            const float w = __int_as_float(__builtin_amdgcn_readlane(weight, s0 + i));
            x += s0 + i < n_split ? v[i].x * w : 0.f;
            y += s0 + i < n_split ? v[i].y * w : 0.f;
          }
        }
        *reinterpret_cast<float2 *>(out + h * kHeadDim + 2 * lane) = make_float2(x, y);
      }
    }
    if (kAligned) return;
    __syncthreads();
  }
}

// Tiles of every sequence (a.tile0, a.tiles), the blocks to spread them over, and the launch.
hipError_t launch_decode(DecodeArgs &a, int n_cu, hipStream_t s) {
  constexpr int kWaves = 4;
  const dim3 block(kWaves * 64);
  int64_t tiles = 0, longest = 1;
  a.tile0[0] = 0;
  for (int b = 0; b < a.n_seq; ++b) {
    const int64_t t = (a.off[b + 1] - a.off[b] + kDecTile - 1) / kDecTile;
    tiles += t;
    longest = std::max(longest, t);
    a.tile0[b + 1] = (int)tiles;
  }
  a.tiles = (int)(tiles * a.Hkv);  // < 2^30: there are less than 2^31 tokens, and 8 KV heads at most
  // Each row cut into pieces of about a CU's share, or left whole, unless that loads the CUs unevenly for long: a share
  // of the line that straddles rows costs a restart of the loads and one more fold, about 5 us.
  //   Whole: rows close to a multiple of the CUs and none much longer than the mean (256 rows of 2048-2560 tokens 50.8
  //   against 56 us, of 1280-2560 45.6 against 48; but 320 rows 54 against 47.7); rows of up to 12 tiles, where a fold
  //   costs more than it saves (160 rows of 250 tokens 7.4 against 13.9).
  //   Pieces: few rows, or few tiles per CU (128 rows of 1000 tokens 14.2 against 17 us; of 5000, 63 against 55.7).
  constexpr int kWholeTiles = 12;
  // Pauses between K requests, for a token-major cache and 40 tiles per block or more.  The heads' blocks read 256 bytes each of the
  // same 2 KiB; all 8 requests of a tile at once (one addition each; a 64-bit product each used to space them) disturb that.
  // With pauses, without, with the products: 32 sequences of 3600-4000 tokens 79.1, 80.3, 79.2 us, 32 of 2048 43.6, 44.5, 43.9, 12 of
  // 7000-8000 65.7, 66.5, 66.2, one of 120000 79.2, 80.3, 80.1.  Fewer tiles and a compact cache are faster without: one sequence of
  // 32768 (32 tiles per block) 25.9, 25.6, 26.7; 48 of 500-1000 31.8, 31.3, 33.6; compact 32 of 3600-4000 76.5, 76.0, 77.1.
  constexpr int kPausesTiles = 40;
  auto pauses = [&](dim3 grid) { return a.tok_stride > kHeadDim && a.tiles >= (int64_t)kPausesTiles * grid.x; };
  const int rows = a.n_seq * a.Hkv;
  const int per_cu = (rows + n_cu - 1) / n_cu;
  const bool even = 10 * rows >= 9 * per_cu * n_cu && 2 * longest * a.n_seq <= 3 * tiles;
  const bool pieces = 4 * rows <= n_cu || (rows <= n_cu && a.tiles <= (int64_t)48 * n_cu);  // <= 1.5 n_cu of them
  if (even || pieces || longest <= kWholeTiles) {
    const int64_t share = std::max<int64_t>(kWaves, ((int64_t)a.tiles + n_cu - 1) / n_cu);
    a.piece0[0] = 0;
    for (int b = 0; b < a.n_seq; ++b) {
      const int64_t t = a.tile0[b + 1] - a.tile0[b];
      int64_t n = even || t <= kWholeTiles ? 1 : std::min<int64_t>((2 * t + share) / (2 * share), kDecodeMaxSplits);
      a.piece0[b + 1] = a.piece0[b] + (int)std::max<int64_t>(n, 1);
    }
    const dim3 grid((unsigned)(a.piece0[a.n_seq] * a.Hkv));
    if (a.block_table)
      hipLaunchKernelGGL((k_decode<true, true, false, kWaves>), grid, block, 0, s, a);
    else if (pauses(grid))
      hipLaunchKernelGGL((k_decode<false, true, true, kWaves>), grid, block, 0, s, a);
    else
      hipLaunchKernelGGL((k_decode<false, true, false, kWaves>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  // Equal shares: one block per CU; two where a block goes through several short rows, as each starts with the latency
  // of its first loads, which the other block then covers.
  const int shares = rows > n_cu && a.tiles <= (int64_t)rows * 16 ? 2 : 1;
  int64_t blocks = std::min<int64_t>(std::min(shares * n_cu, kDecodeMaxBlocks), ((int64_t)a.tiles + kWaves - 1) / kWaves);
  // a row is cut into at most kDecodeMaxSplits pieces: the fold keeps a weight for each
  blocks = std::max<int64_t>(1, std::min<int64_t>(blocks, (int64_t)a.tiles * (kDecodeMaxSplits - 2) / longest));
  const dim3 grid((unsigned)blocks);
  if (a.block_table)
    hipLaunchKernelGGL((k_decode<true, false, false, kWaves>), grid, block, 0, s, a);
  else if (pauses(grid))
    hipLaunchKernelGGL((k_decode<false, false, true, kWaves>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((k_decode<false, false, false, kWaves>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace fkv
