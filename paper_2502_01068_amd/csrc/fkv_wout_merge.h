// Folding the splits that k_wout_partial leaves: the window rows' outputs, and the softmax rows' normalisers.
#pragma once

#include "fkv_dpp.h"
#include "fkv_score_exchange.h"

namespace fkv {

constexpr int kWoRowFloats = kRowsPerGroup * kHeadDim;  // 4096 accumulator values per partial
constexpr int kWoOutputs = kWoRowFloats / 4;            // float4 outputs of a (sequence, group)

// One float4 of the output, `idx` of (sequence, group) bg.  Four lanes (j = 0 .. 3) share it and take every fourth split each
// (eight loads in flight per lane), then meet through two lane exchanges; the order of the sums is fixed.
__device__ __forceinline__ void merge_output(const WoutArgs &a, int bg, int idx, int j) {
  const int b = bg / a.V, g = bg - b * a.V;
  const int row = idx >> 5, chunk = idx & 31;
  const int hl = row >> 3, w = row & 7;
  const bool first = j == 0 && chunk == 0;  // the lane that reports the row's normaliser
  if (hl >= vg_heads(a, g) || w >= a.W) {   // the four lanes of an output leave together
    if (first && a.rowstat) a.rowstat[(size_t)bg * kRowsPerGroup + row] = 0.f;
    return;
  }
  const float2 *ms = a.part_ms + (size_t)bg * a.n_split * kRowsPerGroup + row;
  const float *po = a.part_o + (size_t)bg * a.n_split * kWoRowFloats + row * kHeadDim + chunk * 4;
  constexpr int kBatch = 8;
  const int per = (a.n_split + 3) >> 2;  // splits j, j+4, ... of this lane
  float M = kNegBig;
  for (int i0 = 0; i0 < per; i0 += kBatch) {
    float mx[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) mx[i] = ms[min(4 * (i0 + i) + j, a.n_split - 1) * kRowsPerGroup].x;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) M = fmaxf(M, mx[i]);
  }
  M = fmaxf(M, __shfl_xor(M, 1));
  M = fmaxf(M, __shfl_xor(M, 2));
  float den = 0.f;
  float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int i0 = 0; i0 < per; i0 += kBatch) {
    float2 st[kBatch];
    float4 x[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int sp = min(4 * (i0 + i) + j, a.n_split - 1);
      st[i] = ms[sp * kRowsPerGroup];
      x[i] = *reinterpret_cast<const float4 *>(po + (size_t)sp * kWoRowFloats);
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const float f = 4 * (i0 + i) + j < a.n_split ? fast_exp2(st[i].x - M) : 0.f;
      den += f * st[i].y;
      num.x += f * x[i].x; num.y += f * x[i].y; num.z += f * x[i].z; num.w += f * x[i].w;
    }
  }
#pragma unroll
  for (int d = 1; d <= 2; d <<= 1) {
    den += __shfl_xor(den, d);
    num.x += __shfl_xor(num.x, d); num.y += __shfl_xor(num.y, d);
    num.z += __shfl_xor(num.z, d); num.w += __shfl_xor(num.w, d);
  }
  if (j != 0) return;
  if (first && a.rowstat) a.rowstat[(size_t)bg * kRowsPerGroup + row] = M + __log2f(den);
  const float inv = 1.f / den;
  float *dst = a.out + (((size_t)b * a.W + w) * a.Hq + vg_head0(a, g) + hl) * kHeadDim + chunk * 4;
  *reinterpret_cast<float4 *>(dst) = make_float4(num.x * inv, num.y * inv, num.z * inv, num.w * inv);
}

// The log-sum-exps (log2 units) of the 32 rows of (sequence, group) bg into dst, by one wave: lane group j = lane / 16 takes
// splits j, j + 4, ... of rows lane % 16 and lane % 16 + 16, in merge_output's order of the sums.  Rows that the shape does not
// have get 0.
__device__ __forceinline__ void merge_normalisers(const WoutArgs &a, int bg, int g, int lane, float *dst) {
  const int j = lane >> 4, r0 = lane & 15;
  const float2 *ms = a.part_ms + (size_t)bg * a.n_split * kRowsPerGroup + r0;
  constexpr int kBatch = 8;
  const int per = (a.n_split + 3) >> 2;
  float2 st[2][kBatch];
  auto load = [&](int i0) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const float2 *p = ms + min(4 * (i0 + i) + j, a.n_split - 1) * kRowsPerGroup;
      st[0][i] = p[0];
      st[1][i] = p[16];
    }
  };
  float M[2] = {kNegBig, kNegBig}, den[2] = {0.f, 0.f};
  for (int i0 = 0; i0 < per; i0 += kBatch) {
    load(i0);
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) M[h] = fmaxf(M[h], st[h][i].x);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) M[h] = quarters_max(M[h]);
  for (int i0 = 0; i0 < per; i0 += kBatch) {
    if (per > kBatch) load(i0);  // one batch: still at hand
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) den[h] += (4 * (i0 + i) + j < a.n_split ? fast_exp2(st[h][i].x - M[h]) : 0.f) * st[h][i].y;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float S = quarters_sum(den[h]);
    const int row = r0 + 16 * h;
    const bool ok = (row >> 3) < vg_heads(a, g) && (row & 7) < a.W;
    if (j == 0) dst[row] = ok ? M[h] + __log2f(S) : 0.f;
  }
}

}  // namespace fkv
