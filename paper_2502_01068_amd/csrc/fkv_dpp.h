// Wave-wide reductions and scans on the vector ALU's data-parallel-primitive (DPP) lane routing:
// no LDS crossbar traffic, a few cycles per level instead of a shuffle's LDS round trip.
// A wave is 4 DPP rows of 16 lanes.  Lanes whose source falls outside their row (shifts) or that
// the row mask leaves out keep the `old` operand, which every helper sets to the operation's
// identity.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fkv {

constexpr int kDppRowShr = 0x110;   // + n: lane i reads lane i - n of its row
constexpr int kDppRowRor = 0x120;   // + n: lane i reads lane (i - n) mod 16 of its row
constexpr int kDppQuadXor1 = 0xB1;  // lane i of a quad reads lane i ^ 1,
constexpr int kDppQuadXor2 = 0x4E;  // lane i ^ 2
constexpr int kDppHalfMirror = 0x141;  // lane i of 8 reads lane 7 - i
constexpr int kDppBcast15 = 0x142;  // lane 15 of each row to every lane of the next row
constexpr int kDppBcast31 = 0x143;  // lane 31 to every lane of rows 2 and 3

template <int kCtrl, int kRowMask = 0xF>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t src) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, kCtrl, kRowMask, 0xF, false);
}

// Inclusive prefix sum over the 64 lanes (lane order).
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t x) {
  x += dpp_u32<kDppRowShr + 1>(0u, x);
  x += dpp_u32<kDppRowShr + 2>(0u, x);
  x += dpp_u32<kDppRowShr + 4>(0u, x);
  x += dpp_u32<kDppRowShr + 8>(0u, x);
  x += dpp_u32<kDppBcast15, 0xA>(0u, x);  // rows 1, 3 += total of the row before
  x += dpp_u32<kDppBcast31, 0xC>(0u, x);  // rows 2, 3 += total of rows 0..1
  return x;
}

// Value of lane 63 as a wave-uniform scalar.
__device__ __forceinline__ uint32_t wave_last(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }

// Maximum / minimum over the 64 lanes; the result is valid in lane 63 only (use wave_last to spread it).
__device__ __forceinline__ uint32_t wave_max_to_last(uint32_t x) {  // `old` is the maximum's identity: one instruction a step
  x = max(x, dpp_u32<kDppRowRor + 8>(0u, x));
  x = max(x, dpp_u32<kDppRowRor + 4>(0u, x));
  x = max(x, dpp_u32<kDppRowRor + 2>(0u, x));
  x = max(x, dpp_u32<kDppRowRor + 1>(0u, x));
  x = max(x, dpp_u32<kDppBcast15, 0xA>(0u, x));
  x = max(x, dpp_u32<kDppBcast31, 0xC>(0u, x));
  return x;
}
__device__ __forceinline__ uint32_t wave_min_to_last(uint32_t x) { return ~wave_max_to_last(~x); }

// Sum over the 64 lanes, valid in lane 63 only.
__device__ __forceinline__ uint32_t wave_sum_to_last(uint32_t x) {
  x += dpp_u32<kDppRowRor + 8>(0u, x);
  x += dpp_u32<kDppRowRor + 4>(0u, x);
  x += dpp_u32<kDppRowRor + 2>(0u, x);
  x += dpp_u32<kDppRowRor + 1>(0u, x);
  x += dpp_u32<kDppBcast15, 0xA>(0u, x);
  x += dpp_u32<kDppBcast31, 0xC>(0u, x);
  return x;
}

// ---- fp32 variants --------------------------------------------------------------------------
template <int kCtrl, int kRowMask = 0xF>
__device__ __forceinline__ float dpp_f32(float old, float src) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src), kCtrl, kRowMask, 0xF, false));
}

// Neither the compiler nor its scheduler moves a memory access across this.  A wait that leaves the n youngest loads in
// flight needs it where the order of those loads matters and they do not depend on each other.
__device__ __forceinline__ void keep_access_order() { asm volatile("" ::: "memory"); }

// Lane i reads lane (i - kN) mod 16 of its row.  Every lane has a source, so the routing can become part of the
// instruction that uses it.
template <int kN>
__device__ __forceinline__ float row_ror(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kDppRowRor + kN, 0xF, 0xF, true));
}

// out[q]: maximum of x[q] over the 32 lanes of each wave half (lanes 0-31 and 32-63 separately), in every lane.  A swap of
// odd and even rows lets two registers share one from the first step on; then rotations inside the rows, 8 registers side
// by side.  In asm: in front of a maximum the compiler quietens each operand anew (16 maxima in 100 instructions, not 450).
// The leading and trailing waits are what lane routing needs next to other vector instructions.
__device__ __forceinline__ void half_max16(const float (&x)[16], float (&out)[16]) {
  float m[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[2 * k]), __float_as_uint(x[2 * k + 1]), false, false);
    asm("v_max_f32 %0, %1, %2" : "=v"(m[k]) : "v"(r[0]), "v"(r[1]));
  }
#define FKV_ROW_MAX(n)                                                    \
  "v_max_f32_dpp %0, %0, %0 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %1, %1, %1 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %2, %2, %2 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %3, %3, %3 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %4, %4, %4 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %5, %5, %5 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %6, %6, %6 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %7, %7, %7 row_ror:" n " row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" FKV_ROW_MAX("8") FKV_ROW_MAX("4") FKV_ROW_MAX("2") FKV_ROW_MAX("1") "s_nop 1"
      : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]), "+v"(m[4]), "+v"(m[5]), "+v"(m[6]), "+v"(m[7]));
#undef FKV_ROW_MAX
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(m[k]), __float_as_uint(m[k]), false, false);
    out[2 * k] = __uint_as_float(r[0]);
    out[2 * k + 1] = __uint_as_float(r[1]);
  }
}

// One of two registers by a lane bit.  (Written as a choice between two elements of an array the compiler makes it a
// lane-dependent index and moves the array to LDS.)
__device__ __forceinline__ float lane_pick(bool second, float x, float y) {
  asm("" : "+v"(x), "+v"(y));
  return second ? y : x;
}
// x[lane % 16].
__device__ __forceinline__ float pick16(const float (&x)[16], int lane) {
  float a[8], b[4];
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = lane_pick((lane & 8) != 0, x[k], x[k + 8]);
#pragma unroll
  for (int k = 0; k < 4; ++k) b[k] = lane_pick((lane & 4) != 0, a[k], a[k + 4]);
  return lane_pick((lane & 1) != 0, lane_pick((lane & 2) != 0, b[0], b[2]), lane_pick((lane & 2) != 0, b[1], b[3]));
}

// Sums of 16 products x[q] * y[q] over each wave half: lane q of each 16-lane row returns the q-th.  The tree of a sum is that
// of rotations by 8, 4, 2 and 1 lanes read at lane q, and a product is rounded only on its way to the lane 8 further on,
// which adds it to its own one in a multiply-add; the sums' last bits depend on both.  After the rotation by 4 the tree
// of lane q needs lanes q - 3 .. q of its row: four sums 4 lanes apart share a register from there on.
__device__ __forceinline__ float half_sums_of_products(const float (&x)[16], const float (&y)[16], int lane) {
  float s[16], c[4];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    s[q] = __builtin_fmaf(x[q], y[q], row_ror<8>(x[q] * y[q]));
    s[q] += row_ror<4>(s[q]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int at = lane + 3 - k;  // bits 2 and 3: which of sums k, k + 4, k + 8, k + 12 this lane belongs to
    c[k] = lane_pick((at & 8) != 0, lane_pick((at & 4) != 0, s[k], s[k + 4]), lane_pick((at & 4) != 0, s[k + 8], s[k + 12]));
    c[k] += row_ror<2>(c[k]);
    c[k] += row_ror<1>(c[k]);
  }
  const unsigned u = __float_as_uint(lane_pick((lane & 2) != 0, lane_pick((lane & 1) != 0, c[0], c[1]), lane_pick((lane & 1) != 0, c[2], c[3])));
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Maximum / sum over the 4 lanes that are 16 apart, in every lane; the sum as (0 + 1) + (2 + 3).
__device__ __forceinline__ float quarters_max(float x) {
  unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  u = __float_as_uint(x);
  r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float quarters_sum(float x) {
  unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  u = __float_as_uint(x);
  r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Maximum / sum over the 64 lanes as a wave-uniform value (fixed order: reproducible).
__device__ __forceinline__ float wave_fmax(float x) {
  x = fmaxf(x, dpp_f32<kDppRowRor + 8>(x, x));
  x = fmaxf(x, dpp_f32<kDppRowRor + 4>(x, x));
  x = fmaxf(x, dpp_f32<kDppRowRor + 2>(x, x));
  x = fmaxf(x, dpp_f32<kDppRowRor + 1>(x, x));
  x = fmaxf(x, dpp_f32<kDppBcast15, 0xA>(x, x));
  x = fmaxf(x, dpp_f32<kDppBcast31, 0xC>(x, x));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ float wave_fsum(float x) {
  x += dpp_f32<kDppRowRor + 8>(0.f, x);
  x += dpp_f32<kDppRowRor + 4>(0.f, x);
  x += dpp_f32<kDppRowRor + 2>(0.f, x);
  x += dpp_f32<kDppRowRor + 1>(0.f, x);
  x += dpp_f32<kDppBcast15, 0xA>(0.f, x);
  x += dpp_f32<kDppBcast31, 0xC>(0.f, x);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

}  // namespace fkv
