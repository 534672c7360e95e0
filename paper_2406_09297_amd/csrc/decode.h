// Device helpers shared by the two decode attention kernels (kernels.hip: one
// layer; step.hip: every layer of a step): the rotary rotation of the newest
// token's vectors, the normalisation and the output stores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tile.h"

namespace mlkv {

__device__ __forceinline__ uint16_t f64_to_bf16_bits(double v) {
  // Round to odd into fp32 (24 bits: no double rounding), then to nearest
  // even into bf16.
  const float f = __double2float_rz(v);
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  if (static_cast<double>(f) != v && v == v) u |= 1u;
  return f32_to_bf16_bits(__builtin_bit_cast(float, u));
}

__device__ __forceinline__ double bf16_to_f64(uint16_t x) {
  return __builtin_bit_cast(float, static_cast<uint32_t>(x) << 16);
}

// y = own cos -/+ partner sin with both products and the sum rounded.
template <bool HI>
__device__ __forceinline__ double rotate_one(double own, double partner, double c, double s) {
#pragma clang fp contract(off)
  return HI ? own * c + partner * s : own * c - partner * s;
}

// The rotated chunk of channels c0 .. c0+7 (c0 a multiple of 8): `own` holds
// them, `partner` channels c0 + half (c0 < half) or c0 - half (half <= c0 <
// 2*half); cs = the table entries (cos, sin) of pairs c0 % half ... Chunks at
// or past 2*half are returned unchanged.
template <typename CS>
__device__ __forceinline__ u16x8 rotate_chunk(u16x8 own, u16x8 partner, int c0, int half, CS cs) {
  if (c0 >= 2 * half) return own;
  const bool hi = c0 >= half;
  const int j0 = hi ? c0 - half : c0;
  u16x8 y;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double2 t = cs(j0 + e);
    const double u = bf16_to_f64(own[e]), w = bf16_to_f64(partner[e]);
    y[e] = f64_to_bf16_bits(hi ? rotate_one<true>(u, w, t.x, t.y) : rotate_one<false>(u, w, t.x, t.y));
  }
  return y;
}

// Offset of the channel chunk paired with chunk c0 (see rotate_chunk).
__device__ __forceinline__ int partner_chunk(int c0, int half) {
  return c0 < half ? c0 + half : c0 - half;
}

// What partial results of a row are weighed against: their largest maximum M.
// Where it is -inf no part has a score above that: against 0 an empty part
// counts nothing (2^-inf = 0, times sums of 0), and the non-finite sums of a
// part whose scores were NaN or -inf stay non-finite (0 * NaN).
__device__ __forceinline__ float merge_reference(float M) { return M == -INFINITY ? 0.f : M; }

// acc / den with one reciprocal (within one ulp) for the four channels; zeros
// for an empty row (den = 0).  A row with any attended position has den >= 1
// (its largest weight is at least one), and den = 1 leaves acc exact;
// non-finite inputs give a non-finite den, which propagates as in the
// definition rather than being taken for an empty row.
__device__ __forceinline__ f32x4 normalize4(f32x4 acc, float den) {
  return den != 0.f ? acc * __builtin_amdgcn_rcpf(den) : f32x4{0.f, 0.f, 0.f, 0.f};
}

// Four consecutive channels d..d+3 of output row `row` (d a multiple of 4),
// fp32 or bf16.
template <int D>
__device__ __forceinline__ void store4_as(void* out, int out_bf16, size_t row, int d, f32x4 v) {
  if (out_bf16) {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    const u16x4 bits = {f32_to_bf16_bits(v[0]), f32_to_bf16_bits(v[1]), f32_to_bf16_bits(v[2]),
                        f32_to_bf16_bits(v[3])};
    *reinterpret_cast<u16x4*>(static_cast<uint16_t*>(out) + row * D + d) = bits;
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(out) + row * D + d) = v;
  }
}

}  // namespace mlkv
