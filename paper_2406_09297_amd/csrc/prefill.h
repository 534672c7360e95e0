// Device helpers of the prefill kernels: where a query row stands, direct
// global-to-LDS loads, output stores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "tile.h"

namespace mlkv {

// Wait until this wave's vector memory loads, the direct loads included,
// have landed (vmcnt(0); the other counters are left alone).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8)); }

// 16 bytes of every lane from base + off (base wave-uniform) to LDS at the
// wave-uniform dst + 16 lane.
// (The host pass knows neither the builtin's size 16 nor LDS pointers, and a
// template that names them cannot be instantiated twice there.)
__device__ __forceinline__ void load_lds16(const char* base, unsigned off, uint16_t* dst) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_global_load_lds(static_cast<const void*>(base + off),
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
#endif
}

// Query row rho of unit (b, r): its token and its place in q and out
// (elements); rows past the end are not valid and stand at token 0.
struct RowPlace {
  size_t offset;
  int tok;
  bool valid;
};
__device__ __forceinline__ RowPlace row_place(const PrefillParams& p, int rho, int rows, int b,
                                              int group, int r, int D) {
  RowPlace at;
  const int R = p.layers * p.G;
  at.valid = rho < rows;
  at.tok = at.valid ? rho / R : 0;
  const int c = at.valid ? rho - at.tok * R : 0;
  const int layer = c / p.G;
  const int head = (r - group * p.kv_per_layer) * p.G + c - layer * p.G;
  at.offset = (((static_cast<size_t>(group * p.layers + layer) * p.B + b) * p.T + at.tok) * p.h +
               head) * D;
  return at;
}

// Four channels at element `off` of the output, fp32 or bf16.
__device__ __forceinline__ void store4(const PrefillParams& p, size_t off, f32x4 o) {
  if (p.out_bf16) {
    const uint32_t lo = f32_to_bf16_bits(o[0]) | (static_cast<uint32_t>(f32_to_bf16_bits(o[1])) << 16);
    const uint32_t hi = f32_to_bf16_bits(o[2]) | (static_cast<uint32_t>(f32_to_bf16_bits(o[3])) << 16);
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + off) = make_uint2(lo, hi);
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + off) = o;
  }
}

}  // namespace mlkv
