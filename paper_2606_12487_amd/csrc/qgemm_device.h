// Device helpers shared by the int8-MFMA GEMM kernels: MFMA operands from packed
// codes, the dequantization epilogue, and the workgroup-to-XCD mapping.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

namespace dptq {
namespace qg {

typedef int v4i __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t nib_lo(uint32_t v) { return (v << 4) & 0xF0F0F0F0u; }
__device__ __forceinline__ uint32_t nib_hi(uint32_t v) { return v & 0xF0F0F0F0u; }

// Even-k bytes of an 8-byte run (d0 = k0..3, d1 = k4..7): [k0, k2, k4, k6].
__device__ __forceinline__ uint32_t even_bytes(uint32_t d0, uint32_t d1) {
  return __builtin_amdgcn_perm(d1, d0, 0x06040200u);
}
// Odd-k bytes: [k1, k3, k5, k7].
__device__ __forceinline__ uint32_t odd_bytes(uint32_t d0, uint32_t d1) {
  return __builtin_amdgcn_perm(d1, d0, 0x07050301u);
}

// MFMA operand for one 64-k step from two packed 4-bit dwords (k 0..7, 8..15
// of this lane's 16-k slice).
__device__ __forceinline__ v4i op_from_nibbles(uint32_t v0, uint32_t v1) {
  v4i r;
  r.x = (int)nib_lo(v0);
  r.y = (int)nib_hi(v0);
  r.z = (int)nib_lo(v1);
  r.w = (int)nib_hi(v1);
  return r;
}
// Same k order from 16 int8 codes d0..d3 (k 0..15).
__device__ __forceinline__ v4i op_from_bytes(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3) {
  v4i r;
  r.x = (int)even_bytes(d0, d1);
  r.y = (int)odd_bytes(d0, d1);
  r.z = (int)even_bytes(d2, d3);
  r.w = (int)odd_bytes(d2, d3);
  return r;
}

// 8-bit activation operand of one 32-k step.  Against weights in the
// canonical nibble order the activation bytes are regrouped like the nibble
// unpack (even k, then odd k).  Weights in the 8-bit order (each dword holds
// k0..k3 in its low nibbles and k4..k7 in its high ones, pack_w4_a8_kernel)
// unpack to natural k order, so the activation dwords are the operand as
// they stand.
template <bool WA8>
__device__ __forceinline__ v4i op_a8(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3) {
  if constexpr (WA8) {
    v4i r;
    r.x = (int)d0;
    r.y = (int)d1;
    r.z = (int)d2;
    r.w = (int)d3;
    return r;
  } else {
    return op_from_bytes(d0, d1, d2, d3);
  }
}

__device__ __forceinline__ v4i mfma(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

template <int BITS>
__device__ __forceinline__ int unscale(int v) { return BITS == 4 ? (v >> 8) : (v >> 4); }

// fl16(fl32(fl32(fl32(acc) * as) * ws)).  The empty asm pins t2 as an fp32
// value: without it the backend folds the last multiply and the fp16
// conversion into one mixed-precision FMA (a single rounding to fp16), which
// differs from the two roundings the epilogue is defined with.
__device__ __forceinline__ __half dequant(int acc, float as, float ws) {
  const float t0 = (float)acc;
  const float t1 = t0 * as;
  float t2 = t1 * ws;
  asm("" : "+v"(t2));
  return __float2half_rn(t2);
}

// Four accumulators of one lane (rows n .. n+3 of one column m), unscaled,
// with the zero-point correction off * wz when ZP, dequantized and packed as
// fp16.
template <int BITS, bool ZP>
__device__ __forceinline__ uint2 dequant4z(int a0, int a1, int a2, int a3, float as, float4 ws,
                                           int off, int4 wz) {
  int c0 = unscale<BITS>(a0), c1 = unscale<BITS>(a1), c2 = unscale<BITS>(a2), c3 = unscale<BITS>(a3);
  if constexpr (ZP) {
    c0 += off * wz.x;
    c1 += off * wz.y;
    c2 += off * wz.z;
    c3 += off * wz.w;
  }
  const __half h0 = dequant(c0, as, ws.x), h1 = dequant(c1, as, ws.y);
  const __half h2 = dequant(c2, as, ws.z), h3 = dequant(c3, as, ws.w);
  uint2 pk;
  pk.x = (uint32_t)__half_as_ushort(h0) | ((uint32_t)__half_as_ushort(h1) << 16);
  pk.y = (uint32_t)__half_as_ushort(h2) | ((uint32_t)__half_as_ushort(h3) << 16);
  return pk;
}

// Logical tile of workgroup bid: the workgroups of one XCD (bid mod 8) take
// consecutive logical tiles.
__device__ __forceinline__ int xcd_remap(int bid, int total) {
  const int per = total >> 3, rem = total & 7;
  const int x = bid & 7, idx = bid >> 3;
  return x * per + (x < rem ? x : rem) + idx;
}

}  // namespace qg
}  // namespace dptq
