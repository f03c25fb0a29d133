// Device helpers shared by the FP6 GEMM kernels (the layout is described in
// qgemm_fp6.hip): direct loads, the MFMA step and the dequantization epilogue.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

namespace dptq {
namespace f6 {

typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef float v16f_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) uint8_t* lds_ptr_t;

constexpr int kF6Block = 3072;   // bytes of one 32-row x 128-k block

// Wavefront-wide direct load of 1 KiB (16 bytes per lane) from sbase + voff
// into LDS at lds_off + 16 * lane.
__device__ __forceinline__ void f6_dma16(const void* sbase, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_off)
               : "memory", "m0");
}
__device__ __forceinline__ int f6_xcd_remap(int bid, int total) {
  const int per = total >> 3, rem = total & 7;
  const int x = bid & 7, idx = bid >> 3;
  return x * per + (x < rem ? x : rem) + idx;
}

// One MFMA step: fp6 x fp6, E8M0 scale 128 (= 2) on both operands.
__device__ __forceinline__ v16f_t mfma_f6(const uint32_t* w, const uint32_t* a, v16f_t c) {
  const v8i_t wa = {(int)w[0], (int)w[1], (int)w[2], (int)w[3], (int)w[4], (int)w[5], 0, 0};
  const v8i_t ab = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)a[4], (int)a[5], 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wa, ab, c, 2, 2, 0, 128, 0, 128);
}

// fl16(fl32(fl32(acc) * as) * ws); acc is an exact integer held in fp32.  The
// empty asm keeps the second product an fp32 value (see the int8 kernels).
__device__ __forceinline__ __half f6_dequant(float acc, float as, float ws) {
  const float t1 = acc * as;
  float t2 = t1 * ws;
  asm("" : "+v"(t2));
  return __float2half_rn(t2);
}

__device__ __forceinline__ uint2 f6_dequant4(float a0, float a1, float a2, float a3, float as,
                                             float4 ws) {
  const __half h0 = f6_dequant(a0, as, ws.x), h1 = f6_dequant(a1, as, ws.y);
  const __half h2 = f6_dequant(a2, as, ws.z), h3 = f6_dequant(a3, as, ws.w);
  uint2 pk;
  pk.x = (uint32_t)__half_as_ushort(h0) | ((uint32_t)__half_as_ushort(h1) << 16);
  pk.y = (uint32_t)__half_as_ushort(h2) | ((uint32_t)__half_as_ushort(h3) << 16);
  return pk;
}

}  // namespace f6
}  // namespace dptq
