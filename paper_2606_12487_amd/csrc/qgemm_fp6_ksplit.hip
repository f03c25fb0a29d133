// W4A4 GEMM on the FP6 matrix cores for medium batches (gfx950): shapes whose
// 192 x 256 output tiles would leave most compute units idle.  Same product,
// operand layout, epilogue and bits as qgemm_fp6.hip.
//
// One workgroup computes an output tile of 32 TI (n) x 32 TJ (m) and its
// wavefronts split K between them, each streaming its own blocks through a
// piece of LDS of its own (no barrier in the k loop).  The partial tiles are
// exact integers below 2^24 held in fp32, so their sum, taken through LDS at
// the end, is exact in any order.
//
// What bounds it: latency below about 10 us (the first stages come from
// memory), above that the rate at which a compute unit pulls lines from its
// L2: about 45 bytes a clock in the k loop, 26 over a whole launch of long rows
// with the weights from memory.  So the tile is chosen for as few bytes a
// compute unit as fill the chip once: M = 500, N = 4096, K = 4096 on 2 x 4
// blocks (256 workgroups) 22.2 -> 11.6 us against the 192 x 256 kernel on its
// 44; M = 333, N = 4096, K = 14336 63.8 -> 23.4 us; M = 64, N = 2048,
// K = 14336 80.4 -> 9.9 us.  Where that kernel has tiles for most compute
// units it is the faster (M = 1536, N = 4096, K = 4096: 25.2 against 28.1 us).

#include "fp6_device.h"
#include "internal.h"

namespace dptq {
namespace {

using namespace f6;

// Four scales from a pointer that is 4-byte aligned, as the entry point takes it.
typedef float v4f_dw __attribute__((ext_vector_type(4), aligned(4)));

// Waits that no memory access moves across.
template <int N>
__device__ __forceinline__ void wait_vmcnt_fence() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" : : "i"(N) : "memory");
}
__device__ __forceinline__ void wait_lgkm0_fence() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// A stage is 128 k of the tile: TI weight and TJ activation blocks; each
// wavefront has BUFS stages of its own.
template <int TI, int TJ, int WAVES, int BUFS, bool ACC_OUT>
__global__ void __launch_bounds__(WAVES * 64)
qgemm_fp6_ksplit(const uint8_t* __restrict__ a6, const float* __restrict__ a_scales,
                 const uint8_t* __restrict__ w6, const float* __restrict__ w_scales, int M, int N,
                 int K, __half* __restrict__ y, int32_t* __restrict__ acc_out) {
  constexpr int kLoads = 3 * (TI + TJ);                 // 1 KiB each, per stage
  constexpr int kStage = kLoads * 1024;
  constexpr int kRing = WAVES * BUFS * kStage;
  constexpr int kFrags = TI * TJ;
  constexpr int kFragPart = WAVES * 4096;               // the partial tiles of one 32 x 32 block
  constexpr int kLds = kRing > kFragPart ? kRing : kFragPart;
  constexpr int kPass = kLds / kFragPart < kFrags ? kLds / kFragPart : kFrags;   // blocks summed at a time
  static_assert(kLds <= 160 * 1024, "LDS budget");
  static_assert((BUFS - 1) * kLoads < 64, "loads in flight fit the wait count");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kLds];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  const int mblk = (M + 31) / 32, nblk = (N + 31) / 32;
  const int tiles_m = (mblk + TJ - 1) / TJ;
  const int logical = f6_xcd_remap(blockIdx.x, gridDim.x);
  const int tn = logical / tiles_m, tm = logical - tn * tiles_m;
  const int nkb = K / 128;
  const int s_begin = (int)((long)nkb * wave / WAVES);
  const int s_end = (int)((long)nkb * (wave + 1) / WAVES);

  // Per-lane offsets of the tile's blocks within one k block.  Blocks past
  // the matrix repeat its last one (their products are never stored).
  uint32_t wofs[TI], aofs[TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i) wofs[i] = (uint32_t)min(tn * TI + i, nblk - 1) * kF6Block + lane * 16;
#pragma unroll
  for (int j = 0; j < TJ; ++j) aofs[j] = (uint32_t)min(tm * TJ + j, mblk - 1) * kF6Block + lane * 16;
  const size_t wstride = (size_t)nblk * kF6Block, astride = (size_t)mblk * kF6Block;

  uint8_t* ring = smem + wave * (BUFS * kStage);
  const uint32_t base = (uint32_t)(uintptr_t)(lds_ptr_t)ring;
  auto load = [&](int s, int buf) __attribute__((always_inline)) {
    const uint8_t* wk = w6 + (size_t)s * wstride;
    const uint8_t* ak = a6 + (size_t)s * astride;
    const uint32_t b = base + buf * kStage;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) f6_dma16(wk, wofs[i] + c * 1024, b + (3 * i + c) * 1024);
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int c = 0; c < 3; ++c) f6_dma16(ak, aofs[j] + c * 1024, b + (3 * (TI + j) + c) * 1024);
  };
  struct Frag {
    uint32_t w[2][TI][6], a[2][TJ][6];
  };
  auto read_op = [&](const uint8_t* p, uint32_t* d) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint2 v = *reinterpret_cast<const uint2*>(p + 512 * c + lane * 8);
      d[2 * c] = v.x;
      d[2 * c + 1] = v.y;
    }
  };
  v16f_t acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = v16f_t{};

#pragma unroll
  for (int b = 0; b < BUFS; ++b)
    if (s_begin + b < s_end) load(s_begin + b, b);
  int buf = 0;
  for (int s = s_begin; s < s_end; ++s) {
    // Stage s has landed once only the BUFS - 1 stages after it are in flight.
    if (s + BUFS - 1 < s_end) wait_vmcnt_fence<(BUFS - 1) * kLoads>();
    else wait_vmcnt_fence<0>();
    const uint8_t* st = ring + buf * kStage;
    Frag f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < TI; ++i) read_op(st + i * kF6Block + h * 1536, f.w[h][i]);
#pragma unroll
      for (int j = 0; j < TJ; ++j) read_op(st + (TI + j) * kF6Block + h * 1536, f.a[h][j]);
    }
    wait_lgkm0_fence();   // the stage is refilled after its reads have returned
    if (s + BUFS < s_end) load(s + BUFS, buf);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = mfma_f6(f.w[h][i], f.a[h][j], acc[i][j]);
    buf = buf + 1 == BUFS ? 0 : buf + 1;
  }

  // Sum the partial tiles, kPass blocks at a time.  A unit of the sum is half
  // p of a block: registers 8 p .. 8 p + 7, i.e. two groups of four
  // consecutive n (16 p + 4 g and 16 p + 8 + 4 g, g = lane >> 5) of column
  // m = lane & 31, joined across the half-wavefronts into 16-byte stores.
  float4 (*part)[WAVES][4][64] = reinterpret_cast<float4 (*)[WAVES][4][64]>(smem);
  const int fr = lane & 31, fg = lane >> 5;
#pragma unroll
  for (int f0 = 0; f0 < kFrags; f0 += kPass) {
    __syncthreads();   // every wavefront is done with the ring, or with the last pass
#pragma unroll
    for (int g = 0; g < kPass; ++g) {
      if (f0 + g >= kFrags) continue;
      const v16f_t& c = acc[(f0 + g) / TJ][(f0 + g) % TJ];
#pragma unroll
      for (int b = 0; b < 4; ++b)
        part[g][wave][b][lane] = make_float4(c[4 * b], c[4 * b + 1], c[4 * b + 2], c[4 * b + 3]);
    }
    __syncthreads();
    const int units = 2 * min(kPass, kFrags - f0);
    for (int u = wave; u < units; u += WAVES) {
      const int g = u >> 1, p = u & 1;
      float4 t0 = part[g][0][2 * p][lane], t1 = part[g][0][2 * p + 1][lane];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) {
        const float4 p0 = part[g][w][2 * p][lane], p1 = part[g][w][2 * p + 1][lane];
        t0.x += p0.x; t0.y += p0.y; t0.z += p0.z; t0.w += p0.w;
        t1.x += p1.x; t1.y += p1.y; t1.z += p1.z; t1.w += p1.w;
      }
      const int f = f0 + g, i = f / TJ, j = f - i * TJ;
      const int m = (tm * TJ + j) * 32 + fr, nb = (tn * TI + i) * 32 + 16 * p;
      if (nb >= N) continue;   // whole units: N is a multiple of 16
      if constexpr (ACC_OUT) {
        if (m >= M) continue;
        int32_t* o = acc_out + (size_t)m * N + nb + 4 * fg;
        *reinterpret_cast<int4*>(o) = make_int4((int)t0.x, (int)t0.y, (int)t0.z, (int)t0.w);
        *reinterpret_cast<int4*>(o + 8) = make_int4((int)t1.x, (int)t1.y, (int)t1.z, (int)t1.w);
      } else {
        const float as = a_scales[min(m, M - 1)];
        const v4f_dw v0 = *reinterpret_cast<const v4f_dw*>(w_scales + nb + 4 * fg);
        const v4f_dw v1 = *reinterpret_cast<const v4f_dw*>(w_scales + nb + 8 + 4 * fg);
        const float4 ws0 = make_float4(v0.x, v0.y, v0.z, v0.w), ws1 = make_float4(v1.x, v1.y, v1.z, v1.w);
        const uint2 x0 = f6_dequant4(t0.x, t0.y, t0.z, t0.w, as, ws0);
        const uint2 x1 = f6_dequant4(t1.x, t1.y, t1.z, t1.w, as, ws1);
        const auto s0 = __builtin_amdgcn_permlane32_swap(x0.x, x1.x, false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(x0.y, x1.y, false, false);
        if (m < M)
          *reinterpret_cast<uint4*>(y + (size_t)m * N + nb + 8 * fg) =
              make_uint4(s0[0], s1[0], s0[1], s1[1]);
      }
    }
  }
}

template <bool ACC_OUT, int I = 0>
void launch_tile(int tile, const uint8_t* a6, const float* a_scales, int64_t M, int K, const uint8_t* w6,
                 const float* w_scales, int64_t N, __half* y, int32_t* acc, hipStream_t stream) {
  if constexpr (I < rules::kNumFp6KsplitTiles) {
    if (tile != I) {
      launch_tile<ACC_OUT, I + 1>(tile, a6, a_scales, M, K, w6, w_scales, N, y, acc, stream);
      return;
    }
    constexpr rules::Fp6KsplitTile t = rules::kFp6KsplitTiles[I];
    const int64_t mblk = (M + 31) / 32, nblk = (N + 31) / 32;
    const int64_t grid = ((mblk + t.tj - 1) / t.tj) * ((nblk + t.ti - 1) / t.ti);
    hipLaunchKernelGGL((qgemm_fp6_ksplit<t.ti, t.tj, t.waves, t.bufs, ACC_OUT>), dim3((unsigned)grid),
                       dim3(t.waves * 64), 0, stream, a6, a_scales, w6, w_scales, (int)M, (int)N, K, y, acc);
  }
}

}  // namespace

hipError_t launch_fp6_ksplit(int tile, const uint8_t* a6, const float* a_scales, int64_t M, int K,
                             const uint8_t* w6, const float* w_scales, int64_t N, void* y, int32_t* acc,
                             hipStream_t stream) {
  __half* yh = static_cast<__half*>(y);
  if (acc) launch_tile<true>(tile, a6, a_scales, M, K, w6, w_scales, N, yh, acc, stream);
  else launch_tile<false>(tile, a6, a_scales, M, K, w6, w_scales, N, yh, nullptr, stream);
  return hipGetLastError();
}

}  // namespace dptq
