// W4A4 / W4A8 GEMM for at most 16 tokens (gfx950) that streams the weights
// straight into registers: the kernel for the decode shapes where the K-split
// kernel's way through LDS costs more than it gives.  Same product and epilogue,
// same bits.
//
// One workgroup per NB blocks of 16 output channels; its 8 wavefronts split K,
// stream the weight rows once with 16-byte loads, and the int32 partial tiles
// are summed exactly in LDS.  Every workgroup reads all M activation rows of its
// K range, so when those rows are as many bytes as its weights two blocks share
// them (NB = 2).
//
// What bounds it is latency, one batch of chunks after the other, where K is
// short, and the rate of the loads where it is long: in the decode layout a load
// instruction covers one contiguous KiB, which suits registers as well as LDS,
// while with canonical rows it touches 16 lines (gemm_rules.h has the line
// between the two kernels and both sides' times).

#include "internal.h"
#include "qgemm_device.h"

namespace dptq {
namespace {

using namespace qg;

constexpr int kDecWaves = 8;
constexpr int kDecBatch = 4;

// ZP: the range quantizer's zero-point correction in the epilogue,
// acc + (2^(BITS-1) - a_zeros[m]) * w_sums[n] (exact int32), before the
// dequantization.  WDEC: weights in the decode layout, where the 16 rows x 64
// bytes of a block's 128-k chunk are one contiguous KiB in lane order.
// BATCH: chunks per wavefront in flight.
template <int BITS, bool ACC_OUT, bool ZP = false, bool WA8 = false, int NB = 1, bool WDEC = false,
          int BATCH = kDecBatch>
__global__ void __launch_bounds__(kDecWaves * 64)
qgemm_decode(const uint8_t* __restrict__ a_codes, const float* __restrict__ a_scales,
             const uint8_t* __restrict__ w_packed, const float* __restrict__ w_scales,
             int M, int N, int K, __half* __restrict__ y, int32_t* __restrict__ acc_out,
             const int32_t* __restrict__ a_zeros = nullptr,
             const int32_t* __restrict__ w_sums = nullptr) {
  static_assert(NB == 1 || NB == 2, "blocks per workgroup");
  __shared__ v4i part[NB][kDecWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = blockIdx.x * 16 * NB;
  const int fr = lane & 15, fg = lane >> 4;
  const int nck = K / 128;
  const int c_begin = (int)((long)nck * wave / kDecWaves);
  const int c_end = (int)((long)nck * (wave + 1) / kDecWaves);
  const bool mvalid = fr < M;

  const size_t wrow = (size_t)K / 2;
  // Chunk ck of weight block nb (16 rows) at wp + nb * 16 * wrow + ck * kChunk.
  constexpr size_t kChunk = WDEC ? 1024 : 64;
  const uint8_t* wp = WDEC ? w_packed + (size_t)n0 * wrow + lane * 16
                           : w_packed + (size_t)(n0 + fr) * wrow + fg * 16;
  const size_t arow = BITS == 4 ? (size_t)K / 2 : (size_t)K;
  const uint8_t* ap = a_codes + (size_t)(mvalid ? fr : 0) * arow + (BITS == 4 ? fg * 16 : fg * 32);

  v4i acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = v4i{0, 0, 0, 0};
  for (int c = c_begin; c < c_end; c += BATCH) {
    uint4 wv[NB][BATCH], av[BATCH], av2[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int ck = c + b;
      const bool ok = ck < c_end;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        wv[nb][b] = ok ? *reinterpret_cast<const uint4*>(wp + (size_t)nb * 16 * wrow + (size_t)ck * kChunk)
                       : make_uint4(0, 0, 0, 0);
      if (BITS == 4) {
        av[b] = (ok && mvalid) ? *reinterpret_cast<const uint4*>(ap + (size_t)ck * 64)
                               : make_uint4(0, 0, 0, 0);
      } else {
        av[b] = (ok && mvalid) ? *reinterpret_cast<const uint4*>(ap + (size_t)ck * 128)
                               : make_uint4(0, 0, 0, 0);
        av2[b] = (ok && mvalid) ? *reinterpret_cast<const uint4*>(ap + (size_t)ck * 128 + 16)
                                : make_uint4(0, 0, 0, 0);
      }
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      v4i b0, b1;
      if (BITS == 4) {
        b0 = op_from_nibbles(av[b].x, av[b].y);
        b1 = op_from_nibbles(av[b].z, av[b].w);
      } else {
        b0 = op_a8<WA8>(av[b].x, av[b].y, av[b].z, av[b].w);
        b1 = op_a8<WA8>(av2[b].x, av2[b].y, av2[b].z, av2[b].w);
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        acc[nb] = mfma(op_from_nibbles(wv[nb][b].x, wv[nb][b].y), b0, acc[nb]);
        acc[nb] = mfma(op_from_nibbles(wv[nb][b].z, wv[nb][b].w), b1, acc[nb]);
      }
    }
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) part[nb][wave][lane] = acc[nb];
  __syncthreads();
  // Wavefront nb < NB sums and writes block nb.
  if (wave >= NB) return;
  v4i tot = part[wave][0][lane];
#pragma unroll
  for (int w = 1; w < kDecWaves; ++w) {
    const v4i p = part[wave][w][lane];
    tot.x += p.x; tot.y += p.y; tot.z += p.z; tot.w += p.w;
  }
  if (!mvalid) return;
  const int m = fr, n = n0 + wave * 16 + fg * 4;
  int c0 = unscale<BITS>(tot.x), c1 = unscale<BITS>(tot.y);
  int c2 = unscale<BITS>(tot.z), c3 = unscale<BITS>(tot.w);
  if constexpr (ZP) {
    const int off = (1 << (BITS - 1)) - a_zeros[m];
    const int4 ws = *reinterpret_cast<const int4*>(w_sums + n);
    c0 += off * ws.x;
    c1 += off * ws.y;
    c2 += off * ws.z;
    c3 += off * ws.w;
  }
  if (ACC_OUT) {
    *reinterpret_cast<int4*>(acc_out + (size_t)m * N + n) = make_int4(c0, c1, c2, c3);
  } else {
    const float as = a_scales[m];
    const float4 wsv = *reinterpret_cast<const float4*>(w_scales + n);
    const __half h0 = dequant(c0, as, wsv.x), h1 = dequant(c1, as, wsv.y);
    const __half h2 = dequant(c2, as, wsv.z), h3 = dequant(c3, as, wsv.w);
    uint2 pk;
    pk.x = (uint32_t)__half_as_ushort(h0) | ((uint32_t)__half_as_ushort(h1) << 16);
    pk.y = (uint32_t)__half_as_ushort(h2) | ((uint32_t)__half_as_ushort(h3) << 16);
    *reinterpret_cast<uint2*>(y + (size_t)m * N + n) = pk;
  }
}

template <int BITS, bool ACC_OUT, bool ZP, bool WA8, bool WDEC, int NB, int BATCH>
void launch_t(const KsplitCall& c, hipStream_t stream) {
  hipLaunchKernelGGL((qgemm_decode<BITS, ACC_OUT, ZP, WA8, NB, WDEC, BATCH>), dim3((unsigned)(c.N / (16 * NB))),
                     dim3(kDecWaves * 64), 0, stream, c.a, c.a_scales, c.w, c.w_scales, (int)c.M, (int)c.N, c.K,
                     c.y, c.acc, c.a_zeros, c.w_sums);
}

template <int BITS, bool ACC_OUT, bool ZP, bool WA8, bool WDEC>
void launch(const KsplitCall& c, hipStream_t stream) {
  const int blocks = rules::decode_blocks(c.M, c.N, BITS, c.cus);
  if (blocks == 2)
    launch_t<BITS, ACC_OUT, ZP, WA8, WDEC, 2, kDecBatch>(c, stream);
  else if (WDEC && rules::decode_batch(c.M, c.N, c.K, blocks, c.cus) == 8)
    launch_t<BITS, ACC_OUT, ZP, WA8, WDEC, 1, WDEC ? 8 : kDecBatch>(c, stream);
  else
    launch_t<BITS, ACC_OUT, ZP, WA8, WDEC, 1, kDecBatch>(c, stream);
}

}  // namespace

hipError_t launch_decode_regs(const KsplitCall& c, int bits, int weights, hipStream_t stream) {
  const bool acc = c.acc != nullptr, zp = c.a_zeros != nullptr;
  if (weights == kWeightsDecode) {
    if (bits == 4) acc ? launch<4, true, false, false, true>(c, stream) : launch<4, false, false, false, true>(c, stream);
    else acc ? launch<8, true, false, false, true>(c, stream) : launch<8, false, false, false, true>(c, stream);
  } else if (weights == kWeightsA8Order) {
    launch<8, false, false, true, false>(c, stream);
  } else if (bits == 4) {
    if (acc) launch<4, true, false, false, false>(c, stream);
    else if (zp) launch<4, false, true, false, false>(c, stream);
    else launch<4, false, false, false, false>(c, stream);
  } else {
    if (acc) launch<8, true, false, false, false>(c, stream);
    else if (zp) launch<8, false, true, false, false>(c, stream);
    else launch<8, false, false, false, false>(c, stream);
  }
  return hipGetLastError();
}

}  // namespace dptq
