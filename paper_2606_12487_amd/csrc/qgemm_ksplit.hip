// W4A4 / W4A8 GEMM for few tokens (gfx950): every decode batch (M <= 16), and
// larger batches up to several hundred tokens whose 256 x 128 or 192 x 256
// output tiles would leave most compute units idle.  Same product and epilogue
// as the tile kernels, same bits.
//
// One workgroup computes a small output tile of 16 TI (n) x 16 TJ (m) and its
// wavefronts split K between them.  Each wavefront streams its own k range of
// the tile's weight and activation rows through a piece of LDS of its own
// (no barrier in the k loop, since no two wavefronts read the same bytes),
// feeds 16 x 16 x 64 int8 MFMAs, and the exact int32 partial tiles are summed
// in LDS at the end.
//
// What bounds it is the rate at which a compute unit pulls lines from its L2,
// so the loads are shaped for that.  Loading MFMA fragments straight into
// registers puts consecutive lanes in different rows: measured 16 bytes per
// clock and compute unit.  A direct global->LDS load whose consecutive lanes
// cover 64 bytes of a row reached about 29, and whole 128-byte lines (256 k of
// a 4-bit row at a time; half lines are fetched twice) about 40 to 50.
// M = 128, K = 14336, N = 4096 at 8 bits (32 x 64 tiles, 256 workgroups):
// 27.5 us, 17.0 us and 13.8 us for the three, against 75 us for the 256 x 128
// tile kernel on its 16 workgroups.

#include <type_traits>

#include "internal.h"
#include "qgemm_device.h"

namespace dptq {
namespace {

using namespace qg;

typedef __attribute__((address_space(3))) uint8_t* lds_ptr;

// Wavefront-wide direct load of 1 KiB (16 bytes per lane) from sbase + voff
// into LDS at lds_off + 16 * lane.
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_off)
               : "memory", "m0");
}
// Waits that no memory access moves across.
__device__ __forceinline__ void wait_vmcnt0_fence() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wait_lgkm0_fence() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// 16-byte-piece swizzles of 128-byte LDS rows r = 0..15: physical piece p
// holds logical piece p ^ s(r).  A 16-byte LDS read is served 16 lanes at a
// time, {0-3, 12-15, 20-23, 24-27} and so on, from 64 banks; these spread each
// such group of fragment reads over all of them.  In 4-bit rows lane l reads
// piece 4 h + (l >> 4) of row l & 15, in 8-bit rows piece 2 (l >> 4) + h.
__device__ __forceinline__ int swz_nib(int r) { return 2 * ((r >> 1) & 1) + 4 * (r >> 3); }
__device__ __forceinline__ int swz_byte(int r) { return 2 * ((-(r >> 2)) & 3) + ((r >> 1) & 1); }

// TI x TJ blocks of 16 x 16 per workgroup on WAVES wavefronts.  WA8: weights in
// the 8-bit activation order; WDEC: weights in the decode layout; ZP: the range
// quantizer's zero-point correction acc + (2^(BITS-1) - a_zeros[m]) * w_sums[n].
//
// A wavefront has one stage (256 k) in flight: 16 KiB for 4 x 4 blocks at 4
// bits, so the eight or more wavefronts of a compute unit keep 64 to 144 KiB
// on the way, as much as its LDS holds; two or more smaller stages each were
// no faster (M = 20, K = 14336, N = 4096 at 4 bits: 7.0 us with one, 7.8 us
// with two).
template <int BITS, int TI, int TJ, int WAVES, bool ACC_OUT, bool WA8, bool ZP, bool WDEC>
__global__ void __launch_bounds__(WAVES * 64)
qgemm_ksplit(const uint8_t* __restrict__ a_codes, const float* __restrict__ a_scales,
             const uint8_t* __restrict__ w_packed, const float* __restrict__ w_scales, int M, int N,
             int K, __half* __restrict__ y, int32_t* __restrict__ acc_out,
             const int32_t* __restrict__ a_zeros, const int32_t* __restrict__ w_sums) {
  constexpr int kAB = BITS == 4 ? 2 : 4;         // KiB of an activation block per stage
  constexpr int kLoads = 2 * TI + kAB * TJ;      // 1 KiB each, per stage
  constexpr int kStage = kLoads * 1024;
  constexpr int kRing = WAVES * kStage, kPart = WAVES * WAVES * 1024;
  constexpr int kFrags = TI * TJ;
  static_assert(kRing <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kRing > kPart ? kRing : kPart];
  v4i (*part)[WAVES][64] = reinterpret_cast<v4i (*)[WAVES][64]>(smem);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;

  const int tiles_m = (M + 16 * TJ - 1) / (16 * TJ);
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int tn = logical / tiles_m, tm = logical - tn * tiles_m;
  const int m0 = tm * 16 * TJ, n0 = tn * 16 * TI;

  // Stages of 256 k (a whole 128-byte line of a 4-bit row), the last one of K
  // % 256 == 128 holding 128.
  const int nst = (K + 255) / 256;
  const int s_begin = (int)((long)nst * wave / WAVES);
  const int s_end = (int)((long)nst * (wave + 1) / WAVES);
  const int half_stage = (K & 128) ? nst - 1 : nst;   // the stage without a second half

  // Loads: one direct global->LDS instruction moves 1 KiB, 8 rows x 128 bytes,
  // consecutive lanes covering a row's bytes (a load whose consecutive lanes
  // lie in different rows runs at a fraction of the rate).  Lane l fills
  // physical piece l & 7 of its row.  Rows past the matrix repeat the last
  // one (their products are never stored).
  const int wrow = K / 2, arow = BITS == 4 ? K / 2 : K;
  const uint8_t* wt = w_packed + (size_t)n0 * wrow;
  const uint8_t* at = a_codes + (size_t)m0 * arow;
  uint32_t wofs[2 * TI], aofs[2 * TJ];
  uint32_t hi[2];   // per lane: 64 where it reads a 4-bit row's second half, else 0
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = 8 * q + (lane >> 3);
    const int pn = ((lane & 7) ^ swz_nib(r)) * 16;
    const int pa = BITS == 4 ? pn : ((lane & 7) ^ swz_byte(r)) * 16;
    hi[q] = pn & 64;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      // Decode layout: blocks of 16 rows, K / 128 chunks of 1 KiB each (n0 and
      // N are multiples of 16); half q of a stage is one chunk.
      wofs[2 * i + q] = WDEC ? (uint32_t)(min(16 * i, N - 16 - n0) * wrow + q * 1024 + lane * 16)
                             : (uint32_t)(min(16 * i + r, N - 1 - n0) * wrow + pn);
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) aofs[2 * j + q] = (uint32_t)(min(16 * j + r, M - 1 - m0) * arow + pa);
  }
  uint8_t* stage = smem + wave * kStage;   // this wavefront's own
  const uint32_t base = (uint32_t)(uintptr_t)(lds_ptr)stage;
  // Stage s: blocks of 16 weight rows, then of 16 activation
  // rows (8 bits: its two 128-k halves).  TAIL: the stage without a second
  // half reads its first half twice (the copy is never used).
  auto load_stage = [&](auto tail, int s) __attribute__((always_inline)) {
    constexpr bool TAIL = decltype(tail)::value;
    const uint8_t* wc = wt + (size_t)s * (WDEC ? 2048 : 128);
    const uint8_t* ac = at + (size_t)s * (64 * kAB);
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t o = !TAIL ? wofs[2 * i + q] : WDEC ? wofs[2 * i] : wofs[2 * i + q] - hi[q];
        dma16(wc, o, base + (2 * i + q) * 1024);
      }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t la = base + (2 * TI + kAB * j + q) * 1024;
        if constexpr (BITS == 4) {
          dma16(ac, TAIL ? aofs[2 * j + q] - hi[q] : aofs[2 * j + q], la);
        } else {
          dma16(ac, aofs[2 * j + q], la);
          dma16(TAIL ? ac : ac + 128, aofs[2 * j + q], la + 2048);
        }
      }
    }
  };
  auto load = [&](int s) __attribute__((always_inline)) {
    if (s < min(s_end, half_stage)) load_stage(std::false_type{}, s);
    else if (s < s_end) load_stage(std::true_type{}, s);
  };
  // Fragments of half h (128 k): lane l has row l & 15 of a block.
  struct Half {
    uint4 w[TI];
    uint4 a[TJ * (BITS == 4 ? 1 : 2)];
  };
  auto read = [&](int h, Half& b) __attribute__((always_inline)) {
    const uint32_t rn = (uint32_t)(fr * 128 + ((4 * h + fg) ^ swz_nib(fr)) * 16);
#pragma unroll
    for (int i = 0; i < TI; ++i) b.w[i] = *reinterpret_cast<const uint4*>(stage + i * 2048 + (WDEC ? h * 1024 + lane * 16 : rn));
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const uint8_t* sa = stage + (2 * TI + kAB * j) * 1024;
      if constexpr (BITS == 4) {
        b.a[j] = *reinterpret_cast<const uint4*>(sa + rn);
      } else {
#pragma unroll
        for (int q = 0; q < 2; ++q)
          b.a[2 * j + q] = *reinterpret_cast<const uint4*>(sa + h * 2048 + fr * 128 +
                                                           ((2 * fg + q) ^ swz_byte(fr)) * 16);
      }
    }
  };
  v4i acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = v4i{0, 0, 0, 0};
  auto compute = [&](const Half& b) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v4i aop[TJ];
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        if constexpr (BITS == 4) {
          aop[j] = h == 0 ? op_from_nibbles(b.a[j].x, b.a[j].y) : op_from_nibbles(b.a[j].z, b.a[j].w);
        } else {
          const uint4 u = b.a[2 * j + h];
          aop[j] = op_a8<WA8>(u.x, u.y, u.z, u.w);
        }
      }
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const v4i wop = h == 0 ? op_from_nibbles(b.w[i].x, b.w[i].y) : op_from_nibbles(b.w[i].z, b.w[i].w);
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = mfma(wop, aop[j], acc[i][j]);
      }
    }
  };

  // No barrier: the stage is the wavefront's own, and is refilled after its
  // reads have returned, while the MFMAs run.
  load(s_begin);
  for (int s = s_begin; s < s_end; ++s) {
    wait_vmcnt0_fence();
    Half b0, b1;
    read(0, b0);
    read(1, b1);
    wait_lgkm0_fence();
    load(s + 1);
    compute(b0);
    if (s < half_stage) compute(b1);
  }
  __syncthreads();   // every wavefront is done with its stage

  // Sum the partial tiles, WAVES fragments at a time: every wavefront adds
  // one of them over all wavefronts and writes it.
#pragma unroll
  for (int f0 = 0; f0 < kFrags; f0 += WAVES) {
    if (f0 > 0) __syncthreads();
#pragma unroll
    for (int g = 0; g < WAVES; ++g)
      if (f0 + g < kFrags) part[g][wave][lane] = acc[(f0 + g) / TJ][(f0 + g) % TJ];
    __syncthreads();
    const int f = f0 + wave;
    if (f >= kFrags) continue;
    v4i tot = part[wave][0][lane];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      const v4i p = part[wave][w][lane];
      tot.x += p.x; tot.y += p.y; tot.z += p.z; tot.w += p.w;
    }
    const int i = f / TJ, j = f - i * TJ;
    const int m = m0 + 16 * j + fr, n = n0 + 16 * i + 4 * fg;
    if (m >= M || n >= N) continue;
    if constexpr (ACC_OUT) {
      *reinterpret_cast<int4*>(acc_out + (size_t)m * N + n) =
          make_int4(unscale<BITS>(tot.x), unscale<BITS>(tot.y), unscale<BITS>(tot.z), unscale<BITS>(tot.w));
    } else {
      const int off = ZP ? (1 << (BITS - 1)) - a_zeros[m] : 0;
      const int4 wz = ZP ? *reinterpret_cast<const int4*>(w_sums + n) : make_int4(0, 0, 0, 0);
      *reinterpret_cast<uint2*>(y + (size_t)m * N + n) =
          dequant4z<BITS, ZP>(tot.x, tot.y, tot.z, tot.w, a_scales[m],
                              *reinterpret_cast<const float4*>(w_scales + n), off, wz);
    }
  }
}

template <int BITS, int TI, int TJ, int WAVES, bool ACC_OUT, bool WA8, bool ZP, bool WDEC>
void launch_cfg(const KsplitCall& c, hipStream_t stream) {
  const int64_t tiles = ((c.M + 16 * TJ - 1) / (16 * TJ)) * ((c.N + 16 * TI - 1) / (16 * TI));
  hipLaunchKernelGGL((qgemm_ksplit<BITS, TI, TJ, WAVES, ACC_OUT, WA8, ZP, WDEC>), dim3((unsigned)tiles),
                     dim3(WAVES * 64), 0, stream, c.a, c.a_scales, c.w, c.w_scales, (int)c.M, (int)c.N, c.K,
                     c.y, c.acc, c.a_zeros, c.w_sums);
}

// Tiles for M > 16, as TI, TJ and the wavefronts that split K: eight while
// their stages and partial tiles fit a compute unit, else four.  The last two
// only pay at 8 bits, where an activation row is twice a weight row's bytes.
struct Tile {
  int ti, tj, waves;
};
constexpr Tile kTiles[] = {{1, 1, 8}, {1, 2, 8}, {2, 2, 8}, {2, 3, 8}, {4, 2, 8}, {4, 3, 8},
                           {4, 4, 4}, {4, 6, 4}, {6, 4, 4}, {6, 6, 4}, {8, 4, 4}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
constexpr int num_tiles(int bits) { return bits == 4 ? kNumTiles - 2 : kNumTiles; }

template <int BITS, bool ACC_OUT, bool WA8, bool ZP, int I = 0>
void launch_tile(int tile, const KsplitCall& c, hipStream_t stream) {
  if constexpr (I < num_tiles(BITS)) {
    if (tile == I)
      launch_cfg<BITS, kTiles[I].ti, kTiles[I].tj, kTiles[I].waves, ACC_OUT, WA8, ZP, false>(c, stream);
    else
      launch_tile<BITS, ACC_OUT, WA8, ZP, I + 1>(tile, c, stream);
  }
}

// One row of 16 tokens: one block of 16 channels per workgroup while these fit
// the compute units (about) once, two on eight wavefronts while those do, then
// two on four wavefronts (several workgroups per compute unit keep the loads
// going) up to four blocks per compute unit, and two on eight beyond.
// Measured at M = 8, 4 bits, canonical weights: N = 4096, K = 4096: 3.71 us
// against 3.92 and 4.6 us for the other two; N = 8192, K = 8192: 8.0-8.3 us
// for eight wavefronts against 9.6; N = 10240, K = 8192: 10.7, 11.3 and
// 10.0 us; N = 57344, K = 8192: 46, 41.4 and 42.4 us.
template <int BITS, bool ACC_OUT, bool WA8, bool ZP, bool WDEC>
void launch_decode(const KsplitCall& c, hipStream_t stream) {
  const int64_t nb = c.N / 16, cus = device_cus();
  if (8 * nb <= 9 * cus) launch_cfg<BITS, 1, 1, 8, ACC_OUT, WA8, ZP, WDEC>(c, stream);
  else if (nb > 2 * cus && nb <= 4 * cus) launch_cfg<BITS, 2, 1, 4, ACC_OUT, WA8, ZP, WDEC>(c, stream);
  else launch_cfg<BITS, 2, 1, 8, ACC_OUT, WA8, ZP, WDEC>(c, stream);
}

// Estimated microseconds of a tile: a start, then for each tile of the fullest
// compute unit the bytes it pulls per k (TI and TJ terms), its MFMAs and its
// reduction (TI * TJ terms), and the weights' way from memory.  Fitted to 15
// tiles over 1024 shapes (M 17-1024, N 1024-28672, K 2048-14336); the
// estimate is within 12% (one standard deviation) of the measured time.
double tile_cost(Tile t, int64_t M, int64_t N, int K, int bits, int64_t cus) {
  const int64_t tiles = ((M + 16 * t.tj - 1) / (16 * t.tj)) * ((N + 16 * t.ti - 1) / (16 * t.ti));
  const double rounds = (double)((tiles + cus - 1) / cus);
  const double area = (double)(t.ti * t.tj), k = (double)K;
  if (bits == 4)
    return 2.4 + rounds * (0.135 * area + k * (7.8e-5 * t.ti + 6.2e-5 * t.tj + 2.0e-5 * area)) +
           2.4e-8 * k * (double)N;
  return 1.9 + rounds * (0.2 * area + k * (7.8e-5 * t.ti + 1.85e-4 * t.tj + 1.7e-6 * area)) +
         2.0e-8 * k * (double)N;
}

int best_tile(int64_t M, int64_t N, int K, int bits, double* cost) {
  const int64_t cus = device_cus();
  int best = 0;
  *cost = 0.0;
  for (int i = 0; i < num_tiles(bits); ++i) {
    const double t = tile_cost(kTiles[i], M, N, K, bits, cus);
    if (i == 0 || t < *cost) {
      best = i;
      *cost = t;
    }
  }
  return best;
}

template <int BITS, bool ACC_OUT, bool WA8, bool ZP>
void launch_canonical(const KsplitCall& c, hipStream_t stream) {
  if (c.M <= 16) {
    launch_decode<BITS, ACC_OUT, WA8, ZP, false>(c, stream);
    return;
  }
  double cost;
  launch_tile<BITS, ACC_OUT, WA8, ZP>(best_tile(c.M, c.N, c.K, BITS, &cost), c, stream);
}

}  // namespace

double ksplit_cost(int64_t M, int64_t N, int K, int bits) {
  double cost;
  best_tile(M, N, K, bits, &cost);
  return cost;
}

hipError_t launch_ksplit(const KsplitCall& c, int bits, int weights, hipStream_t stream) {
  if (c.M == 0) return hipSuccess;
  const bool acc = c.acc != nullptr, zp = c.a_zeros != nullptr;
  if (weights == kWeightsDecode) {
    if (bits == 4) acc ? launch_decode<4, true, false, false, true>(c, stream)
                       : launch_decode<4, false, false, false, true>(c, stream);
    else acc ? launch_decode<8, true, false, false, true>(c, stream)
             : launch_decode<8, false, false, false, true>(c, stream);
  } else if (weights == kWeightsA8Order) {
    launch_canonical<8, false, true, false>(c, stream);
  } else if (bits == 4) {
    if (acc) launch_canonical<4, true, false, false>(c, stream);
    else if (zp) launch_canonical<4, false, false, true>(c, stream);
    else launch_canonical<4, false, false, false>(c, stream);
  } else {
    if (acc) launch_canonical<8, true, false, false>(c, stream);
    else if (zp) launch_canonical<8, false, false, true>(c, stream);
    else launch_canonical<8, false, false, false>(c, stream);
  }
  return hipGetLastError();
}

}  // namespace dptq
