// W4A4 / W4A8 GEMM for few tokens (gfx950): decode batches (M <= 16; some run on
// qgemm_decode.hip), and larger batches up to several hundred tokens whose 256 x
// 128 or 192 x 256 output tiles would leave most compute units idle.  Same
// product and epilogue as the tile kernels, same bits.
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
// a 4-bit row at a time; half lines are fetched twice) about 40 to 50, in the k
// loop and with the operands in the caches; whole launches with the weights from
// memory, start and sums included, 24 on long rows (19.6 us for this shape).
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
template <int N>
__device__ __forceinline__ void wait_vmcnt_fence() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" : : "i"(N) : "memory");
}
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
// bits, so a compute unit keeps 64 to 160 KiB on the way, as much as its LDS
// holds; two or more smaller stages each were no faster (M = 20, K = 14336,
// N = 4096 at 4 bits: 7.0 us with one, 7.8 us with two).
template <int BITS, int TI, int TJ, int WAVES, bool ACC_OUT, bool WA8, bool ZP, bool WDEC>
__global__ void __launch_bounds__(WAVES * 64)
qgemm_ksplit(const uint8_t* __restrict__ a_codes, const float* __restrict__ a_scales,
             const uint8_t* __restrict__ w_packed, const float* __restrict__ w_scales, int M, int N,
             int K, __half* __restrict__ y, int32_t* __restrict__ acc_out,
             const int32_t* __restrict__ a_zeros, const int32_t* __restrict__ w_sums) {
  constexpr int kAB = BITS == 4 ? 2 : 4;         // KiB of an activation block per stage
  constexpr int kLoads = 2 * TI + kAB * TJ;      // 1 KiB each, per stage
  constexpr int kStage = kLoads * 1024;
  constexpr int kRing = WAVES * kStage;
  constexpr int kFrags = TI * TJ, kFragPart = WAVES * 1024;   // one block's partial tiles
  constexpr int kPart = (kFrags < WAVES ? kFrags : WAVES) * kFragPart;
  constexpr int kLds = kRing > kPart ? kRing : kPart;
  constexpr int kPass = kLds / kFragPart < kFrags ? kLds / kFragPart : kFrags;   // blocks summed at a time
  static_assert(kRing <= 160 * 1024, "LDS budget");
  // Refill the stage part by part (below) where there are MFMAs enough to read
  // under, but not if the second set of fragments costs a resident workgroup:
  // 4 x 4 blocks at 4 bits, two workgroups a compute unit with 256 registers
  // each.  M = 333, K = 14336, N = 4096 at 8 bits (4 x 6 blocks): 31.6 us
  // refilled at once, 26.1 us part by part; M = 512, K = N = 4096 at 4 bits
  // (4 x 4): 13.3 against 15 us; two to six blocks: the same within 1%.
  constexpr bool kStream = WAVES == 4 && kFrags >= 8 && (kRing > 80 * 1024 || kFrags < 16);
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kLds];
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
  auto load_w = [&](auto tail, int s) __attribute__((always_inline)) {
    constexpr bool TAIL = decltype(tail)::value;
    const uint8_t* wc = wt + (size_t)s * (WDEC ? 2048 : 128);
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t o = !TAIL ? wofs[2 * i + q] : WDEC ? wofs[2 * i] : wofs[2 * i + q] - hi[q];
        dma16(wc, o, base + (2 * i + q) * 1024);
      }
  };
  auto load_a = [&](auto tail, int s, int j) __attribute__((always_inline)) {
    constexpr bool TAIL = decltype(tail)::value;
    const uint8_t* ac = at + (size_t)s * (64 * kAB);
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
  };
  auto part_w = [&](int s) __attribute__((always_inline)) {
    if (s < half_stage) load_w(std::false_type{}, s);
    else load_w(std::true_type{}, s);
  };
  auto part_a = [&](int s, int j) __attribute__((always_inline)) {
    if (s < half_stage) load_a(std::false_type{}, s, j);
    else load_a(std::true_type{}, s, j);
  };
  // Fragments of half h (128 k): lane l has row l & 15 of a block.
  struct WFrag {
    uint4 v[2][TI];
  };
  struct AFrag {
    uint4 v[2][BITS == 4 ? 1 : 2];
  };
  auto read_w = [&](WFrag& b) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < TI; ++i)
        b.v[h][i] = *reinterpret_cast<const uint4*>(
            stage + i * 2048 + (WDEC ? h * 1024 + lane * 16 : fr * 128 + ((4 * h + fg) ^ swz_nib(fr)) * 16));
  };
  auto read_a = [&](int j, AFrag& b) __attribute__((always_inline)) {
    const uint8_t* sa = stage + (2 * TI + kAB * j) * 1024;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (BITS == 4) {
        b.v[h][0] = *reinterpret_cast<const uint4*>(sa + fr * 128 + ((4 * h + fg) ^ swz_nib(fr)) * 16);
      } else {
#pragma unroll
        for (int q = 0; q < 2; ++q)
          b.v[h][q] = *reinterpret_cast<const uint4*>(sa + h * 2048 + fr * 128 +
                                                      ((2 * fg + q) ^ swz_byte(fr)) * 16);
      }
    }
  };
  v4i acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = v4i{0, 0, 0, 0};
  // Column j of the tile over half h.
  auto compute = [&](const WFrag& w, const AFrag& a, int j, int h) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      v4i aop;
      if constexpr (BITS == 4) {
        const uint4 u = a.v[h][0];
        aop = e == 0 ? op_from_nibbles(u.x, u.y) : op_from_nibbles(u.z, u.w);
      } else {
        const uint4 u = a.v[h][e];
        aop = op_a8<WA8>(u.x, u.y, u.z, u.w);
      }
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const uint4 u = w.v[h][i];
        acc[i][j] = mfma(e == 0 ? op_from_nibbles(u.x, u.y) : op_from_nibbles(u.z, u.w), aop, acc[i][j]);
      }
    }
  };

  // No barrier: the stage is the wavefront's own.  Small tiles refill it at
  // once, after its reads have returned, while the MFMAs run.
  if constexpr (!kStream) {
    auto load_stage = [&](auto tail, int s) __attribute__((always_inline)) {
      load_w(tail, s);
#pragma unroll
      for (int j = 0; j < TJ; ++j) load_a(tail, s, j);
    };
    auto load = [&](int s) __attribute__((always_inline)) {
      if (s < min(s_end, half_stage)) load_stage(std::false_type{}, s);
      else if (s < s_end) load_stage(std::true_type{}, s);
    };
    load(s_begin);
    for (int s = s_begin; s < s_end; ++s) {
      wait_vmcnt_fence<0>();
      WFrag w;
      AFrag a[TJ];
      read_w(w);
#pragma unroll
      for (int j = 0; j < TJ; ++j) read_a(j, a[j]);
      wait_lgkm0_fence();
      load(s + 1);
#pragma unroll
      for (int j = 0; j < TJ; ++j) compute(w, a[j], j, 0);
      if (s < half_stage) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) compute(w, a[j], j, 1);
      }
    }
  }
  // Larger tiles: the stage is refilled part by part (the weights and the first
  // activation block, then each of the other blocks), each part as soon as its
  // reads have returned, and a part is read while the MFMAs of the one before
  // run; so loads leave all the time.
  // Step j of stage s reads part j + 1 of it (the last step part 0 of stage
  // s + 1); more: whether stage s + 1 exists.
  constexpr int kP0 = 2 * TI + kAB;   // loads of part 0
  if (kStream && s_begin < s_end) {
    part_w(s_begin);
#pragma unroll
    for (int j = 0; j < TJ; ++j) part_a(s_begin, j);
    WFrag w[2];
    AFrag a[2];
    wait_vmcnt_fence<(TJ - 1) * kAB>();
    read_w(w[0]);
    read_a(0, a[0]);
    wait_lgkm0_fence();
    if (s_begin + 1 < s_end) {
      part_w(s_begin + 1);
      part_a(s_begin + 1, 0);
    }
    auto stage_steps = [&](auto morec, int s, const WFrag& wc, WFrag& wn, auto par) __attribute__((always_inline)) {
      constexpr bool more = decltype(morec)::value;
      constexpr int P = decltype(par)::value;   // a[P] holds block 0
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        AFrag& ac = a[(P + j) & 1];
        AFrag& an = a[(P + j + 1) & 1];
        if (j + 1 < TJ) {
          // In flight after it: blocks j + 2 .. of this stage, part 0 and blocks 1 .. j of the next.
          if constexpr (more) wait_vmcnt_fence<(TJ - 2) * kAB + kP0>();
          else wait_vmcnt_fence<0>();
          read_a(j + 1, an);
        } else if constexpr (more) {
          wait_vmcnt_fence<(TJ - 1) * kAB>();
          read_w(wn);
          read_a(0, an);
        }
        __builtin_amdgcn_sched_barrier(0);
        compute(wc, ac, j, 0);
        if (more || s < half_stage) compute(wc, ac, j, 1);
        __builtin_amdgcn_sched_barrier(0);
        wait_lgkm0_fence();
        if constexpr (more) {
          if (j + 1 < TJ) {
            part_a(s + 1, j + 1);
          } else if (s + 2 < s_end) {
            part_w(s + 2);
            part_a(s + 2, 0);
          }
        }
      }
    };
    constexpr std::integral_constant<int, 0> p0{};
    constexpr std::integral_constant<int, TJ & 1> p1{};
    int s = s_begin;
    for (; s + 2 < s_end; s += 2) {
      stage_steps(std::true_type{}, s, w[0], w[1], p0);
      stage_steps(std::true_type{}, s + 1, w[1], w[0], p1);
    }
    if (s + 1 < s_end) {
      stage_steps(std::true_type{}, s, w[0], w[1], p0);
      stage_steps(std::false_type{}, s + 1, w[1], w[0], p1);
    } else {
      stage_steps(std::false_type{}, s, w[0], w[1], p0);
    }
  }
  __syncthreads();   // every wavefront is done with its stage

  // Sum the partial tiles, kPass blocks at a time.  Up to one block per
  // wavefront, a wavefront adds one block over all wavefronts, each lane the
  // four values it holds in its own (n .. n + 3 of one m).  More blocks go two
  // at a time to a wavefront, a lane adding eight consecutive n of one m, so
  // that the stores are 16 bytes.
  auto total = [&](int g, int slot) __attribute__((always_inline)) {
    v4i t = part[g][0][slot];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      const v4i p = part[g][w][slot];
      t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
    }
    return t;
  };
  auto scaled = [&](v4i t, int m, int n) __attribute__((always_inline)) {
    const int off = ZP ? (1 << (BITS - 1)) - a_zeros[m] : 0;
    const int4 wz = ZP ? *reinterpret_cast<const int4*>(w_sums + n) : make_int4(0, 0, 0, 0);
    return dequant4z<BITS, ZP>(t.x, t.y, t.z, t.w, a_scales[m],
                               *reinterpret_cast<const float4*>(w_scales + n), off, wz);
  };
  auto unscaled = [&](v4i t) __attribute__((always_inline)) {
    return make_int4(unscale<BITS>(t.x), unscale<BITS>(t.y), unscale<BITS>(t.z), unscale<BITS>(t.w));
  };
#pragma unroll
  for (int f0 = 0; f0 < kFrags; f0 += kPass) {
    if (f0 > 0) __syncthreads();
#pragma unroll
    for (int g = 0; g < kPass; ++g)
      if (f0 + g < kFrags) part[g][wave][lane] = acc[(f0 + g) / TJ][(f0 + g) % TJ];
    __syncthreads();
    constexpr bool kPairs = kFrags > WAVES;
    const int blocks = min(kPass, kFrags - f0);
    for (int u = wave; u < (kPairs ? (blocks + 1) / 2 : blocks); u += WAVES) {
      const int g = kPairs ? 2 * u + (lane >> 5) : u;
      const int f = f0 + g, i = f / TJ, j = f - i * TJ;
      const int q = kPairs ? (fg & 1) * 2 : fg;           // group of four n
      const int m = m0 + 16 * j + fr, n = n0 + 16 * i + 4 * q;
      if (g >= blocks || m >= M || n >= N) continue;      // whole blocks of n: N is a multiple of 16
      const v4i t0 = total(g, 16 * q + fr);
      if constexpr (kPairs) {
        const v4i t1 = total(g, 16 * q + 16 + fr);
        if constexpr (ACC_OUT) {
          int32_t* o = acc_out + (size_t)m * N + n;
          *reinterpret_cast<int4*>(o) = unscaled(t0);
          *reinterpret_cast<int4*>(o + 4) = unscaled(t1);
        } else {
          const uint2 lo = scaled(t0, m, n), hi2 = scaled(t1, m, n + 4);
          *reinterpret_cast<uint4*>(y + (size_t)m * N + n) = make_uint4(lo.x, lo.y, hi2.x, hi2.y);
        }
      } else if constexpr (ACC_OUT) {
        *reinterpret_cast<int4*>(acc_out + (size_t)m * N + n) = unscaled(t0);
      } else {
        *reinterpret_cast<uint2*>(y + (size_t)m * N + n) = scaled(t0, m, n);
      }
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

template <int BITS, bool ACC_OUT, bool WA8, bool ZP, int I = 0>
void launch_tile(int tile, const KsplitCall& c, hipStream_t stream) {
  if constexpr (I < rules::ksplit_tiles(BITS)) {
    constexpr rules::KsplitTile t = rules::ksplit_tile(BITS, I);
    if (tile == I)
      launch_cfg<BITS, t.ti, t.tj, t.waves, ACC_OUT, WA8, ZP, false>(c, stream);
    else
      launch_tile<BITS, ACC_OUT, WA8, ZP, I + 1>(tile, c, stream);
  }
}

template <int BITS, bool ACC_OUT, bool WA8, bool ZP, bool WDEC>
void launch_decode(const KsplitCall& c, hipStream_t stream) {
  const rules::DecodeTile t = rules::decode_tile(c.N, c.cus);
  if (t.ti == 1) launch_cfg<BITS, 1, 1, 8, ACC_OUT, WA8, ZP, WDEC>(c, stream);
  else if (t.waves == 4) launch_cfg<BITS, 2, 1, 4, ACC_OUT, WA8, ZP, WDEC>(c, stream);
  else launch_cfg<BITS, 2, 1, 8, ACC_OUT, WA8, ZP, WDEC>(c, stream);
}

template <int BITS, bool ACC_OUT, bool WA8, bool ZP>
void launch_canonical(const KsplitCall& c, int tile, hipStream_t stream) {
  if (c.M <= 16) launch_decode<BITS, ACC_OUT, WA8, ZP, false>(c, stream);
  else launch_tile<BITS, ACC_OUT, WA8, ZP>(tile, c, stream);
}

}  // namespace

hipError_t launch_ksplit(const KsplitCall& c, int bits, int weights, int tile, hipStream_t stream) {
  if (c.M == 0) return hipSuccess;
  if (c.M > 16 && tile < 0) return hipErrorInvalidValue;
  if (c.M <= 16 && rules::decode_in_regs(c.M, c.N, c.K, bits, weights == kWeightsDecode, c.cus))
    return launch_decode_regs(c, bits, weights, stream);
  const bool acc = c.acc != nullptr, zp = c.a_zeros != nullptr;
  if (weights == kWeightsDecode) {
    if (bits == 4) acc ? launch_decode<4, true, false, false, true>(c, stream)
                       : launch_decode<4, false, false, false, true>(c, stream);
    else acc ? launch_decode<8, true, false, false, true>(c, stream)
             : launch_decode<8, false, false, false, true>(c, stream);
  } else if (weights == kWeightsA8Order) {
    launch_canonical<8, false, true, false>(c, tile, stream);
  } else if (bits == 4) {
    if (acc) launch_canonical<4, true, false, false>(c, tile, stream);
    else if (zp) launch_canonical<4, false, false, true>(c, tile, stream);
    else launch_canonical<4, false, false, false>(c, tile, stream);
  } else {
    if (acc) launch_canonical<8, true, false, false>(c, tile, stream);
    else if (zp) launch_canonical<8, false, false, true>(c, tile, stream);
    else launch_canonical<8, false, false, false>(c, tile, stream);
  }
  return hipGetLastError();
}

}  // namespace dptq
