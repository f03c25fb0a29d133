// Which kernel and tile a shape runs: pure functions of the sizes and the
// compute units, evaluated once per call (host only, no HIP, so that they can be
// checked without a GPU).  Estimates are in microseconds; the kernels that they
// choose between return the same bits.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace dptq {

// GEMM kernels (values of dptq_gemm_kernel, then kGemmKsplit: the K-split
// kernel that serves kGemmDecode, for M > 16 on a tile the dispatch chose).
constexpr int kGemmAuto = 0, kGemmDecode = 1, kGemmTile = 2, kGemmWide = 3, kGemmKsplit = 4;

namespace rules {

constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// A tile of a K-split kernel (-1: none) and its estimated time.
struct TilePlan {
  int tile;
  double cost;
};

// ---------------------------------------------------------------------------
// K-split int8 GEMM, M > 16.  Tiles (TI, TJ, the wavefronts that split K), and
// the estimate of each: a start, then per round of `resident` workgroups a
// compute unit a fixed part and the k loop, then what grows with every tile a
// compute unit runs, with the weights' way from memory and with the output's.
// Fitted to 288 shapes a bit width (M 20-1024, N 1024-28672, K 2048-28672;
// weights cycling through 300 MB): the tile picked is within 2% of the best of
// 20 on average.
// ---------------------------------------------------------------------------
struct KsplitTile {
  int ti, tj, waves, resident;
  double start, round, round_k, tile_k, kn, mn;
};
constexpr KsplitTile kKsplitTiles4[] = {
    {1, 1, 8, 2, 2.38, 0.00, 9.85e-05, 1.08e-04, 2.16e-08, 2.90e-06},
    {1, 2, 8, 1, 2.57, 0.00, 2.45e-04, 0.00e+00, 2.50e-08, 1.78e-06},
    {2, 2, 8, 1, 2.52, 0.11, 3.35e-04, 0.00e+00, 2.93e-08, 1.51e-06},
    {2, 3, 8, 1, 2.74, 0.27, 4.43e-04, 0.00e+00, 2.02e-08, 1.03e-06},
    {2, 4, 8, 1, 1.79, 1.31, 5.76e-04, 0.00e+00, 1.70e-08, 1.07e-06},
    {4, 3, 8, 1, 1.70, 1.83, 6.98e-04, 0.00e+00, 2.56e-08, 6.68e-07},
    {2, 2, 4, 2, 2.75, 0.00, 3.36e-04, 1.77e-04, 2.87e-08, 5.92e-07},
    {2, 3, 4, 3, 2.95, 0.00, 3.43e-04, 3.31e-04, 1.53e-08, 7.78e-07},
    {2, 4, 4, 2, 3.02, 0.00, 4.13e-04, 3.16e-04, 1.81e-08, 9.85e-07},
    {4, 4, 4, 2, 2.95, 0.86, 4.29e-04, 7.25e-04, 1.87e-08, 7.25e-07},
    {8, 4, 4, 1, 1.68, 4.39, 1.57e-03, 0.00e+00, 1.81e-08, 4.62e-07},
    {4, 8, 4, 1, 1.82, 3.80, 1.66e-03, 0.00e+00, 1.26e-08, 4.27e-07}};
constexpr KsplitTile kKsplitTiles8[] = {
    {1, 1, 8, 1, 2.40, 0.00, 2.27e-04, 0.00e+00, 2.72e-08, 2.63e-06},
    {1, 2, 8, 1, 2.37, 0.00, 3.68e-04, 0.00e+00, 2.37e-08, 2.57e-06},
    {2, 2, 8, 1, 1.72, 0.71, 4.71e-04, 0.00e+00, 2.46e-08, 2.37e-06},
    {2, 3, 8, 1, 1.73, 0.97, 6.26e-04, 0.00e+00, 1.35e-08, 1.63e-06},
    {4, 3, 8, 1, 1.53, 1.57, 8.43e-04, 0.00e+00, 2.26e-08, 9.59e-07},
    {2, 4, 4, 1, 2.56, 0.00, 7.39e-04, 0.00e+00, 1.60e-08, 1.03e-06},
    {4, 2, 4, 2, 2.36, 0.41, 1.03e-04, 5.87e-04, 2.77e-08, 8.12e-07},
    {4, 4, 4, 1, 1.51, 2.06, 1.01e-03, 0.00e+00, 1.69e-08, 8.48e-07},
    {4, 6, 4, 1, 1.58, 2.73, 1.32e-03, 0.00e+00, 1.21e-08, 8.05e-07},
    {4, 8, 4, 1, 1.65, 3.53, 1.63e-03, 0.00e+00, 1.82e-08, 6.65e-07},
    {8, 4, 4, 1, 1.74, 3.79, 1.59e-03, 0.00e+00, 1.90e-08, 6.60e-07}};
constexpr int ksplit_tiles(int bits) {
  return bits == 4 ? sizeof(kKsplitTiles4) / sizeof(kKsplitTiles4[0])
                   : sizeof(kKsplitTiles8) / sizeof(kKsplitTiles8[0]);
}
constexpr KsplitTile ksplit_tile(int bits, int i) { return bits == 4 ? kKsplitTiles4[i] : kKsplitTiles8[i]; }

// The estimate of a tile of which the fullest compute unit runs q.
template <class Tile>
double ksplit_tile_us(const Tile& t, int64_t q, int64_t M, int64_t N, int K) {
  const double rounds = (double)ceil_div(q, t.resident), k = (double)K;
  return t.start + rounds * (t.round + k * t.round_k) + (double)q * k * t.tile_k + t.kn * k * (double)N +
         t.mn * (double)M * (double)N;
}

// The tile with the lowest estimate among those that give a compute unit at most
// three rounds (and at least six tiles), where the fitted shapes lie.
inline TilePlan ksplit_plan(int64_t M, int64_t N, int K, int bits, int cus) {
  TilePlan best{-1, 0.0};
  for (int i = 0; i < ksplit_tiles(bits); ++i) {
    const KsplitTile t = ksplit_tile(bits, i);
    const int64_t q = ceil_div(ceil_div(M, 16 * t.tj) * ceil_div(N, 16 * t.ti), cus);
    if (q > 3 * (t.resident > 2 ? t.resident : 2)) continue;
    const double c = ksplit_tile_us(t, q, M, N, K);
    if (best.tile < 0 || c < best.cost) best = {i, c};
  }
  return best;
}

// Output tiles (n x m) of the two int8 tile kernels; the wide one needs a full
// tile and a ring's worth of k.
constexpr int kTileN = 256, kTileM = 128, kWideN = 192, kWideM = 256;
constexpr int wide_min_k(int bits) { return bits == 4 ? 512 : 384; }
inline bool wide_fits(int64_t M, int64_t N, int K, int bits) {
  return M >= kWideM && N >= kWideN && K >= wide_min_k(bits);
}

// Which of the two: relative time, rounds of one tile per compute unit times the
// tile's area over the measured throughput of the tile shape (large prefill
// shapes).
constexpr double kWideSpeed = 1.3;
inline double tile_launch_cost(int64_t M, int64_t N, int bm, int bn, double speed, int cus) {
  return (double)ceil_div(ceil_div(M, bm) * ceil_div(N, bn), cus) * (double)bm * (double)bn / speed;
}
inline bool wide_is_faster(int64_t M, int64_t N, int K, int bits, int cus) {
  return wide_fits(M, N, K, bits) && tile_launch_cost(M, N, kWideM, kWideN, kWideSpeed, cus) <=
                                         tile_launch_cost(M, N, kTileM, kTileN, 1.0, cus);
}

// Estimate of a 256 x 128 or 192 x 256 tile kernel: a start, then per round of
// one tile per compute unit its k loop (slower when every unit is busy: power)
// and its epilogue.  Fitted to measured times over M 17-1024, N 1024-28672, K
// 2048-14336, within 4%.
inline double tile_kernel_us(int64_t M, int64_t N, int K, int bits, bool wide, int cus) {
  const int64_t bm = wide ? kWideM : kTileM, bn = wide ? kWideN : kTileN;
  const int64_t tiles = ceil_div(M, bm) * ceil_div(N, bn);
  const double rounds = (double)ceil_div(tiles, cus), k = (double)K;
  const double fill = tiles < cus ? (double)tiles / cus : 1.0;
  if (bits == 4)
    return wide ? 3.0 + rounds * (5.85 + k * (5.81e-3 + 1.43e-3 * fill))
                : 1.8 + rounds * (4.35 + k * (5.12e-3 + 0.87e-3 * fill));
  return wide ? 3.9 + rounds * (5.0 + k * (5.55e-3 + 2.17e-3 * fill))
              : 1.4 + rounds * (4.76 + k * (4.59e-3 + 1.45e-3 * fill));
}

// What the estimates leave out beyond the shapes they were fitted to.  Below K =
// 2048: a round's cost besides its k loop (8 bits, N = 6144, K = 256: M = 384 8.7
// against 6.8 us on the tile kernel).  Beyond M = 1024: the activations' way; the
// tiles run along M within an XCD, so up to eight L2s read all of them, and each
// read past the second adds to every element (M = 2853, N = 1456, K = 9216, 8 bits:
// 89 against 54 us).
inline double ksplit_extra_us(int tile, int64_t M, int64_t N, int K, int bits, int cus) {
  const KsplitTile t = ksplit_tile(bits, tile);
  const int64_t tiles_n = ceil_div(N, 16 * t.ti);
  double us = 0.0;
  if (K < 2048) {
    const int64_t rounds = ceil_div(ceil_div(ceil_div(M, 16 * t.tj) * tiles_n, cus), t.resident);
    us += (bits == 4 ? 0.4 : 0.65) * (double)(rounds - 1);
  }
  if (M > 1024 && tiles_n > 2)
    us += (bits == 4 ? 5e-8 : 1.2e-7) * (double)((tiles_n < 8 ? tiles_n : 8) - 2) * (double)K * (double)M;
  return us;
}

// The kernel of a shape, and the K-split kernel's tile.  M <= 16 streams the
// weights; otherwise the K-split kernel where its estimate is at least 8% below
// the tile kernels' (it is the less exact).  At K = 14336, N = 4096, 4 bits it
// takes 8.7 us against 83 us at M = 48, 18.6 against 80 at M = 256, 31.6 against
// 80.5 at M = 512, 64.8 against 83 at M = 1024; at K = 2048, N = 11008 it stops
// paying at M = 384 (17.1 against 17.9 us).
struct GemmRoute {
  int kernel, tile;
};
inline GemmRoute gemm_route(int64_t M, int64_t N, int K, int bits, int cus) {
  if (M <= 16) return {kGemmDecode, -1};
  const bool wide = wide_is_faster(M, N, K, bits, cus);
  const TilePlan p = ksplit_plan(M, N, K, bits, cus);
  if (p.tile >= 0) {
    const double us = p.cost + ksplit_extra_us(p.tile, M, N, K, bits, cus);
    if (1.08 * us < tile_kernel_us(M, N, K, bits, wide, cus)) return {kGemmKsplit, p.tile};
  }
  return {wide ? kGemmWide : kGemmTile, -1};
}

// ---------------------------------------------------------------------------
// At most 16 tokens: the K-split kernel, or the kernel that streams the weights
// into registers (qgemm_decode.hip).
// ---------------------------------------------------------------------------
// Workgroup of the K-split kernel for at most 16 tokens, as blocks of 16 channels
// and wavefronts: one block while these fit the compute units (about) once, two
// on eight wavefronts while those do, then two on four wavefronts (several
// workgroups per compute unit keep the loads going) up to four blocks per
// compute unit, and two on eight beyond.  Measured at M = 8, 4 bits, canonical
// weights: N = 4096, K = 4096: 3.71 us against 3.92 and 4.6 us for the other
// two; N = 8192, K = 8192: 8.0-8.3 us for eight wavefronts against 9.6; N =
// 10240, K = 8192: 10.7, 11.3 and 10.0 us; N = 57344, K = 8192: 46, 41.4 and
// 42.4 us.
struct DecodeTile {
  int ti, waves;
};
inline DecodeTile decode_tile(int64_t N, int cus) {
  const int64_t nb = N / 16;
  if (8 * nb <= 9 * (int64_t)cus) return {1, 8};
  if (nb > 2 * (int64_t)cus && nb <= 4 * (int64_t)cus) return {2, 4};
  return {2, 8};
}

// Blocks of 16 output channels per workgroup of the register kernel.  A
// one-block workgroup reads M * K * bits / 8 activation bytes beside 8 K weight
// bytes; once the activations are as large (M * bits >= 64) two blocks share
// them, provided N still gives two workgroups per compute unit.  (Four blocks
// were slower at 8 tokens and 4 bits, N = 57344.)
inline int decode_blocks(int64_t M, int64_t N, int bits, int cus) {
  return M * bits >= 64 && N % 32 == 0 && N / 32 >= 2 * (int64_t)cus ? 2 : 1;
}
// Its 128-k chunks in flight: eight instead of four where a wavefront streams
// at least 12, the grid is at most one workgroup per compute unit and M <= 4
// (decode layout, K = 14336, N = 4096, 4 bits: M = 1 7.90 -> 7.25 us, M = 4 8.30
// -> 7.40 us); slower with fewer chunks or more workgroups (K = 4096, N = 12288,
// M = 1: 6.53 -> 8.25 us).
inline int decode_batch(int64_t M, int64_t N, int K, int blocks, int cus) {
  return blocks == 1 && M <= 4 && K / 128 >= 12 * 8 && N / 16 <= cus ? 8 : 4;
}

// Estimated microseconds of either on the decode layout: a start, then what grows
// with the workgroups of the fullest compute unit, with their batches of four
// chunks (stages of the K-split kernel), with the rounds of `resident` workgroups
// a compute unit, with a wavefront's chunks (stages), and the weights' and the
// activations' way.  Fitted where they decide (below), to 2128 and 2128 shapes a
// bit width (M 1-16, N 64-57344, K 512-28672; weights cycling through 768 MB),
// within 3 to 7% (one standard deviation).
struct DecodeCost {
  int resident;
  double start, wg, wg_step, round, round_step, step, kn, act;
};
constexpr DecodeCost kDecodeCosts[2][6] = {
    // 4 bits: registers 1 x 4, 1 x 8 and 2 x 4 (blocks x chunks), K split 1 x 8, 2 x 4 and 2 x 8
    {{1, 2.385, 0, 0.2755, 0, 0, 0.0722, 5.77e-8, 7.12e-6},
     {1, 0, 0, 0, 2.04, 0.566, 0.0363, 4.31e-8, 5.68e-6},
     {3, 2.385, 0, 0.2283, 0.2143, 0, 0.0582, 4.46e-8, 2.011e-5},
     {1, 2.467, 0, 0, 0, 0, 0.2914, 6.64e-8, 1.05e-6},
     {1, 0, 1.44, 0.1117, 0, 0, 0, 6.98e-8, 2.55e-6},
     {3, 2.374, 0.0681, 0.1693, 0.2595, 0, 0.0795, 7.07e-8, 3.04e-6}},
    // 8 bits
    {{1, 2.252, 0, 0.3416, 0.0292, 0, 0.1009, 5.19e-8, 1.47e-5},
     {1, 0, 0, 0, 2.049, 0, 0.2089, 5.38e-8, 1.559e-5},
     {2, 1.754, 0, 0, 1.082, 0.2134, 0.1214, 5.96e-8, 1.678e-5},
     {1, 2.498, 0, 0.3315, 0, 0, 0, 6.43e-8, 2.98e-6},
     {1, 0, 1.454, 0.1662, 0, 0, 0, 6.10e-8, 6.96e-6},
     {2, 1.891, 0.1828, 0.2512, 0.5839, 0, 0.1412, 6.11e-8, 6.75e-6}}};
inline double decode_us(const DecodeCost& c, int64_t wgs, int64_t steps, int64_t wg_steps, int64_t M, int64_t N,
                        int K, int cus) {
  const double q = (double)ceil_div(wgs, cus), rounds = (double)ceil_div(wgs, (int64_t)cus * c.resident);
  const double k = (double)K, ws = (double)wg_steps;
  return c.start + q * (c.wg + c.wg_step * ws) + rounds * (c.round + c.round_step * ws) + c.step * (double)steps +
         c.kn * k * (double)N + c.act * q * (double)M * k;
}
inline double decode_regs_us(int64_t M, int64_t N, int K, int bits, int cus) {
  const int blocks = decode_blocks(M, N, bits, cus), batch = decode_batch(M, N, K, blocks, cus);
  const int64_t chunks = ceil_div(K / 128, 8);
  return decode_us(kDecodeCosts[bits == 8][blocks == 2 ? 2 : batch == 8 ? 1 : 0], N / (16 * blocks), chunks,
                   ceil_div(chunks, batch) * (batch / 4), M, N, K, cus);
}
inline double decode_ksplit_us(int64_t M, int64_t N, int K, int bits, int cus) {
  const DecodeTile t = decode_tile(N, cus);
  const int64_t stages = ceil_div(ceil_div(K, 256), t.waves);
  return decode_us(kDecodeCosts[bits == 8][t.ti == 1 ? 3 : t.waves == 4 ? 4 : 5], ceil_div(N / 16, t.ti), stages,
                   stages, M, N, K, cus);
}

// Which of the two.  Where a wavefront has at most half a chunk the way through
// LDS only adds latency: K <= 128, or K <= 512 on at most two blocks of channels
// a compute unit (M = 1, N = 4096, K = 512, 8 bits: 2.75 against 2.99 us), or K <=
// 384 on more than four at 8 bits (M = 4, N = 20480, K = 256: 4.4 against 5.1); but
// three of the register kernel's workgroups fit a compute unit at 8 bits, so
// between three and four blocks it loses a round (M = 4, N = 14336, K = 128: 3.4
// against 3.1 us).  Longer rows of canonical weights take the K-split kernel,
// whose loads cover whole lines (M = 4, N = 4096, K = 14336, 8 bits: 8.7 against
// 10.6 us).  The decode layout gives both kernels whole KiB, so the estimates
// decide (4 bits: M = 1, N = 2560, K = 14336 6.5 us in registers against 7.6 us, M =
// 1, N = 28672, K = 4096 11.6 against 13.7, M = 16, N = K = 8192 10.1 against 8.9),
// but for short rows of many channels, which the K-split kernel takes (M = 1, N =
// 43008, K = 768: 8.1 against 9.5 us), and two kinds of long 4-bit rows that the
// register kernel takes: where it streams eight chunks at a time (M = 1, N = 1024, K
// = 28672: 9.4 against 11.4 us, N = 4096, K = 14336 7.5 against 8.0), and up to eight
// tokens of K > 16384 on at most eight blocks a compute unit, if the last round of
// its workgroups is 85% full or the only one (M = 8, K = 28672, N = 8192: 22.9
// against 24.1 us; a quarter full, N = 5120: 21.2 against 17.1).
inline bool decode_in_regs(int64_t M, int64_t N, int K, int bits, bool decode_layout, int cus) {
  const int64_t nb = N / 16;
  const bool many = nb > 2 * (int64_t)cus;
  if (K <= 128) return !(bits == 8 && nb > 3 * (int64_t)cus && nb <= 4 * (int64_t)cus);
  if (K <= 512 && !many) return true;
  if (bits == 8 && K <= 384 && nb > 4 * (int64_t)cus) return true;
  if (!decode_layout) return false;
  if (K < 2048 && many) return false;
  if (bits == 4 && N >= 1024) {
    if (decode_batch(M, N, K, 1, cus) == 8) return true;
    const int64_t rounds = ceil_div(nb, cus);
    if (M <= 8 && K > 16384 && rounds <= 8 && (rounds == 1 || 20 * nb >= 17 * cus * rounds)) return true;
  }
  return decode_regs_us(M, N, K, bits, cus) < 1.01 * decode_ksplit_us(M, N, K, bits, cus);
}

// Whether the one-launch decode (decode_fused.hip), every workgroup of 16
// channels repeating the rotation of the M rows, beats rotate + quantize and then
// the decode GEMM, for h = f * 2^j.  Measured over 1400 shapes (K 512-20480, N
// 1024-24576, 4 and 8 bits alike, weights cycling through 768 MB), one launch
// against two: M = 1, N = 4096, K = 4096 0.68 of the time, K = 14336 0.74; N =
// 12288, K = 4096 0.82, K = 8192 0.83, K = 2048 0.98, K = 14336 1.22; N = 16384, K =
// 12288 0.90, K = 4096 (one whole segment) 0.87-0.94, K = 5120 1.02.  M = 2, N = 4096 0.74 at K = 4096, 0.91 at 12288;
// N = 12288 0.92 at K = 4096, 1.4 at 12288.  Above K = 12288 a workgroup's staging
// leaves room for one a compute unit.  More rows never gained over 5%, and h = 28 *
// 2^j is slower throughout (the 28-point stage in every workgroup): 1.04-4.
inline bool decode_one_launch(int64_t M, int K, int f, int j, int64_t N, int cus) {
  if (f != 1 || M > 2) return false;
  const int64_t nb = N / 16;   // workgroups
  int per_cu;
  if (M == 1) {
    if (j > 14) return false;
    per_cu = K > 12288 ? 1 : K < 2048 ? 2 : j < 13 && (K >= 8192 || (K > 3072 && K <= 4096)) ? 4 : 3;
  } else {
    if (j > 12 || K > 12288) return false;
    per_cu = K > 4096 || K < 2048 ? 1 : K < 2560 ? 2 : 3;
  }
  return nb <= (int64_t)per_cu * cus;
}

// ---------------------------------------------------------------------------
// K-split FP6 GEMM.  Tiles as above in blocks of 32, with the stages a wavefront
// keeps.  Fitted to 217 shapes (M 64-2048, N 1024-28672, K 2048-28672; weights
// cycling through 300 MB): the estimate is within 10% (one standard deviation),
// and the tile that it picks within 0.3% of the best one on average, 15% at
// worst.
// ---------------------------------------------------------------------------
struct Fp6KsplitTile {
  int ti, tj, waves, bufs, resident;
  double start, round, round_k, tile_k, kn, mn;
};
constexpr Fp6KsplitTile kFp6KsplitTiles[] = {
    {1, 1, 8, 2, 1, 1.33, 0.62, 5.14e-4, 0.0, 2.26e-8, 2.32e-6},
    {1, 2, 8, 2, 1, 1.43, 0.82, 7.42e-4, 0.0, 3.37e-8, 1.57e-6},
    {2, 2, 4, 1, 3, 3.09, 0.23, 1.92e-4, 8.91e-4, 4.00e-8, 5.79e-7},
    {2, 2, 4, 2, 1, 1.72, 0.91, 1.00e-3, 0.0, 3.93e-8, 1.21e-6},
    {2, 3, 4, 2, 1, 1.65, 1.67, 1.21e-3, 0.0, 2.98e-8, 1.06e-6},
    {2, 4, 4, 2, 1, 1.91, 2.03, 1.47e-3, 0.0, 3.17e-8, 1.07e-6},
    {4, 3, 4, 1, 1, 2.16, 3.48, 1.70e-3, 0.0, 3.89e-8, 9.07e-7},
    {4, 4, 4, 1, 1, 1.83, 4.98, 1.99e-3, 0.0, 4.41e-8, 7.70e-7}};
constexpr int kNumFp6KsplitTiles = sizeof(kFp6KsplitTiles) / sizeof(kFp6KsplitTiles[0]);

// The tile with the lowest estimate among those that run at most three rounds,
// where the fitted shapes lie.
inline TilePlan fp6_ksplit_plan(int64_t M, int64_t N, int K, int cus) {
  TilePlan best{-1, 0.0};
  for (int i = 0; i < kNumFp6KsplitTiles; ++i) {
    const Fp6KsplitTile& t = kFp6KsplitTiles[i];
    const int64_t q = ceil_div(ceil_div(ceil_div(M, 32), t.tj) * ceil_div(ceil_div(N, 32), t.ti), cus);
    if (q > 3 * t.resident) continue;
    const double c = ksplit_tile_us(t, q, M, N, K);
    if (best.tile < 0 || c < best.cost) best = {i, c};
  }
  return best;
}

// The K-split kernel's tile where its estimate is below the 192 x 256 kernel's
// (whole rounds of its tiles, 6.9 us + 4.0 ns per k each, and the operands' and
// the output's way) by a margin, or -1 for that kernel.  The margin is 5%, and
// 10% for the shapes below one of its tiles or three of its stages, which run its
// clamped variant: M = 4096, N = 28672, K = 256 72 us there against 131 us on the
// K-split kernel, M = 224, N = 28672, K = 4096 35.6 against 43.5 us, but M = 64,
// N = 2048, K = 14336 80.4 against 9.9 us.
//
// Beyond the fitted M the activations count: the K-split kernel's tiles run
// along M within an XCD, so up to eight L2s read all of them, and each read past
// the second adds 6e-8 us an element (M = 8192, N = 512, K = 2048 20.4 against
// 16.2 us on the 192 x 256 kernel, M = 4096, N = 1024, K = 2048 20.0 against 16.2,
// K = 14336 58 against 80).
inline int fp6_ksplit_or_none(int64_t M, int64_t N, int K, int cus) {
  const bool fits = ceil_div(M, 32) >= 8 && ceil_div(N, 32) >= 6 && K >= 3 * 128;
  const double rounds = (double)ceil_div(ceil_div(M, 256) * ceil_div(N, 192), cus), k = (double)K, n = (double)N;
  const double cost = rounds * (6.91 + 3.99e-3 * k) + 5.98e-8 * k * n + 1.84e-7 * (double)M * n;
  TilePlan p = fp6_ksplit_plan(M, N, K, cus);
  if (p.tile < 0) return -1;
  if (M > 2048) {
    const int64_t tn = ceil_div(ceil_div(N, 32), kFp6KsplitTiles[p.tile].ti), reads = tn < 8 ? tn : 8;
    if (reads > 2) p.cost += 6e-8 * k * (double)M * (double)(reads - 2);
  }
  return p.cost < (fits ? 0.95 : 0.9) * cost ? p.tile : -1;
}

// ---------------------------------------------------------------------------
// Rotate + quantize: whether rows of one block of 28 * 2^j (j = 9, 10; fp16 in,
// codes out) stay in registers (rq28_kernel) or go to the general kernel.  More
// than 64 rows of 28 x 512 (256 rows 7.2 us, against 9.8 us on the general
// kernel's 256 threads a row; its 1024 threads for fewer rows are as fast, 6.6 and
// 6.7 us), and more rows than compute units of 28 x 1024 (256 rows 11.3 us against
// 10.6 us, 300 rows 17.9 us against 19.0 us).  A launch holds less than 2^32
// threads; rows whose 1024 threads are more keep to the general kernel.
// ---------------------------------------------------------------------------
constexpr int kRq28Threads = 1024;
inline bool rotate_in_registers(int64_t M, int K, int f, int j, int cus) {
  if (f != 28 || K != (28 << j) || (M + 31) * kRq28Threads > 0xFFFFFFFFll) return false;
  return (j == 9 && M > 64) || (j == 10 && M > cus);
}

}  // namespace rules
}  // namespace dptq
