// Prints the routes of the GEMM dispatch rules for shapes read from stdin, at 256
// compute units:
//   int8 M N K bits -> the kernel (decode, tile, wide or ksplit), and for ksplit
//                      its tile as TI x TJ x wavefronts;
//   fp6 M N K       -> wide, or TI x TJ x wavefronts x stages;
//   decode M N K bits layout (1: decode layout) -> for M <= 16, "regs" with blocks
//                      x chunks in flight, or "ksplit" with TI x TJ x wavefronts;
//   fused M K f j N -> "one" or "two" launches for h = f * 2^j;
//   rotate M K f j  -> "registers" or "general" for h = f * 2^j;
//   tiles           -> every tile of the tables, one a line, then an empty line.
#include "gemm_rules.h"

#include <cstdio>
#include <cstring>

using namespace dptq;
using namespace dptq::rules;

int main() {
  const int cus = 256;
  char what[16];
  while (std::scanf("%15s", what) == 1) {
    long M = 0, N = 0;
    int K = 0, bits = 0;
    if (!std::strcmp(what, "int8")) {
      if (std::scanf("%ld %ld %d %d", &M, &N, &K, &bits) != 4) return 1;
      const GemmRoute r = gemm_route(M, N, K, bits, cus);
      if (r.kernel == kGemmKsplit) {
        const KsplitTile t = ksplit_tile(bits, r.tile);
        std::printf("ksplit %dx%dx%d\n", t.ti, t.tj, t.waves);
      } else {
        std::printf("%s\n", r.kernel == kGemmDecode ? "decode" : r.kernel == kGemmWide ? "wide" : "tile");
      }
    } else if (!std::strcmp(what, "fp6")) {
      if (std::scanf("%ld %ld %d", &M, &N, &K) != 3) return 1;
      const int i = fp6_ksplit_or_none(M, N, K, cus);
      if (i < 0) {
        std::printf("wide\n");
      } else {
        const Fp6KsplitTile t = kFp6KsplitTiles[i];
        std::printf("ksplit %dx%dx%dx%d\n", t.ti, t.tj, t.waves, t.bufs);
      }
    } else if (!std::strcmp(what, "decode")) {
      int layout = 0;
      if (std::scanf("%ld %ld %d %d %d", &M, &N, &K, &bits, &layout) != 5) return 1;
      if (decode_in_regs(M, N, K, bits, layout != 0, cus)) {
        const int blocks = decode_blocks(M, N, bits, cus);
        std::printf("regs %dx%d\n", blocks, decode_batch(M, N, K, blocks, cus));
      } else {
        const DecodeTile t = decode_tile(N, cus);
        std::printf("ksplit %dx1x%d\n", t.ti, t.waves);
      }
    } else if (!std::strcmp(what, "fused")) {
      int f = 0, j = 0;
      if (std::scanf("%ld %d %d %d %ld", &M, &K, &f, &j, &N) != 5) return 1;
      std::printf("%s\n", decode_one_launch(M, K, f, j, N, cus) ? "one" : "two");
    } else if (!std::strcmp(what, "rotate")) {
      int f = 0, j = 0;
      if (std::scanf("%ld %d %d %d", &M, &K, &f, &j) != 4) return 1;
      std::printf("%s\n", rotate_in_registers(M, K, f, j, cus) ? "registers" : "general");
    } else if (!std::strcmp(what, "tiles")) {
      for (int b = 4; b <= 8; b += 4)
        for (int i = 0; i < ksplit_tiles(b); ++i) {
          const KsplitTile t = ksplit_tile(b, i);
          std::printf("int8 %d %dx%dx%d\n", b, t.ti, t.tj, t.waves);
        }
      for (const Fp6KsplitTile& t : kFp6KsplitTiles)
        std::printf("fp6 4 %dx%dx%dx%d\n", t.ti, t.tj, t.waves, t.bufs);
      std::printf("\n");
    } else {
      return 1;
    }
  }
  return 0;
}
