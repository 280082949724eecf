// Prints the tile that a lone bf16 GEMM launch takes (gemm_tiles.h) for each
// problem on the command line, written as M,N,K,a_trans.
#include <stdio.h>

#include "gemm_tiles.h"

using namespace merak;

int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    GemmBatch b{};
    int a_t = 0;
    b.n_probs = 1;
    if (sscanf(argv[i], "%d,%d,%d,%d", &b.p[0].M, &b.p[0].N, &b.p[0].K, &a_t) != 4) return 2;
    const char* name = "?";
    switch (choose_tile_alone(b, a_t)) {
      case TILE_256x256_W8_S2: name = "256x256"; break;
      case TILE_256x192_W8_S2: name = "256x192"; break;
      case TILE_256x128_W8_S2: name = "256x128"; break;
      case TILE_192x128_W8_S4: name = "192x128"; break;
      case TILE_128x192_W8_S4: name = "128x192"; break;
      case TILE_128x128_W8_S4: name = "128x128"; break;
      case TILE_64x128_W8_S4: name = "64x128"; break;
    }
    printf("%s\n", name);
  }
  return 0;
}
