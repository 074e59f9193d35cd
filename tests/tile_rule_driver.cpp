// Prints what the tile rules of the row GEMM answer: arguments m_cap counted ncols kc, four at a time; one line
// "large medium" each.
#include <cstdio>
#include <cstdlib>

#include "gemm_shape.h"

int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int m = std::atoi(argv[i]), counted = std::atoi(argv[i + 1]), n = std::atoi(argv[i + 2]), k = std::atoi(argv[i + 3]);
    std::printf("%d %d\n", (int)spa::large_tiles(m, counted != 0, n, k), (int)spa::medium_tiles(m, n));
  }
  return 0;
}
