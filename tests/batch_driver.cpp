// Prints the parts that graph replay cuts runs of blocks into: one line per
// "batched blocks" pair on stdin.
#include <cstdio>

#include "batch.hpp"

int main() {
  int batched, n;
  while (std::scanf("%d %d", &batched, &n) == 2) {
    for (int j = 0, nb; j < n; j += nb) std::printf("%d ", nb = rta::graph_run(batched != 0, n - j));
    std::printf("\n");
  }
  return 0;
}
