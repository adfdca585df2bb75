// Prints what csrc/tile_rules.h picks: one line in, one number out.
#include <cstdio>
#include <cstring>
#include "tile_rules.h"

int main() {
  char rule[16];
  while (std::scanf("%15s", rule) == 1) {
    int np, M, N, K;
    if (!std::strcmp(rule, "f32")) {
      if (std::scanf("%d %d %d %d", &np, &M, &N, &K) != 4) return 1;
      std::printf("%d\n", (int)pahq::pick_f32_tile(np, M, N, K));
    } else if (!std::strcmp(rule, "exact")) {
      int b16, kl, wide, residual;
      if (std::scanf("%d %d %d %d %d %d %d %d", &np, &M, &N, &K, &b16, &kl, &wide, &residual) != 8) return 1;
      std::printf("%d\n", (int)pahq::pick_exact_tile(np, M, N, K, b16, kl, wide, residual));
    } else return 1;
  }
  return 0;
}
