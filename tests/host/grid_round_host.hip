// Host driver for the library's exact rounding of Phi0 + delta: reads lines
// "code f delta_bits_hex" (delta as float64 bits) and prints the decision.
#include <cstdio>
#include <cstring>

#include "common.h"

int main() {
  int code, f;
  unsigned long long bits;
  while (std::scanf("%d %d %llx", &code, &f, &bits) == 3) {
    double delta;
    std::memcpy(&delta, &bits, 8);
    std::printf("%d\n", lrqat::grid_round_f64(code, f, delta));
  }
  return 0;
}
