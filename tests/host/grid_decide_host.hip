// Host driver for the float32 decisions of the grid pass: reads lines
// "f b tz d0 c0 d1 c1 d2 c2 d3 c3" (four codes with their deltas; floats as
// hex bits) and prints, for the byte-parallel path, its regime, the word of
// results, the clip marks and a mask of the certain elements, and for the
// rounding path four integers and a mask of the certain ones.
#include <cmath>
#include <cstdio>
#include <cstring>

#include "grid_swar.h"

using namespace lrqat;

static float flt(unsigned bits) {
  float x;
  std::memcpy(&x, &bits, 4);
  return x;
}

int main() {
  int f, b, code[4];
  unsigned tb, db[4];
  while (std::scanf("%d %d %x %x %d %x %d %x %d %x %d", &f, &b, &tb, &db[0], &code[0], &db[1], &code[1], &db[2], &code[2],
                    &db[3], &code[3]) == 11) {
    const float tz = flt(tb);
    uint32_t word = 0, carry = 0, clip = 0;
    int sure1 = 0, sure2 = 0, v2[4];
    float amx = 0.f, vab = 0.f, u[4], v[4];
    for (int j = 0; j < 4; ++j) {
      word |= uint32_t(code[j] & 255) << (8 * j);
      amx = std::fmax(amx, std::fabs(flt(db[j])));
    }
    for (int j = 0; j < 4; ++j) {
      if (f) {
        const float w = grid_w(word, j, f, flt(db[j]), 1.f);
        carry |= uint32_t(!std::signbit(w)) << (8 * j);
        sure1 |= int(std::fabs(w) > tz) << j;
      }
      u[j] = __builtin_fmaf(flt(db[j]), 1.f, float(code[j]) * std::ldexp(1.f, -f));
      const float vm = u[j] + kGridMagic;
      uint32_t bits;
      std::memcpy(&bits, &vm, 4);
      v2[j] = int(bits << 10) >> 10;
      v[j] = vm - kGridMagic;
      vab = std::fmax(vab, std::fabs(v[j]));
    }
    const float thr = grid_certain(tz, vab);
    for (int j = 0; j < 4; ++j) sure2 |= int(std::fabs(u[j] - v[j]) < thr) << j;
    const uint32_t q = f ? swar_carry_q8(word, carry, f, b, clip) : 0;
    std::printf("%d %x %x %x %d %d %d %d %x\n", int(f != 0 && amx < 0.5f - tz - 0x1p-20f), q, clip, sure1, v2[0], v2[1], v2[2],
                v2[3], sure2);
  }
  return 0;
}
