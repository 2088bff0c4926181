// Which GEMM kernel runs at which sizes: variants, tiles and the rules that choose them (host code, shared
// with its test).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace lrqat {

// bf16 MFMA GEMM family.  C[M][N] = sum_K a(M, K) b(K, N) with the operand
// sources and epilogue chosen by the kernel variant.
enum GemmVariant { kFwd = 0, kDx = 1, kDw = 2 };

// Work split of a GEMM: block tiles of tm x tn outputs (256 or 128 each); for dW in 128 x 128 tiles `split`
// blocks per tile, each for a range of the tokens.
struct GemmPlan {
  int tm = 256, tn = 256;
  int split = 1;
};

// int8 tokens run on the int8 MFMA with one scale per output channel, and where int32 sums of products
// up to 2^14 (16 q n) cannot wrap
inline bool fwd_int8(bool act, bool grouped, int64_t K) { return act && !grouped && K <= (int64_t(1) << 16); }
// what gemm_plan takes as al16
inline bool gemm_al16(GemmVariant v, bool act, int64_t K, int64_t lda, int64_t ldb) {
  if (v == kDw) return lda % 8 == 0 && ldb % 8 == 0;
  return act || (lda % 8 == 0 && K % 64 == 0);
}

// Few tokens: the weights streamed (gemm_small.hip) against the tiles of the general GEMM.  Up to 64 tokens
// the streaming kernel reads them once; past that each 64 tokens read them again, which pays while its
// blocks (32 rows by 64 tokens) are few.  Streamed / tiled, in us: 4096 x 4096, T = 128 (256 blocks) 28 / 33, with groups
// of 128 29 / 46, int8 14 / 24, int8 with groups 20 / 55; T = 256 (512) 46 / 33, 50 / 46, 24 / 24, 33 / 55.  The length
// of K changes both alike (1024 x 14336, T = 512, 256 blocks: 83 / 138; 1024 x 1024: 11 / 13).  The widest layers
// come out even near 64 tokens: 14336 x 4096, T = 48 36 / 38, T = 64 43 / 38, with groups 45 / 47, int8 23 / 22, rows off 16
// bytes 47 / 94.
inline bool fwd_small(int64_t T, int64_t m) { return T <= 64 || (T <= 512 && ((m + 31) / 32) * ((T + 63) / 64) < 384); }

// Tiles: the time of a launch is its rounds over the chip (256 CUs; two 128 x 128 blocks share one) times
// the time of a round, and a 256 x 256 tile has the best rate but leaves CUs idle when an output has few
// of them.  The weights below are rounds of each tile against a round of 256 x 256 tiles, measured on
// outputs that fill the chip (4096 x 4096, T = 8192: forward 226 us with 256 x 256 tiles, 251 / 286 / 279 with
// 256 x 128, 128 x 256, 128 x 128; dX 246, 289 / 312 / 347) or at most once.  What the choice gives: forward of
// 640 tokens through 11008 x 4096 (129 tiles of 256 x 256) 98 -> 70 us, of 4096 tokens through 1024 x 4096 94 ->
// 49; dX of 2048 tokens through 14336 x 4096 (128 tiles) 339 -> 254.
//
// dW: its epilogue and its partial sums grow with the number of tiles, so an output of more than 128 tiles of
// 256 x 256 keeps them.  A smaller one, which would leave half the chip without a tile, takes 128 x 128 tiles if one
// per CU covers it, else 256 x 128 (T = 4096: 1024 x 4096, 256 small tiles, 146 -> 70 us; 2048 x 2500, 153 -> 96 in
// 256 x 128, 105 in 128 x 128).  Where even 128 x 128 tiles are at most half the CUs, the blocks of a tile share its
// tokens, and a second launch adds their float32 sums before anything is rounded: at least eight K-tiles for
// each, which is what that launch costs (1024 x 1024: T = 2048 42 -> 30 us in four ranges, T = 512 21 -> 23 in
// two), and 16 ranges at most, which one block adds in turn (256 x 256, T = 8192: 124 us, 36 in 16, 42 in 32).
//
// Against every other tile on 110 drawn layers (m and k 256 .. 14336, T 576 .. 8192, every form of the weights; 330
// GEMMs) the choice is the best or within 4% of it but for 17.  Most of those would be faster in 128 x 128:
// forwards of short rows (chosen / 128 x 128: 5120 x 320, T = 7104 48 / 39 us; 13824 x 640, T = 1280 with groups 46 / 41) and dW of few
// tokens in 130 to 350 large tiles (640 x 12224, T = 704 53 / 37; 5120 x 4096, T = 1152 127 / 111).
// al16: the bfloat16 rows start on 16 bytes (and a K-contiguous one has no partial K-tile)
inline GemmPlan gemm_plan(GemmVariant v, bool act, bool grouped, bool al16, int64_t M, int64_t N, int64_t K) {
  GemmPlan g;
  auto tiles = [&](int tm, int tn) { return ((M + tm - 1) / tm) * ((N + tn - 1) / tn); };
  if (v == kDw) {
    const int64_t n22 = tiles(128, 128);
    if (n22 <= 256) {
      g.tm = g.tn = 128;
      g.split = int(std::max<int64_t>(1, std::min<int64_t>({256 / n22, (K + 63) / 64 / 8, 16})));
    } else if (tiles(256, 256) <= 128) {
      g.tn = 128;
    }
    return g;
  }
  if (!al16) {  // rows off 16 bytes: the small tile, whose second block per CU hides the loads that cross lines
    g.tm = g.tn = 128;
    return g;
  }
  struct Cost { double t42, t24, t22, t22_one; };  // a round of 256 x 128, 128 x 256, 128 x 128 (two and one per CU)
  constexpr double never = 1e30;  // the other tiles are ahead wherever it could be taken
  const Cost c = v == kFwd ? (act ? Cost{never, never, 0.54, 0.46} : Cost{0.57, never, 0.63, 0.44})
                           : (grouped ? Cost{0.78, 0.74, 0.88, 0.55} : Cost{0.59, 0.63, 0.70, 0.45});
  auto rounds = [](int64_t n, int64_t slots) { return double((n + slots - 1) / slots); };
  double best = rounds(tiles(256, 256), 256);
  auto offer = [&](int tm, int tn, double cost) {
    if (cost < best) {
      best = cost;
      g.tm = tm;
      g.tn = tn;
    }
  };
  offer(256, 128, rounds(tiles(256, 128), 256) * c.t42);
  offer(128, 256, rounds(tiles(128, 256), 256) * c.t24);
  const int64_t n22 = tiles(128, 128);
  offer(128, 128, n22 <= 256 ? c.t22_one : rounds(n22, 512) * c.t22);
  return g;
}

}  // namespace lrqat
