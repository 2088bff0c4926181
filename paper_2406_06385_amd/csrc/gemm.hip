// Dispatch of the bf16 MFMA GEMM variants (one translation unit per variant
// family, see gemm_impl.h) and the deterministic reduction of the rank-r
// partial products.
#include <algorithm>

#include "kernels.h"

namespace lrqat {

// Deterministic sum of partial buffers: out = (accumulate ? out : 0) + c * sum_p part[p].
__global__ __launch_bounds__(256) void k_reduce(const float* __restrict__ part, int64_t nparts, int64_t n,
                                                float* __restrict__ out, float c, int accumulate) {
  const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= n) return;
  float s = 0.f;
  for (int64_t q = 0; q < nparts; ++q) s += part[q * n + idx];
  out[idx] = (accumulate ? out[idx] : 0.f) + c * s;
}

// ds[row][grp] = (accumulate ? ds : 0) + the partials of the group's 32-column chunks.
// 2^lg consecutive lanes share a (row, group): each takes every 2^lg-th chunk (coalesced), and their sums
// meet in a fixed tree, so the result is deterministic.  (One thread per row, whose loads are a row apart,
// took 47 us for 4096 rows of 344 chunks.)
template <class I>
__device__ __forceinline__ void reduce_ds(const Reduce2Args& ra, int64_t t) {
  const int64_t idx = t >> ra.lg;
  const bool in = idx < ra.m * ra.ngroups;
  const int l = int(t & ((1 << ra.lg) - 1));
  float s = 0.f;
  if (in) {
    const int64_t row = int64_t(I(idx) / I(ra.ngroups)), grp = idx - row * ra.ngroups;
    const int64_t c0 = grp * ra.cpg, c1 = min(ra.nchunks, c0 + ra.cpg);
    const float* src = ra.ds_part + row * ra.ldds;
    for (int64_t c = c0 + l; c < c1; c += int64_t(1) << ra.lg) s += src[c];
  }
  for (int off = (1 << ra.lg) >> 1; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (in && l == 0) ra.ds[idx] = (ra.accumulate ? ra.ds[idx] : 0.f) + s;
}

// The gradients of A, B and s in one launch: out = (accumulate ? out : 0) + c * sum_p part[p] for
// dA (side 0) and dB (side 1), then the blocks of ds.  Four consecutive elements per thread; the partial
// buffers are summed in a fixed order (two interleaved running sums), so results are deterministic.
__global__ __launch_bounds__(256) void k_reduce2(Reduce2Args ra) {
  if (int64_t(blockIdx.x) >= ra.nblocks) {  // block-uniform
    const int64_t td = (int64_t(blockIdx.x) - ra.nblocks) * 256 + threadIdx.x;
    if (ra.m * ra.ngroups < (int64_t(1) << 31)) reduce_ds<uint32_t>(ra, td);
    else reduce_ds<int64_t>(ra, td);
    return;
  }
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t nt0 = (ra.n[0] + 3) / 4;
  const int side = t < nt0 ? 0 : 1;
  const int64_t idx = 4 * (side ? t - nt0 : t);
  const int64_t n = ra.n[side], np = ra.nparts[side];
  if (idx >= n) return;
  const float* part = ra.part[side] + idx;
  float* out = ra.out[side] + idx;
  if (ra.vec[side] && idx + 4 <= n) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
    int64_t q = 0;
    for (; q + 2 <= np; q += 2) {
      s0 += *reinterpret_cast<const f32x4*>(part + q * n);
      s1 += *reinterpret_cast<const f32x4*>(part + (q + 1) * n);
    }
    if (q < np) s0 += *reinterpret_cast<const f32x4*>(part + q * n);
    const f32x4 prev = ra.accumulate ? *reinterpret_cast<const f32x4*>(out) : f32x4{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<f32x4*>(out) = prev + ra.c * (s0 + s1);
  } else {
    for (int64_t e = 0; e < 4 && idx + e < n; ++e) {
      float s0 = 0.f, s1 = 0.f;
      int64_t q = 0;
      for (; q + 2 <= np; q += 2) {
        s0 += part[q * n + e];
        s1 += part[(q + 1) * n + e];
      }
      if (q < np) s0 += part[q * n + e];
      out[e] = (ra.accumulate ? out[e] : 0.f) + ra.c * (s0 + s1);
    }
  }
}

hipError_t launch_reduce2(const Reduce2Args& ra0, hipStream_t st) {
  Reduce2Args ra = ra0;
  ra.nblocks = ((ra.n[0] + 3) / 4 + (ra.n[1] + 3) / 4 + 255) / 256;
  int64_t nds = 0;
  if (ra.ds) {
    ra.lg = 0;  // lanes per sum of ds: up to a wave, no more than its chunks
    while (ra.lg < 6 && (int64_t(2) << ra.lg) <= ra.cpg) ++ra.lg;
    nds = (((ra.m * ra.ngroups) << ra.lg) + 255) / 256;
  }
  k_reduce2<<<unsigned(ra.nblocks + nds), 256, 0, st>>>(ra);
  return hipGetLastError();
}

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
GemmPlan gemm_plan(GemmVariant v, bool act, bool grouped, bool al16, int64_t M, int64_t N, int64_t K) {
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

hipError_t launch_gemm(GemmVariant v, bool act, bool grouped, int opt, const GemmArgs& p, hipStream_t st) {
  const bool zp = (opt & kOptZ) != 0, i8 = (opt & kOptQ8) != 0;
  switch (v) {
    case kFwd:
      if (fwd_int8(act, grouped, p.K)) return launch_fwd_int8(i8, zp, p, st);
      if (act) return i8 ? launch_fwd_act_i8(grouped, zp, p, st) : launch_fwd_act_i4(grouped, zp, p, st);
      return i8 ? launch_fwd_i8(grouped, zp, p, st) : launch_fwd_i4(grouped, zp, p, st);
    case kDx:
      return i8 ? launch_dx_i8(grouped, zp, p, st) : launch_dx_i4(grouped, zp, p, st);
    case kDw:  // W4A8 runs the dW GEMM on X_hat in bfloat16
      if (act) return hipErrorInvalidValue;
      return grouped ? launch_dw_grp(p, st) : launch_dw_pc(p, st);
  }
  return hipErrorInvalidValue;
}

// dst[row][0 .. ldd) = src[row][0 .. w) followed by zeros; one thread per destination byte.
__global__ __launch_bounds__(256) void k_repack_rows(const uint8_t* __restrict__ src, int64_t m, int64_t w,
                                                     uint8_t* __restrict__ dst, int64_t ldd) {
  const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= m * ldd) return;
  const int64_t row = idx / ldd, col = idx % ldd;
  dst[idx] = col < w ? src[row * w + col] : uint8_t(0);
}

hipError_t launch_repack_rows(const uint8_t* src, int64_t m, int64_t w, uint8_t* dst, int64_t ldd, hipStream_t st) {
  const int64_t n = m * ldd;
  if (n == 0) return hipSuccess;
  k_repack_rows<<<unsigned((n + 255) / 256), 256, 0, st>>>(src, m, w, dst, ldd);
  return hipGetLastError();
}

hipError_t launch_reduce(const float* part, int64_t nparts, int64_t n, float* out, float c, int accumulate,
                         hipStream_t st) {
  k_reduce<<<unsigned((n + 255) / 256), 256, 0, st>>>(part, nparts, n, out, c, accumulate);
  return hipGetLastError();
}

}  // namespace lrqat
