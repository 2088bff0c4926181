// bf16 MFMA GEMMs of the LR-QAT layer on gfx950.
//
//   kFwd  Y  = X_hat W_hat^T      M = T, N = m, K = k   (Section 3, Eq. lr_qat)
//   kDx   dX = dY W_hat           M = T, N = k, K = m
//   kDw   dW = dY^T X_hat         M = m, N = k, K = T, never stored: the
//         epilogue forms G = s * M * dW and the rank-r partial products
//         G B^T and A^T G (Section 3, STE gradients w.r.t. A and B).
//
// W_hat enters as the integer grid q written by the grid pass (packed int4, or
// int8 for grids of 5..7 bits); the operand loaders unpack it into bfloat16
// tiles in LDS (q - z is exact in bfloat16 for |q - z| <= 256), with the scale
// s applied in the epilogue (forward, per channel) or folded into the tile
// (dX, and the forward with group-wise scales).
//
// Block tile 256 x 256 x 64, or 256 x 128, 128 x 256, 128 x 128 where that fills the
// chip better; four waves in a 2 x 2 arrangement, each wave a quarter of it in
// MFMA 32x32x16 blocks.  Two LDS stages of bfloat16 tiles; the next K-tile is
// fetched into registers while the current one feeds the MFMAs.  The forward
// and dX output tiles leave through LDS as whole row segments.
//
// The W4A8 forward with one scale per output channel runs on the int8 MFMA
// (32x32x32, twice the bf16 rate, K-tiles of 128): token codes and q are int8
// operands, the sums exact in int32, and s, s_x and a zero offset (through the
// token's sum of codes) enter in the epilogue.
#pragma once

#include "kernels.h"

namespace lrqat {

// Operand tiles in LDS are [256 rows][64] bfloat16 (128-byte rows of eight
// 16-byte chunks).  Chunk c of row r sits at chunk slot c ^ g(r) with
// g(r) = (r & 7) ^ ((r >> 3) & 1): any 8 consecutive rows read at one chunk
// hit 8 different slots (32 banks), any 16 consecutive rows hit 16 different
// (row parity, slot) pairs (64 banks).  g depends on r mod 16 only, so the
// fragments of row blocks 32 apart are constant offsets of one address.
__device__ __forceinline__ int tile_g(int row) { return (row & 7) ^ ((row >> 3) & 1); }
__device__ __forceinline__ int tile_off(int row, int chunk) { return row * 64 + ((chunk ^ tile_g(row)) << 3); }

// ------------------------------------------------------------------ buffer resources
// Operands are read with raw buffer loads.  A load whose per-lane offset is
// at or past the resource's num_records returns zeros, so a tile that
// overhangs the end of a tensor needs no per-lane branch: each resource
// starts at the tile's origin and all strides stay in the per-lane offset.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, int64_t bytes) {
  const int64_t n = bytes < 0 ? 0 : (bytes > int64_t(0xFFFFFFFF) ? int64_t(0xFFFFFFFF) : bytes);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), short(0), int(uint32_t(n)), 0x00020000);
}
__device__ __forceinline__ u32x4 ld128(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, int(off), 0, 0));
}
__device__ __forceinline__ u32x2 ld64(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, int(off), 0, 0));
}
__device__ __forceinline__ uint32_t ld32(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, int(off), 0, 0);
}
__device__ __forceinline__ uint32_t ld16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b16(r, int(off), 0, 0);
}
__device__ __forceinline__ float ldf(__amdgpu_buffer_rsrc_t r, uint32_t off) { return __uint_as_float(ld32(r, off)); }

// Zero the elements of an 8-wide bfloat16 chunk at column kk that lie at or past K.
__device__ __forceinline__ u32x4 mask_tail(u32x4 v, int kk, int K) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = (kk + 2 * q < K) ? 0x0000FFFFu : 0u, hi = (kk + 2 * q + 1 < K) ? 0xFFFF0000u : 0u;
    v[q] &= lo | hi;
  }
  return v;
}

// Alignment of the bfloat16 rows of an operand (its leading dimension ld): rows that start on 16 bytes
// and have no partial K-tile; rows that start on dwords (ld even); odd ld, where every other row starts in
// the middle of a dword and is loaded from the dword before and shifted into place when it is stored.
enum : int { kAlDword = 0, kAl16 = 1, kAlOdd = 2 };

// Resource over `bytes` bytes, rounded up to whole dwords: the range check of a multi-dword load works
// per dword, so the last element of an odd count would read as zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc4(const void* base, int64_t bytes) { return rsrc(base, (bytes + 3) & ~int64_t(3)); }

// v shifted right by two bytes, x supplying the top half word.
__device__ __forceinline__ u32x4 shift_half(const u32x4& v, uint32_t x, uint32_t bytes) {
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = __builtin_amdgcn_alignbyte(q < 3 ? v[(q + 1) & 3] : x, v[q], bytes);
  return o;
}

// ------------------------------------------------------------------ K-contiguous bf16 source
// 32 NR x 64 tile of a row-major [rows][K] bfloat16 matrix (forward X, dX's dY);
// thread t loads chunk t%8 of rows t/8 + 32 i.  Off the 16-byte path, columns
// >= K are masked (they hold the next row's values).
template <int AL, int NR>
struct RegsKc {
  u32x4 v[NR];
  uint32_t x[AL == kAlOdd ? NR : 1];
  u32x4 msk;
  uint32_t sh;
};

template <int AL, int NR>
__device__ __forceinline__ void load_kc_bf16(RegsKc<AL, NR>& R, const uint16_t* __restrict__ src, int64_t ld,
                                             int64_t row0, int64_t nrows, int64_t k0, int64_t K, int w0, int w1) {
  const int t = threadIdx.x;
  const auto r = rsrc4(src + row0 * ld, (nrows - row0) * ld * 2);
  const int kk = int(k0) + 8 * (t & 7);
  const uint32_t at = uint32_t(((t >> 3) * ld + kk) * 2), step = uint32_t(32 * ld * 2);
  const uint32_t base = AL == kAlOdd ? at & ~3u : at;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    if (i < w0 || i >= w1) continue;
    R.v[i] = ld128(r, base + i * step);
    if constexpr (AL == kAlOdd) R.x[i] = ld32(r, base + i * step + 16);
  }
  if (w0 > 0 || w1 <= 0) return;
  if constexpr (AL == kAlOdd) R.sh = at & 3u;
  if constexpr (AL != kAl16) R.msk = mask_tail(u32x4{~0u, ~0u, ~0u, ~0u}, kk, int(K));
}

// Each operand tile is written to LDS as 16-byte stores per thread; the *_one
// functions do store number w, so the main loop can spread them between MFMA
// groups.
template <int AL, int NR>
__device__ __forceinline__ void store_kc_one(uint16_t* tile, const RegsKc<AL, NR>& R, int i) {
  const int t = threadIdx.x;
  u32x4 v = R.v[i];
  if constexpr (AL == kAlOdd) v = shift_half(v, R.x[i], R.sh);
  if constexpr (AL != kAl16) v &= R.msk;
  *reinterpret_cast<u32x4*>(tile + tile_off((t >> 3) + 32 * i, t & 7)) = v;
}

// ------------------------------------------------------------------ K-contiguous int8 source (W4A8 codes, widened to bf16)
// n [T][ld] is zero beyond column k, so no K mask is needed.
template <int NR>
struct RegsKc8 {
  u32x2 v[NR];
};

template <int NR>
__device__ __forceinline__ void load_kc_i8(RegsKc8<NR>& R, const int8_t* __restrict__ src, int64_t ld,
                                           int64_t row0, int64_t nrows, int64_t k0, int w0, int w1) {
  const int t = threadIdx.x;
  const auto r = rsrc(src + row0 * ld, (nrows - row0) * ld);
  const uint32_t base = uint32_t((t >> 3) * ld + k0 + 8 * (t & 7)), step = uint32_t(32 * ld);
#pragma unroll
  for (int i = 0; i < NR; ++i)
    if (i >= w0 && i < w1) R.v[i] = ld64(r, base + i * step);
}

template <int NR>
__device__ __forceinline__ void store_kc_i8_one(uint16_t* tile, const RegsKc8<NR>& R, int i) {
  const int t = threadIdx.x;
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t w = R.v[i][q >> 1];
    o[q] = pack_bf16x2(float(sbyte(w, 2 * (q & 1))), float(sbyte(w, 2 * (q & 1) + 1)));
  }
  *reinterpret_cast<u32x4*>(tile + tile_off((t >> 3) + 32 * i, t & 7)) = o;
}

// ------------------------------------------------------------------ zero offsets
// z[row][grp] (z shaped like s; grp = 0 for one offset per row) as an int;
// rows past the end read 0.
__device__ __forceinline__ int ld_z(__amdgpu_buffer_rsrc_t rz, int64_t idx) { return int(ld32(rz, uint32_t(idx * 4))); }

// ------------------------------------------------------------------ packed q, K-contiguous (forward B)
// 128 NH weight rows x 64 K-values (32 bytes); thread t takes 16 bytes
// (32 values) of rows t/2 + 128 i.  q is zero past column k.
template <int NH>
struct RegsQKc {
  u32x4 v[NH];
  float sc[NH];
  int zi[NH];
};

template <bool GRP, bool ZP, int NH>
__device__ __forceinline__ void load_q_kc(RegsQKc<NH>& R, const GemmArgs& p, int64_t row0, int64_t k0, int w0, int w1) {
  const int t = threadIdx.x;
  const int64_t kk = k0 + 32 * (t & 1);
  const auto rq = rsrc(static_cast<const uint8_t*>(p.b) + row0 * p.ldb, (p.N - row0) * p.ldb);
  const uint32_t base = uint32_t((t >> 1) * p.ldb + (kk >> 1)), step = uint32_t(128 * p.ldb);
#pragma unroll
  for (int i = 0; i < NH; ++i)
    if (i >= w0 && i < w1) R.v[i] = ld128(rq, base + i * step);
  if (w0 > 0 || w1 <= 0) return;  // scales and offsets with the first load
  const int64_t grp = GRP ? kk / p.gsize : 0;
  if (GRP) {
    const auto rs = rsrc(p.s + row0 * p.ngroups, (p.N - row0) * p.ngroups * 4);
    const uint32_t sb = uint32_t(((t >> 1) * p.ngroups + grp) * 4), sstep = uint32_t(128 * p.ngroups * 4);
#pragma unroll
    for (int i = 0; i < NH; ++i) R.sc[i] = ldf(rs, sb + i * sstep);
  }
  if (ZP) {
    const auto rz = rsrc(p.z + row0 * p.ngroups, (p.N - row0) * p.ngroups * 4);
#pragma unroll
    for (int i = 0; i < NH; ++i) R.zi[i] = ld_z(rz, ((t >> 1) + 128 * i) * p.ngroups + grp);
  }
}

template <bool GRP, bool ZP, int NH>
__device__ __forceinline__ void store_q_kc_one(uint16_t* tile, const RegsQKc<NH>& R, int w8) {
  const int t = threadIdx.x;
  const int i = w8 >> 2, c = w8 & 3;  // row half, 16-byte chunk
  const int row = (t >> 1) + 128 * i;
  const uint32_t w = R.v[i][c];
  u32x4 o;
  if constexpr (!GRP && !ZP) {
    o = unpack_q16(w);  // q / 16: the epilogue's scale has the factor back
  } else
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int na = nibble(w, 2 * q), nb = nibble(w, 2 * q + 1);
    if (ZP) {
      na -= R.zi[i];
      nb -= R.zi[i];
    }
    float a = float(na), b = float(nb);
    if (GRP) {
      a *= R.sc[i];
      b *= R.sc[i];
    }
    o[q] = pack_bf16x2(a, b);
  }
  *reinterpret_cast<u32x4*>(tile + tile_off(row, 4 * (t & 1) + c)) = o;
}

// ------------------------------------------------------------------ int8 q, K-contiguous (forward B, 5..7-bit grids)
// 32 NR weight rows x 64 bytes: thread t loads 8 bytes of rows t/8 + 32 i; q is zero past column k.
template <int NR>
struct RegsQKc8 {
  u32x2 v[NR];
  float sc[NR];
  int zi[NR];
};

template <bool GRP, bool ZP, int NR>
__device__ __forceinline__ void load_q_kc8(RegsQKc8<NR>& R, const GemmArgs& p, int64_t row0, int64_t k0, int w0, int w1) {
  const int t = threadIdx.x;
  const auto rq = rsrc(static_cast<const uint8_t*>(p.b) + row0 * p.ldb, (p.N - row0) * p.ldb);
  const int64_t kk = k0 + 8 * (t & 7);
  const uint32_t base = uint32_t((t >> 3) * p.ldb + kk), step = uint32_t(32 * p.ldb);
#pragma unroll
  for (int i = 0; i < NR; ++i)
    if (i >= w0 && i < w1) R.v[i] = ld64(rq, base + i * step);
  if (w0 > 0 || w1 <= 0) return;
  const int64_t grp = GRP ? kk / p.gsize : 0;
  if (GRP) {
    const auto rs = rsrc(p.s + row0 * p.ngroups, (p.N - row0) * p.ngroups * 4);
#pragma unroll
    for (int i = 0; i < NR; ++i) R.sc[i] = ldf(rs, uint32_t((((t >> 3) + 32 * i) * p.ngroups + grp) * 4));
  }
  if (ZP) {
    const auto rz = rsrc(p.z + row0 * p.ngroups, (p.N - row0) * p.ngroups * 4);
#pragma unroll
    for (int i = 0; i < NR; ++i) R.zi[i] = ld_z(rz, ((t >> 3) + 32 * i) * p.ngroups + grp);
  }
}

template <bool GRP, bool ZP, int NR>
__device__ __forceinline__ void store_q_kc8_one(uint16_t* tile, const RegsQKc8<NR>& R, int i) {
  const int t = threadIdx.x;
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t w = R.v[i][q >> 1];
    int na = sbyte(w, 2 * (q & 1)), nb = sbyte(w, 2 * (q & 1) + 1);
    if (ZP) {
      na -= R.zi[i];
      nb -= R.zi[i];
    }
    float a = float(na), b = float(nb);
    if (GRP) {
      a *= R.sc[i];
      b *= R.sc[i];
    }
    o[q] = pack_bf16x2(a, b);
  }
  *reinterpret_cast<u32x4*>(tile + tile_off((t >> 3) + 32 * i, t & 7)) = o;
}

// ------------------------------------------------------------------ operands of the int8 MFMA (W4A8 forward)
// A K-tile holds 128 int8 values in the 128 bytes of a tile row.  The token
// codes are copied as they are (their rows are zero-padded to whole tiles), an
// int8 grid too; packed q becomes bytes 16 q (two ANDs and a shift for eight
// values, two byte permutes to bring them into column order), and the int32 sum
// is shifted back in the epilogue.  Thread t takes 16 bytes (32 values) of rows
// t/4 + 64 i.
template <int NQ>
struct RegsQ16 {
  u32x4 v[NQ];
};

template <int NQ>
__device__ __forceinline__ void load_q_x16(RegsQ16<NQ>& R, const GemmArgs& p, int64_t row0, int64_t k0, int w0, int w1) {
  const int t = threadIdx.x;
  const auto rq = rsrc(static_cast<const uint8_t*>(p.b) + row0 * p.ldb, (p.N - row0) * p.ldb);
  const uint32_t base = uint32_t((t >> 2) * p.ldb + (k0 >> 1) + 16 * (t & 3)), step = uint32_t(64 * p.ldb);
#pragma unroll
  for (int i = 0; i < NQ; ++i)
    if (i >= w0 && i < w1) R.v[i] = ld128(rq, base + i * step);
}

template <int NQ>
__device__ __forceinline__ void store_q_x16_one(uint16_t* tile, const RegsQ16<NQ>& R, int w) {
  const int t = threadIdx.x;
  const int i = w >> 1, h = w & 1;  // row group, 16-byte half of the 32 values
  u32x4 o;
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    const uint32_t x = R.v[i][2 * h + d];
    const uint32_t ev = (x << 4) & 0xF0F0F0F0u, od = x & 0xF0F0F0F0u;
    o[2 * d] = __builtin_amdgcn_perm(od, ev, 0x05010400u);
    o[2 * d + 1] = __builtin_amdgcn_perm(od, ev, 0x07030602u);
  }
  *reinterpret_cast<u32x4*>(tile + tile_off((t >> 2) + 64 * i, 2 * (t & 3) + h)) = o;
}

// ------------------------------------------------------------------ K-strided sources
// Tile rows are the index contiguous in memory, K the strided one.  Thread t
// covers RW consecutive tile rows RW (t/8) .. (one vector per K-line; RW = 8
// for a 256-row tile, 4 for 128 rows of q) of the 8 K-lines 8 (t%8) .. +7 and
// transposes them in registers into RW chunks; the 8 lanes of a K-group fill
// one 128-byte row segment of LDS.  128 rows of bfloat16 keep the 16-byte
// vectors (8 tile rows 8 (t/16) ..) and take 4 K-lines 4 (t%16) .. +3 each, in
// chunks of 8 bytes.
// Columns past a tensor's width only feed output rows/columns that the
// epilogue discards; K-lines past the end read as zeros.

// packed q (dX B): K = weight rows (m), tile rows = weight columns (k).
// Values are scaled by their row's (or row-group's) s before rounding to bf16.
struct RegsQKs {
  uint32_t w[8];
  float sc[8];
  int zi[8];
};

// Scales (and zero offsets) of the 8 K-lines (weight rows) k0 + 8 kg .. +7 at column col.
template <bool GRP, bool ZP>
__device__ __forceinline__ void load_ks_scales(float (&sc)[8], int (&zi)[8], const GemmArgs& p, int64_t k0, int kg,
                                               int64_t col) {
  const int64_t grp = GRP ? col / p.gsize : 0;
  if (GRP) {
    const auto rs = rsrc(p.s + k0 * p.ngroups, (p.K - k0) * p.ngroups * 4);
    const uint32_t sb = uint32_t((8 * kg * p.ngroups + grp) * 4), sstep = uint32_t(p.ngroups * 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) sc[e] = ldf(rs, sb + e * sstep);
  } else {
    // the 8 rows' scales are consecutive: two 16-byte loads (rows past K read as zeros)
    const auto rs = rsrc(p.s + k0, (p.K - k0) * 4);
    const u32x4 s0 = ld128(rs, uint32_t(8 * kg * 4)), s1 = ld128(rs, uint32_t((8 * kg + 4) * 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[e] = __uint_as_float(s0[e]);
      sc[4 + e] = __uint_as_float(s1[e]);
    }
  }
  if (ZP) {
    const auto rz = rsrc(p.z + k0 * p.ngroups, (p.K - k0) * p.ngroups * 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) zi[e] = ld_z(rz, (8 * kg + e) * p.ngroups + grp);
  }
}

template <bool GRP, bool ZP, int RW>
__device__ __forceinline__ void load_q_ks(RegsQKs& R, const GemmArgs& p, int64_t n0, int64_t k0, int w0, int w1) {
  const int t = threadIdx.x;
  const int kg = t & 7, a = t >> 3;
  const int64_t col = n0 + RW * a;
  const auto rq = rsrc(static_cast<const uint8_t*>(p.b) + k0 * p.ldb, (p.K - k0) * p.ldb);
  const uint32_t base = uint32_t(8 * kg * p.ldb + (col >> 1)), step = uint32_t(p.ldb);
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (e >= w0 && e < w1) R.w[e] = RW == 8 ? ld32(rq, base + e * step) : ld16(rq, base + e * step);
  if (w0 <= 0 && w1 > 0) load_ks_scales<GRP, ZP>(R.sc, R.zi, p, k0, kg, col);
}

template <bool ZP, int RW>
__device__ __forceinline__ void store_q_ks_one(uint16_t* tile, const RegsQKs& R, int c) {
  const int t = threadIdx.x;
  const int kg = t & 7, a = t >> 3;
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int na = nibble(R.w[2 * q], c), nb = nibble(R.w[2 * q + 1], c);
    if (ZP) {
      na -= R.zi[2 * q];
      nb -= R.zi[2 * q + 1];
    }
    o[q] = pack_bf16x2(float(na) * R.sc[2 * q], float(nb) * R.sc[2 * q + 1]);
  }
  *reinterpret_cast<u32x4*>(tile + tile_off(RW * a + c, kg)) = o;
}

// int8 q (dX B, 5..7-bit grids): RW bytes of each K-line.
struct RegsQKs8 {
  u32x2 v[8];
  float sc[8];
  int zi[8];
};

template <bool GRP, bool ZP, int RW>
__device__ __forceinline__ void load_q_ks8(RegsQKs8& R, const GemmArgs& p, int64_t n0, int64_t k0, int w0, int w1) {
  const int t = threadIdx.x;
  const int kg = t & 7, a = t >> 3;
  const int64_t col = n0 + RW * a;
  const auto rq = rsrc(static_cast<const uint8_t*>(p.b) + k0 * p.ldb, (p.K - k0) * p.ldb);
  const uint32_t base = uint32_t(8 * kg * p.ldb + col), step = uint32_t(p.ldb);
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (e >= w0 && e < w1) R.v[e] = RW == 8 ? ld64(rq, base + e * step) : u32x2{ld32(rq, base + e * step), 0u};
  if (w0 <= 0 && w1 > 0) load_ks_scales<GRP, ZP>(R.sc, R.zi, p, k0, kg, col);
}

template <bool ZP, int RW>
__device__ __forceinline__ void store_q_ks8_one(uint16_t* tile, const RegsQKs8& R, int c) {
  const int t = threadIdx.x;
  const int kg = t & 7, a = t >> 3;
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int na = sbyte(R.v[2 * q][c >> 2], c & 3), nb = sbyte(R.v[2 * q + 1][c >> 2], c & 3);
    if (ZP) {
      na -= R.zi[2 * q];
      nb -= R.zi[2 * q + 1];
    }
    o[q] = pack_bf16x2(float(na) * R.sc[2 * q], float(nb) * R.sc[2 * q + 1]);
  }
  *reinterpret_cast<u32x4*>(tile + tile_off(RW * a + c, kg)) = o;
}

// bfloat16 (dW A = dY, dW B = X): a 16-byte vector per K-line; with an odd
// ld the odd K-lines start in the middle of a dword (an extra dword each).
// kAlOdd: at least one of the two operands has an odd ld (`odd` is uniform).
// KL: K-lines per thread (8 for a 256-row tile, 4 for 128 rows).
template <int AL, int KL>
struct RegsKs {
  u32x4 v[KL];
  uint32_t x[AL == kAlOdd ? KL / 2 : 1];
  bool odd;
};

template <int AL, int KL>
__device__ __forceinline__ void load_ks_bf16(RegsKs<AL, KL>& R, const uint16_t* __restrict__ src, int64_t ld,
                                             int64_t c0, int64_t k0, int64_t K, int w0, int w1) {
  const int t = threadIdx.x;
  const int kg = t & (64 / KL - 1), a = t / (64 / KL);
  const auto r = rsrc4(src + k0 * ld + c0, (K - k0) * ld * 2 - c0 * 2);
  const uint32_t base = uint32_t((KL * kg * ld + 8 * a) * 2), step = uint32_t(ld * 2);
  R.odd = AL == kAlOdd && (ld & 1);
#pragma unroll
  for (int e = 0; e < KL; ++e) {
    if (e < w0 || e >= w1) continue;
    // a K-line past the end must read zeros: with an odd count of elements the first one's leading dword
    // holds the last element and two bytes beyond the tensor
    const uint32_t off = AL == kAlOdd ? (k0 + KL * kg + e < K ? (base + e * step) & ~3u : 0xFFFFFF00u) : base + e * step;
    R.v[e] = ld128(r, off);
    if constexpr (AL == kAlOdd)
      if (e & 1) R.x[e >> 1] = ld32(r, off + 16);
  }
}

template <int AL, int KL>
__device__ __forceinline__ void store_ks_bf16_one(uint16_t* tile, const RegsKs<AL, KL>& R, int c) {
  const int t = threadIdx.x;
  const int kg = t & (64 / KL - 1), a = t / (64 / KL);
  typename std::conditional<KL == 8, u32x4, u32x2>::type o;
#pragma unroll
  for (int q = 0; q < KL / 2; ++q) {
    const uint32_t x = R.v[2 * q][c >> 1];
    if constexpr (AL == kAlOdd) {
      // element c of the odd line is half word c (odd ld: c + 1) of its loaded dwords
      const uint32_t ye = R.v[2 * q + 1][c >> 1], yo = c < 7 ? R.v[2 * q + 1][((c + 1) >> 1) & 3] : R.x[q];
      if (c & 1) o[q] = __builtin_amdgcn_perm(R.odd ? yo : ye, x, R.odd ? 0x05040302u : 0x07060302u);
      else o[q] = __builtin_amdgcn_perm(ye, x, R.odd ? 0x07060100u : 0x05040100u);
    } else {
      const uint32_t y = R.v[2 * q + 1][c >> 1];
      o[q] = (c & 1) ? perm_hi16(x, y) : perm_lo16(x, y);
    }
  }
  *reinterpret_cast<decltype(o)*>(tile + tile_off(8 * a + c, KL * kg >> 3) + (KL * kg & 7)) = o;
}

// ------------------------------------------------------------------ the kernel

template <int V, int ACT, bool GRP, int AL, int OPT, int MI, int NJ>
struct Loader;

// load(.., w0, w1): global loads w0 .. w1 - 1 of the NLD of a tile, the A operand's first (the scales and
// zero offsets of the B operand ride on its first one).
// store_one(w): LDS store w of the NST of the tile held in registers, the A operand's first (2 MI and 2 NJ; dW
// 8 and 8).
template <int ACT, bool GRP, int AL, int OPT, int MI, int NJ>
struct Loader<kFwd, ACT, GRP, AL, OPT, MI, NJ> {
  static constexpr bool ZP = (OPT & kOptZ) != 0, Q8 = (OPT & kOptQ8) != 0;
  typename std::conditional<ACT == kActWide, RegsKc8<2 * MI>, RegsKc<ACT == kActI8 ? kAl16 : AL, 2 * MI>>::type ra;
  typename std::conditional<ACT == kActI8, typename std::conditional<Q8, RegsKc<kAl16, 2 * NJ>, RegsQ16<NJ>>::type,
                            typename std::conditional<Q8, RegsQKc8<2 * NJ>, RegsQKc<NJ / 2>>::type>::type rb;
  static constexpr int NA = 2 * MI, NB = Q8 ? 2 * NJ : ACT == kActI8 ? NJ : NJ / 2, NLD = NA + NB, NST = 2 * (MI + NJ);
  __device__ __forceinline__ void load(const GemmArgs& p, int64_t m0, int64_t n0, int64_t k0, int w0, int w1) {
    if constexpr (ACT == kActI8) {
      // rows of bytes as rows of half as many 16-bit values
      load_kc_bf16<kAl16, 2 * MI>(ra, static_cast<const uint16_t*>(p.a), p.lda / 2, m0, p.M, k0 / 2, p.lda / 2, w0, w1);
      if constexpr (Q8) load_kc_bf16<kAl16, 2 * NJ>(rb, static_cast<const uint16_t*>(p.b), p.ldb / 2, n0, p.N, k0 / 2, p.ldb / 2, w0 - NA, w1 - NA);
      else load_q_x16<NJ>(rb, p, n0, k0, w0 - NA, w1 - NA);
    } else {
      if constexpr (ACT == kActWide) load_kc_i8<2 * MI>(ra, static_cast<const int8_t*>(p.a), p.lda, m0, p.M, k0, w0, w1);
      else load_kc_bf16<AL, 2 * MI>(ra, static_cast<const uint16_t*>(p.a), p.lda, m0, p.M, k0, p.K, w0, w1);
      if constexpr (Q8) load_q_kc8<GRP, ZP, 2 * NJ>(rb, p, n0, k0, w0 - NA, w1 - NA);
      else load_q_kc<GRP, ZP, NJ / 2>(rb, p, n0, k0, w0 - NA, w1 - NA);
    }
  }
  __device__ __forceinline__ void store_one(uint16_t* As, uint16_t* Bs, int w) {
    if (w < 2 * MI) {
      if constexpr (ACT == kActWide) store_kc_i8_one<2 * MI>(As, ra, w);
      else store_kc_one(As, ra, w);
    } else if constexpr (ACT == kActI8) {
      if constexpr (Q8) store_kc_one(Bs, rb, w - 2 * MI);
      else store_q_x16_one<NJ>(Bs, rb, w - 2 * MI);
    } else {
      if constexpr (Q8) store_q_kc8_one<GRP, ZP, 2 * NJ>(Bs, rb, w - 2 * MI);
      else store_q_kc_one<GRP, ZP, NJ / 2>(Bs, rb, w - 2 * MI);
    }
  }
};

template <int ACT, bool GRP, int AL, int OPT, int MI, int NJ>
struct Loader<kDx, ACT, GRP, AL, OPT, MI, NJ> {
  static constexpr bool ZP = (OPT & kOptZ) != 0, Q8 = (OPT & kOptQ8) != 0;
  static constexpr int RW = 2 * NJ;
  RegsKc<AL, 2 * MI> ra;
  typename std::conditional<Q8, RegsQKs8, RegsQKs>::type rb;
  static constexpr int NA = 2 * MI, NLD = NA + 8, NST = 2 * (MI + NJ);
  __device__ __forceinline__ void load(const GemmArgs& p, int64_t m0, int64_t n0, int64_t k0, int w0, int w1) {
    load_kc_bf16<AL, 2 * MI>(ra, static_cast<const uint16_t*>(p.a), p.lda, m0, p.M, k0, p.K, w0, w1);
    if constexpr (Q8) load_q_ks8<GRP, ZP, RW>(rb, p, n0, k0, w0 - NA, w1 - NA);
    else load_q_ks<GRP, ZP, RW>(rb, p, n0, k0, w0 - NA, w1 - NA);
  }
  __device__ __forceinline__ void store_one(uint16_t* As, uint16_t* Bs, int w) {
    if (w < 2 * MI) {
      store_kc_one(As, ra, w);
    } else {
      if constexpr (Q8) store_q_ks8_one<ZP, RW>(Bs, rb, w - 2 * MI);
      else store_q_ks_one<ZP, RW>(Bs, rb, w - 2 * MI);
    }
  }
};

template <int ACT, bool GRP, int AL, int OPT, int MI, int NJ>
struct Loader<kDw, ACT, GRP, AL, OPT, MI, NJ> {
  static_assert(ACT == kActNone, "the dW GEMM reads bfloat16 operands (W4A8: X_hat)");
  static constexpr int KA = 2 * MI, KB = 2 * NJ, NLD = KA + KB, NST = 16;
  RegsKs<AL, KA> ra;
  RegsKs<AL, KB> rb;
  __device__ __forceinline__ void load(const GemmArgs& p, int64_t m0, int64_t n0, int64_t k0, int w0, int w1) {
    load_ks_bf16<AL, KA>(ra, static_cast<const uint16_t*>(p.a), p.lda, m0, k0, p.K, w0, w1);
    load_ks_bf16<AL, KB>(rb, static_cast<const uint16_t*>(p.b), p.ldb, n0, k0, p.K, w0 - KA, w1 - KA);
  }
  __device__ __forceinline__ void store_one(uint16_t* As, uint16_t* Bs, int w) {
    if (w < 8) store_ks_bf16_one(As, ra, w);
    else store_ks_bf16_one(Bs, rb, w - 8);
  }
};

// Offset of element (i, j) in a [rows][W] bfloat16 staging tile of an epilogue
// (the output tile; dW's G and its A/B blocks): the W / 8 16-byte chunks of a row
// are permuted by i mod W / 8, so that consecutive rows read at one column hit
// different chunk slots.
template <int W>
__device__ __forceinline__ int g_off(int i, int j) { return i * W + ((((j >> 3) ^ (i & (W / 8 - 1)))) << 3) + (j & 7); }

// LDS transpose load (gfx950): lane i of each 16-lane group receives the 4
// values in column i % 4 of the 4-element rows that lanes 4 e + i / 4 address
// (e = 0..3).
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 ld_tr16(const uint16_t* p) {
  const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(const_cast<uint16_t*>(p)));
  return __builtin_bit_cast(u32x2, v);
}

// MFMA operand from a [K][W] staging tile laid out by g_off: lane l gets
// column c0 + l % 32 at the 8 K rows k0 + 8 (l / 32) .. +7.  Lanes 4 e + q of
// each 16-lane group point at K row k0 + 8 (l / 32) + e (+4 for the second
// half) and columns c0 + 16 ((l / 16) % 2) + 4 q, so lane i of the group
// receives column c0 + 16 ((l / 16) % 2) + i.
template <int W>
__device__ __forceinline__ u32x4 frag_tr_g(const uint16_t* tile, int c0, int k0, int lane) {
  const int g = lane >> 4, r = lane & 15;
  const int c = c0 + 16 * (g & 1) + 4 * (r & 3);
  const int k = k0 + 8 * (g >> 1) + (r >> 2);
  const u32x2 lo = ld_tr16(tile + g_off<W>(k, c));
  const u32x2 hi = ld_tr16(tile + g_off<W>(k + 4, c));
  return u32x4{lo[0], lo[1], hi[0], hi[1]};
}

// Instruction interleave of one k-step (MI NJ MFMAs, one scheduling region
// closed by a sched_barrier): each MFMA is followed by a few VALU ops of the
// next tile's conversion; the fragment reads of the following k-step ride on
// the first MFMAs, the LDS stores of the next tile and the global loads of
// the tile after it are spread over the sequence.
enum : int { SG_VALU = 0x2, SG_MFMA = 0x8, SG_VMEM_READ = 0x20, SG_DS_READ = 0x100, SG_DS_WRITE = 0x200 };

// Schedule of the main loop, chosen by timing variants against each other in
// turn on one card: the k-steps over which the next tile's global loads are
// spread, and the VALU ops after each MFMA.  The loads of all four waves in one
// k-step queue up at the CU's address unit and hold the waves, so they are
// spread over two k-steps (forward: three): dX of 2048 tokens through 5120 x
// 13824 with groups of 128 433 -> 371 us, 14336 x 4096 377 -> 339, forward of the
// former 296 -> 276, dW 510 -> 491.
template <int V>
struct Sched {
  static constexpr int kLoadStep0 = 0, kLoadStep1 = V == kFwd ? 2 : 1;  // the k-steps that issue global loads
  static constexpr int kValu = V == kFwd ? 4 : 3;
};

// NLD global loads, NWR LDS stores and MI + NJ fragment reads over MI NJ MFMAs.
template <class S, int NLD, int NWR, int MI, int NJ>
__device__ __forceinline__ void interleave_kstep() {
  constexpr int NM = MI * NJ, NR = MI + NJ;
  constexpr int RP = (2 * NR + NM - 1) / NM;  // fragment reads per MFMA, in the first half
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
    if (m * RP < NR) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, RP, 0);
    __builtin_amdgcn_sched_group_barrier(SG_VALU, S::kValu, 0);
    const int w = (m + 1) * NWR / NM - m * NWR / NM, l = (m + 1) * NLD / NM - m * NLD / NM;
    if (w == 1) __builtin_amdgcn_sched_group_barrier(SG_DS_WRITE, 1, 0);
    if (w == 2) __builtin_amdgcn_sched_group_barrier(SG_DS_WRITE, 2, 0);
    if (w > 2) __builtin_amdgcn_sched_group_barrier(SG_DS_WRITE, 3, 0);
    if (l == 1) __builtin_amdgcn_sched_group_barrier(SG_VMEM_READ, 1, 0);
    if (l == 2) __builtin_amdgcn_sched_group_barrier(SG_VMEM_READ, 2, 0);
    if (l > 2) __builtin_amdgcn_sched_group_barrier(SG_VMEM_READ, 4, 0);
  }
}

// The k-step after the barrier: the next tile's first fragment reads first,
// then the MFMAs of this tile's last k-step.
template <int MI, int NJ>
__device__ __forceinline__ void interleave_last() {
  __builtin_amdgcn_sched_group_barrier(SG_DS_READ, MI + NJ, 0);
  __builtin_amdgcn_sched_group_barrier(SG_MFMA, MI * NJ, 0);
}

// Block -> tile order.  Blocks are dealt round-robin to the 8 XCDs (each with
// its own L2), so block b is renumbered to v = (b % 8) * (nt / 8) + b / 8: the
// blocks an XCD runs get consecutive numbers.  v then walks the tiles in
// groups of 4 tile rows (all columns of a group before the next group), so an
// XCD's concurrent blocks cover a compact 4 x 8 patch of tiles and share
// operand strips in its L2.
__device__ __forceinline__ void tile_of(int64_t b, int64_t ntm, int64_t ntn, int64_t& tm, int64_t& tn) {
  const int64_t nt = ntm * ntn, per = nt / 8;
  const int64_t v = b < per * 8 ? (b % 8) * per + b / 8 : b;
  constexpr int64_t GM = 4;
  const int64_t gsz = GM * ntn;
  const int64_t first = (v / gsz) * GM;
  const int64_t gm = ntm - first < GM ? ntm - first : GM;
  const int64_t off = v % gsz;
  tm = first + off % gm;
  tn = off / gm;
}

// Element n of a lane's accumulators in a tile's buffer of a split dW: 16 bytes a lane, 1 KiB a wave.
template <int MI, int NJ>
__device__ __forceinline__ f32x4* part_at(float* tiles, int64_t tile, int wave, int lane, int n) {
  return reinterpret_cast<f32x4*>(tiles) + ((tile * 4 + wave) * (MI * NJ * 4) + n) * 64 + lane;
}

// A block's tile is 64 MI x 64 NJ.  The 256 x 256 tile (one wave per SIMD, 256
// accumulator registers a wave) reads the fewest LDS bytes per MFMA; the 128 x
// 128 tile (two blocks a CU) quarters the unit of work for outputs that would
// leave CUs without a tile.
template <int V, int ACT, bool GRP, int AL, int OPT, int MI, int NJ>
__global__ __launch_bounds__(256, MI * NJ <= 4 ? 2 : 1) __attribute__((amdgpu_waves_per_eu(MI * NJ <= 4 ? 2 : 1, MI * NJ <= 4 ? 2 : 1)))
void k_gemm(GemmArgs p) {
  constexpr int BM = 64 * MI, BN = 64 * NJ, BK = ACT == kActI8 ? 128 : 64;  // K values of a tile (128 bytes a row)
  constexpr int TA = BM * 64, TB = BN * 64;
  // A stages 0, 1 then B stages 0, 1; the epilogues reuse all of it.
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * (TA + TB)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t ntm = (p.M + BM - 1) / BM, ntn = (p.N + BN - 1) / BN;
  int64_t tm, tn;
  constexpr bool kJoin = V == kDw && (OPT & kOptJoin) != 0, kSplit = V == kDw && MI == 2 && NJ == 2 && !kJoin;
  const int sp = kSplit ? int(blockIdx.x / uint32_t(ntm * ntn)) : 0;  // token range of the tile (plan.split of them)
  tile_of(int64_t(blockIdx.x) - int64_t(sp) * ntm * ntn, ntm, ntn, tm, tn);
  const int64_t m0 = tm * BM, n0 = tn * BN;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);

  f32x16 acc[MI][NJ];
  #pragma unroll
  for (int a = 0; a < MI; ++a)
    #pragma unroll
    for (int b = 0; b < NJ; ++b)
      #pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  if constexpr (kJoin) {
    // the token ranges' sums, added in float32 and in order before anything is rounded
    for (int q = 0; q < p.plan.split; ++q)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 v = *part_at<MI, NJ>(p.tile_part, (q * ntm + tm) * ntn + tn, wave, lane, (i * NJ + j) * 4 + g);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][4 * g + e] += v[e];
          }
  } else {
    // Software pipeline over K-tiles.  While the MFMAs consume LDS stage kt%2,
    // the registers holding tile kt+1 are written to the other stage (spread over
    // k-steps 0..2) and the tile kt+2 is fetched into a second register set from
    // k-step kLoadStep on.  The one barrier per tile sits before k-step 3, whose
    // fragments are already in registers, so the first fragments of tile kt+1
    // are read right after it and their latency hides behind k-step 3's MFMAs.
    // Loads past the last tile read zeros or unused data and are never
    // consumed, so the body has no branches.
    using Ld = Loader<V, ACT, GRP, AL, OPT, MI, NJ>;
    using S = Sched<V>;
    constexpr int NST = Ld::NST;  // LDS stores of a tile per thread
    // the block's K-tiles: nk of them from kb on
    int nk = int((p.K + BK - 1) / BK);
    int64_t kb = 0;
    if constexpr (kSplit) {
      const int first = int(int64_t(nk) * sp / p.plan.split);
      nk = int(int64_t(nk) * (sp + 1) / p.plan.split) - first;
      kb = int64_t(first) * BK;
    }
    u32x4 fa[2][MI], fb[2][NJ];
    auto read = [&](u32x4 (&a)[MI], u32x4 (&b)[NJ], const uint16_t* As, const uint16_t* Bs, int s) {
      const int ch = 2 * s + (lane >> 5);
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = *reinterpret_cast<const u32x4*>(As + tile_off(wm + 32 * i + (lane & 31), ch));
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[j] = *reinterpret_cast<const u32x4*>(Bs + tile_off(wn + 32 * j + (lane & 31), ch));
    };
    auto mfmas = [&](const u32x4 (&a)[MI], const u32x4 (&b)[NJ]) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          // D = B-tile x A-tile^T: a lane's accumulator holds 4 consecutive output
          // columns of one output row (8-byte stores; dW: 4 columns of one weight row)
          acc[i][j] = ACT == kActI8 ? mfma32_i8(b[j], a[i], acc[i][j]) : mfma32(b[j], a[i], acc[i][j]);
    };
    // store n of a tile in order: the operands alternate
    auto order = [](int n) { return MI == NJ ? (n & 1) * (NST / 2) + (n >> 1) : n; };
    Ld L0, L1;
    L0.load(p, m0, n0, kb, 0, Ld::NLD);
    L1.load(p, m0, n0, kb + BK, 0, Ld::NLD);
#pragma unroll
    for (int w = 0; w < NST; ++w) L0.store_one(lds, lds + 2 * TA, w);
    __syncthreads();
    read(fa[0], fb[0], lds, lds + 2 * TA, 0);
    auto step = [&](int kt, Ld& Lnext, Ld& Lfree) {
      const uint16_t* As = lds + (kt & 1) * TA;
      const uint16_t* Bs = lds + 2 * TA + (kt & 1) * TB;
      uint16_t* Asn = lds + ((kt + 1) & 1) * TA;
      uint16_t* Bsn = lds + 2 * TA + ((kt + 1) & 1) * TB;
      auto kstep = [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        constexpr int nls = S::kLoadStep1 - S::kLoadStep0 + 1;
        constexpr int l0 = s < S::kLoadStep0 ? 0 : s > S::kLoadStep1 ? Ld::NLD : (s - S::kLoadStep0) * Ld::NLD / nls;
        constexpr int l1 = s < S::kLoadStep0 ? 0 : s >= S::kLoadStep1 ? Ld::NLD : (s + 1 - S::kLoadStep0) * Ld::NLD / nls;
        constexpr int w0 = s == 0 ? 0 : s == 1 ? (3 * NST + 7) / 8 : (11 * NST + 15) / 16;
        constexpr int w1 = s == 0 ? (3 * NST + 7) / 8 : s == 1 ? (11 * NST + 15) / 16 : NST;
        if constexpr (l1 > l0) Lfree.load(p, m0, n0, kb + int64_t(kt + 2) * BK, l0, l1);
        read(fa[(s + 1) & 1], fb[(s + 1) & 1], As, Bs, s + 1);
        mfmas(fa[s & 1], fb[s & 1]);
#pragma unroll
        for (int w = w0; w < w1; ++w) Lnext.store_one(Asn, Bsn, order(w));
        interleave_kstep<S, l1 - l0, w1 - w0, MI, NJ>();
        __builtin_amdgcn_sched_barrier(0);
      };
      kstep(std::integral_constant<int, 0>{});
      kstep(std::integral_constant<int, 1>{});
      kstep(std::integral_constant<int, 2>{});
      // the last k-step of tile kt (after the barrier) with the first fragment reads of tile kt+1
      __syncthreads();
      read(fa[0], fb[0], Asn, Bsn, 0);
      mfmas(fa[1], fb[1]);
      interleave_last<MI, NJ>();
      __builtin_amdgcn_sched_barrier(0);
    };
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
      step(kt, L1, L0);
      step(kt + 1, L0, L1);
    }
    if (kt < nk) step(kt, L1, L0);
  }

  // acc[i][j][4g + e] = C[m0 + wm + 32 i + lane % 32][n0 + wn + 32 j + 8 g + 4 (lane / 32) + e]
  if constexpr (V == kFwd || V == kDx) {
    uint16_t* out = static_cast<uint16_t*>(p.out);
    const int64_t col_l = n0 + wn + 4 * (lane >> 5);
    // per-channel forward scales of the lane's columns (packed q without zero offsets entered as q / 16)
    constexpr float kQScale = V == kFwd && !GRP && (OPT & (kOptZ | kOptQ8)) == 0 && ACT != kActI8 ? 16.f : 1.f;
    // The tile goes through LDS (bf16 [BM][BN], 16-byte chunks permuted by row
    // as in g_off) and back to memory as whole row segments: a store
    // instruction then covers whole lines instead of 16 bytes of 32 rows, which
    // shortens the burst of output writes that ends the kernel.
    __syncthreads();  // every wave has read its last fragments
    uint16_t* Cs = lds;
    if constexpr (V == kFwd && !GRP && ACT == kActNone) {
      // a column block's scales are loaded when it is stored: all of them beside the accumulators spilled 16
      // registers of the 256 x 256 tile
      const auto rs = rsrc(p.s + n0, (p.N - n0) * 4);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        u32x4 cs[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) cs[g] = ld128(rs, uint32_t((wn + 32 * j + 8 * g + 4 * (lane >> 5)) * 4));
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const int lr = wm + 32 * i + (lane & 31);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            float val[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = acc[i][j][4 * g + e] * (__uint_as_float(cs[g][e]) * kQScale);
            *reinterpret_cast<u32x2*>(Cs + g_off<BN>(lr, wn + 32 * j + 8 * g + 4 * (lane >> 5))) =
                u32x2{pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3])};
          }
        }
      }
    } else {
      f32x4 cs[NJ][4];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int64_t c = col_l + 32 * j + 8 * g;
#pragma unroll
          for (int e = 0; e < 4; ++e) cs[j][g][e] = (V == kFwd && !GRP && c + e < p.N) ? p.s[c + e] * kQScale : 1.f;
        }
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int lr = wm + 32 * i + (lane & 31);
        const float rs = (V == kFwd && ACT != kActNone && m0 + lr < p.M) ? p.sx[m0 + lr] : 1.f;
        const double sn = (V == kFwd && ACT == kActI8 && (OPT & kOptZ) && m0 + lr < p.M) ? double(p.nsum[m0 + lr]) : 0.0;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            float val[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float x = acc[i][j][4 * g + e];
              if constexpr (ACT == kActI8) {
                // the exact integer sum of n q (packed q entered as 16 q), less z times the sum of n
                const int v = __float_as_int(x) >> ((OPT & kOptQ8) ? 0 : 4);
                x = float(v);
                if constexpr ((OPT & kOptZ) != 0) {
                  const int64_t c = col_l + 32 * j + 8 * g + e;
                  if (c < p.N) x = float(double(v) - double(p.z[c]) * sn);
                }
              }
              val[e] = x * cs[j][g][e] * rs;
            }
            *reinterpret_cast<u32x2*>(Cs + g_off<BN>(lr, wn + 32 * j + 8 * g + 4 * (lane >> 5))) =
                u32x2{pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3])};
          }
      }
    }
    __syncthreads();
    constexpr int CH = BN / 8, RPP = 256 / CH;  // chunks of a row, rows per pass
    if ((p.ldo & 7) == 0) {  // N = ldo here: whole 16-byte chunks
      // thread t writes 16-byte chunk t % CH of rows RPP ps + t / CH
      const int ch = threadIdx.x & (CH - 1);
      const int64_t col = n0 + 8 * ch;
      if (col < p.N) {
#pragma unroll 8
        for (int ps = 0; ps < BM / RPP; ++ps) {
          const int lr = RPP * ps + int(threadIdx.x) / CH;
          const u32x4 v = *reinterpret_cast<const u32x4*>(Cs + g_off<BN>(lr, 8 * ch));
          if (m0 + lr < p.M) *reinterpret_cast<u32x4*>(out + (m0 + lr) * p.ldo + col) = v;
        }
      }
    } else {
      // rows that are not 16-byte aligned: each thread writes the dwords of a row segment that start on
      // dwords (a row that begins in the middle of one has a half word at each end)
      const int dw = threadIdx.x & (BN / 2 - 1);  // dword of the row segment
      for (int lr = int(threadIdx.x) / (BN / 2); lr < BM; lr += 512 / BN) {
        if (m0 + lr >= p.M) break;
        const int sh = int(((m0 + lr) * p.ldo) & 1);  // n0 is even
        uint16_t* dst = out + (m0 + lr) * p.ldo + n0;
        const int c = 2 * dw + sh;  // columns c, c + 1
        const int64_t left = p.N - n0;
        if (c + 1 < BN && c + 1 < left) {
          const uint32_t w = uint32_t(Cs[g_off<BN>(lr, c)]) | (uint32_t(Cs[g_off<BN>(lr, c + 1)]) << 16);
          *reinterpret_cast<uint32_t*>(dst + c) = w;
        } else if (c < BN && c < left) {
          dst[c] = Cs[g_off<BN>(lr, c)];
        }
        if (sh && dw == 0) dst[0] = Cs[g_off<BN>(lr, 0)];
      }
    }
  } else {
    if constexpr (kSplit)
      if (p.plan.split > 1) {  // uniform: the sums of the block's tokens, for the launch that joins them
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              *part_at<MI, NJ>(p.tile_part, (sp * ntm + tm) * ntn + tn, wave, lane, (i * NJ + j) * 4 + g) =
                  f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        return;
      }
    __shared__ float s_tile[BM];                                      // per-channel scales
    __shared__ __attribute__((aligned(16))) uint16_t rt_tile[32 * (BM > BN ? BM : BN)];  // A or B rank block (bf16)
    // ---- dW epilogue: G = s * M * dW staged in LDS as bf16 [row][col], then both
    // rank-r products from LDS; the accumulators are dead once G is staged.
    // The lane holds rows R_i = m0 + wm + 32 i + lane % 32 and, in chunk j (32
    // columns from n0 + wn + 32 j), the columns 8 g + 4 h + e (h = lane / 32).
    const int r = p.r;
    const int nrb = (r + 31) / 32;
    const int half = lane >> 5;
    const int lrow = wm + (lane & 31);  // local row of i = 0
    uint16_t* Gs = lds;

    // columns of chunk j inside N, as a 32-bit mask over the chunk
    uint32_t colok[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int64_t left = p.N - (n0 + wn + 32 * j);
      colok[j] = left >= 32 ? 0xFFFFFFFFu : left <= 0 ? 0u : (1u << left) - 1u;
    }
    // clip-mask bits of chunk j of row R_i: two adjacent 16-bit words, one 4-byte load (rows >= M read 0)
    uint32_t mw[MI][NJ];
    {
      const auto rm = rsrc(p.mask + (m0 + wm) * p.ldm, (p.M - m0 - wm) * p.ldm * 2);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int64_t word = (((lane & 31) + 32 * i) * p.ldm + ((n0 + wn + 32 * j) >> 4)) * 2;
          mw[i][j] = ld32(rm, uint32_t(word)) & colok[j];
        }
    }
    // scales: per channel through LDS, group-wise per (row, chunk) (groups hold whole chunks)
    const auto rsg = rsrc(p.s + m0 * p.ngroups, (p.M - m0) * p.ngroups * 4);  // rows >= M read 0
    if constexpr (!GRP) {
      if (threadIdx.x < BM) s_tile[threadIdx.x] = ldf(rsg, uint32_t(threadIdx.x * 4));
      __syncthreads();
    }
    float sc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if constexpr (GRP)
          sc[i][j] = ldf(rsg, uint32_t(((lrow + 32 * i) * p.ngroups + (n0 + wn + 32 * j) / p.gsize) * 4));
        else
          sc[i][j] = s_tile[lrow + 32 * i];
      }

    // scale-gradient partials: ds_part[R_i][chunk] = sum over the chunk of dW (q - z); the lane
    // sums its 16 columns, the lane 32 apart the other 16
    if (p.ds_part) {
      const auto rq = rsrc(p.qd + (m0 + wm) * p.ldqd, (p.M - m0 - wm) * p.ldqd);  // rows >= M read 0
      // without a zero offset the resource is empty and every z reads 0
      const auto rz = p.z ? rsrc(p.z + (m0 + wm) * p.ngroups, (p.M - m0 - wm) * p.ngroups * 4) : rsrc(p.ds_part, 0);
      const auto rd = rsrc(p.ds_part + (m0 + wm) * p.ldds, (p.M - m0 - wm) * p.ldds * 4);
      const bool q8 = p.qd8 != 0;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int rl = (lane & 31) + 32 * i;  // row relative to m0 + wm
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int64_t c0 = n0 + wn + 32 * j;
          const int zi = ld_z(rz, int64_t(rl) * p.ngroups + (GRP ? c0 / p.gsize : 0));
          float sum = 0.f;
          if (q8) {
            // bytes c0 .. c0 + 31 of the row; column 8 g + 4 h + e is byte e of word 2 g + h
            const u32x4 qa = ld128(rq, uint32_t(rl * p.ldqd + c0)), qb = ld128(rq, uint32_t(rl * p.ldqd + c0 + 16));
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const uint32_t w = (2 * g + half) < 4 ? qa[(2 * g + half) & 3] : qb[(2 * g + half) & 3];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const bool ok = (colok[j] >> (8 * g + 4 * half + e)) & 1u;
                sum = __builtin_fmaf(ok ? acc[i][j][4 * g + e] : 0.f, float(sbyte(w, e) - zi), sum);
              }
            }
          } else {
            // nibbles c0 .. c0 + 31 of the row: column 8 g + 4 h + e is nibble 4 h + e of word g
            const u32x4 qv = ld128(rq, uint32_t(rl * p.ldqd + (c0 >> 1)));
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const bool ok = (colok[j] >> (8 * g + 4 * half + e)) & 1u;
                sum = __builtin_fmaf(ok ? acc[i][j][4 * g + e] : 0.f, float(nibble(qv[g], 4 * half + e) - zi), sum);
              }
          }
          sum += __shfl_xor(sum, 32);
          if (half == 0 && colok[j])
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sum), rd,
                                                  int(uint32_t((rl * p.ldds + (c0 >> 5)) * 4)), 0, 0);
        }
      }
    }

    // G staged as Gs[row][col]: the lane's 4 consecutive columns are one 8-byte write
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int lr = lrow + 32 * i;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint32_t bits = mw[i][j] >> (8 * g + 4 * half);
          float gv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) gv[e] = (bits >> e) & 1u ? acc[i][j][4 * g + e] * sc[i][j] : 0.f;
          *reinterpret_cast<u32x2*>(Gs + g_off<BN>(lr, wn + 32 * j + 8 * g + 4 * half)) =
              u32x2{pack_bf16x2(gv[0], gv[1]), pack_bf16x2(gv[2], gv[3])};
        }
    }

    // stage rank block rb of A (transposed, W = BM) or B (W = BN) as bf16 [32][W] in `rt_tile`
    auto stage = [&](const float* __restrict__ src, auto is_a_c, int rb) {
      constexpr bool is_a = decltype(is_a_c)::value;
      constexpr int W = is_a ? BM : BN, PT = W / 8;  // values per thread
      // unconditional buffer loads, all in flight at once: rows of A past M and ranks of B past r
      // lie outside the resource and read 0; ranks of A past r and columns of B past N are zeroed
      const auto rs = is_a ? rsrc(src + m0 * r, (p.M - m0) * int64_t(r) * 4) : rsrc(src + n0, (int64_t(r) * p.N - n0) * 4);
      if (is_a && (r & 3) == 0) {
        // thread t takes PT ranks of row m0 + t % W as 16-byte loads, written transposed
        const int c = threadIdx.x & (W - 1), rl0 = PT * (int(threadIdx.x) / W);
        float xv[PT];
#pragma unroll
        for (int q = 0; q < PT / 4; ++q) {
          const u32x4 v = ld128(rs, uint32_t((c * r + 32 * rb + rl0 + 4 * q) * 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) xv[4 * q + e] = __uint_as_float(v[e]);
        }
#pragma unroll
        for (int q = 0; q < PT; ++q)
          rt_tile[g_off<W>(rl0 + q, c)] = uint16_t(pack_bf16x2(32 * rb + rl0 + q < r ? xv[q] : 0.f, 0.f) & 0xFFFFu);
        return;
      }
      const int rho_l = threadIdx.x >> 3, c0 = PT * (threadIdx.x & 7);
      const int rho = 32 * rb + rho_l;
      float xv[PT];
      if (!is_a && (p.N & 3) == 0) {
        // B[rho][n0 + c0 ..]: 16-byte loads
#pragma unroll
        for (int q = 0; q < PT / 4; ++q) {
          const u32x4 v = ld128(rs, uint32_t((int64_t(rho) * p.N + c0 + 4 * q) * 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) xv[4 * q + e] = __uint_as_float(v[e]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < PT; ++i) {
          const int c = c0 + i;
          xv[i] = ldf(rs, is_a ? uint32_t((c * r + rho) * 4) : uint32_t((int64_t(rho) * p.N + c) * 4));
        }
      }
#pragma unroll
      for (int q = 0; q < PT / 8; ++q) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int c = c0 + 8 * q + e;
          x[e] = (rho < r && (is_a || n0 + c < p.N)) ? xv[8 * q + e] : 0.f;  // A[m0 + c][rho] or B[rho][n0 + c]
        }
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = pack_bf16x2(x[2 * e], x[2 * e + 1]);
        *reinterpret_cast<u32x4*>(&rt_tile[g_off<W>(rho_l, c0 + 8 * q)]) = o;
      }
    };

    // dB partial [tm][rho][n0 + j] = sum_i A[m0 + i][rho] G[i][j]; dA partial [tn][m0 + i][rho] = sum_j G[i][j] B[rho][n0 + j]
    const auto rdb = rsrc(p.dB_part + tm * r * p.N + n0, (int64_t(r) * p.N - n0) * 4);
    const auto rda = rsrc(p.dA_part + (tn * p.M + m0) * r, (p.M - m0) * int64_t(r) * 4);
    for (int rb = 0; rb < nrb; ++rb) {
      const int rho = 32 * rb + (lane & 31);
      __syncthreads();  // G staged / previous rank block consumed
      stage(p.Am, std::true_type{}, rb);
      __syncthreads();
      // dB: A operand = A^T rows (rt_tile), B operand = 8 consecutive rows of a G column (LDS transpose loads)
#pragma unroll
      for (int cb2 = 0; cb2 < BN / 128; ++cb2) {
        const int cb = (BN / 128) * wave + cb2;   // column block of 32
        const int lj = 32 * cb + (lane & 31);
        f32x16 d;
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll 4
        for (int s2 = 0; s2 < BM / 16; ++s2) {
          const u32x4 aa = *reinterpret_cast<const u32x4*>(&rt_tile[g_off<BM>(lane & 31, 16 * s2 + 8 * half)]);
          const u32x4 gb = frag_tr_g<BN>(Gs, 32 * cb, 16 * s2, lane);  // G[16 s2 + 8 half .. +7][32 cb + l % 32]
          d = mfma32(aa, gb, d);
        }
        if (n0 + lj < p.N) {
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int rr = 32 * rb + acc_row(v, lane);
            if (rr < r)
              __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d[v]), rdb, int(uint32_t((int64_t(rr) * p.N + lj) * 4)), 0, 0);
          }
        }
      }
      __syncthreads();
      stage(p.Bm, std::false_type{}, rb);
      __syncthreads();
      // dA: A operand = 8 consecutive columns of a G row (one read), B operand = B rows (rt_tile)
#pragma unroll
      for (int h2 = 0; h2 < BM / 128; ++h2) {
        const int rowblk = (BM / 128) * wave + h2;
        f32x16 d;
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll 4
        for (int s2 = 0; s2 < BN / 16; ++s2) {
          const u32x4 ga = *reinterpret_cast<const u32x4*>(Gs + g_off<BN>(32 * rowblk + (lane & 31), 16 * s2 + 8 * half));
          const u32x4 bb = *reinterpret_cast<const u32x4*>(&rt_tile[g_off<BN>(lane & 31, 16 * s2 + 8 * half)]);
          d = mfma32(ga, bb, d);
        }
        if (rho < r) {
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int row = 32 * rowblk + acc_row(v, lane);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d[v]), rda, int(uint32_t((row * r + rho) * 4)), 0, 0);
          }
        }
      }
    }
  }
}

// Launch one instantiation.
template <int V, int ACT, bool GRP, int AL, int OPT, int MI, int NJ>
hipError_t launch_tile(const GemmArgs& p, hipStream_t st) {
  const int64_t ntm = (p.M + 64 * MI - 1) / (64 * MI), ntn = (p.N + 64 * NJ - 1) / (64 * NJ);
  k_gemm<V, ACT, GRP, AL, OPT, MI, NJ><<<unsigned(ntm * ntn * p.plan.split), 256, 0, st>>>(p);
  return hipGetLastError();
}

// The instantiation for a plan (the forward and dX variants share this helper).
template <int V, int ACT, bool GRP, int OPT>
hipError_t launch_variant(const GemmArgs& p, hipStream_t st) {
  if constexpr (ACT == kActNone) {
    if (!gemm_al16(GemmVariant(V), false, p.K, p.lda, p.ldb))
      return p.lda & 1 ? launch_tile<V, ACT, GRP, kAlOdd, OPT, 2, 2>(p, st) : launch_tile<V, ACT, GRP, kAlDword, OPT, 2, 2>(p, st);
  }
  if constexpr (V == kDx)
    if (p.plan.tm == 128 && p.plan.tn == 256) return launch_tile<V, ACT, GRP, kAl16, OPT, 2, 4>(p, st);
  if constexpr (ACT == kActNone)
    if (p.plan.tm == 256 && p.plan.tn == 128) return launch_tile<V, ACT, GRP, kAl16, OPT, 4, 2>(p, st);
  if (p.plan.tm == 128 && p.plan.tn == 128) return launch_tile<V, ACT, GRP, kAl16, OPT, 2, 2>(p, st);
  if (p.plan.tm != 256 || p.plan.tn != 256) return hipErrorInvalidValue;
  return launch_tile<V, ACT, GRP, kAl16, OPT, 4, 4>(p, st);
}

// dW in tiles of 64 MI x 64 NJ.
template <bool GRP, int MI, int NJ>
hipError_t launch_dw_tile(const GemmArgs& p, hipStream_t st) {
  if (gemm_al16(kDw, false, p.K, p.lda, p.ldb)) return launch_tile<kDw, kActNone, GRP, kAl16, 0, MI, NJ>(p, st);
  if ((p.lda | p.ldb) & 1) return launch_tile<kDw, kActNone, GRP, kAlOdd, 0, MI, NJ>(p, st);
  return launch_tile<kDw, kActNone, GRP, kAlDword, 0, MI, NJ>(p, st);
}
template <bool GRP>
hipError_t launch_dw(const GemmArgs& p, hipStream_t st) {
  const GemmPlan& g = p.plan;
  if (g.split == 1) {
    if (g.tm == 256 && g.tn == 256) return launch_dw_tile<GRP, 4, 4>(p, st);
    if (g.tm == 256 && g.tn == 128) return launch_dw_tile<GRP, 4, 2>(p, st);
    if (g.tm == 128 && g.tn == 128) return launch_dw_tile<GRP, 2, 2>(p, st);
  }
  if (g.tm != 128 || g.tn != 128 || g.split < 1 || !p.tile_part) return hipErrorInvalidValue;
  const hipError_t e = launch_dw_tile<GRP, 2, 2>(p, st);
  if (e != hipSuccess) return e;
  k_gemm<kDw, kActNone, GRP, kAl16, kOptJoin, 2, 2><<<unsigned(((p.M + 127) / 128) * ((p.N + 127) / 128)), 256, 0, st>>>(p);
  return hipGetLastError();
}

// Run-time choice of the grouped-scale and zero-offset instantiations of one
// family (OPT_BASE: 0 or kOptQ8).
template <int V, int ACT, int OPT_BASE>
hipError_t launch_zg(bool grouped, bool zp, const GemmArgs& p, hipStream_t st) {
  if (zp) return grouped ? launch_variant<V, ACT, true, OPT_BASE | kOptZ>(p, st) : launch_variant<V, ACT, false, OPT_BASE | kOptZ>(p, st);
  return grouped ? launch_variant<V, ACT, true, OPT_BASE>(p, st) : launch_variant<V, ACT, false, OPT_BASE>(p, st);
}

}  // namespace lrqat
