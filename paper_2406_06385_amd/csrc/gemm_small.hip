// Y = X_hat W_hat^T for few tokens (decoding, small batches).
//
// With T tokens the layer reads m k / 2 bytes of weights for 2 T m k flops, so
// below about a hundred tokens it is bound by how fast the weights stream in,
// and the 256 x 256 tiles of the general GEMM leave the chip idle (m / 256
// blocks, each walking all of K alone).  Here a block owns 16 RG weight rows and
// its waves split K between them (chunks of 128 columns, dealt round-robin), so
// that m / (16 RG) blocks of up to 16 waves are in flight; the waves' partial
// sums meet in LDS and are added in a fixed order.  Operands are not staged: the
// K order inside an MFMA is free as long as both operands use the same one, so
// lane l takes the 32 consecutive columns 32 (l / 16) .. +31 of weight row
// l % 16 (one 16-byte load of packed q) and the same columns of token l % 16,
// straight from memory (every block reads the same few token rows, from L2).
//
// Int8 tokens (W4A8) with one scale per output channel run on the int8 MFMA:
// sums of integer products are exact in int32, s and s_x are applied once at
// the end, and a zero offset as (sum n q) - z (sum n).
//
// Measured (HIP-graph replays, weights of several layers in turn; 256 x 256 tiles
// -> this kernel), bf16 tokens: 4096 x 4096, T = 1 84 -> 7.2 us, T = 128 84 -> 26;
// 14336 x 4096, T = 1 85 -> 18, T = 64 86 -> 39; int8 tokens with their
// quantisation: 14336 x 4096, T = 24 104 -> 16, 4096 x 14336, T = 128 331 -> 45.
#include "gemm_impl.h"

namespace lrqat {

namespace {

enum SmallMode { kSmallBf16 = 0, kSmallI8 = 1, kSmallI8Wide = 2 };  // X in bf16; codes on the int8 MFMA; codes widened to bf16

__device__ __forceinline__ f32x4 mfma16_bf16(const u32x4& p, const u32x4& q, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, p), __builtin_bit_cast(bf16x8, q), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16_i8(const u32x4& p, const u32x4& q, const f32x4& c) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, p), __builtin_bit_cast(i32x4, q),
                                                                        __builtin_bit_cast(i32x4, c), 0, 0, 0));
}

// 16 bytes at any byte offset: dword-aligned loads, shifted into place.
__device__ __forceinline__ u32x4 ld128_any(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const uint32_t o = off & ~3u;
  const u32x4 a = ld128(r, o);
  const uint32_t b = ld32(r, o + 16);
  u32x4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_alignbyte(i < 3 ? a[(i + 1) & 3] : b, a[i], off & 3u);
  return v;
}

template <int MODE, bool GRP, bool Q8, int TG, int RG>
__global__ __launch_bounds__(1024) void k_small(GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t small_lds[];
  f32x4* red = reinterpret_cast<f32x4*>(small_lds);  // [waves][RG * TG][64]
  const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), nw = int(blockDim.x >> 6);
  const int64_t n0 = int64_t(blockIdx.x) * 16 * RG, t0 = int64_t(blockIdx.y) * 16 * TG;
  const int nch = int((p.K + 127) / 128);
  constexpr int NQ = Q8 ? 2 : 1;           // 16-byte loads of q per lane and chunk
  constexpr bool Q16 = MODE != kSmallI8 && !GRP && !Q8;  // without zero offsets q enters as q / 16
  constexpr int PF = RG * NQ * TG <= 2 ? 4 : 2;  // chunks whose weights are in flight together

  const auto rq = rsrc4(static_cast<const uint8_t*>(p.b) + n0 * p.ldb, (p.N - n0) * p.ldb);
  const bool qdw = (p.ldb & 3) == 0;  // uniform: weight rows start on dwords
  const auto rx = rsrc4(static_cast<const uint8_t*>(p.a) + t0 * p.lda * (MODE == kSmallBf16 ? 2 : 1),
                        (p.M - t0) * p.lda * (MODE == kSmallBf16 ? 2 : 1));
  const bool xdw = (p.lda & 1) == 0;  // uniform: token rows start on dwords
  const auto rs = rsrc(p.s + n0 * p.ngroups, (p.N - n0) * p.ngroups * 4);
  const auto rz = p.z ? rsrc(p.z + n0 * p.ngroups, (p.N - n0) * p.ngroups * 4) : rsrc(p.s, 0);  // empty: z reads 0

  f32x4 acc[RG][TG];
#pragma unroll
  for (int r = 0; r < RG; ++r)
#pragma unroll
    for (int t = 0; t < TG; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int cb = wave; cb < nch; cb += PF * nw) {
    u32x4 qv[PF][RG][NQ];
#pragma unroll
    for (int f = 0; f < PF; ++f) {
      const int c = cb + f * nw;
#pragma unroll
      for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int h = 0; h < NQ; ++h) {
          // chunks past the last one load far off (zeros, or values that nothing uses): no branch around a load
          const uint32_t off = c < nch ? uint32_t((16 * r + i16) * p.ldb) + uint32_t(64 * NQ * c + 16 * NQ * g + 16 * h) : 0xFFFF0000u;
          qv[f][r][h] = qdw ? ld128(rq, off) : ld128_any(rq, off);
        }
    }
#pragma unroll
    for (int f = 0; f < PF; ++f) {
      const int c = cb + f * nw;
      if (c >= nch) break;  // wave-uniform
      const int kk = 128 * c + 32 * g;  // the lane's first column
      float sc[RG];
      int zi[RG];
      if constexpr (MODE != kSmallI8) {
        // columns past K have zero tokens; their group index is clamped into the row
        const int64_t grp = GRP ? min<int64_t>(kk / p.gsize, p.ngroups - 1) : 0;
#pragma unroll
        for (int r = 0; r < RG; ++r) {
          sc[r] = GRP ? ldf(rs, uint32_t(((16 * r + i16) * p.ngroups + grp) * 4)) : 1.f;
          zi[r] = ld_z(rz, (16 * r + i16) * p.ngroups + grp);
        }
      }
      if constexpr (MODE == kSmallI8) {
        // natural column order in both operands: 16 columns (bytes) per 16x16x64 MFMA
        u32x4 wb[RG][2];
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if constexpr (Q8) {
              wb[r][h] = qv[f][r][h];
            } else {
#pragma unroll
              for (int d = 0; d < 2; ++d) {  // eight nibbles -> eight bytes 16 q (the sum is shifted back at the end)
                const uint32_t w = qv[f][r][0][2 * h + d];
                const uint32_t e = (w << 4) & 0xF0F0F0F0u, o = w & 0xF0F0F0F0u;
                wb[r][h][2 * d] = __builtin_amdgcn_perm(o, e, 0x05010400u);
                wb[r][h][2 * d + 1] = __builtin_amdgcn_perm(o, e, 0x07030602u);
              }
            }
          }
#pragma unroll
        for (int t = 0; t < TG; ++t)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const u32x4 xv = ld128(rx, uint32_t((16 * t + i16) * p.lda + kk + 16 * h));
#pragma unroll
            for (int r = 0; r < RG; ++r) acc[r][t] = mfma16_i8(wb[r][h], xv, acc[r][t]);
          }
      } else {
        const bool whole = 128 * c + 128 <= int(p.K);  // wave-uniform
#pragma unroll
        for (int w8 = 0; w8 < 4; ++w8) {
          u32x4 wv[RG];
          if (Q16 && !p.z) {  // uniform
#pragma unroll
            for (int r = 0; r < RG; ++r) wv[r] = unpack_q16(qv[f][r][0][w8]);
          } else
#pragma unroll
          for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              int na, nb;
              if constexpr (Q8) {
                const uint32_t w = qv[f][r][w8 >> 1][2 * (w8 & 1) + (q >> 1)];
                na = sbyte(w, 2 * (q & 1));
                nb = sbyte(w, 2 * (q & 1) + 1);
              } else {
                const uint32_t w = qv[f][r][0][w8];
                na = nibble(w, 2 * q);
                nb = nibble(w, 2 * q + 1);
              }
              float a = float(na - zi[r]), b = float(nb - zi[r]);
              if constexpr (GRP) {
                a *= sc[r];
                b *= sc[r];
              }
              wv[r][q] = pack_bf16x2(a, b);
            }
#pragma unroll
          for (int t = 0; t < TG; ++t) {
            u32x4 xv;
            if constexpr (MODE == kSmallBf16) {
              const uint32_t off = uint32_t(((16 * t + i16) * p.lda + kk + 8 * w8) * 2);
              xv = xdw ? ld128(rx, off) : ld128_any(rx, off);
              if (!whole) xv = mask_tail(xv, kk + 8 * w8, int(p.K));
            } else {
              const u32x2 cv = ld64(rx, uint32_t((16 * t + i16) * p.lda + kk + 8 * w8));
#pragma unroll
              for (int q = 0; q < 4; ++q)
                xv[q] = pack_bf16x2(float(sbyte(cv[q >> 1], 2 * (q & 1))), float(sbyte(cv[q >> 1], 2 * (q & 1) + 1)));
            }
#pragma unroll
            for (int r = 0; r < RG; ++r) acc[r][t] = mfma16_bf16(wv[r], xv, acc[r][t]);
          }
        }
      }
    }
  }

  // the waves' sums: tile i is finished by wave i % nw, its parts added in wave order
#pragma unroll
  for (int r = 0; r < RG; ++r)
#pragma unroll
    for (int t = 0; t < TG; ++t) red[(wave * RG * TG + r * TG + t) * 64 + lane] = acc[r][t];
  __syncthreads();
  for (int i = wave; i < RG * TG; i += nw) {
    const int r = i / TG, t = i % TG;
    float val[4];
    // acc element v of the lane: weight row n0 + 16 r + 4 (l / 16) + v, token t0 + 16 t + l % 16
    const int64_t tok = t0 + 16 * t + i16, c = n0 + 16 * r + 4 * g;
    if constexpr (MODE == kSmallI8) {
      i32x4 s = {0, 0, 0, 0};
      for (int w = 0; w < nw; ++w) s += __builtin_bit_cast(i32x4, red[(w * RG * TG + i) * 64 + lane]);
#pragma unroll
      for (int e = 0; e < 4; ++e) val[e] = float(Q8 ? s[e] : s[e] >> 4);
      if (p.z && tok < p.M) {
        const double sn = double(p.nsum[tok]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          val[e] = float(double(Q8 ? s[e] : s[e] >> 4) - double(ld_z(rz, 16 * r + 4 * g + e)) * sn);
      }
    } else {
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
      for (int w = 0; w < nw; ++w) s += red[(w * RG * TG + i) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) val[e] = Q16 && !p.z ? 16.f * s[e] : s[e];
    }
    if (tok >= p.M) continue;
    const float rsx = MODE != kSmallBf16 ? p.sx[tok] : 1.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) val[e] = val[e] * (GRP ? 1.f : ldf(rs, uint32_t((16 * r + 4 * g + e) * 4))) * rsx;
    uint16_t* dst = static_cast<uint16_t*>(p.out) + tok * p.ldo + c;
    if (c + 4 <= p.N && (p.ldo & 3) == 0) {
      *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3])};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < p.N) dst[e] = __builtin_bit_cast(uint16_t, (__bf16)val[e]);
    }
  }
}

template <int MODE, bool GRP, bool Q8, int TG, int RG>
hipError_t launch_rg(const GemmArgs& p, hipStream_t st) {
  const int64_t nb = (p.N + 16 * RG - 1) / (16 * RG), nt = (p.M + 16 * TG - 1) / (16 * TG), nch = (p.K + 127) / 128;
  // waves per block: enough for 16 waves on each of the 256 CUs (8 with more than 16 tokens: more only
  // add partial sums), at most one per chunk of K, and at most 64 KiB of partial sums
  int64_t w = 4;
  while (w < 16 && nb * nt * w < (TG == 1 ? 4096 : 2048) && 2 * w * RG * TG <= 64) w *= 2;
  while (w > 1 && w > nch) w /= 2;
  k_small<MODE, GRP, Q8, TG, RG><<<dim3(unsigned(nb), unsigned(nt)), unsigned(64 * w), size_t(w) * RG * TG * 1024, st>>>(p);
  return hipGetLastError();
}

// Token groups of 16 per block by the token count, four at most (eight held too many registers: 128
// tokens through 4096 x 4096 took 51 us, 26 as two blocks of four).  A second row group halves the
// token loads per weight: with four token groups, and with two where groups of 16 rows are more blocks than
// CUs (K = 4096, T = 32, one -> two row groups: m = 4096 16 -> 14 us, and group-wise 17 -> 16, int8 9 -> 10, int8
// group-wise 13 -> 14; 6144 21 -> 14, 24 -> 17, 14 -> 10, 17 -> 14; 14336 36 -> 25; 1024 13 -> 14).
template <int MODE, bool GRP, bool Q8>
hipError_t launch_mode(const GemmArgs& p, hipStream_t st) {
  if (p.M <= 16) return launch_rg<MODE, GRP, Q8, 1, 1>(p, st);
  if (p.M <= 32) return p.N > 4096 ? launch_rg<MODE, GRP, Q8, 2, 2>(p, st) : launch_rg<MODE, GRP, Q8, 2, 1>(p, st);
  return launch_rg<MODE, GRP, Q8, 4, 2>(p, st);
}

}  // namespace

hipError_t launch_fwd_small(bool act, bool grouped, bool q8, const GemmArgs& p, hipStream_t st) {
  if (!act) {
    if (grouped) return q8 ? launch_mode<kSmallBf16, true, true>(p, st) : launch_mode<kSmallBf16, true, false>(p, st);
    return q8 ? launch_mode<kSmallBf16, false, true>(p, st) : launch_mode<kSmallBf16, false, false>(p, st);
  }
  if (!fwd_int8(act, grouped, p.K)) {
    if (grouped) return q8 ? launch_mode<kSmallI8Wide, true, true>(p, st) : launch_mode<kSmallI8Wide, true, false>(p, st);
    return q8 ? launch_mode<kSmallI8Wide, false, true>(p, st) : launch_mode<kSmallI8Wide, false, false>(p, st);
  }
  return q8 ? launch_mode<kSmallI8, false, true>(p, st) : launch_mode<kSmallI8, false, false>(p, st);
}

}  // namespace lrqat
