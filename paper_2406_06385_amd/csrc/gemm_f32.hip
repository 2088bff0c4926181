// float32-activation path of the LR-QAT layer ("FP32 compute data type",
// Section 4.2): the same integer grid and clip mask as the bfloat16 path.
//
// The three large contractions run on the bfloat16 matrix cores with float32
// accuracy.  A float32 x of at least 2^-110 is the exact sum of three bfloat16 pieces x = h + m + l
// of 8 significant bits each, and products of bfloat16 values are exact in float32, so
//   X W_hat^T  = s (.) (Xh + Xm + Xl) q^T            three products: q is exact in bfloat16
//   dY W_hat   = ((dY s)h + (dY s)m + (dY s)l) q
//   dY^T X     ~ hh + hm + mh + mm + hl + lh           six; ml, lm, ll are below 2^-21 |x||y|
// With group-wise scales or a zero offset W_hat = fl32(s (q - z)) is split too and
// both others take six products.  The products with an l or m piece have an
// accumulator of their own, so the main sum sees one addition per 16 terms.
// The matrix cores take bfloat16 subnormals as zero, so below 2^-110 the pieces l and then m are lost: a sum
// whose terms are all of that size is off by 2e-6 of itself at 2^-116, 4e-5 at 2^-120, 2e-3 at 2^-126, and
// float32 subnormals count as zero.
// The rank-r contractions of G = s M dW (dW is kept in the workspace) use the
// float32 MFMA: they are bound by reading dW.
//
// A 32x32x16 bf16 MFMA does 16 times the work per cycle of a float32 one, so
// even six products leave 2.7 times its rate; measured on 4096 x 4096, T = 1024
// (before: float32 FMA tiles of 64 x 64): forward 1123 -> 119 us, dX 994 -> 167 us, dW with
// both rank-r products and ds 3320 -> 342 us; the errors against float64 fall from
// 1.0e-6 .. 1.3e-6 to 0.7e-7 (Y, dX) and 3.5e-7 (dA, dB).
#include "gemm_impl.h"

namespace lrqat {

namespace {

constexpr int FB = 128, FK = 32;                 // block tile 128 x 128, 32 terms of K per stage
constexpr int F_PLANE = FB * FK;                 // elements of one bfloat16 plane of an operand tile
constexpr int F_THREADS = 512;

// A plane is [128 rows][32] bfloat16 (64-byte rows of four 16-byte chunks);
// chunk c of row r sits at slot c ^ ((r / 2) % 4), so that 8 consecutive rows
// read at one chunk hit 8 different 16-byte slots of 128 bytes.
__device__ __forceinline__ int plane_off(int row, int chunk) { return row * FK + ((chunk ^ ((row >> 1) & 3)) << 3); }

// Eight floats -> their three bfloat16 pieces: h truncated (a finite x stays finite), m and l
// rounded.  An infinite x gives m = l = NaN, which reaches the second accumulator only.  NaNs are made quiet
// first: one whose payload lies in the low half alone would be truncated to an infinity.
__device__ __forceinline__ void split3(const float (&x)[8], u32x4& h, u32x4& m, u32x4& l) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float a = __builtin_canonicalizef(x[2 * p]), b = __builtin_canonicalizef(x[2 * p + 1]);
    const float a1 = a - bf16_hi(__float_as_uint(a)), b1 = b - bf16_hi(__float_as_uint(b));
    const uint32_t mm = pack_bf16x2(a1, b1);
    h[p] = perm_hi16(__float_as_uint(a), __float_as_uint(b));
    m[p] = mm;
    l[p] = pack_bf16x2(a1 - bf16_lo(mm), b1 - bf16_hi(mm));
  }
}

// Eight consecutive floats at byte offset off (dword-aligned rows; past the end reads 0).
__device__ __forceinline__ void ld8f(float (&x)[8], __amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x4 a = ld128(r, off), b = ld128(r, off + 16);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[e] = __uint_as_float(a[e]);
    x[4 + e] = __uint_as_float(b[e]);
  }
}

// C[M][N] = sum_K a(i, kk) b(j, kk) on split operands.
//   kFwd: a = X, b = W_hat rows;  kDx: a = dY (times s where W_hat is not split), b = W_hat columns;
//   kDw: a = dY columns, b = X columns, C = dW.
// Thread t holds 8 consecutive K values of one row of each operand tile: K-contiguous sources
// (X, dY, q rows) take row t / 4, chunk t % 4; K-strided ones row t % 128, chunk t / 128.
template <int V, bool W3, bool Q8>
struct F32Regs {
  float a[8];
  float b[8];       // kDw
  uint32_t q[8];    // kFwd: 1 (packed) or 2 words of the row; kDx: one byte or nibble per K line
  float sc[8];      // scales: kFwd with W3 one, kDx eight
  int zi[8];
};

template <int V, bool W3, bool Q8>
__device__ __forceinline__ void f32_load(F32Regs<V, W3, Q8>& R, const F32Args& p, int64_t m0, int64_t n0, int64_t k0,
                                         int64_t M, int64_t N, int64_t K) {
  const int t = threadIdx.x;
  if constexpr (V == kDw) {
    const int row = t & 127, kc = t >> 7;
    // K lines (tokens) past the end lie outside the resources and read 0; rows past M or N feed
    // outputs that are not stored
    const auto ra = rsrc(p.dY + k0 * M + m0, ((K - k0) * M - m0) * 4);
    const auto rb = rsrc(p.X + k0 * N + n0, ((K - k0) * N - n0) * 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      R.a[e] = ldf(ra, uint32_t(((8 * kc + e) * M + row) * 4));
      R.b[e] = ldf(rb, uint32_t(((8 * kc + e) * N + row) * 4));
    }
  } else {
    const float* src = V == kFwd ? p.X : p.dY;
    {
      const int row = t >> 2;
      const int64_t kk = k0 + 8 * (t & 3);
      ld8f(R.a, rsrc(src + m0 * K, (M - m0) * K * 4), uint32_t((row * K + kk) * 4));
      if (k0 + FK > K) {  // uniform: the last, partial tile
#pragma unroll
        for (int e = 0; e < 8; ++e) R.a[e] = kk + e < K ? R.a[e] : 0.f;
      }
      if constexpr (V == kDx && !W3) {
        float s[8];
        ld8f(s, rsrc(p.s, K * 4), uint32_t(kk * 4));
#pragma unroll
        for (int e = 0; e < 8; ++e) R.a[e] *= s[e];
      }
    }
    if constexpr (V == kFwd) {
      const int row = t >> 2;
      const int64_t kk = k0 + 8 * (t & 3);  // q is zero past column k
      const auto rq = rsrc(p.q + n0 * p.ldq, (N - n0) * p.ldq);
      if constexpr (Q8) {
        const u32x2 v = ld64(rq, uint32_t(row * p.ldq + kk));
        R.q[0] = v[0];
        R.q[1] = v[1];
      } else {
        R.q[0] = ld32(rq, uint32_t(row * p.ldq + (kk >> 1)));
      }
      if constexpr (W3) {
        const int64_t at = row * p.ngroups + (p.gsize ? min<int64_t>(kk / p.gsize, p.ngroups - 1) : 0);
        R.sc[0] = ldf(rsrc(p.s + n0 * p.ngroups, (N - n0) * p.ngroups * 4), uint32_t(at * 4));
        R.zi[0] = p.z ? ld_z(rsrc(p.z + n0 * p.ngroups, (N - n0) * p.ngroups * 4), at) : 0;
      }
    } else {
      const int row = t & 127, kc = t >> 7;
      const int64_t col = n0 + row;
      const auto rq = rsrc(p.q + k0 * p.ldq, (K - k0) * p.ldq);
      const int64_t byte = Q8 ? col : col >> 1;
#pragma unroll
      for (int e = 0; e < 8; ++e)  // columns past the padded row read a neighbour's; they are not stored
        R.q[e] = __builtin_amdgcn_raw_buffer_load_b8(rq, int(uint32_t((8 * kc + e) * p.ldq + byte)), 0, 0);
      if constexpr (W3) {
        const int64_t grp = p.gsize ? min<int64_t>(col / p.gsize, p.ngroups - 1) : 0;
        const auto rs = rsrc(p.s + k0 * p.ngroups, (K - k0) * p.ngroups * 4);
        const auto rz = p.z ? rsrc(p.z + k0 * p.ngroups, (K - k0) * p.ngroups * 4) : rsrc(p.s, 0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          R.sc[e] = ldf(rs, uint32_t(((8 * kc + e) * p.ngroups + grp) * 4));
          R.zi[e] = ld_z(rz, (8 * kc + e) * p.ngroups + grp);
        }
      }
    }
  }
}

template <int V, bool W3, bool Q8>
__device__ __forceinline__ void f32_store(uint16_t* As, uint16_t* Bs, const F32Regs<V, W3, Q8>& R, int64_t n0) {
  const int t = threadIdx.x;
  const int okc = plane_off(t >> 2, t & 3), oks = plane_off(t & 127, t >> 7);
  auto put3 = [](uint16_t* P, int off, const float (&x)[8]) {
    u32x4 h, m, l;
    split3(x, h, m, l);
    *reinterpret_cast<u32x4*>(P + off) = h;
    *reinterpret_cast<u32x4*>(P + F_PLANE + off) = m;
    *reinterpret_cast<u32x4*>(P + 2 * F_PLANE + off) = l;
  };
  put3(As, V == kDw ? oks : okc, R.a);
  if constexpr (V == kDw) {
    put3(Bs, oks, R.b);
  } else {
    float w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      int q;
      if constexpr (V == kFwd) q = Q8 ? sbyte(R.q[e >> 2], e & 3) : nibble(R.q[0], e);
      else q = Q8 ? sbyte(R.q[e], 0) : (int(R.q[e] << (28 - 4 * ((n0 + (t & 127)) & 1))) >> 28);
      if constexpr (W3) w[e] = float(q - R.zi[V == kFwd ? 0 : e]) * R.sc[V == kFwd ? 0 : e];
      else w[e] = float(q);
    }
    const int off = V == kFwd ? okc : oks;
    if constexpr (W3) {
      put3(Bs, off, w);
    } else {
      u32x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = pack_bf16x2(w[2 * q], w[2 * q + 1]);
      *reinterpret_cast<u32x4*>(Bs + off) = o;
    }
  }
}

template <int V, bool W3, bool Q8>
__global__ __launch_bounds__(F_THREADS) void k_f32(F32Args p, float* __restrict__ C, int64_t M, int64_t N, int64_t K) {
  constexpr int PB = (V == kDw || W3) ? 3 : 1;  // planes of the second operand
  __shared__ __attribute__((aligned(16))) uint16_t lds[2][(3 + PB) * F_PLANE];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  int64_t tm, tn;
  tile_of(int64_t(blockIdx.x), (M + FB - 1) / FB, (N + FB - 1) / FB, tm, tn);
  const int64_t m0 = tm * FB, n0 = tn * FB;
  const int wm = (wave >> 2) * 64, wn = (wave & 3) * 32;  // the wave's 64 x 32 part
  f32x16 hi[2], lo[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) hi[i][v] = lo[i][v] = 0.f;

  F32Regs<V, W3, Q8> R;
  f32_load<V, W3, Q8>(R, p, m0, n0, 0, M, N, K);
  f32_store<V, W3, Q8>(lds[0], lds[0] + 3 * F_PLANE, R, n0);
  const int nk = int((K + FK - 1) / FK);
  for (int kt = 0; kt < nk; ++kt) {
    __syncthreads();  // stage kt % 2 is written, and nobody reads the other one any more
    const bool more = kt + 1 < nk;
    if (more) f32_load<V, W3, Q8>(R, p, m0, n0, int64_t(kt + 1) * FK, M, N, K);
    const uint16_t* As = lds[kt & 1];
    const uint16_t* Bs = As + 3 * F_PLANE;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int ch = 2 * s + (lane >> 5);
      u32x4 a[2][3], b[PB];
#pragma unroll
      for (int q = 0; q < PB; ++q) b[q] = *reinterpret_cast<const u32x4*>(Bs + q * F_PLANE + plane_off(wn + (lane & 31), ch));
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          a[i][q] = *reinterpret_cast<const u32x4*>(As + q * F_PLANE + plane_off(wm + 32 * i + (lane & 31), ch));
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        lo[i] = mfma32(a[i][2], b[0], lo[i]);
        lo[i] = mfma32(a[i][1], b[0], lo[i]);
        if constexpr (PB == 3) {
          lo[i] = mfma32(a[i][0], b[2], lo[i]);
          lo[i] = mfma32(a[i][1], b[1], lo[i]);
          lo[i] = mfma32(a[i][0], b[1], lo[i]);
        }
        hi[i] = mfma32(a[i][0], b[0], hi[i]);
      }
    }
    if (more) f32_store<V, W3, Q8>(lds[(kt + 1) & 1], lds[(kt + 1) & 1] + 3 * F_PLANE, R, n0);
  }
  const int64_t col = n0 + wn + (lane & 31);
  if (col >= N) return;
  const float sc = V == kFwd && !W3 ? p.s[col] : 1.f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t row = m0 + wm + 32 * i + acc_row(v, lane);
      // the main sum alone decides infinities and NaNs: the small pieces of an infinite operand are NaN
      const float sum = __builtin_isinf(hi[i][v]) ? hi[i][v] : hi[i][v] + lo[i][v];
      if (row < M) C[row * N + col] = sum * sc;
    }
}

// ------------------------------------------------------------------ rank-r gradients from the stored dW

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int F_WAVES = 16;  // waves of a block; they split the contracted dimension
constexpr int F_RG = 2;      // groups of 16 ranks per pass over dW

// dA[i][rho] = c sum_j G[i][j] B[rho][j].  A block owns 16 rows; wave w takes the 16-column steps
// w, w + 16, ...; lane l holds columns 4 (l / 16) .. +3 of row l % 16 (one 16-byte load), element e of
// which is the K index of the e-th 16x16x4 MFMA.
__global__ __launch_bounds__(64 * F_WAVES) void k_f32_da(F32Args p, float* __restrict__ dA, int accumulate) {
  __shared__ f32x4 red[F_WAVES][F_RG][64];
  const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int64_t i0 = int64_t(blockIdx.x) * 16;
  const int rho0 = int(blockIdx.y) * 16 * F_RG;
  const auto rg = rsrc(p.dW + i0 * p.k, (p.m - i0) * p.k * 4);
  const auto rm = rsrc(p.mask + i0 * p.ldm, (p.m - i0) * p.ldm * 2);
  const auto rs = rsrc(p.s + i0 * p.ngroups, (p.m - i0) * p.ngroups * 4);
  const auto rb = rsrc(p.B + rho0 * p.k, (int64_t(p.r) - rho0) * p.k * 4);  // ranks past r read 0
  f32x4 acc[F_RG];
#pragma unroll
  for (int q = 0; q < F_RG; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nst = int((p.k + 15) / 16);
  const float s_row = p.gsize ? 0.f : ldf(rs, uint32_t(i16 * 4));
  for (int st = wave; st < nst; st += F_WAVES) {
    const int col = 16 * st + 4 * g;
    const u32x4 w = ld128(rg, uint32_t((i16 * p.k + col) * 4));
    const uint32_t mb = ld16(rm, uint32_t((i16 * p.ldm + st) * 2)) >> (4 * g);
    const float sc = p.gsize ? ldf(rs, uint32_t((i16 * p.ngroups + min<int64_t>(col / p.gsize, p.ngroups - 1)) * 4)) : s_row;
    u32x4 bv[F_RG];
#pragma unroll
    for (int q = 0; q < F_RG; ++q) bv[q] = ld128(rb, uint32_t(((16 * q + i16) * p.k + col) * 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = col + e < p.k;  // the last step's columns past k hold the next row's values
      const float gv = in && ((mb >> e) & 1u) ? __uint_as_float(w[e]) * sc : 0.f;
#pragma unroll
      for (int q = 0; q < F_RG; ++q) acc[q] = mfma_f32(gv, in ? __uint_as_float(bv[q][e]) : 0.f, acc[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < F_RG; ++q) red[wave][q][lane] = acc[q];
  __syncthreads();
  if (wave >= F_RG) return;
  f32x4 s = red[0][wave][lane];
  for (int w = 1; w < F_WAVES; ++w) s += red[w][wave][lane];
  const int rho = rho0 + 16 * wave + i16;
  if (rho >= p.r) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t row = i0 + 4 * g + v;
    if (row < p.m) {
      float* d = dA + row * p.r + rho;
      *d = (accumulate ? *d : 0.f) + p.c * s[v];
    }
  }
}

// dB[rho][j] = c sum_i A[i][rho] G[i][j].  A block owns 64 columns; wave w takes the 4-row steps w,
// w + 16, ...; lane l holds columns 4 (l % 16) .. +3 of row l / 16, element e of which belongs to the
// e-th MFMA (its column l % 16 stands for column 4 (l % 16) + e).
__global__ __launch_bounds__(64 * F_WAVES) void k_f32_db(F32Args p, float* __restrict__ dB, int accumulate) {
  __shared__ f32x4 red[F_WAVES][F_RG][64];
  const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int64_t j0 = int64_t(blockIdx.x) * 64, col = j0 + 4 * i16;
  const int rho0 = int(blockIdx.y) * 16 * F_RG;
  f32x4 acc[F_RG][4];
#pragma unroll
  for (int q = 0; q < F_RG; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[q][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int64_t nst = (p.m + 3) / 4;
  const int64_t grp = p.gsize ? min<int64_t>(col / p.gsize, p.ngroups - 1) : 0;
  for (int64_t st = wave; st < nst; st += F_WAVES) {
    const int64_t r0 = 4 * st;  // rows past m lie outside the resources and read 0
    const u32x4 w = ld128(rsrc(p.dW + r0 * p.k + j0, ((p.m - r0) * p.k - j0) * 4), uint32_t((g * p.k + 4 * i16) * 4));
    const uint32_t mb = ld16(rsrc(p.mask + r0 * p.ldm, (p.m - r0) * p.ldm * 2), uint32_t((g * p.ldm + (col >> 4)) * 2)) >> (col & 15);
    const float sc = ldf(rsrc(p.s + r0 * p.ngroups, (p.m - r0) * p.ngroups * 4), uint32_t((g * p.ngroups + grp) * 4));
    const auto ra = rsrc(p.A + r0 * p.r, (p.m - r0) * int64_t(p.r) * 4);
    float av[F_RG];
#pragma unroll
    for (int q = 0; q < F_RG; ++q) {
      const int rho = rho0 + 16 * q + i16;
      const float v = ldf(ra, uint32_t((g * p.r + rho) * 4));
      av[q] = rho < p.r ? v : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gv = (mb >> e) & 1u ? __uint_as_float(w[e]) * sc : 0.f;  // columns past k are not stored
#pragma unroll
      for (int q = 0; q < F_RG; ++q) acc[q][e] = mfma_f32(av[q], gv, acc[q][e]);
    }
  }
  for (int e = 0; e < 4; ++e) {  // four passes over the shared sums
#pragma unroll
    for (int q = 0; q < F_RG; ++q) red[wave][q][lane] = e == 0 ? acc[q][0] : e == 1 ? acc[q][1] : e == 2 ? acc[q][2] : acc[q][3];
    __syncthreads();
    if (wave < F_RG && col + e < p.k) {
      f32x4 s = red[0][wave][lane];
      for (int w = 1; w < F_WAVES; ++w) s += red[w][wave][lane];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int rho = rho0 + 16 * wave + 4 * g + v;
        if (rho < p.r) {
          float* d = dB + rho * p.k + col + e;
          *d = (accumulate ? *d : 0.f) + p.c * s[v];
        }
      }
    }
    __syncthreads();
  }
}

// ds[i][grp] = (accumulate ? ds : 0) + sum over the group's columns of dW (q - z); one wave per (row, group).
__global__ __launch_bounds__(256) void k_f32_ds(F32Args p, float* __restrict__ ds, int accumulate) {
  const int64_t ng = p.gsize ? p.ngroups : 1;
  const int64_t idx = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (idx >= p.m * ng) return;  // wave-uniform
  const int64_t i = idx / ng, grp = idx % ng;
  const int64_t j0 = p.gsize ? grp * p.gsize : 0, j1 = p.gsize ? j0 + p.gsize : p.k;
  const int zz = p.z ? p.z[idx] : 0;
  const float* dw = p.dW + i * p.k;
  const uint8_t* q = p.q + i * p.ldq;
  float acc = 0.f;
  for (int64_t j = j0 + lane; j < j1; j += 64) {
    const int v = p.q8 ? int(int8_t(q[j])) : int(uint32_t(q[j >> 1]) << (28 - 4 * int(j & 1))) >> 28;
    acc = __builtin_fmaf(dw[j], float(v - zz), acc);
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) ds[idx] = (accumulate ? ds[idx] : 0.f) + acc;
}

template <int V>
hipError_t run(const F32Args& a, float* C, int64_t M, int64_t N, int64_t K, hipStream_t st) {
  const unsigned nb = unsigned(((M + FB - 1) / FB) * ((N + FB - 1) / FB));
  if constexpr (V == kDw) {
    k_f32<V, true, false><<<nb, F_THREADS, 0, st>>>(a, C, M, N, K);
  } else {
    const bool w3 = a.gsize != 0 || a.z;
    if (w3) {
      if (a.q8) k_f32<V, true, true><<<nb, F_THREADS, 0, st>>>(a, C, M, N, K);
      else k_f32<V, true, false><<<nb, F_THREADS, 0, st>>>(a, C, M, N, K);
    } else {
      if (a.q8) k_f32<V, false, true><<<nb, F_THREADS, 0, st>>>(a, C, M, N, K);
      else k_f32<V, false, false><<<nb, F_THREADS, 0, st>>>(a, C, M, N, K);
    }
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_f32_forward(const F32Args& a, float* Y, hipStream_t st) { return run<kFwd>(a, Y, a.T, a.m, a.k, st); }

hipError_t launch_f32_dx(const F32Args& a, float* dX, hipStream_t st) { return run<kDx>(a, dX, a.T, a.k, a.m, st); }

hipError_t launch_f32_dw(const F32Args& a, float* dA, float* dB, float* ds, int accumulate, hipStream_t st) {
  hipError_t e = run<kDw>(a, a.dW, a.m, a.k, a.T, st);
  if (e != hipSuccess) return e;
  const unsigned nr = unsigned((a.r + 16 * F_RG - 1) / (16 * F_RG));
  k_f32_da<<<dim3(unsigned((a.m + 15) / 16), nr), 64 * F_WAVES, 0, st>>>(a, dA, accumulate);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_f32_db<<<dim3(unsigned((a.k + 63) / 64), nr), 64 * F_WAVES, 0, st>>>(a, dB, accumulate);
  e = hipGetLastError();
  if (e != hipSuccess || !ds) return e;
  const int64_t n = a.m * (a.gsize ? a.ngroups : 1);
  k_f32_ds<<<unsigned((n + 3) / 4), 256, 0, st>>>(a, ds, accumulate);
  return hipGetLastError();
}

}  // namespace lrqat
