// Dense contractions on the matrix cores (gfx950).
//
// Both GEMMs here are "NT": D[m][n] = sum_k A[m][k] B[n][k], both operands
// with k contiguous, which is how the batched charge step Q0 = B S^T (frames
// x atoms times the symmetric atoms x atoms S) and the k-space part of the
// elastance, 2 C C^T, are stored.
//
// FP64: v_mfma_f64_16x16x4 (the path's FP64 arithmetic, unchanged).  A
// 256-thread workgroup owns a 64 x 64 tile of D, each wavefront a 32 x 32
// quarter as 2 x 2 MFMA blocks; operand slabs of 64 rows x 16 k go through
// LDS with two buffers, the next slab's global loads in flight while the
// current one is multiplied (one barrier per slab).
//
// Mixed form: the three-term bf16 split of both operands (x = x0 + x1 + x2,
// six products x_a y_b with a + b <= 2, FP32 accumulation), on
// v_mfma_f32_16x16x32_bf16: slabs of 64 rows x 32 k per split term, 16-byte
// global and LDS accesses, the same tiling and double buffering.
//
// MFMA lane layouts (16 x 16 blocks): operand lane l carries row (or column)
// l % 16 and the k values (l / 16) * kw .. (l / 16) * kw + kw - 1 (kw = 1 for
// f64 x4, 8 for bf16 x32).  Result lane l holds column l % 16 in four
// values t = 0..3: rows 4 t + l / 16 for f64 (interleaved), rows
// 4 (l / 16) + t for the f32 results of the bf16 products (measured with a
// one-wavefront probe of each builtin).
#include "common.h"

namespace cpm {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

static_assert(ELAST_TILE == 64 && ELAST_SLAB == 16, "the padded lists match the tiles here");
constexpr int G64_TILE = 64, G64_K = 16, G64_LD = G64_K + 1;   // LDS rows padded against bank conflicts

// (row, column) of tile t of a lower triangle listed row by row
__device__ __forceinline__ void tri_tile(int t, int& row, int& col) {
  row = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while (row * (row + 1) / 2 > t) --row;                 // the estimate may be one off
  while ((row + 1) * (row + 2) / 2 <= t) ++row;
  col = t - row * (row + 1) / 2;
}

// D = A B^T.  SYM: A and B are the same matrix, D += A A^T, whose product part
// is symmetric: only the tiles of the lower triangle are computed (blockIdx.x
// lists them) and each is added at both places, half the matrix work.
template <bool SYM>
__global__ __launch_bounds__(256) void k_gemm_f64_mfma(int M, int N, int K, const double* __restrict__ A, int lda,
                                                       const double* __restrict__ B, int ldb, double* __restrict__ D,
                                                       int ldd) {
  __shared__ double sA[2][G64_TILE * G64_LD], sB[2][G64_TILE * G64_LD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int tm = blockIdx.y, tn = blockIdx.x;
  if (SYM) tri_tile(blockIdx.x, tm, tn);
  const int m0 = tm * G64_TILE, n0 = tn * G64_TILE;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  // loader: thread t moves 4 consecutive k of row t / 4 of each operand
  const int lrow = threadIdx.x >> 2, lk = (threadIdx.x & 3) * 4;
  const int ga = m0 + lrow, gb = n0 + lrow;
  const bool vec = ((lda | ldb) & 1) == 0 && ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 15) == 0;
  double ra[4], rb[4];
  auto load = [&](int k0) {
    const int k = k0 + lk;
    if (vec && k + 3 < K) {
      if (ga < M) {
        const double2 v0 = *reinterpret_cast<const double2*>(A + (size_t)ga * lda + k);
        const double2 v1 = *reinterpret_cast<const double2*>(A + (size_t)ga * lda + k + 2);
        ra[0] = v0.x; ra[1] = v0.y; ra[2] = v1.x; ra[3] = v1.y;
      } else {
        ra[0] = ra[1] = ra[2] = ra[3] = 0.0;
      }
      if (gb < N) {
        const double2 v0 = *reinterpret_cast<const double2*>(B + (size_t)gb * ldb + k);
        const double2 v1 = *reinterpret_cast<const double2*>(B + (size_t)gb * ldb + k + 2);
        rb[0] = v0.x; rb[1] = v0.y; rb[2] = v1.x; rb[3] = v1.y;
      } else {
        rb[0] = rb[1] = rb[2] = rb[3] = 0.0;
      }
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        ra[t] = (ga < M && k + t < K) ? A[(size_t)ga * lda + k + t] : 0.0;
        rb[t] = (gb < N && k + t < K) ? B[(size_t)gb * ldb + k + t] : 0.0;
      }
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      sA[buf][lrow * G64_LD + lk + t] = ra[t];
      sB[buf][lrow * G64_LD + lk + t] = rb[t];
    }
  };
  double4_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int r = lane & 15, kq = lane >> 4;
  const int n_slabs = (K + G64_K - 1) / G64_K;
  load(0);
  store(0);
  __syncthreads();
  for (int s = 0; s < n_slabs; ++s) {
    const int buf = s & 1;
    if (s + 1 < n_slabs) load((s + 1) * G64_K);
    const double* pa = sA[buf];
    const double* pb = sB[buf];
#pragma unroll
    for (int kk = 0; kk < G64_K; kk += 4) {
      double av[2], bv[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) av[a] = pa[(wm + 16 * a + r) * G64_LD + kk + kq];
#pragma unroll
      for (int b = 0; b < 2; ++b) bv[b] = pb[(wn + 16 * b + r) * G64_LD + kk + kq];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    if (s + 1 < n_slabs) store(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int gm = m0 + wm + 16 * a + 4 * t + kq, gn = n0 + wn + 16 * b + r;
        if (gm < M && gn < N) {
          double* d = D + (size_t)gm * ldd + gn;
          *d = (SYM ? *d : 0.0) + acc[a][b][t];
          if (SYM && tm != tn) {
            d = D + (size_t)gn * ldd + gm;
            *d += acc[a][b][t];
          }
        }
      }
}

// The same product where its 64 x 64 tiles would leave most of the chip idle
// (few frames): a 16 x 16 tile per workgroup, whose GS_WAVES wavefronts take a
// share of K each and join their blocks through LDS.  Operands come straight
// from global memory, two consecutive k per lane and load (the two MFMAs of a
// step take the even and the odd ones), GS_AHEAD steps in flight.  Bound by
// the latency of one wavefront's K / GS_WAVES chain: 37 frames of 936 atoms
// take 15 tiles of 64 x 64 and 57 us, or 177 small ones.
constexpr int GS_TILE = 16, GS_WAVES = 8, GS_AHEAD = 4;
constexpr int GS_MAX_TILES = 64;           // 64 x 64 tiles up to which this form is taken

__global__ __launch_bounds__(GS_WAVES * 64) void k_gemm_f64_small(int M, int N, int K, const double* __restrict__ A,
                                                                  int lda, const double* __restrict__ B, int ldb,
                                                                  double* __restrict__ D, int ldd) {
  __shared__ double red[GS_WAVES][GS_TILE * GS_TILE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.y * GS_TILE, n0 = blockIdx.x * GS_TILE;
  const int r = lane & 15, kq = lane >> 4;
  // rows past the end repeat the last one (their results are not stored)
  const double* a = A + (size_t)min(m0 + r, M - 1) * lda;
  const double* b = B + (size_t)min(n0 + r, N - 1) * ldb;
  const int steps = (K + 7) / 8;                       // of 8 k: lane quarter kq has k = 8 s + 2 kq and the next
  const int s0 = steps * wave / GS_WAVES, s1 = steps * (wave + 1) / GS_WAVES;
  const bool vec = ((lda | ldb) & 1) == 0 && ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 15) == 0;
  double2 av[GS_AHEAD], bv[GS_AHEAD];
  auto load = [&](int s, double2& x, double2& y) {
    const int k = 8 * s + 2 * kq;
    x = y = double2{0.0, 0.0};
    if (s >= s1) return;
    if (vec && k + 1 < K) {
      x = *reinterpret_cast<const double2*>(a + k);
      y = *reinterpret_cast<const double2*>(b + k);
    } else {
      if (k < K) { x.x = a[k]; y.x = b[k]; }
      if (k + 1 < K) { x.y = a[k + 1]; y.y = b[k + 1]; }
    }
  };
  double4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < GS_AHEAD; ++u) load(s0 + u, av[u], bv[u]);
  for (int s = s0; s < s1; s += GS_AHEAD) {
#pragma unroll
    for (int u = 0; u < GS_AHEAD; ++u) {
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].x, bv[u].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].y, bv[u].y, acc, 0, 0, 0);
      load(s + u + GS_AHEAD, av[u], bv[u]);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) red[wave][(4 * t + kq) * GS_TILE + r] = acc[t];
  __syncthreads();
  for (int e = threadIdx.x; e < GS_TILE * GS_TILE; e += GS_WAVES * 64) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < GS_WAVES; ++w) v += red[w][e];
    const int gm = m0 + e / GS_TILE, gn = n0 + e % GS_TILE;
    if (gm < M && gn < N) D[(size_t)gm * ldd + gn] = v;
  }
}

// ------------------------------------------------ elastance, k space by heights

// For electrode atoms that share a few heights z_h (flat sheets) the k-space
// part of A is separable: with the k-vectors grouped by their x-y part,
//   sum_k 2 k_e w(k) cos(k.(r_i - r_j))
//     = sum_kxy W[h_i][h_j][kxy] (c_i c_j + s_i s_j),
// c, s the cos and sin of kxy.r, W the sum over k_z of 2 k_e w cos(k_z (z_h -
// z_h')) (k and -k of one kxy paired, so the sin terms of z cancel).  The
// inner dimension falls from twice the k-vectors to twice the x-y parts: at
// the doubled paper cell (n = 1760) 2 x 36.6 k to 2 x 288, and the build's
// k-space part from 12.4 ms of FP64 matrix products to ~0.1 ms.

// W[h][h'][c] of the x-y parts c0 .. c0 + nkp; kxy[2][nk], nz[c]: the largest
// |n_z| with |k| <= kcut of that x-y part; entries past nk are zero.  The first
// x-y part is 0, whose half space holds n_z > 0 only.
// Sixteen lanes share an entry's k_z (an exp and a cos each, ~100 of them in
// a chain cost 34 us at the doubled paper cell with one lane per entry).  The
// workgroups are listed along x alone: H^2 pairs pass the grid's y limit of
// 65535 from 256 heights on.
__global__ __launch_bounds__(256) void k_height_weights(int H, int c0, int nk, int nkp,
                                                        const double* __restrict__ heights,
                                                        const double* __restrict__ kxy, const int* __restrict__ nz,
                                                        double dkz, double inv4a2, double scale,
                                                        double* __restrict__ W) {
  const int per = nkp / 16;                              // workgroups of a pair (nkp is a multiple of 16)
  const int pair = blockIdx.x / per;
  const int cl = (blockIdx.x - pair * per) * 16 + (threadIdx.x >> 4), c = c0 + cl;
  double acc = 0.0, k2 = 0.0;
  if (c < nk) {
    const double dz = heights[pair / H] - heights[pair % H];
    k2 = kxy[c] * kxy[c] + kxy[nk + c] * kxy[nk + c];
    for (int m = 1 + (threadIdx.x & 15); m <= nz[c]; m += 16) {
      const double kz = dkz * m, kk = k2 + kz * kz;
      acc += exp(-kk * inv4a2) / kk * cos(kz * dz);
    }
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (c > 0 && c < nk) acc = 2.0 * acc + exp(-k2 * inv4a2) / k2;
  if ((threadIdx.x & 15) == 0) W[(size_t)pair * nkp + cl] = scale * acc;
}

// P[a][c] = cos(kxy_c . r_a), P[a][nkp + c] = sin, of the same x-y parts, for
// the atoms listed by height (atom < 0: padding, zeros)
__global__ __launch_bounds__(256) void k_phase_xy(int c0, int nk, int nkp, const int* __restrict__ atoms,
                                                  const double* __restrict__ kxy, const double* __restrict__ ex,
                                                  const double* __restrict__ ey, double* __restrict__ P) {
  const int cl = blockIdx.y * blockDim.x + threadIdx.x, c = c0 + cl;
  if (cl >= nkp) return;
  const int a = atoms[blockIdx.x];
  double s = 0.0, co = 0.0;
  if (a >= 0 && c < nk) sincos(kxy[c] * ex[a] + kxy[nk + c] * ey[a], &s, &co);
  double* row = P + (size_t)blockIdx.x * 2 * nkp;
  row[cl] = co;
  row[nkp + cl] = s;
}

// A[i][j] += sum_c W[h_i][h_j][c] (c_i c_j + s_i s_j) over the tiles of the
// lower triangle of the height-sorted atom list (64 atoms of one height per
// tile, so W is one vector per tile), added at both places; MFMA tiling and
// double buffering as in k_gemm_f64_mfma, W applied to the row operand as it
// is staged.
__global__ __launch_bounds__(256) void k_elastance_kspace(int n, int H, int nkp, const int* __restrict__ atoms,
                                                          const int* __restrict__ tile_h,
                                                          const double* __restrict__ P, const double* __restrict__ W,
                                                          double* __restrict__ A) {
  __shared__ double sA[2][G64_TILE * G64_LD], sB[2][G64_TILE * G64_LD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int tm, tn;
  tri_tile(blockIdx.x, tm, tn);
  const int m0 = tm * G64_TILE, n0 = tn * G64_TILE;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int lrow = threadIdx.x >> 2, lk = (threadIdx.x & 3) * 4;
  const double* pa0 = P + (size_t)(m0 + lrow) * 2 * nkp + lk;
  const double* pb0 = P + (size_t)(n0 + lrow) * 2 * nkp + lk;
  const double* w0 = W + (size_t)(tile_h[tm] * H + tile_h[tn]) * nkp + lk;
  double2 ra[2], rb[2], rw[2];
  auto load = [&](int k0) {
    const int c0 = k0 < nkp ? k0 : k0 - nkp;             // nkp is a multiple of the slab
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      ra[t] = *reinterpret_cast<const double2*>(pa0 + k0 + 2 * t);
      rb[t] = *reinterpret_cast<const double2*>(pb0 + k0 + 2 * t);
      rw[t] = *reinterpret_cast<const double2*>(w0 + c0 + 2 * t);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      sA[buf][lrow * G64_LD + lk + 2 * t] = ra[t].x * rw[t].x;
      sA[buf][lrow * G64_LD + lk + 2 * t + 1] = ra[t].y * rw[t].y;
      sB[buf][lrow * G64_LD + lk + 2 * t] = rb[t].x;
      sB[buf][lrow * G64_LD + lk + 2 * t + 1] = rb[t].y;
    }
  };
  double4_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int r = lane & 15, kq = lane >> 4;
  const int n_slabs = 2 * nkp / G64_K;
  load(0);
  store(0);
  __syncthreads();
  for (int s = 0; s < n_slabs; ++s) {
    const int buf = s & 1;
    if (s + 1 < n_slabs) load((s + 1) * G64_K);
    const double* pa = sA[buf];
    const double* pb = sB[buf];
#pragma unroll
    for (int kk = 0; kk < G64_K; kk += 4) {
      double av[2], bv[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) av[a] = pa[(wm + 16 * a + r) * G64_LD + kk + kq];
#pragma unroll
      for (int b = 0; b < 2; ++b) bv[b] = pb[(wn + 16 * b + r) * G64_LD + kk + kq];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    if (s + 1 < n_slabs) store(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = atoms[m0 + wm + 16 * a + 4 * t + kq], j = atoms[n0 + wn + 16 * b + r];
        if (i < 0 || j < 0) continue;
        A[(size_t)i * n + j] += acc[a][b][t];
        if (tm != tn) A[(size_t)j * n + i] += acc[a][b][t];
      }
}

// ---------------------------------------------------------- bf16 x 6 products

constexpr int GB_TILE = 64, GB_K = 32, GB_LD = GB_K + 8;   // rows of 40 bf16 (80 B): 16-byte aligned, skewed banks

__global__ __launch_bounds__(256) void k_gemm_bf16x6_mfma(int M, int N, int K, const unsigned short* __restrict__ A,
                                                          size_t a_plane, const unsigned short* __restrict__ B,
                                                          size_t b_plane, double* __restrict__ D, int ldd) {
  // [buffer][term][row * GB_LD + k]
  __shared__ __align__(16) unsigned short sA[2][3][GB_TILE * GB_LD], sB[2][3][GB_TILE * GB_LD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.y * GB_TILE, n0 = blockIdx.x * GB_TILE;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  // loader: thread t moves 8 consecutive k (16 bytes) of row t / 4 of each term of each operand
  const int lrow = threadIdx.x >> 2, lk = (threadIdx.x & 3) * 8;
  const int ga = m0 + lrow, gb = n0 + lrow;
  uint4 ra[3], rb[3];
  auto load = [&](int k0) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      ra[p] = ga < M ? *reinterpret_cast<const uint4*>(A + p * a_plane + (size_t)ga * K + k0 + lk) : uint4{0, 0, 0, 0};
      rb[p] = gb < N ? *reinterpret_cast<const uint4*>(B + p * b_plane + (size_t)gb * K + k0 + lk) : uint4{0, 0, 0, 0};
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      *reinterpret_cast<uint4*>(&sA[buf][p][lrow * GB_LD + lk]) = ra[p];
      *reinterpret_cast<uint4*>(&sB[buf][p][lrow * GB_LD + lk]) = rb[p];
    }
  };
  float4_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = float4_t{0.f, 0.f, 0.f, 0.f};
  const int r = lane & 15, kq = (lane >> 4) * 8;
  const int n_slabs = K / GB_K;
  load(0);
  store(0);
  __syncthreads();
  for (int s = 0; s < n_slabs; ++s) {
    const int buf = s & 1;
    if (s + 1 < n_slabs) load((s + 1) * GB_K);
    bf16x8_t av[3][2], bv[3][2];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
        av[p][a] = *reinterpret_cast<const bf16x8_t*>(&sA[buf][p][(wm + 16 * a + r) * GB_LD + kq]);
#pragma unroll
      for (int b = 0; b < 2; ++b)
        bv[p][b] = *reinterpret_cast<const bf16x8_t*>(&sB[buf][p][(wn + 16 * b + r) * GB_LD + kq]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // smallest products first
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[1][a], bv[1][b], acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[2][a], bv[0][b], acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[0][a], bv[2][b], acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[1][a], bv[0][b], acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[0][a], bv[1][b], acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[0][a], bv[0][b], acc[a][b], 0, 0, 0);
      }
    if (s + 1 < n_slabs) store(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int gm = m0 + wm + 16 * a + 4 * (lane >> 4) + t, gn = n0 + wn + 16 * b + r;
        if (gm < M && gn < N) D[(size_t)gm * ldd + gn] = (double)acc[a][b][t];
      }
}

void launch_gemm_nt(hipStream_t s, int M, int N, int K, const double* A, int lda, const double* B, int ldb, double* D,
                    int ldd) {
  if (M <= 0 || N <= 0) return;
  const dim3 grid((N + G64_TILE - 1) / G64_TILE, (M + G64_TILE - 1) / G64_TILE);
  if (grid.x * grid.y <= GS_MAX_TILES)
    hipLaunchKernelGGL(k_gemm_f64_small, dim3((N + GS_TILE - 1) / GS_TILE, (M + GS_TILE - 1) / GS_TILE),
                       dim3(GS_WAVES * 64), 0, s, M, N, K, A, lda, B, ldb, D, ldd);
  else
    hipLaunchKernelGGL(k_gemm_f64_mfma<false>, grid, dim3(256), 0, s, M, N, K, A, lda, B, ldb, D, ldd);
}

void launch_syrk_nt(hipStream_t s, int M, int K, const double* A, int lda, double* D, int ldd) {
  if (M <= 0) return;
  const int t = (M + G64_TILE - 1) / G64_TILE;
  hipLaunchKernelGGL(k_gemm_f64_mfma<true>, dim3(t * (t + 1) / 2), dim3(256), 0, s, M, M, K, A, lda, A, lda, D,
                     ldd);
}

void launch_elastance_kspace(hipStream_t s, int n, int n_list, const int* atoms, const int* tile_h, int H,
                             const double* heights, int c0, int nk, int nkp, const double* kxy, const int* nz,
                             double dkz, double inv4a2, double scale, const double* ex, const double* ey, double* W,
                             double* P, double* A) {
  const int t = n_list / ELAST_TILE;
  hipLaunchKernelGGL(k_height_weights, dim3((size_t)H * H * (nkp / 16)), dim3(256), 0, s, H, c0, nk, nkp, heights, kxy,
                     nz, dkz, inv4a2, scale, W);
  hipLaunchKernelGGL(k_phase_xy, dim3(n_list, (nkp + 255) / 256), dim3(256), 0, s, c0, nk, nkp, atoms, kxy, ex, ey, P);
  hipLaunchKernelGGL(k_elastance_kspace, dim3(t * (t + 1) / 2), dim3(256), 0, s, n, H, nkp, atoms, tile_h, P, W, A);
}

void launch_gemm_bf16x6(hipStream_t s, int M, int N, int K, const unsigned short* A, size_t a_plane,
                        const unsigned short* B, size_t b_plane, double* D, int ldd) {
  if (M <= 0 || N <= 0) return;
  hipLaunchKernelGGL(k_gemm_bf16x6_mfma, dim3((N + GB_TILE - 1) / GB_TILE, (M + GB_TILE - 1) / GB_TILE), dim3(256), 0,
                     s, M, N, K, A, a_plane, B, b_plane, D, ldd);
}

}  // namespace cpm
