// Dense linear algebra of the constant-potential solve, all FP64:
//   * elastance matrix A (paper Eq. 3): Gaussian-Gaussian real-space pairs,
//     k-space as 2 k_e C C^T from the cos/sin factor matrix, self term;
//   * its inverse by blocked Gauss-Jordan elimination without pivoting (A is
//     symmetric positive definite for alpha < eta/sqrt2, so every pivot block
//     is too; a non-positive pivot reports CPM_ENOTSPD);
//   * the projections S = A^-1 - u u^T/(e.u), u = A^-1 e (Eq. 8-9), and for
//     the doubled cell S <- S - w w^T/(e1.w), w = S e1 (Eq. 14-15);
//   * the per-step charge solve q = S b + dV S c (one wavefront per row,
//     streaming S once) and the energy reductions.
#include "common.h"

namespace cpm {

// ------------------------------------------------------------ elastance

__global__ __launch_bounds__(256) void k_elastance_real(int n, const double* __restrict__ ex,
                                                        const double* __restrict__ ey, const double* __restrict__ ez,
                                                        Cell cell, double alpha, double eta, double rc2,
                                                        double self_term, double* __restrict__ A) {
  const int j = blockIdx.x * 16 + (threadIdx.x & 15);
  const int i = blockIdx.y * 16 + (threadIdx.x >> 4);
  if (i >= n || j >= n) return;
  const double eta2 = eta * 0.70710678118654752;   // eta / sqrt(2)
  double dx0 = min_image(ex[i] - ex[j], cell.L[0], cell.invL[0]);
  double dy0 = min_image(ey[i] - ey[j], cell.L[1], cell.invL[1]);
  double dz0 = min_image(ez[i] - ez[j], cell.L[2], cell.invL[2]);
  double acc = 0.0;
  for (int a = -cell.img[0]; a <= cell.img[0]; ++a)
    for (int b = -cell.img[1]; b <= cell.img[1]; ++b)
      for (int c = -cell.img[2]; c <= cell.img[2]; ++c) {
        if (i == j && a == 0 && b == 0 && c == 0) continue;
        double dx = dx0 + a * cell.L[0], dy = dy0 + b * cell.L[1], dz = dz0 + c * cell.L[2];
        double r2 = dx * dx + dy * dy + dz * dz;
        if (r2 < rc2) {
          double r = sqrt(r2);
          acc += (erfc(alpha * r) - erfc(eta2 * r)) / r;
        }
      }
  if (i == j) acc += self_term;
  A[(size_t)i * n + j] = KE * acc;
}

// C[i][c] for the k-vectors k0 .. k0+nkc-1: c < nkc -> s_k cos(k.r_i),
// c >= nkc -> s_k sin(k.r_i), s_k = sqrt(2 k_e w(k)); row-major n x 2 nkc
__global__ __launch_bounds__(256) void k_phase_matrix(int n, int nkc, int k0, int nk, const double* __restrict__ kv,
                                                      const double* __restrict__ sk, const double* __restrict__ ex,
                                                      const double* __restrict__ ey, const double* __restrict__ ez,
                                                      double* __restrict__ C) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = blockIdx.y;
  if (c >= nkc) return;
  const int k = k0 + c;
  double s, co;
  sincos(kv[k] * ex[i] + kv[nk + k] * ey[i] + kv[2 * nk + k] * ez[i], &s, &co);
  C[(size_t)i * 2 * nkc + c] = sk[k] * co;
  C[(size_t)i * 2 * nkc + nkc + c] = sk[k] * s;
}

__global__ void k_symmetrize(int n, double* __restrict__ A) {
  const int j = blockIdx.x * 16 + (threadIdx.x & 15);
  const int i = blockIdx.y * 16 + (threadIdx.x >> 4);
  if (i >= n || j >= n || j <= i) return;
  double a = A[(size_t)i * n + j], b = A[(size_t)j * n + i];
  double m = 0.5 * (a + b);
  A[(size_t)i * n + j] = m;
  A[(size_t)j * n + i] = m;
}

// ---------------------------------------------------- Gauss-Jordan inverse

constexpr int GJ_NB = GJ_BLOCK;
constexpr int GJ_TILE = 64;            // update tile
static_assert(GJ_NB == 32, "the thread maps below are written for 32 x 32 pivot blocks");

typedef double gj_double4 __attribute__((ext_vector_type(4)));

// Scratch of the pivot inversion: the pivot row and column of the current
// and the next elimination step.
struct GJPivotLds {
  double prow[2][GJ_NB], pcol[2][GJ_NB];
};

// Invert an nb x nb pivot block (Gauss-Jordan, no pivoting) held four
// consecutive elements of a row per thread (v, row threadIdx.x / 8): inverse
// to dinv, flag on a non-positive or non-finite pivot.  256 threads.
// Bound by the latency of its nb dependent steps (a reciprocal, two LDS
// reads, a barrier): the elements stay in registers and the next step's row
// and column go to the other LDS buffer, so a step has one barrier instead
// of three and no pass over the block in LDS.
__device__ __forceinline__ void gj_invert_block(double v[4], int nb, double* __restrict__ dinv, int* __restrict__ flag,
                                                GJPivotLds& l) {
  const int r = threadIdx.x >> 3, c0 = (threadIdx.x & 7) * 4;
  if (r == 0)
#pragma unroll
    for (int k = 0; k < 4; ++k) l.prow[0][c0 + k] = v[k];
  if (c0 == 0) l.pcol[0][r] = v[0];
  __syncthreads();
  // (four steps per trip: the column to publish is then a fixed element)
  for (int p0 = 0; p0 < nb; p0 += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int p = p0 + q;
      if (p >= nb) break;
      const int buf = q & 1;
      double piv = l.prow[buf][p];
      if (!(piv > 0.0) || !isfinite(piv)) {
        if (threadIdx.x == 0) atomicOr(flag, 1);
        piv = 1.0;
      }
      const double ip = 1.0 / piv;
      const double pc = l.pcol[buf][r];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // (selected, not branched: 16 short divergent paths a step cost more than the step)
        const int c = c0 + k;
        const double pr = l.prow[buf][c];
        const double in_row = c == p ? ip : pr * ip;
        const double in_col = -pc * ip, rest = v[k] - pc * pr * ip;
        const double off_row = c == p ? in_col : rest;
        v[k] = r == p ? in_row : off_row;
      }
      if (r == p + 1)
#pragma unroll
        for (int k = 0; k < 4; ++k) l.prow[buf ^ 1][c0 + k] = v[k];
      if (c0 == (q < 3 ? p0 : p0 + 4)) l.pcol[buf ^ 1][r] = v[(q + 1) & 3];
      __syncthreads();
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (r < nb && c0 + k < nb) dinv[r * nb + c0 + k] = v[k];
}

// The first pivot block (the later ones are inverted by k_gj_update).
__global__ __launch_bounds__(256) void k_gj_pivot(int n, int nb, const double* __restrict__ A,
                                                  double* __restrict__ dinv, int* __restrict__ flag) {
  __shared__ GJPivotLds l;
  const int r = threadIdx.x >> 3, c0 = (threadIdx.x & 7) * 4;
  double v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = (r < nb && c0 + k < nb) ? A[(size_t)r * n + c0 + k] : 0.0;
  gj_invert_block(v, nb, dinv, flag, l);
}

// Panels: pc[i][t] = A[i][k0+t] (column block, i outside the pivot rows is
// what the update needs) and rx[t][j] = (Dinv A[k0.., j]) for j outside the
// block, Dinv[t][j-k0] inside it.  A workgroup takes 32 columns j, thread
// (j, g) the four rows t = g, g + 8, g + 16, g + 24 (four independent
// chains).  Latency of one load and 32 dependent FMAs; a thread per column
// with the whole 32 x 32 product took 152 us at n = 1760 (7 workgroups); 7 us
// like this.
constexpr int GJ_PCOLS = 32;
__global__ __launch_bounds__(256) void k_gj_panels(int n, int k0, int nb, const double* __restrict__ A,
                                                   const double* __restrict__ dinv, double* __restrict__ pc,
                                                   double* __restrict__ rx) {
  __shared__ double Ds[GJ_NB][GJ_NB + 1], Cs[GJ_NB][GJ_PCOLS + 1];
  const int j0 = blockIdx.x * GJ_PCOLS;
  for (int e = threadIdx.x; e < GJ_NB * GJ_PCOLS; e += 256) {
    const int t = e / GJ_PCOLS, c = e % GJ_PCOLS;
    Cs[t][c] = (t < nb && j0 + c < n) ? A[(size_t)(k0 + t) * n + j0 + c] : 0.0;
    // the same thread map transposed: column block row j0 + t, entry c
    if (j0 + t < n && c < nb) pc[(size_t)(j0 + t) * nb + c] = A[(size_t)(j0 + t) * n + k0 + c];
    Ds[t][c] = (t < nb && c < nb) ? dinv[t * nb + c] : 0.0;
  }
  __syncthreads();
  const int c = threadIdx.x % GJ_PCOLS, g = threadIdx.x / GJ_PCOLS, j = j0 + c;
  if (j >= n) return;
  if (j >= k0 && j < k0 + nb) {
    for (int t = g; t < nb; t += 8) rx[(size_t)t * n + j] = Ds[t][j - k0];
  } else {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int u = 0; u < nb; ++u) {
      const double a = Cs[u][c];
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] = fma(Ds[g + 8 * k][u], a, s[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (g + 8 * k < nb) rx[(size_t)(g + 8 * k) * n + j] = s[k];
  }
}

// A[i][j] = rx[i-k0][j] for i in the block, else (j in block ? 0 : A[i][j]) - sum_t pc[i][t] rx[t][j].
// A 64 x 64 tile per workgroup on v_mfma_f64_16x16x4 (the tiling and lane
// layout of k_gemm.hip).  Workgroup 0 takes the next pivot block alone (the
// tile around it leaves it out) and inverts it into dinv, beside the other
// tiles' work: a step is two launches, and the pivot's latency is hidden by
// the update (n = 1760: pivot 43 us and update 36 apart, 20 together).
__global__ __launch_bounds__(256) void k_gj_update(int n, int k0, int nb, int k1, int nb1, double* __restrict__ A,
                                                   const double* __restrict__ pc, const double* __restrict__ rx,
                                                   double* __restrict__ dinv, int* __restrict__ flag) {
  // (row strides of 72 and 160 dwords: the operand reads meet every bank twice)
  __shared__ double Ps[GJ_TILE][GJ_NB + 4];
  __shared__ double Rs[GJ_NB][GJ_TILE + 16];
  if (blockIdx.x == 0) {
    // rows and columns k1 .. k1 + nb1 - 1, four elements of a row per thread
    // (all beyond the pivot block, so the update's general case)
    __shared__ GJPivotLds l;
    if (nb1 <= 0) return;
    const int r = threadIdx.x >> 3, c0 = (threadIdx.x & 7) * 4;
    double v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (r < nb1 && c0 + k < nb1) ? A[(size_t)(k1 + r) * n + k1 + c0 + k] : 0.0;
    for (int e = threadIdx.x; e < GJ_NB * GJ_NB; e += 256) {
      const int a = e / GJ_NB, b = e % GJ_NB;
      Ps[a][b] = (a < nb1 && b < nb) ? pc[(size_t)(k1 + a) * nb + b] : 0.0;
      Rs[a][b] = (a < nb && b < nb1) ? rx[(size_t)a * n + k1 + b] : 0.0;
    }
    __syncthreads();
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int t = 0; t < nb; ++t) {
      const double a = Ps[r][t];
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] = fma(a, Rs[t][c0 + k], s[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = v[k] - s[k];
      if (r < nb1 && c0 + k < nb1) A[(size_t)(k1 + r) * n + k1 + c0 + k] = v[k];
    }
    gj_invert_block(v, nb1, dinv, flag, l);
    return;
  }
  const int nt = (n + GJ_TILE - 1) / GJ_TILE, tile = blockIdx.x - 1;
  const int i0 = (tile / nt) * GJ_TILE, j0 = (tile % nt) * GJ_TILE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32, lr = lane & 15, kq = lane >> 4;
  // the elements of this lane (MFMA result layout), in flight during staging
  double base[2][2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int gi = i0 + wm + 16 * a + 4 * t + kq, gj = j0 + wn + 16 * b + lr;
        base[a][b][t] = (gi < n && gj < n && !(gj >= k0 && gj < k0 + nb)) ? A[(size_t)gi * n + gj] : 0.0;
      }
  for (int t = threadIdx.x; t < GJ_TILE * GJ_NB; t += 256) {
    const int r = t / GJ_NB, c = t % GJ_NB;
    Ps[r][c] = (i0 + r < n && c < nb) ? pc[(size_t)(i0 + r) * nb + c] : 0.0;
    const int tr = t / GJ_TILE, tc = t % GJ_TILE;
    Rs[tr][tc] = (j0 + tc < n && tr < nb) ? rx[(size_t)tr * n + j0 + tc] : 0.0;
  }
  __syncthreads();
  gj_double4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = gj_double4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kk = 0; kk < GJ_NB; kk += 4) {
    double av[2], bv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) av[a] = Ps[wm + 16 * a + lr][kk + kq];
#pragma unroll
    for (int b = 0; b < 2; ++b) bv[b] = Rs[kk + kq][wn + 16 * b + lr];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int gi = i0 + wm + 16 * a + 4 * t + kq, lj = wn + 16 * b + lr, gj = j0 + lj;
        const bool next = gi >= k1 && gi < k1 + nb1 && gj >= k1 && gj < k1 + nb1;   // workgroup 0's
        if (gi < n && gj < n && !next)
          A[(size_t)gi * n + gj] = (gi >= k0 && gi < k0 + nb) ? Rs[gi - k0][lj] : base[a][b][t] - acc[a][b][t];
      }
}

// ------------------------------------------------------------ projections

// y[i] = sum_j M[i][j] x[j] (x == nullptr: x = 1); one wavefront per row
__global__ __launch_bounds__(256) void k_matvec(int n, const double* __restrict__ Mx, const double* __restrict__ x,
                                                double* __restrict__ y) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int i = blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x >> 6);
  if (i >= n) return;
  const double* row = Mx + (size_t)i * n;
  double acc = 0.0;
  for (int j = lane; j < n; j += WAVE) acc += row[j] * (x ? x[j] : 1.0);
  acc = wave_sum(acc);
  if (lane == 0) y[i] = acc;
}

// out[0] = sum_i a[i] * (b ? b[i] : 1)  (one workgroup)
__global__ __launch_bounds__(256) void k_dot(int n, const double* __restrict__ a, const double* __restrict__ b,
                                             double* __restrict__ out) {
  __shared__ double red[4];
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) acc += a[i] * (b ? b[i] : 1.0);
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = red[0] + red[1] + red[2] + red[3];
}

// S[i][j] -= u_i u_j / s
__global__ void k_rank1(int n, double* __restrict__ S, const double* __restrict__ u, const double* __restrict__ s) {
  const int j = blockIdx.x * 16 + (threadIdx.x & 15);
  const int i = blockIdx.y * 16 + (threadIdx.x >> 4);
  if (i >= n || j >= n) return;
  S[(size_t)i * n + j] -= u[i] * u[j] / s[0];
}

// ------------------------------------------------------------ charge solve

// Q0 = S b (per frame), q = Q0 + dv Sc; one wavefront per row, four
// independent accumulators so that four row loads per lane are in flight
// (the body; k_charges and k_charges_tail below are its launches)
template <bool TAIL>
__device__ __forceinline__ void charges_body(int n, const double* __restrict__ S, const double* __restrict__ b_all,
                                             const double* __restrict__ Sc, double dv, double* __restrict__ Q0_all,
                                             double* __restrict__ q_all, const int* __restrict__ epos,
                                             double* __restrict__ qs_all, const ChargeTail& tail) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int i = blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x >> 6);
  const int frame = blockIdx.y;
  if (i >= n) return;
  const double* b = b_all + (size_t)frame * n;
  const int ep = qs_all ? epos[i] : 0;      // read now, used at the end
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  if ((n & 1) == 0) {       // rows are 16-byte aligned: stream them as double2
    const double2* row = reinterpret_cast<const double2*>(S + (size_t)i * n);
    const double2* b2 = reinterpret_cast<const double2*>(b);
    const int n2 = n >> 1;
    int j = lane;
    for (; j + 3 * WAVE < n2; j += 4 * WAVE) {
      const double2 s0 = row[j], s1 = row[j + WAVE], s2 = row[j + 2 * WAVE], s3 = row[j + 3 * WAVE];
      const double2 v0 = b2[j], v1 = b2[j + WAVE], v2 = b2[j + 2 * WAVE], v3 = b2[j + 3 * WAVE];
      a0 = fma(s0.x, v0.x, fma(s0.y, v0.y, a0));
      a1 = fma(s1.x, v1.x, fma(s1.y, v1.y, a1));
      a2 = fma(s2.x, v2.x, fma(s2.y, v2.y, a2));
      a3 = fma(s3.x, v3.x, fma(s3.y, v3.y, a3));
    }
    for (; j < n2; j += WAVE) {
      const double2 s0 = row[j], v0 = b2[j];
      a0 = fma(s0.x, v0.x, fma(s0.y, v0.y, a0));
    }
  } else {
    const double* row = S + (size_t)i * n;
    for (int j = lane; j < n; j += WAVE) a0 = fma(row[j], b[j], a0);
  }
  const double acc = wave_sum((a0 + a1) + (a2 + a3));
  if (lane == 0) {
    const size_t o = (size_t)frame * n + i;
    double qv = acc + dv * Sc[i];
    if (Q0_all) Q0_all[o] = acc;
    if (q_all) q_all[o] = qv;
    if (TAIL && tail.g) tail.g[i] = 2.0 * (qv - tail.t[i]) + dv * tail.c[i];
    if (TAIL && tail.qa) {
      qv = tail.q_of[i] - acc;
      tail.qa[i] = qv;
    }
    if (qs_all) qs_all[(size_t)frame * n + ep] = qv;      // cell-sorted copy
  }
}

__global__ __launch_bounds__(256) void k_charges(int n, const double* __restrict__ S, const double* __restrict__ b,
                                                 const double* __restrict__ Sc, double dv, double* __restrict__ Q0,
                                                 double* __restrict__ q, const int* __restrict__ epos,
                                                 double* __restrict__ qs) {
  charges_body<false>(n, S, b, Sc, dv, Q0, q, epos, qs, ChargeTail{});
}
__global__ __launch_bounds__(256) void k_charges_tail(int n, const double* __restrict__ S, const double* __restrict__ b,
                                                      const double* __restrict__ Sc, double dv, double* __restrict__ Q0,
                                                      double* __restrict__ q, const int* __restrict__ epos,
                                                      double* __restrict__ qs, ChargeTail tail) {
  charges_body<true>(n, S, b, Sc, dv, Q0, q, epos, qs, tail);
}

// dst[f][epos[i]] = src[f][i]: charges of every frame in the electrodes'
// cell-sorted order (what the pair walkers stream)
__global__ __launch_bounds__(256) void k_permute(int n, const int* __restrict__ epos, const double* __restrict__ src,
                                                 double* __restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const size_t f = blockIdx.y;
  if (i < n) dst[f * n + epos[i]] = src[f * n + i];
}

// q[f][v][i] = Q0[f][i] + dv[v] Sc[i], and qs[f][epos[i]] = Q0[f][i] (the
// charges the force pass reads, in the electrodes' cell-sorted order)
__global__ __launch_bounds__(256) void k_expand_charges(int n_elec, int n_dv, const double* __restrict__ dv,
                                                        const double* __restrict__ Q0, const double* __restrict__ Sc,
                                                        double* __restrict__ q, const int* __restrict__ epos,
                                                        double* __restrict__ qs) {
  // a thread takes atom i of frame f over the whole sweep (its two inputs
  // read once, every store a run of consecutive atoms)
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int f = blockIdx.y;
  if (i >= n_elec) return;
  const double a = Q0[(size_t)f * n_elec + i], b = Sc[i];
  if (qs) qs[(size_t)f * n_elec + epos[i]] = a;
  double* o = q + (size_t)f * n_dv * n_elec + i;
  for (int v = 0; v < n_dv; ++v) o[(size_t)v * n_elec] = a + dv[v] * b;
}

// out[f][v][k] = comp[f][0][k] + dv[v] comp[f][1][k], k < n3: the forces are
// affine in dV, so the sweep is written from two vectors per frame, every
// store a full run of consecutive values
__global__ __launch_bounds__(256) void k_expand_forces(int n3, int n_dv, const double* __restrict__ dv,
                                                       const double* __restrict__ comp, double* __restrict__ out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int f = blockIdx.y;
  if (k >= n3) return;
  const double a = comp[(size_t)f * 2 * n3 + k];
  const double b = comp[(size_t)f * 2 * n3 + n3 + k];
  double* o = out + (size_t)f * n_dv * n3 + k;
  for (int v = 0; v < n_dv; ++v) o[(size_t)v * n3] = a + dv[v] * b;
}

// ------------------------------------------------------------ launchers

void launch_elastance_real(hipStream_t s, int n, const double* ex, const double* ey, const double* ez,
                           const Cell& cell, double alpha, double eta, double rcut, double self_term, double* A) {
  dim3 grid((n + 15) / 16, (n + 15) / 16);
  hipLaunchKernelGGL(k_elastance_real, grid, dim3(256), 0, s, n, ex, ey, ez, cell, alpha, eta, rcut * rcut,
                     self_term, A);
}
void launch_phase_matrix(hipStream_t s, int n, int nkc, int k0, int nk, const double* kv, const double* sk,
                         const double* ex, const double* ey, const double* ez, double* C) {
  hipLaunchKernelGGL(k_phase_matrix, dim3((nkc + 255) / 256, n), dim3(256), 0, s, n, nkc, k0, nk, kv, sk, ex, ey,
                     ez, C);
}
void launch_symmetrize(hipStream_t s, int n, double* A) {
  hipLaunchKernelGGL(k_symmetrize, dim3((n + 15) / 16, (n + 15) / 16), dim3(256), 0, s, n, A);
}
void launch_gj_invert(hipStream_t s, int n, double* A, double* dinv, double* pc, double* rx, int* flag) {
  const int nt = (n + GJ_TILE - 1) / GJ_TILE;
  hipLaunchKernelGGL(k_gj_pivot, dim3(1), dim3(256), 0, s, n, n < GJ_NB ? n : GJ_NB, A, dinv, flag);
  for (int k0 = 0; k0 < n; k0 += GJ_NB) {
    const int nb = n - k0 < GJ_NB ? n - k0 : GJ_NB;
    const int k1 = k0 + nb, nb1 = n - k1 < GJ_NB ? n - k1 : GJ_NB;
    hipLaunchKernelGGL(k_gj_panels, dim3((n + GJ_PCOLS - 1) / GJ_PCOLS), dim3(256), 0, s, n, k0, nb, A, dinv, pc, rx);
    hipLaunchKernelGGL(k_gj_update, dim3(1 + nt * nt), dim3(256), 0, s, n, k0, nb, k1, nb1, A, pc, rx, dinv, flag);
  }
}
void launch_matvec(hipStream_t s, int n, const double* Mx, const double* x, double* y) {
  hipLaunchKernelGGL(k_matvec, dim3((n + 3) / 4), dim3(256), 0, s, n, Mx, x, y);
}
void launch_dot(hipStream_t s, int n, const double* a, const double* b, double* out) {
  hipLaunchKernelGGL(k_dot, dim3(1), dim3(256), 0, s, n, a, b, out);
}
void launch_rank1(hipStream_t s, int n, double* S, const double* u, const double* sc) {
  hipLaunchKernelGGL(k_rank1, dim3((n + 15) / 16, (n + 15) / 16), dim3(256), 0, s, n, S, u, sc);
}
void launch_charges(hipStream_t s, int n_frames, int n, const double* S, const double* b, const double* Sc, double dv,
                    double* Q0, double* q, const int* epos, double* qs, const ChargeTail* tail) {
  const dim3 grid((n + 3) / 4, n_frames);
  if (tail)
    hipLaunchKernelGGL(k_charges_tail, grid, dim3(256), 0, s, n, S, b, Sc, dv, Q0, q, epos, qs, *tail);
  else
    hipLaunchKernelGGL(k_charges, grid, dim3(256), 0, s, n, S, b, Sc, dv, Q0, q, epos, qs);
}
void launch_permute(hipStream_t s, int n_frames, int n, const int* epos, const double* src, double* dst) {
  if (n == 0 || n_frames == 0) return;
  hipLaunchKernelGGL(k_permute, dim3((n + 255) / 256, n_frames), dim3(256), 0, s, n, epos, src, dst);
}
void launch_expand_forces(hipStream_t s, int n_frames, int n_site, int n_dv, const double* dv, const double* comp,
                          double* out) {
  const int n3 = 3 * n_site;
  if (n3 == 0 || n_frames == 0) return;
  hipLaunchKernelGGL(k_expand_forces, dim3((n3 + 255) / 256, n_frames), dim3(256), 0, s, n3, n_dv, dv, comp, out);
}
void launch_expand_charges(hipStream_t s, int n_frames, int n_elec, int n_dv, const double* dv, const double* Q0,
                           const double* Sc, double* q, const int* epos, double* qs) {
  hipLaunchKernelGGL(k_expand_charges, dim3((n_elec + 255) / 256, n_frames), dim3(256), 0, s, n_elec, n_dv, dv, Q0, Sc,
                     q, epos, qs);
}

}  // namespace cpm
