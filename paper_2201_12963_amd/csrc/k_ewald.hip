// Explicit Ewald reciprocal sums over a list of half-space wavevectors
// (k and -k contribute complex conjugates, so each listed k carries the
// doubled weight ew = 2 k_e w(k), w(k) = (4 pi/V) exp(-k^2/4 alpha^2)/k^2).
// Used for small cells, where a k-sphere of ~10^3 vectors is cheaper and
// more accurate than a mesh.
//   structure factor   rho(k) = sum_j Q_j e^{i k.R_j}       (one wave per k)
//   potential at the electrodes  sum_k ew Re(e^{-i k.r_i} rho(k))
//   all-charge factor  rho_all(k) = rho(k) + sum_i q_i e^{i k.r_i}
//   field at the sites E_j = -sum_k ew k Im(e^{-i k.R_j} rho_all(k))
//                      (k_site_forces_ewald, with the rest of the force)
// The electrode phases e^{i k.r_i} are a fixed table [k][atom].
//
// A step of such a cell is launch-bound: its kernels are microseconds of
// latency each, so whatever does not wait for each other shares a launch.
//   k_ewald_sf   the binning, and beside it the structure factor from the
//                unsorted positions;
//   k_ewald_b    b, real and reciprocal part of an atom in one workgroup,
//                and beside it the site-site sums;
//   (charges)    k_linalg.hip
//   k_ewald_rho_all
//   k_site_forces_ewald.
// At 144 atoms, 100 sites and 1327 k-vectors: nine launches of 62.5 us in all
// before, five now.
#include "bin.h"
#include "pairs.h"

namespace cpm {

constexpr int EWALD_SF_THREADS = 1024;     // the binning workgroups' width

__global__ __launch_bounds__(EWALD_SF_THREADS) void k_ewald_sf(BinArgs ba, int n_bin, int nk,
                                                               const double* __restrict__ kv,
                                                               const double* __restrict__ ew,
                                                               double2* __restrict__ rho, double* __restrict__ ek) {
  extern __shared__ __align__(16) int lds[];
  if ((int)blockIdx.x < n_bin) {
    bin_layers_block<EWALD_SF_THREADS>(ba, blockIdx.x, n_bin, lds);
    return;
  }
  const int lane = threadIdx.x & (WAVE - 1);
  const int k = (blockIdx.x - n_bin) * (EWALD_SF_THREADS / WAVE) + (threadIdx.x >> 6);
  if (k >= nk) return;
  const int n = ba.n_site;
  const double kx = kv[k], ky = kv[nk + k], kz = kv[2 * nk + k];
  const double* x = ba.xyz_all;
  // wrapped into the box like the binning's copies (a non-finite coordinate
  // counts as 0 there too)
  auto wrap = [](double v, double L, double rL) { return isfinite(v) ? v - L * floor(v * rL) : 0.0; };
  double re = 0.0, im = 0.0;
  for (int j = lane; j < n; j += WAVE) {
    const double px = wrap(x[j], ba.cell.L[0], ba.cell.invL[0]), py = wrap(x[n + j], ba.cell.L[1], ba.cell.invL[1]);
    const double pz = wrap(x[2 * (size_t)n + j], ba.cell.L[2], ba.cell.invL[2]), q = ba.site_q[j];
    double s, c;
    sincos(kx * px + ky * py + kz * pz, &s, &c);
    re += q * c;
    im += q * s;
  }
  re = wave_sum(re);
  im = wave_sum(im);
  if (lane == 0) {
    rho[k] = double2{re, im};
    if (ek) ek[k] = 0.5 * ew[k] * (re * re + im * im);
  }
}

// Workgroups 0 .. n_elec - 1: b of one electrode atom, the real-space part by
// the first wavefront, a third of the k-vectors by each of the others (the
// phase table is read across its rows, a line per lane: many loads in flight
// rather than one wavefront's chain).  Further workgroups: the site-site sums
// of four sites each.
__global__ __launch_bounds__(256) void k_ewald_b(int nk, const double* __restrict__ ew,
                                                 const double2* __restrict__ eph, const double2* __restrict__ rho,
                                                 RealBArgs<double> rb, double* __restrict__ b, SlabTerms sl,
                                                 PairArgs<double> pa) {
  __shared__ __align__(16) unsigned char scratch[4 * wave_scratch_bytes<double>()];
  __shared__ double part[4];
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x >> 6;
  double* ws = reinterpret_cast<double*>(scratch + wv * wave_scratch_bytes<double>());
  const int n_elec = rb.el.n;
  if ((int)blockIdx.x >= n_elec) {
    const int j = ((int)blockIdx.x - n_elec) * 4 + wv;
    if (j < pa.st.n) site_pairs_wave(pa.cell, pa.st, pa.alpha, pa.rc2, pa.f_pair, pa.u_site, j, 0, ws);
    return;
  }
  const int i = rb.el.orig[blockIdx.x];
  if (wv == 0) {
    const double phi = real_b_wave(rb.cell, rb.alpha, rb.eta, rb.rc2, rb.el, rb.st, rb.phi_out, blockIdx.x, 0, ws);
    if (lane == 0) part[0] = phi;
  } else {
    double acc = 0.0;
#pragma unroll 4
    for (int k = (wv - 1) * WAVE + lane; k < nk; k += 3 * WAVE) {
      const double2 e = eph[(size_t)k * n_elec + i], r = rho[k];
      acc += ew[k] * (e.x * r.x + e.y * r.y);       // Re(conj(e) rho)
    }
    acc = wave_sum(acc);
    if (lane == 0) part[wv] = acc;
  }
  __syncthreads();
  if (threadIdx.x == 0) b[i] = -(part[0] + ((part[1] + part[2]) + part[3])) - slab_b_term(sl, i, 0);
}

__global__ __launch_bounds__(256) void k_ewald_rho_all(int nk, int n_elec, const double2* __restrict__ eph,
                                                       const double* __restrict__ q, const double2* __restrict__ rho,
                                                       double2* __restrict__ out) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int k = blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x >> 6);
  if (k >= nk) return;
  const double2 r = rho[k];
  double re = 0.0, im = 0.0;
  for (int i = lane; i < n_elec; i += WAVE) {
    double2 e = eph[(size_t)k * n_elec + i];
    re += q[i] * e.x;
    im += q[i] * e.y;
  }
  re = wave_sum(re);
  im = wave_sum(im);
  if (lane == 0) out[k] = double2{r.x + re, r.y + im};
}

void launch_ewald_sf(hipStream_t s, const BinArgs& ba, int nk, const double* kv, const double* ew, double2* rho,
                     double* ek) {
  const int nb = bin_layer_wgs(ba.cell), per = EWALD_SF_THREADS / WAVE;
  const size_t lds = bin_layers_lds<EWALD_SF_THREADS>(ba.n_site, ba.cell);
  hipLaunchKernelGGL(k_ewald_sf, dim3(nb + (nk + per - 1) / per), dim3(EWALD_SF_THREADS), lds, s, ba, nb, nk, kv, ew,
                     rho, ek);
}
void launch_ewald_b(hipStream_t s, int nk, const double* ew, const double2* eph, const double2* rho,
                    const RealBArgs<double>& rb, double* b, const SlabTerms& sl, const PairArgs<double>* pa) {
  const PairArgs<double> p = pa ? *pa : PairArgs<double>{};
  hipLaunchKernelGGL(k_ewald_b, dim3(rb.el.n + p.n_blocks), dim3(256), 0, s, nk, ew, eph, rho, rb, b, sl, p);
}
void launch_ewald_rho_all(hipStream_t s, int nk, int n_elec, const double2* eph, const double* q, const double2* rho,
                          double2* out) {
  hipLaunchKernelGGL(k_ewald_rho_all, dim3((nk + 3) / 4), dim3(256), 0, s, nk, n_elec, eph, q, rho, out);
}

}  // namespace cpm
