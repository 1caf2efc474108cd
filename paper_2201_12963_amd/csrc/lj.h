// Lennard-Jones forces and energy share of one electrolyte site, by one
// workgroup of LJ_WAVES wavefronts whose threads share the partners: the sites and
// graphene atoms of the z layers within the cutoff (the layers of the
// electrostatic cell grid, whose binning of the same positions has run),
// minimum image, pairs of one molecule excluded, energy shifted to zero at
// the cutoff, Lorentz-Berthelot mixing from the stored square roots of
// epsilon.  A kernel of its own (k_lj) or extra workgroups of the MD loop's
// field z pass.
#pragma once
#include "common.h"
#include "bin.h"
#include "pairs.h"

namespace cpm {

// Bound by latency and by the field pass's occupancy (its pair walk leaves 3
// waves per SIMD): a chain of dependent reads per site, so the partners come
// from the binning's sorted copies, coalesced, LJ_AHEAD per thread in flight
// with their parameters (one by one through the sort's index, an MD step of
// 1280 sites takes 57.7 us; so, 54.8).  Two wavefronts per site or one: 55.9,
// 56.3, fewer reads in flight.  No FP64 divisions: 1 / r^2 is the hardware's
// estimate with two Newton steps.
constexpr int LJ_AHEAD = 4;

__device__ __forceinline__ void lj_site(const LJArgs& a, int is) {
  constexpr int NT = LJ_WAVES * WAVE;
  __shared__ double red[LJ_WAVES][4];
  const double xi = a.sx[is], yi = a.sy[is], zi = a.sz[is];
  const int i = a.order[is];
  const double2 pi = a.par[i];
  const int mi = a.mol_of[i];
  const double rc2 = a.rc2, irc2 = a.irc2;
  double fx = 0.0, fy = 0.0, fz = 0.0, u = 0.0;
  // squared minimum-image distance, the displacement in d
  auto dist2 = [&](double (&d)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] -= a.box[k] * rint(d[k] * a.inv_box[k]);
    return d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
  };
  // eps4: 4 epsilon; uw: the site's share of the pair's energy (half of a
  // site-site pair's)
  auto pair = [&](const double (&d)[3], double r2, double sig, double eps4, double uw) {
    const double ir2 = recip_nr(r2), s2 = sig * sig;
    const double t = s2 * ir2, s6 = t * t * t, tc = s2 * irc2, c6 = tc * tc * tc;
    const double e = s6 * s6 - s6;
    const double fr = 6.0 * eps4 * fma(s6, s6, e) * ir2;
    fx = fma(fr, d[0], fx); fy = fma(fr, d[1], fy); fz = fma(fr, d[2], fz);
    u = fma(uw * eps4, e - (c6 * c6 - c6), u);
  };
  // the z layer of the site and the sorted-site ranges of the layers within
  // lj_reach (its margin covers a coordinate on a layer's face)
  int cz;
  wrap_and_cell(zi, a.box[2], a.nc_z, cz);
  const int* cs = a.cell_start;
  int lo0 = 0, hi0 = a.n_site, lo1 = 0, hi1 = 0;
  if (2 * a.lj_reach + 1 < a.nc_z) {
    const int la = cz - a.lj_reach, lb = cz + a.lj_reach;
    if (la < 0) { lo0 = cs[(la + a.nc_z) * a.nxy]; hi1 = cs[(lb + 1) * a.nxy]; }
    else if (lb >= a.nc_z) { lo0 = cs[la * a.nxy]; hi1 = cs[(lb + 1 - a.nc_z) * a.nxy]; }
    else { lo0 = cs[la * a.nxy]; hi0 = cs[(lb + 1) * a.nxy]; }
  }
  const int* cr = a.carbon_run + 4 * cz;
  const int c0 = cr[0], c1 = cr[2], m0 = cr[1] - c0, m = m0 + cr[3] - c1;
  // the four ranges as one run of partners, LJ_AHEAD of them per thread
  // loaded together, then their parameters together: two latencies a chunk
  const int n0 = hi0 - lo0, n = n0 + hi1 - lo1;
  for (int t0 = threadIdx.x; t0 < n + m; t0 += LJ_AHEAD * NT) {
    double p[LJ_AHEAD][3];
    int id[LJ_AHEAD];                          // the site's index, or -1
#pragma unroll
    for (int k = 0; k < LJ_AHEAD; ++k) {
      const int t = t0 + k * NT;
      id[k] = -1;
      if (t < n) {
        const int s = t < n0 ? lo0 + t : lo1 + t - n0;
        p[k][0] = a.sx[s]; p[k][1] = a.sy[s]; p[k][2] = a.sz[s]; id[k] = a.order[s];
      } else if (t < n + m) {
        const int q = t - n, j = q < m0 ? c0 + q : c1 + q - m0;
        p[k][0] = a.cx[j]; p[k][1] = a.cx[a.n_lj_elec + j]; p[k][2] = a.cx[2 * a.n_lj_elec + j];
      }
    }
    double2 pj[LJ_AHEAD];
    int mj[LJ_AHEAD];
#pragma unroll
    for (int k = 0; k < LJ_AHEAD; ++k) {
      pj[k] = double2{a.carbon_sigma, a.carbon_sqeps};
      mj[k] = -1;
      if (id[k] >= 0) { pj[k] = a.par[id[k]]; mj[k] = a.mol_of[id[k]]; }
    }
#pragma unroll
    for (int k = 0; k < LJ_AHEAD; ++k) {
      if (t0 + k * NT >= n + m) break;
      double d[3] = {xi - p[k][0], yi - p[k][1], zi - p[k][2]};
      const double r2 = dist2(d);
      if (r2 < rc2 && r2 > 0.0 && mj[k] != mi)
        pair(d, r2, 0.5 * (pi.x + pj[k].x), 4.0 * pi.y * pj[k].y, mj[k] < 0 ? 1.0 : 0.5);
    }
  }
  const double v[4] = {fx, fy, fz, u};
  const double tot = wave_sum4(v);             // lane l: value l >> 4
  const int w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  if ((lane & 15) == 0) red[w][lane >> 4] = tot;
  __syncthreads();
  if (threadIdx.x < 4) {
    double t = red[0][threadIdx.x];
#pragma unroll
    for (int k = 1; k < LJ_WAVES; ++k) t += red[k][threadIdx.x];
    if (threadIdx.x < 3) a.f_lj[threadIdx.x * a.n_site + i] = t;
    else a.u_lj[i] = t;
  }
}

}  // namespace cpm
