// Cell binning of the electrolyte sites (the neighbour-list stage of an MD
// step, one of the itemised costs of the paper's timing breakdown), as the
// body of one workgroup of NT threads per frame:
//   1. cell id of every site (double precision, bit-identical to the integer
//      reference), kept in LDS; non-finite coordinates raise a status flag
//      and count as 0;
//   2. each wave owns a contiguous range of sites and walks it 64 at a time;
//      lanes with equal keys are grouped by AND-ing one ballot per key bit
//      (no atomics), every site records its rank among the earlier sites of
//      its wave and cell, and the lowest lane of each group advances the
//      wave's count of that cell;
//   3. a scan over (cell, wave) gives every wave its write offset per cell and
//      the cell_start array;
//   4. every site goes to offset + rank, all sites in parallel, so the sites
//      of a cell appear in increasing original index (a stable counting sort).
// The wrapped coordinates come from the same quotient x/L as the cell index,
// computed once in step 1 and carried to step 4 in a scratch array in global
// memory, which keeps the register count (and the occupancy of the many-frame
// launches) down.
// One frame takes bin_layers_block instead: the same sort split by z layers
// over up to BIN_LAYER_WGS workgroups.
// The sorted FP64 SoA copies (wrapped x, y, z and the charge) are what the
// later kernels stream; the body also sums Q_j Z_j for the finite-field energy.
#pragma once
#include "common.h"

namespace cpm {


// sites per thread whose loads are issued together
constexpr int BIN_BATCH = 6;

// LDS of the body (ints): cell ids, ranks, per-wave histograms, cell totals
template <int NT>
size_t bin_body_lds(int n_site, int n_cells) {
  return sizeof(int) * (2 * (size_t)n_site + (size_t)(NT / WAVE + 1) * n_cells);
}

// wrapped coordinate x - L floor(x/L) and cell index min(floor(f n), n - 1),
// f = x/L - floor(x/L), from one quotient (the same operations as
// cell_coord)
__device__ __forceinline__ double wrap_and_cell(double x, double L, int n, int& c) {
  const double t = x / L;
  const double fl = floor(t);
  const int ci = (int)floor((t - fl) * (double)n);
  c = ci < n - 1 ? ci : n - 1;
  return x - L * fl;
}

template <int NT, int BATCH>
__device__ __forceinline__ void bin_block(const BinArgs& a, int frame, int* lds) {
  constexpr int NW = NT / WAVE;
  const int n_site = a.n_site;
  const Cell& cell = a.cell;
  const int n_cells = cell.n_cells;
  int* cid = lds;                              // [n_site]
  int* rnk = cid + n_site;                     // [n_site]
  int* hist = rnk + n_site;                    // [NW][n_cells]
  int* tot = hist + NW * n_cells;              // [n_cells]
  __shared__ double red[NW];

  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = tid >> 6;
  const double* x = a.xyz_all + frame * a.frame_stride;
  const double* y = x + n_site;
  const double* z = y + n_site;
  int* cell_start = a.cell_start_all + (size_t)frame * (n_cells + 1);
  int* order = a.order_all + (size_t)frame * n_site;

  double* wx = a.wrap_all + (size_t)frame * 3 * n_site;
  double* wy = wx + n_site;
  double* wz = wy + n_site;

  // 1. cell ids and wrapped coordinates; the loads of BATCH sites per
  // thread are issued together
  double zd = 0.0;
  int bad = 0;
  for (int i0 = tid; i0 < n_site; i0 += BATCH * NT) {
    double xv[BATCH], yv[BATCH], zv[BATCH], qv[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int i = i0 + u * NT;
      xv[u] = yv[u] = zv[u] = qv[u] = 0.0;
      if (i < n_site) { xv[u] = x[i]; yv[u] = y[i]; zv[u] = z[i]; qv[u] = a.site_q[i]; }
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int i = i0 + u * NT;
      double ax = 0.0, ay = 0.0, az = 0.0;
      if (i < n_site) {
        double xi = xv[u], yi = yv[u], zi = zv[u];
        if (!isfinite(xi) || !isfinite(yi) || !isfinite(zi)) { bad = 1; xi = yi = zi = 0.0; }
        int cx, cy, cz;
        ax = wrap_and_cell(xi, cell.L[0], cell.nc[0], cx);
        ay = wrap_and_cell(yi, cell.L[1], cell.nc[1], cy);
        az = wrap_and_cell(zi, cell.L[2], cell.nc[2], cz);
        cid[i] = (cz * cell.nc[1] + cy) * cell.nc[0] + cx;
        wx[i] = ax; wy[i] = ay; wz[i] = az;
        zd += qv[u] * az;
      }
    }
  }
  if (bad) atomicOr(a.status, 1);
  for (int i = tid; i < NW * n_cells; i += NT) hist[i] = 0;
  zd = wave_sum(zd);
  if (lane == 0) red[wave] = zd;
  __syncthreads();
  if (tid == 0 && a.zdip_all) {
    double s = 0.0;
    for (int w = 0; w < NW; ++w) s += red[w];
    a.zdip_all[frame] = s;
  }

  // 2. ranks within (wave, cell) and per-wave counts; keys 0..n_cells
  // (n_cells pads the last batch)
  const int nbits = 32 - __clz(n_cells);
  const unsigned long long lt = (1ull << lane) - 1ull;
  const int per_wave = ((n_site + NW - 1) / NW + WAVE - 1) / WAVE * WAVE;
  const int lo = wave * per_wave;
  const int hi = min(n_site, lo + per_wave);
  // (the next batch's keys are read before this batch's ballots, so that
  // their LDS latency overlaps them)
  int key_next = (lo + lane < hi) ? cid[lo + lane] : n_cells;
  for (int base = lo; base < hi; base += WAVE) {
    const int i = base + lane;
    const int key = key_next;
    key_next = (i + WAVE < hi) ? cid[i + WAVE] : n_cells;
    unsigned long long eq = ~0ull;
    for (int b = 0; b < nbits; ++b) {
      const unsigned long long bb = __ballot((key >> b) & 1);
      eq &= ((key >> b) & 1) ? bb : ~bb;
    }
    const int r = __popcll(eq & lt);
    // rank in the low 24 bits, owning wave above (no division by per_wave later)
    if (key < n_cells) rnk[i] = (wave << 24) | (hist[wave * n_cells + key] + r);
    // every lane has read the count; the group leader advances it
    __builtin_amdgcn_wave_barrier();
    if (key < n_cells && r == 0) hist[wave * n_cells + key] += __popcll(eq);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();

  // 3. offsets: per cell, exclusive over waves (hist); then exclusive scan
  // over cells (tot); a site goes to tot + hist + rank
  for (int c = tid; c < n_cells; c += NT) {
    int run = 0;
    for (int w = 0; w < NW; ++w) {
      const int h = hist[w * n_cells + c];
      hist[w * n_cells + c] = run;
      run += h;
    }
    tot[c] = run;
  }
  __syncthreads();
  if (wave == 0) {
    int carry = 0;
    for (int c0 = 0; c0 < n_cells; c0 += WAVE) {
      const int c = c0 + lane;
      const int v = (c < n_cells) ? tot[c] : 0;
      int incl = v;
      for (int off = 1; off < WAVE; off <<= 1) {
        const int t = __shfl_up(incl, off, WAVE);
        if (lane >= off) incl += t;
      }
      if (c < n_cells) {
        tot[c] = carry + incl - v;     // exclusive start
        cell_start[c] = carry + incl - v;
      }
      carry += __shfl(incl, WAVE - 1, WAVE);
    }
    if (lane == 0) cell_start[n_cells] = carry;
  }
  __syncthreads();
  // (the cell starts folded into the offsets here, one register fewer in
  // step 4, which keeps the spread's occupancy)
  for (int i = tid; i < NW * n_cells; i += NT) hist[i] += tot[i % n_cells];
  __syncthreads();

  // 4. placement, every site independently
  double* sx = a.sx_all + (size_t)frame * n_site;
  double* sy = a.sy_all + (size_t)frame * n_site;
  double* sz = a.sz_all + (size_t)frame * n_site;
  double* sq = a.sq_all + (size_t)frame * n_site;
  // (all loads of a batch before any store: the output may not be assumed
  // apart from the input)
  for (int i0 = tid; i0 < n_site; i0 += BATCH * NT) {
    double xv[BATCH], yv[BATCH], zv[BATCH], qv[BATCH];
    int pv[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int i = i0 + u * NT;
      xv[u] = yv[u] = zv[u] = qv[u] = 0.0;
      pv[u] = 0;
      if (i < n_site) {
        xv[u] = wx[i]; yv[u] = wy[i]; zv[u] = wz[i]; qv[u] = a.site_q[i];
        const int rw = rnk[i];
        pv[u] = hist[(rw >> 24) * n_cells + cid[i]] + (rw & 0xffffff);
      }
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int i = i0 + u * NT;
      if (i < n_site) {
        const int pos = pv[u];
        order[pos] = i;
        sx[pos] = xv[u]; sy[pos] = yv[u]; sz[pos] = zv[u]; sq[pos] = qv[u];
      }
    }
  }
}

// ------------------------------------------------- one frame, by z layers

// The same sort for one frame, where the latency of a single workgroup is the
// launch's (7.6 / 11.7 / 24 us at 1280 / 2560 / 5120 sites): workgroup g of
// n_wg takes the z layers [nc_z g / n_wg, nc_z (g + 1) / n_wg), a contiguous
// range of cells.  Every workgroup reads every z; it keeps the sites of its
// layers in index order (ballots, each wavefront its own contiguous range of
// sites) and counts those of lower layers, which is where its part of the
// sorted arrays begins.  The rest is the counting sort above over its own
// sites and cells, so no workgroup waits for another.  A non-finite
// coordinate counts as 0 (and raises the status flag).
constexpr int BIN_LAYER_WGS = 16;        // workgroups at most
constexpr int BIN_LAYER_BATCH = 2;       // rounds of a wavefront's own sites held in registers
constexpr int BIN_SITE_BITS = 15;        // a list entry: site index, local cell above (binning limit: 19200 sites)

inline __host__ __device__ int bin_layer_wgs(const Cell& cell) {
  return cell.nc[2] < BIN_LAYER_WGS ? cell.nc[2] : BIN_LAYER_WGS;
}
template <int NT>
size_t bin_layers_lds(int n_site, const Cell& cell) {
  const int n_wg = bin_layer_wgs(cell), layers = (cell.nc[2] + n_wg - 1) / n_wg;
  return sizeof(int) * (2 * (size_t)n_site + (size_t)(NT / WAVE + 1) * layers * cell.nc[0] * cell.nc[1]);
}

template <int NT>
__device__ __forceinline__ void bin_layers_block(const BinArgs& a, int g, int n_wg, int* lds) {
  constexpr int NW = NT / WAVE, B = BIN_LAYER_BATCH;
  const int n_site = a.n_site;
  const Cell& cell = a.cell;
  const int nxy = cell.nc[0] * cell.nc[1];
  const int l0 = cell.nc[2] * g / n_wg, l1 = cell.nc[2] * (g + 1) / n_wg;
  const int nlc = (l1 - l0) * nxy, c_lo = l0 * nxy;
  int* ent = lds;                              // [n_site] a wavefront's sites from its range's start
  int* rnk = ent + n_site;                     // [n_site]
  int* hist = rnk + n_site;                    // [NW][nlc]
  int* tot = hist + NW * nlc;                  // [nlc]
  __shared__ int below[NW];
  __shared__ double red[NW];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
  const double* x = a.xyz_all;
  const double* y = x + n_site;
  const double* z = y + n_site;
  const int per_wave = ((n_site + NW - 1) / NW + WAVE - 1) / WAVE * WAVE;
  const int lo = min(n_site, wave * per_wave), hi = min(n_site, lo + per_wave);
  const unsigned long long lt = (1ull << lane) - 1ull;
  int* wh = hist + wave * nlc;
  for (int c = lane; c < nlc; c += WAVE) wh[c] = 0;

  // 1. the sites of the layers, and the count below them
  constexpr int U = 4;
  int cnt = 0, low = 0;
  double zd = 0.0;
  for (int b0 = lo; b0 < hi; b0 += U * WAVE) {
    double zv[U], qv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = b0 + u * WAVE + lane;
      zv[u] = i < hi ? z[i] : 0.0;
      qv[u] = g == 0 && i < hi ? a.site_q[i] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = b0 + u * WAVE + lane;
      if (b0 + u * WAVE >= hi) break;
      int cz;
      const double az = wrap_and_cell(isfinite(zv[u]) ? zv[u] : 0.0, cell.L[2], cell.nc[2], cz);
      zd += qv[u] * az;
      const bool in = i < hi && cz >= l0 && cz < l1;
      low += __popcll(__ballot(i < hi && cz < l0));
      const unsigned long long m = __ballot(in);
      if (in) ent[lo + cnt + __popcll(m & lt)] = i;
      cnt += __popcll(m);
    }
  }
  if (lane == 0) below[wave] = low;
  if (g == 0) {
    zd = wave_sum(zd);
    if (lane == 0) red[wave] = zd;
  }
  __builtin_amdgcn_wave_barrier();             // a wavefront's LDS operations complete in order

  // 2. coordinates, cells and ranks of the wavefront's sites
  double kx[B], ky[B], kz[B], kq[B];
  const int nbits = 32 - __clz(nlc);
  int bad = 0;
  auto load = [&](int j, double& px, double& py, double& pz, double& pq) {
    px = x[j]; py = y[j]; pz = z[j]; pq = a.site_q[j];
  };
  auto place = [&](double& px, double& py, double& pz) -> int {
    if (!isfinite(px) || !isfinite(py) || !isfinite(pz)) bad = 1;
    int cx, cy, cz;
    px = wrap_and_cell(isfinite(px) ? px : 0.0, cell.L[0], cell.nc[0], cx);
    py = wrap_and_cell(isfinite(py) ? py : 0.0, cell.L[1], cell.nc[1], cy);
    pz = wrap_and_cell(isfinite(pz) ? pz : 0.0, cell.L[2], cell.nc[2], cz);
    return ((cz - l0) * cell.nc[1] + cy) * cell.nc[0] + cx;
  };
  auto rank = [&](int e, int key, int j) {
    unsigned long long eq = ~0ull;
    for (int b = 0; b < nbits; ++b) {
      const unsigned long long bb = __ballot((key >> b) & 1);
      eq &= ((key >> b) & 1) ? bb : ~bb;
    }
    const int r = __popcll(eq & lt);
    if (key < nlc) {
      ent[lo + e] = j | key << BIN_SITE_BITS;
      rnk[lo + e] = wh[key] + r;
    }
    // every lane has read the count; the group leader advances it
    __builtin_amdgcn_wave_barrier();
    if (key < nlc && r == 0) wh[key] += __popcll(eq);
    __builtin_amdgcn_wave_barrier();
  };
  int kj[B];
#pragma unroll
  for (int u = 0; u < B; ++u) {
    const int e = u * WAVE + lane;
    kx[u] = ky[u] = kz[u] = kq[u] = 0.0;
    kj[u] = e < cnt ? ent[lo + e] : 0;
    if (e < cnt) load(kj[u], kx[u], ky[u], kz[u], kq[u]);
  }
#pragma unroll
  for (int u = 0; u < B; ++u) {
    if (u * WAVE >= cnt) break;
    const int e = u * WAVE + lane;
    int key = nlc;                             // (pads the round: nlc < 2^nbits)
    if (e < cnt) key = place(kx[u], ky[u], kz[u]);
    rank(e, key, kj[u]);
  }
  for (int e0 = B * WAVE; e0 < cnt; e0 += WAVE) {
    const int e = e0 + lane;
    int key = nlc, j = 0;
    if (e < cnt) {
      double px, py, pz, pq;
      j = ent[lo + e];
      load(j, px, py, pz, pq);
      key = place(px, py, pz);
    }
    rank(e, key, j);
  }
  if (bad) atomicOr(a.status, 1);
  __syncthreads();

  // 3. offsets: per cell, exclusive over waves; then over cells, from the
  // number of sites below
  for (int c = tid; c < nlc; c += NT) {
    int run = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int h = hist[w * nlc + c];
      hist[w * nlc + c] = run;
      run += h;
    }
    tot[c] = run;
  }
  __syncthreads();
  if (wave == 0) {
    int carry = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) carry += below[w];
    for (int c0 = 0; c0 < nlc; c0 += WAVE) {
      const int c = c0 + lane;
      const int v = (c < nlc) ? tot[c] : 0;
      int incl = v;
      for (int off = 1; off < WAVE; off <<= 1) {
        const int t = __shfl_up(incl, off, WAVE);
        if (lane >= off) incl += t;
      }
      if (c < nlc) {
        tot[c] = carry + incl - v;
        a.cell_start_all[c_lo + c] = carry + incl - v;
      }
      carry += __shfl(incl, WAVE - 1, WAVE);
    }
    if (lane == 0 && g == n_wg - 1) a.cell_start_all[cell.n_cells] = carry;
    if (lane == 0 && g == 0 && a.zdip_all) {
      double s = 0.0;
      for (int w = 0; w < NW; ++w) s += red[w];
      a.zdip_all[0] = s;
    }
  }
  __syncthreads();

  // 4. placement
  auto put = [&](int e, double px, double py, double pz, double pq) {
    const int v = ent[lo + e];
    const int c = v >> BIN_SITE_BITS;
    const int pos = tot[c] + wh[c] + rnk[lo + e];
    a.order_all[pos] = v & ((1 << BIN_SITE_BITS) - 1);
    a.sx_all[pos] = px; a.sy_all[pos] = py; a.sz_all[pos] = pz; a.sq_all[pos] = pq;
  };
#pragma unroll
  for (int u = 0; u < B; ++u)
    if (u * WAVE + lane < cnt) put(u * WAVE + lane, kx[u], ky[u], kz[u], kq[u]);
  for (int e = B * WAVE + lane; e < cnt; e += WAVE) {
    double px, py, pz, pq;
    load(ent[lo + e] & ((1 << BIN_SITE_BITS) - 1), px, py, pz, pq);
    place(px, py, pz);
    put(e, px, py, pz, pq);
  }
}

}  // namespace cpm
