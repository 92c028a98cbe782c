// Restart remap, Galilean boost and frame-acceleration estimate
// (Sec. Domain remapping and frame conversion, eqs remap-state-vector,
// remap-cell-average, galilean-boost; Sec. Moving-frame dynamics and BH
// treatment, eq frame-acceleration).
//
// Remap: a target cell inside the excision
// sphere takes the sink state and one whose centre lies outside the source
// domain along a non-periodic axis the floor state; within kBand source cells
// inside a source face beyond which the target domain extends, the remapped
// density, momentum and thermal energy density are blended toward the floor
// state (at rest) with the weight s = 3u^2 - 2u^3 of the distance u to the
// nearest such face in band widths, so density and pressure reach the floor
// smoothly at the old domain's edge; on a target grid that
// coincides with the source grid (same spacing, origin a whole number of
// cells away) the source cell's conserved values are copied; otherwise the
// cell averages the trilinear interpolant of the source density, momentum and
// thermal energy density (the auxiliary energy with dual energy on,
// E - |m|^2/2rho otherwise) over its eight sub-cell midpoints, and rebuilds
// E = U + |m|^2/2rho (and U_aux = U).  Source neighbours are found through the
// source mesh's lattice map and read in place from its current buffers;
// stencils clamp at non-periodic source edges and wrap across periodic ones.
//
// The mean of the interpolant over the eight sub-cell points is a product of
// one-dimensional weights: along each axis the two points' linear weights give
// a target cell three taps on the source cells (four where a target cell is
// 1.95 source cells wide or more).  A workgroup takes a tile of target cells,
// stages the five fields of the source cells under it in LDS once, and each
// thread sums its cell's taps along x, then y, then z.  What bounds it: LDS
// reads (135 per target cell) and HBM (a target cell writes nv doubles).
// Gathering each of the 8 x 8 stencil cells from global memory, with a block
// look-up each, took 4.0 ms for 128^3 onto 256^3 cells (table EOS, six
// variables) against 0.9 GB to move.  The taps' sums round otherwise than the
// eight points' mean one after the other: results differ from it by about 3e-16.
#include "tdh_internal.hpp"

namespace tdh {

namespace {
constexpr int kRmThreads = 256;

struct SrcView {
  MeshDev m;
  const int *par;
  const double *Qa, *Qb;
};

__device__ __forceinline__ int src_axis(int i, int n, int periodic) {
  if (periodic) return i < 0 ? i + n * ((-i + n - 1) / n) : i % n;
  return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

// conserved values (nv) of global source cell (i, j, k), in-range indices
template <int NV>
__device__ __forceinline__ void src_cell(const SrcView &S, int i, int j, int k, double *q) {
  const MeshDev &m = S.m;
  const int b = m.lmap[((k >> m.lat_shift) * m.ly + (j >> m.lat_shift)) * m.lx + (i >> m.lat_shift)];
  const BlockInfo B = m.blocks[b];
  const double *Q = S.par[b] ? S.Qb : S.Qa;
  const long long n3 = (long long)B.n * B.n * B.n;
  const long long l = ((long long)(k - B.oz) * B.n + (j - B.oy)) * B.n + (i - B.ox);
#pragma unroll
  for (int v = 0; v < NV; ++v) q[v] = Q[B.off + v * n3 + l];
}

// rho, mx, my, mz, U_th of a source cell
template <int NV>
__device__ __forceinline__ void src_fields(const SrcView &S, int i, int j, int k, double *f) {
#pragma clang fp contract(off)
  double q[6];
  src_cell<NV>(S, i, j, k, q);
  f[0] = q[0];
  f[1] = q[1];
  f[2] = q[2];
  f[3] = q[3];
  if (NV > 5) {
    f[4] = q[5];
  } else {
    const double K = 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) / q[0];
    f[4] = q[4] - K;
  }
}

// trilinear interpolant of the five fields at point r (x, then y, then z)
template <int NV>
__device__ __forceinline__ void trilinear5(const SrcView &S, const double *r, double *out) {
#pragma clang fp contract(off)
  const int N[3] = {S.m.nx, S.m.ny, S.m.nz};
  int i0[3], i1[3];
  double w[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double xi = (r[d] - S.m.x0[d]) / S.m.dx[d] - 0.5;
    const double fl = floor(xi);
    w[d] = xi - fl;
    const int il = (int)fmin(fmax(fl, -1e9), 1e9);  // far-off points stay in int range (and NaN too)
    i0[d] = src_axis(il, N[d], S.m.bc[d] == 0);
    i1[d] = src_axis(il + 1, N[d], S.m.bc[d] == 0);
  }
  double c000[5], c100[5], c010[5], c110[5], c001[5], c101[5], c011[5], c111[5];
  src_fields<NV>(S, i0[0], i0[1], i0[2], c000);
  src_fields<NV>(S, i1[0], i0[1], i0[2], c100);
  src_fields<NV>(S, i0[0], i1[1], i0[2], c010);
  src_fields<NV>(S, i1[0], i1[1], i0[2], c110);
  src_fields<NV>(S, i0[0], i0[1], i1[2], c001);
  src_fields<NV>(S, i1[0], i0[1], i1[2], c101);
  src_fields<NV>(S, i0[0], i1[1], i1[2], c011);
  src_fields<NV>(S, i1[0], i1[1], i1[2], c111);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double a00 = (1.0 - w[0]) * c000[v] + w[0] * c100[v];
    const double a10 = (1.0 - w[0]) * c010[v] + w[0] * c110[v];
    const double a01 = (1.0 - w[0]) * c001[v] + w[0] * c101[v];
    const double a11 = (1.0 - w[0]) * c011[v] + w[0] * c111[v];
    const double b0 = (1.0 - w[1]) * a00 + w[1] * a10;
    const double b1 = (1.0 - w[1]) * a01 + w[1] * a11;
    out[v] = (1.0 - w[2]) * b0 + w[2] * b1;
  }
}

__device__ __forceinline__ bool excised_at(const Phys &p, const double *r, double t) {
  if (p.grav_kind != 2 || !(p.r_exc > 0.0)) return false;
  double s = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double q = r[d] - (p.bh_x0[d] - p.v_frame[d] * t);
    s += q * q;
  }
  return s < p.r_exc * p.r_exc;
}

__device__ __forceinline__ double u_floor_of(const Phys &p, double rho) {
  return p.eos_kind == 0 ? p.p_floor / (p.gamma - 1.0) : rho * p.e_floor;
}

constexpr double kBand = 2.0;  // width of the blending band in source cells

// blending weight of target centre c (inside the source domain): 1 away from the
// source faces the target domain extends beyond, falling smoothly to 0 at them
__device__ __forceinline__ double band_weight(const MeshDev &S, const MeshDev &D, const double *c) {
#pragma clang fp contract(off)
  const int NS[3] = {S.nx, S.ny, S.nz}, ND[3] = {D.nx, D.ny, D.nz};
  double u = 1.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (S.bc[a] == 0) continue;
    const double lo = S.x0[a], hi = S.x0[a] + NS[a] * S.dx[a];
    const double dlo = D.x0[a], dhi = D.x0[a] + ND[a] * D.dx[a];
    const double w = kBand * S.dx[a];
    if (dlo < lo) u = fmin(u, (c[a] - lo) / w);
    if (dhi > hi) u = fmin(u, (hi - c[a]) / w);
  }
  if (u <= 0.0) return 0.0;
  if (u >= 1.0) return 1.0;
  return u * u * (3.0 - 2.0 * u);
}
}  // namespace

// Floor (or sink) state, blending and the store of target cell gi with centre
// c: q holds its remapped conserved state, uth0 its thermal energy density.
template <int NV>
__device__ __forceinline__ void finish_target(const SrcView &S, const MeshDev &D, double *Qd, const Phys &p,
                                              const int *gi, const double *c, bool floored, double *q, double uth0) {
  if (floored) {
    const double uf = u_floor_of(p, p.rho_floor);
    q[0] = p.rho_floor;
    q[1] = q[2] = q[3] = 0.0;
    q[4] = uf;
    q[5] = uf;
  } else {
#pragma clang fp contract(off)
    const double w = band_weight(S.m, D, c);
    if (w < 1.0) {
      const double uf = u_floor_of(p, p.rho_floor);
      const double rho = w * q[0] + (1.0 - w) * p.rho_floor;
      const double m0 = w * q[1], m1 = w * q[2], m2 = w * q[3];
      const double uth = w * uth0 + (1.0 - w) * uf;
      q[0] = rho;
      q[1] = m0;
      q[2] = m1;
      q[3] = m2;
      q[4] = uth + 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) / rho;
      q[5] = uth;
    }
  }
  const int b = D.lmap[((gi[2] >> D.lat_shift) * D.ly + (gi[1] >> D.lat_shift)) * D.lx + (gi[0] >> D.lat_shift)];
  const BlockInfo B = D.blocks[b];
  const long long n3 = (long long)B.n * B.n * B.n;
  const long long l = ((long long)(gi[2] - B.oz) * B.n + (gi[1] - B.oy)) * B.n + (gi[0] - B.ox);
#pragma unroll
  for (int v = 0; v < NV; ++v) Qd[B.off + v * n3 + l] = q[v];
}

// whether target centre c lies outside the source domain along a non-periodic axis
__device__ __forceinline__ bool outside_source(const MeshDev &S, const double *c) {
  const int N[3] = {S.nx, S.ny, S.nz};
  bool out = false;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double lo = S.x0[d], hi = S.x0[d] + N[d] * S.dx[d];
    if (S.bc[d] != 0 && (c[d] < lo || c[d] >= hi)) out = true;
  }
  return out;
}

constexpr long long kRmBeyond = 1 << 17;  // cells outside the tiles worth a launch of their own

// A box of target cells, lo up to (not including) hi.
struct RemapBox {
  int lo[3], hi[3];
};

// One thread per target cell, reading the source in place: the copy onto a
// coincident grid, targets too coarse for the tiled form, and the cells beyond
// the source around the tiled form's box (left out).
template <int NV>
__global__ __launch_bounds__(kRmThreads) void remap_kernel(SrcView S, MeshDev D, double *Qd, Phys p, double t,
                                                            int coincident, int sx, int sy, int sz, RemapBox out) {
  const long long n = (long long)D.nx * D.ny * D.nz;
  for (long long g = blockIdx.x * (long long)kRmThreads + threadIdx.x; g < n; g += (long long)gridDim.x * kRmThreads) {
    const int gi[3] = {(int)(g % D.nx), (int)((g / D.nx) % D.ny), (int)(g / ((long long)D.nx * D.ny))};
    if (gi[0] >= out.lo[0] && gi[0] < out.hi[0] && gi[1] >= out.lo[1] && gi[1] < out.hi[1] && gi[2] >= out.lo[2] &&
        gi[2] < out.hi[2])
      continue;
    double c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) c[d] = D.x0[d] + (gi[d] + 0.5) * D.dx[d];
    const int NS[3] = {S.m.nx, S.m.ny, S.m.nz};
    double q[6], uth0 = 0.0;  // conserved state; its thermal energy density
    const bool floored = excised_at(p, c, t) || outside_source(S.m, c);
    if (floored) {
    } else if (coincident) {
      const int sh[3] = {sx, sy, sz};
      int si[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) si[d] = src_axis(gi[d] + sh[d], NS[d], S.m.bc[d] == 0);
      src_cell<NV>(S, si[0], si[1], si[2], q);
      uth0 = NV > 5 ? q[5] : q[4] - 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) / q[0];
    } else {
#pragma clang fp contract(off)
      double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
      for (int s = 0; s < 8; ++s) {
        const int ox = s & 1, oy = (s >> 1) & 1, oz = s >> 2;  // z outer, x inner
        const double r[3] = {c[0] + (ox ? 0.25 : -0.25) * D.dx[0], c[1] + (oy ? 0.25 : -0.25) * D.dx[1],
                             c[2] + (oz ? 0.25 : -0.25) * D.dx[2]};
        double f[5];
        trilinear5<NV>(S, r, f);
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v] += f[v];
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[v] *= 0.125;
      q[0] = acc[0];
      q[1] = acc[1];
      q[2] = acc[2];
      q[3] = acc[3];
      q[4] = acc[4] + 0.5 * (acc[1] * acc[1] + acc[2] * acc[2] + acc[3] * acc[3]) / acc[0];
      q[5] = acc[4];
      uth0 = acc[4];
    }
    finish_target<NV>(S, D, Qd, p, gi, c, floored, q, uth0);
  }
}

// Index of the source cell whose centre is at or below sub-cell point o (0:
// -1/4, 1: +1/4) of target cell g along axis d, and the weight of the next one.
__device__ __forceinline__ int source_point(const SrcView &S, const MeshDev &D, int d, int g, int o, double &w) {
#pragma clang fp contract(off)
  const double c = D.x0[d] + (g + 0.5) * D.dx[d];
  const double r = c + (o ? 0.25 : -0.25) * D.dx[d];
  const double xi = (r - S.m.x0[d]) / S.m.dx[d] - 0.5;
  const double fl = floor(xi);
  w = xi - fl;
  return (int)fmin(fmax(fl, -1e9), 1e9);  // far-off points stay in int range (and NaN too)
}

// Tile of target cells of a workgroup and the source cells it stages along each
// axis (the tile's first sub-cell point's cell onwards).
struct RemapTile {
  int t[3], s[3];
  int nt[3];  // tiles per axis
  RemapBox box;  // of the target cells they cover
};

template <int NV, int TAPS>
__global__ __launch_bounds__(kRmThreads) void remap_tiled_kernel(SrcView S, MeshDev D, double *Qd, Phys p, double t,
                                                                 RemapTile T) {
  extern __shared__ double sf[];  // five fields of the staged source cells
  const int ns = T.s[0] * T.s[1] * T.s[2];
  const int tile = blockIdx.x;
  const int o[3] = {T.box.lo[0] + tile % T.nt[0] * T.t[0], T.box.lo[1] + tile / T.nt[0] % T.nt[1] * T.t[1],
                    T.box.lo[2] + tile / (T.nt[0] * T.nt[1]) * T.t[2]};
  const int NS[3] = {S.m.nx, S.m.ny, S.m.nz};
  int base[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double w;
    base[d] = source_point(S, D, d, o[d], 0, w);
  }
  for (int e = threadIdx.x; e < ns; e += kRmThreads) {
    const int l[3] = {e % T.s[0], e / T.s[0] % T.s[1], e / (T.s[0] * T.s[1])};
    int si[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) si[d] = src_axis(base[d] + l[d], NS[d], S.m.bc[d] == 0);
    double f[5];
    src_fields<NV>(S, si[0], si[1], si[2], f);
#pragma unroll
    for (int v = 0; v < 5; ++v) sf[v * ns + e] = f[v];
  }
  __syncthreads();
  const int lt = threadIdx.x;
  const int gi[3] = {o[0] + lt % T.t[0], o[1] + lt / T.t[0] % T.t[1], o[2] + lt / (T.t[0] * T.t[1])};
  if (lt >= T.t[0] * T.t[1] * T.t[2] || gi[0] >= T.box.hi[0] || gi[1] >= T.box.hi[1] ||
      gi[2] >= T.box.hi[2])
    return;
  double c[3], W[3][TAPS];
  int l0[3], off[3][TAPS];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    c[d] = D.x0[d] + (gi[d] + 0.5) * D.dx[d];
    double w0, w1;
    const int i0 = source_point(S, D, d, gi[d], 0, w0), i1 = source_point(S, D, d, gi[d], 1, w1);
    l0[d] = min(max(i0 - base[d], 0), T.s[d] - TAPS);
    const int k1 = min(max(i1 - i0, 0), TAPS - 2);  // tap of the second point's cell
#pragma unroll
    for (int k = 0; k < TAPS; ++k) {
      W[d][k] = 0.5 * ((k == 0 ? 1.0 - w0 : (k == 1 ? w0 : 0.0)) + (k == k1 ? 1.0 - w1 : (k == k1 + 1 ? w1 : 0.0)));
      // taps past the second point's stencil have no weight and read a cell of
      // it again, so that a value outside it (infinite, NaN) never enters
      off[d][k] = (k < 2 ? k : min(k, k1 + 1)) * (d == 0 ? 1 : (d == 1 ? T.s[0] : T.s[0] * T.s[1]));
    }
  }
  double acc[5];
  const double *f0 = sf + l0[0] + T.s[0] * (l0[1] + T.s[1] * l0[2]);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double az = 0.0;
#pragma unroll
    for (int kz = 0; kz < TAPS; ++kz) {
      double ay = 0.0;
#pragma unroll
      for (int ky = 0; ky < TAPS; ++ky) {
        const double *r = f0 + v * ns + off[1][ky] + off[2][kz];
        double ax = W[0][0] * r[0];
#pragma unroll
        for (int kx = 1; kx < TAPS; ++kx) ax = fma(W[0][kx], r[off[0][kx]], ax);
        ay = ky ? fma(W[1][ky], ax, ay) : W[1][0] * ax;
      }
      az = kz ? fma(W[2][kz], ay, az) : W[2][0] * ay;
    }
    acc[v] = az;
  }
  double q[6] = {acc[0], acc[1], acc[2], acc[3], 0.0, acc[4]};
  q[4] = acc[4] + 0.5 * (acc[1] * acc[1] + acc[2] * acc[2] + acc[3] * acc[3]) / acc[0];
  finish_target<NV>(S, D, Qd, p, gi, c, excised_at(p, c, t) || outside_source(S.m, c), q, acc[4]);
}

// Galilean boost of the current state, in place (floor-density cells skipped)
template <int NV>
__global__ __launch_bounds__(kRmThreads) void boost_kernel(MeshDev m, const int *par, double *Qa, double *Qb,
                                                           double V0, double V1, double V2, double rho_skip) {
  const long long n = (long long)m.nx * m.ny * m.nz;
  for (long long g = blockIdx.x * (long long)kRmThreads + threadIdx.x; g < n; g += (long long)gridDim.x * kRmThreads) {
    const int i = (int)(g % m.nx), j = (int)((g / m.nx) % m.ny), k = (int)(g / ((long long)m.nx * m.ny));
    const int b = m.lmap[((k >> m.lat_shift) * m.ly + (j >> m.lat_shift)) * m.lx + (i >> m.lat_shift)];
    const BlockInfo B = m.blocks[b];
    double *Q = (par[b] ? Qb : Qa) + B.off;
    const long long n3 = (long long)B.n * B.n * B.n;
    const long long l = ((long long)(k - B.oz) * B.n + (j - B.oy)) * B.n + (i - B.ox);
    const double rho = Q[l];
    if (!(rho > rho_skip)) continue;
    const double mx = Q[n3 + l], my = Q[2 * n3 + l], mz = Q[3 * n3 + l];
    const double mv = (mx * V0 + my * V1) + mz * V2;
    const double v2 = (V0 * V0 + V1 * V1) + V2 * V2;
    Q[4 * n3 + l] = (Q[4 * n3 + l] + mv) + 0.5 * rho * v2;
    Q[n3 + l] = mx + rho * V0;
    Q[2 * n3 + l] = my + rho * V1;
    Q[3 * n3 + l] = mz + rho * V2;
  }
}

// partial sums of rho, rho g (x, y, z) over dense non-excised cells; a fixed
// grid of kRmParts workgroups, then one workgroup sums the partials
constexpr int kRmParts = 1024;
__global__ __launch_bounds__(kRmThreads) void frame_acc_partial_kernel(MeshDev m, const int *par, const double *Qa,
                                                                       const double *Qb, Phys p, double t,
                                                                       double rho_min, double *part) {
  __shared__ double red[4][kRmThreads];
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  const long long n = (long long)m.nx * m.ny * m.nz;
  for (long long g = blockIdx.x * (long long)kRmThreads + threadIdx.x; g < n; g += (long long)gridDim.x * kRmThreads) {
    const int i = (int)(g % m.nx), j = (int)((g / m.nx) % m.ny), k = (int)(g / ((long long)m.nx * m.ny));
    const int b = m.lmap[((k >> m.lat_shift) * m.ly + (j >> m.lat_shift)) * m.lx + (i >> m.lat_shift)];
    const BlockInfo B = m.blocks[b];
    const double *Q = (par[b] ? Qb : Qa) + B.off;
    const double rho = Q[((long long)(k - B.oz) * B.n + (j - B.oy)) * B.n + (i - B.ox)];
    const double c[3] = {m.x0[0] + (i + 0.5) * m.dx[0], m.x0[1] + (j + 0.5) * m.dx[1], m.x0[2] + (k + 0.5) * m.dx[2]};
    if (!(rho > rho_min) || excised_at(p, c, t)) continue;
    double dr[3], r2 = p.r_soft * p.r_soft;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      dr[d] = c[d] - (p.bh_x0[d] - p.v_frame[d] * t);
      r2 += dr[d] * dr[d];
    }
    const double f = -p.gm_bh / (r2 * sqrt(r2));
    s[0] += rho;
#pragma unroll
    for (int d = 0; d < 3; ++d) s[1 + d] += rho * (f * dr[d]);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[v][threadIdx.x] = s[v];
  __syncthreads();
  for (int w = kRmThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[v][threadIdx.x] += red[v][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[threadIdx.x * kRmParts + blockIdx.x] = red[threadIdx.x][0];
}

__global__ __launch_bounds__(kRmThreads) void frame_acc_final_kernel(const double *part, double *out) {
  __shared__ double red[4][kRmThreads];
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int q = threadIdx.x; q < kRmParts; q += kRmThreads)
#pragma unroll
    for (int v = 0; v < 4; ++v) s[v] += part[v * kRmParts + q];
#pragma unroll
  for (int v = 0; v < 4; ++v) red[v][threadIdx.x] = s[v];
  __syncthreads();
  for (int w = kRmThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[v][threadIdx.x] += red[v][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 3) out[threadIdx.x] = red[0][0] > 0.0 ? red[1 + threadIdx.x][0] / red[0][0] : 0.0;
}

static int rm_grid(long long n) {
  const long long g = (n + kRmThreads - 1) / kRmThreads;
  return (int)(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

hipError_t launch_remap(const MeshDev &src, const int *src_par, const double *sQa, const double *sQb,
                        const MeshDev &dst, double *Qd, const Phys &p, double t, int nv, int coincident,
                        const int *shift, hipStream_t s) {
  SrcView S{src, src_par, sQa, sQb};
  const int ND[3] = {dst.nx, dst.ny, dst.nz}, NS[3] = {src.nx, src.ny, src.nz};
  const long long n = (long long)dst.nx * dst.ny * dst.nz;
  auto cell_by_cell = [&](const RemapBox &out) {
    if (nv == 6)
      hipLaunchKernelGGL((remap_kernel<6>), dim3(rm_grid(n)), dim3(kRmThreads), 0, s, S, dst, Qd, p, t, coincident,
                         shift[0], shift[1], shift[2], out);
    else
      hipLaunchKernelGGL((remap_kernel<5>), dim3(rm_grid(n)), dim3(kRmThreads), 0, s, S, dst, Qd, p, t, coincident,
                         shift[0], shift[1], shift[2], out);
    return hipGetLastError();
  };
  // The tiled form takes targets up to nearly four source cells wide (three
  // taps cover two points less than one source cell apart, four taps less than
  // two), with the first tile whose staged cells fit 64 KB of LDS: 16 x 4 x 4
  // targets (whole 128-byte lines) to 1.3 source cells, smaller ones above.  The
  // copy onto a coincident grid reads each source cell once and needs no tile.
  double most = 0.0;
  for (int d = 0; d < 3; ++d) most = fmax(most, dst.dx[d] / src.dx[d]);
  if (!coincident && most < 3.9) {
    const int taps = most < 1.95 ? 3 : 4;
    const int shapes[3][3] = {{16, 4, 4}, {8, 4, 4}, {4, 4, 4}};
    for (const int *sh : shapes) {
      // Tiles cover the target cells inside the source (whole tiles from the
      // first such cell on), unless that leaves out less than a quarter of the
      // target or 2^17 cells (a launch more, 4 of 28 us for 24^3 cells): a cell beyond the source is a floor state, which the cell-by-cell
      // kernel writes at memory speed while a tile would stage source cells for
      // it.  192^3 targets of which the source holds 2 to 6 %, 1.3, 1.5 and 1.9
      // source cells wide: 538, 638 and 890 us by tiles everywhere, 135, 123 and
      // 111 this way, 289, 230 and 200 cell by cell.
      RemapTile T;
      long long cells = 1, tiles = 1, held = 1;
      for (int d = 0; d < 3; ++d) {
        T.box.lo[d] = 0;
        T.box.hi[d] = ND[d];
        if (src.bc[d] != 0) {
          const double end = src.x0[d] + NS[d] * src.dx[d];
          auto centre = [&](int g) { return dst.x0[d] + (g + 0.5) * dst.dx[d]; };
          while (T.box.lo[d] < ND[d] && centre(T.box.lo[d]) < src.x0[d]) ++T.box.lo[d];
          while (T.box.hi[d] > T.box.lo[d] && centre(T.box.hi[d] - 1) >= end) --T.box.hi[d];
          T.box.lo[d] -= T.box.lo[d] % sh[d];
        }
        held *= T.box.hi[d] - T.box.lo[d];
      }
      const bool whole = held > 0 && (4 * held > 3 * n || n - held < kRmBeyond);
      for (int d = 0; d < 3; ++d) {
        if (whole) {
          T.box.lo[d] = 0;
          T.box.hi[d] = ND[d];
        }
        T.t[d] = sh[d];
        T.nt[d] = (T.box.hi[d] - T.box.lo[d] + sh[d] - 1) / sh[d];
        T.s[d] = (int)floor((sh[d] - 0.5) * (dst.dx[d] / src.dx[d])) + taps + 1;
        cells *= T.s[d];
        tiles *= T.nt[d];
      }
      const size_t bytes = (size_t)cells * 5 * sizeof(double);
      if (bytes > 65536 || tiles > (1LL << 30)) continue;
      if (!whole) {
        const hipError_t e = cell_by_cell(T.box);
        if (e != hipSuccess || tiles == 0) return e;
      }
      const dim3 grid((unsigned)tiles), block(kRmThreads);
      if (nv == 6 && taps == 3) hipLaunchKernelGGL((remap_tiled_kernel<6, 3>), grid, block, bytes, s, S, dst, Qd, p, t, T);
      else if (nv == 6) hipLaunchKernelGGL((remap_tiled_kernel<6, 4>), grid, block, bytes, s, S, dst, Qd, p, t, T);
      else if (taps == 3) hipLaunchKernelGGL((remap_tiled_kernel<5, 3>), grid, block, bytes, s, S, dst, Qd, p, t, T);
      else hipLaunchKernelGGL((remap_tiled_kernel<5, 4>), grid, block, bytes, s, S, dst, Qd, p, t, T);
      return hipGetLastError();
    }
  }
  return cell_by_cell(RemapBox{});
}

hipError_t launch_boost(const MeshDev &m, const int *par, double *Qa, double *Qb, int nv, const double *V,
                        double rho_skip, hipStream_t s) {
  const long long n = (long long)m.nx * m.ny * m.nz;
  if (nv == 6)
    hipLaunchKernelGGL((boost_kernel<6>), dim3(rm_grid(n)), dim3(kRmThreads), 0, s, m, par, Qa, Qb, V[0], V[1], V[2],
                       rho_skip);
  else
    hipLaunchKernelGGL((boost_kernel<5>), dim3(rm_grid(n)), dim3(kRmThreads), 0, s, m, par, Qa, Qb, V[0], V[1], V[2],
                       rho_skip);
  return hipGetLastError();
}

hipError_t launch_frame_acceleration(const MeshDev &m, const int *par, const double *Qa, const double *Qb,
                                     const Phys &p, double t, double rho_min, double *part, double *out,
                                     hipStream_t s) {
  hipLaunchKernelGGL(frame_acc_partial_kernel, dim3(kRmParts), dim3(kRmThreads), 0, s, m, par, Qa, Qb, p, t, rho_min,
                     part);
  hipLaunchKernelGGL(frame_acc_final_kernel, dim3(1), dim3(kRmThreads), 0, s, part, out);
  return hipGetLastError();
}

int frame_acceleration_parts() { return kRmParts; }

}  // namespace tdh
