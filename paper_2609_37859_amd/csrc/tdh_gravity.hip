// Self-gravity (Sec. Self-gravity solver): geometric multigrid for the
// periodic Poisson problem A phi = S on the mesh's uniform grid, A = -lap_h the
// seven-point operator with the anisotropic weights the paper states
// (wy = (dx/dy)^2, wz = (dx/dz)^2, centre 2 (1 + wy + wz)) and
// S = -4 pi G (rho - mean rho) (eq selfgrav-poisson; the mean is removed so the
// periodic problem is solvable).
//
// V-cycle (the paper's order): two red-black Gauss-Seidel sweeps with
// over-relaxation 1.15, the defect d = S - A phi (eq selfgrav-defect) averaged
// over the eight children onto the coarser level, full-approximation coarse
// problem (start R phi, source R d + A_c R phi), the correction returned by
// tricubic interpolation, two post-sweeps; the coarsest level takes
// 2 (nx+ny+nz)^2 sweeps in one workgroup's LDS; one extra finest sweep ends
// each cycle.
//
// Every level is stored in red-black order: the red cells (i+j+k even) first,
// then the black ones, each colour as [nz][ny][nx/2] with x fastest, and
// addressed periodically (no ghost cells, so no ghost-fill launches).  Each
// level has even dimensions, so the colours are a true 2-colouring and a
// colour's cells update independently: one thread per cell of the colour,
// the same values as a sequential sweep, reading and writing its colour's
// half contiguously and its neighbours from the other half.  Levels are HBM-bound stencils
// (about 24 bytes per cell and sweep at the finest level); the levels that fit
// one workgroup's LDS run there in one launch, and the host captures a cycle in
// a graph.
// Sums (mean density, defect norm, mean potential) use a fixed grid and a
// fixed tree, so they are deterministic.
#include "tdh_internal.hpp"

namespace tdh {

namespace {

constexpr double kOmegaGS = 1.15;
constexpr int kMgThreads = 256;

__device__ __forceinline__ int pwrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

__device__ __forceinline__ long long ncell(const MgLevel &L) { return (long long)L.nx * L.ny * L.nz; }

// storage index of cell (i, j, k), offsets of up to two cells wrapped
__device__ __forceinline__ long long at(const MgLevel &L, int i, int j, int k) {
  i = pwrap(i, L.nx);
  j = pwrap(j, L.ny);
  k = pwrap(k, L.nz);
  const long long nat = ((long long)k * L.ny + j) * L.nx + i;
  return ((i + j + k) & 1) * (ncell(L) >> 1) + (nat >> 1);
}

// cell of storage index q
__device__ __forceinline__ void cell_of(const MgLevel &L, long long q, int &i, int &j, int &k) {
  const long long half = ncell(L) >> 1;
  const int color = q >= half;
  const long long r = q - color * half;
  const int hx = L.nx >> 1;
  const long long row = r / hx;
  j = (int)(row % L.ny);
  k = (int)(row / L.ny);
  i = 2 * (int)(r % hx) + ((j + k + color) & 1);
}

// ((x- + x+) + wy (y- + y+)) + wz (z- + z+)
__device__ __forceinline__ double nbsum(const MgLevel &L, const double *f, int i, int j, int k) {
#pragma clang fp contract(off)
  const double sx = f[at(L, i - 1, j, k)] + f[at(L, i + 1, j, k)];
  const double sy = f[at(L, i, j - 1, k)] + f[at(L, i, j + 1, k)];
  const double sz = f[at(L, i, j, k - 1)] + f[at(L, i, j, k + 1)];
  return (sx + L.wy * sy) + L.wz * sz;
}

// x / c0 by the reciprocal and one correction: the rounded quotient in three
// dependent operations instead of a division's eleven
__device__ __forceinline__ double over_c0(double c0, double r0, double x) {
  const double q = x * r0;
  return fma(fma(-c0, q, x), r0, q);
}
__device__ __forceinline__ double apply_A(const MgLevel &L, const double *f, int i, int j, int k) {
#pragma clang fp contract(off)
  return (L.c0 * f[at(L, i, j, k)] - nbsum(L, f, i, j, k)) / L.hx2;
}

__device__ __forceinline__ double gs_value(const MgLevel &L, const double *phi, double src, int i, int j, int k,
                                           double old) {
#pragma clang fp contract(off)
  const double gs = (nbsum(L, phi, i, j, k) + L.hx2 * src) / L.c0;
  return (1.0 - kOmegaGS) * old + kOmegaGS * gs;
}

__device__ __forceinline__ double child_mean(const MgLevel &F, const double *f, int i, int j, int k) {
#pragma clang fp contract(off)
  const int I = 2 * i, J = 2 * j, K = 2 * k;
  const double a = f[at(F, I, J, K)] + f[at(F, I + 1, J, K)];
  const double b = f[at(F, I, J + 1, K)] + f[at(F, I + 1, J + 1, K)];
  const double c = f[at(F, I, J, K + 1)] + f[at(F, I + 1, J, K + 1)];
  const double d = f[at(F, I, J + 1, K + 1)] + f[at(F, I + 1, J + 1, K + 1)];
  return 0.125 * ((a + b) + (c + d));
}


}  // namespace

// the density of every cell into the finest level's source array
__global__ __launch_bounds__(kMgThreads) void mg_gather_kernel(MeshDev m, const int *par, const double *Qa,
                                                                  const double *Qb, MgLevel F) {
  const long long n = ncell(F);
  for (long long q = blockIdx.x * (long long)kMgThreads + threadIdx.x; q < n; q += (long long)gridDim.x * kMgThreads) {
    int i, j, k;
    cell_of(F, q, i, j, k);
    const int b = m.lmap[((k >> m.lat_shift) * m.ly + (j >> m.lat_shift)) * m.lx + (i >> m.lat_shift)];
    const BlockInfo B = m.blocks[b];
    const double *Q = par[b] ? Qb : Qa;
    F.src[q] = Q[B.off + ((long long)(k - B.oz) * B.n + (j - B.oy)) * B.n + (i - B.ox)];
  }
}

// per-workgroup partial sums of x (or x^2) over a fixed grid-stride share
__global__ __launch_bounds__(kMgThreads) void mg_partial_sum_kernel(const double *x, long long n, int square,
                                                                       double *part) {
  __shared__ double red[kMgThreads];
  double s = 0.0;
  for (long long p = blockIdx.x * (long long)kMgThreads + threadIdx.x; p < n; p += (long long)gridDim.x * kMgThreads) {
    const double v = x[p];
    s += square ? v * v : v;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = kMgThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// out = sum(part) * scale (op 0) or sqrt(sum(part) * scale) (op 1); one workgroup
__global__ __launch_bounds__(kMgThreads) void mg_final_sum_kernel(const double *part, int nparts, double scale,
                                                                     int op, double *out) {
  __shared__ double red[kMgThreads];
  double s = 0.0;
  for (int p = threadIdx.x; p < nparts; p += kMgThreads) s += part[p];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = kMgThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = op == 0 ? red[0] * scale : sqrt(red[0] * scale);
}

// src = -4 pi G (rho - mean); rho arrives in src
__global__ __launch_bounds__(kMgThreads) void mg_source_kernel(double *src, const double *mean, double four_pi_G,
                                                                  long long n) {
  const double mu = mean[0];
  for (long long p = blockIdx.x * (long long)kMgThreads + threadIdx.x; p < n; p += (long long)gridDim.x * kMgThreads)
    src[p] = -four_pi_G * (src[p] - mu);
}

__global__ __launch_bounds__(kMgThreads) void mg_affine_kernel(double *x, const double *shift, double zero_fill,
                                                                  long long n) {
  // x -= shift[0] (shift non-null) or x = zero_fill
  for (long long p = blockIdx.x * (long long)kMgThreads + threadIdx.x; p < n; p += (long long)gridDim.x * kMgThreads)
    x[p] = shift ? x[p] - shift[0] : zero_fill;
}

__global__ __launch_bounds__(kMgThreads) void mg_rbgs_kernel(MgLevel L, int color) {
  const long long half = ncell(L) >> 1;
  for (long long t = blockIdx.x * (long long)kMgThreads + threadIdx.x; t < half; t += (long long)gridDim.x * kMgThreads) {
    const long long q = color * half + t;
    int i, j, k;
    cell_of(L, q, i, j, k);
    L.phi[q] = gs_value(L, L.phi, L.src[q], i, j, k, L.phi[q]);
  }
}

__device__ __forceinline__ double defect_at(const MgLevel &L, int i, int j, int k) {
  return L.src[at(L, i, j, k)] - apply_A(L, L.phi, i, j, k);
}

// per-workgroup partial sums of the squared defect over the same fixed
// grid-stride shares as mg_partial_sum_kernel (the defect is not stored)
__global__ __launch_bounds__(kMgThreads) void mg_defect_sq_partial_kernel(MgLevel L, double *part) {
  __shared__ double red[kMgThreads];
  const long long n = ncell(L);
  double s = 0.0;
  for (long long q = blockIdx.x * (long long)kMgThreads + threadIdx.x; q < n; q += (long long)gridDim.x * kMgThreads) {
    int i, j, k;
    cell_of(L, q, i, j, k);
    const double d = L.src[q] - apply_A(L, L.phi, i, j, k);
    s += d * d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = kMgThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------------------
// Red-black sweeps of a large level in one pass over memory: S half-sweeps (two
// or four) from L.phi to `out`, and then the squared defect of the result or the
// coarse level's start (mg_restrict_kernel's values).
// One colour's kernel reads and writes four half-arrays, so that two sweeps move
// eight times the level's potential and the defect twice more; here they move
// three (potential and source in, potential out) and the halo.  A workgroup
// holds 32 x 32 columns of cell pairs (one red, one black) and marches along z:
// in step z it loads plane z and updates plane z - s by half-sweep s, each from
// the previous half-sweep's three planes in registers and its plane's neighbours
// in LDS, published one step before; one barrier per plane.  A half-sweep spoils
// one more cell at the columns' edge, which the tiles overlap by (28 x 24 pairs
// of the 32 x 32 are written by two sweeps, 28 x 26 by one with the defect), and
// one more plane at the ends of a z chunk.  The values are the one-colour
// kernel's, the defect's sum is taken in another order.
// 256^3: two sweeps 131 us against 250 (with the restriction 156 against 365), a
// sweep and the defect 104 us against 258;
// registers held to 64 for two workgroups on a compute unit spill (twice as slow).
// Levels of 2^20 cells and more: ten cycles of 256^3 12.7 -> 9.0 ms, 128^3 3.24 ->
// 2.68, 128 x 128 x 64 2.50 -> 2.19; below, the tiles and z chunks are too few to
// pay for their edges (64^3 1.74 ms plain, 1.77 this way; 128 x 64 x 32 1.70, 1.78).
// ---------------------------------------------------------------------------
constexpr int kMgSmoothThreads = 1024, kMgEdge = 32;
constexpr long long kMgSmoothCells = 1 << 20;
enum { kMgPlain, kMgNorm, kMgRestrict };  // after the sweeps: nothing, the squared defect, the coarse level's start
template <int S, int TAIL>
struct MgSmooth {
  static constexpr int H = S + (TAIL == kMgPlain ? 0 : 1);   // spoiled cells at every edge
  static constexpr int PX = (H + 1) / 2, PY = H;             // in pairs and rows
  static constexpr int OX = kMgEdge - 2 * PX, OY = kMgEdge - 2 * PY;
};

__device__ __forceinline__ int modulo(int a, int n) {
  a %= n;
  return a < 0 ? a + n : a;
}

template <int S, int TAIL>
__global__ __launch_bounds__(kMgSmoothThreads) void mg_smooth_kernel(MgLevel L, double *out, int tx, int ty, int nc,
                                                                     double *part, MgLevel C) {
#pragma clang fp contract(off)
  using G = MgSmooth<S, TAIL>;
  static_assert(S == 2 ? TAIL != kMgRestrict : S == 4 && TAIL != kMgNorm, "the planes kept below");
  constexpr bool NORM = TAIL == kMgNorm, REST = TAIL == kMgRestrict;
  __shared__ double sh[2][REST ? 6 : 4][kMgSmoothThreads];
  __shared__ double rows[REST ? 2 : 1][2][REST ? kMgSmoothThreads : 1];  // a plane's pair sums of potential and defect
  // workgroups of one XCD take consecutive tiles: neighbours share its L2
  const int per = gridDim.x / 8, id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (id >= tx * ty * nc) return;
  const int ti = id % tx, tj = (id / tx) % ty, tc = id / (tx * ty);
  const int k0 = 2 * (int)((long long)(L.nz / 2) * tc / nc), k1 = 2 * (int)((long long)(L.nz / 2) * (tc + 1) / nc);
  const int t = threadIdx.x, lane = t & (kMgEdge - 1), row = t / kMgEdge;
  const int hx = L.nx >> 1;
  const int pi = ti * G::OX + lane - G::PX, pj = tj * G::OY + row - G::PY;
  const bool mine = lane >= G::PX && lane < kMgEdge - G::PX && row >= G::PY && row < kMgEdge - G::PY && pi < hx &&
                    pj < L.ny;
  const int j = modulo(pj, L.ny);
  const long long plane = (long long)hx * L.ny, half = ncell(L) >> 1;
  const long long col = (long long)j * hx + modulo(pi, hx);
  // neighbours in the plane: the edge's own value beyond the columns (spoiled cells)
  const int tl = lane ? t - 1 : t, tr = lane < kMgEdge - 1 ? t + 1 : t;
  const int tm = row ? t - kMgEdge : t, tp = row < kMgEdge - 1 ? t + kMgEdge : t;
  const double rc0 = 1.0 / L.c0, rh = 1.0 / L.hx2;
  auto nb = [&](const double *f, int side, double own, double below, double above) {
    const double sx = own + f[side];
    const double sy = f[tm] + f[tp];
    const double sz = below + above;
    return (sx + L.wy * sy) + L.wz * sz;
  };
  auto relax = [&](double n, double src, double old) {
    return (1.0 - kOmegaGS) * old + kOmegaGS * over_c0(L.c0, rc0, n + L.hx2 * src);
  };
  auto defect = [&](double n, double src, double f) { return src - over_c0(L.hx2, rh, L.c0 * f - n); };

  // planes z, z-1, ...: potential of both colours as loaded (0), after the first
  // sweep (1) and the second (2), whose newest plane is z - (half-sweeps done); sources
  double R0[2] = {}, B0[3] = {}, R1[4] = {}, B1[3] = {}, R2[4] = {}, B2[3] = {}, SR[6] = {}, SB[6] = {};
  int zl = modulo(k0 - G::H, L.nz);
  long long at0 = zl * plane + col;
  double nr = L.phi[at0], nbk = L.phi[half + at0], nsr = L.src[at0], nsb = L.src[half + at0];
  double sum = 0.0, f0 = 0.0, d0 = 0.0;
  for (int z = k0 - G::H; z < k1 + G::H + (REST ? 1 : 0); ++z) {
    R0[1] = R0[0]; R0[0] = nr;
    B0[2] = B0[1]; B0[1] = B0[0]; B0[0] = nbk;
    SR[5] = SR[4]; SR[4] = SR[3]; SR[3] = SR[2]; SR[2] = SR[1]; SR[1] = SR[0]; SR[0] = nsr;
    SB[5] = SB[4]; SB[4] = SB[3]; SB[3] = SB[2]; SB[2] = SB[1]; SB[1] = SB[0]; SB[0] = nsb;
    if (z + 1 < k1 + G::H) {  // the next plane, under way during this one
      zl = zl + 1 == L.nz ? 0 : zl + 1;
      at0 = zl * plane + col;
      nr = L.phi[at0];
      nbk = L.phi[half + at0];
      nsr = L.src[at0];
      nsb = L.src[half + at0];
    }
    const double(*f)[kMgSmoothThreads] = sh[(z & 1) ^ 1];
    double(*g)[kMgSmoothThreads] = sh[z & 1];
    // of a pair in row j of plane k the red cell is the right one if j + k is odd,
    // and a cell's other neighbour along x is in the pair beside it: that of plane
    // z-1's red, plane z-2's black, plane z-3's red and plane z-4's black cell
    const int side = (j + z) & 1 ? tl : tr, other = (j + z) & 1 ? tr : tl;
    const double r1 = relax(nb(f[0], side, B0[1], B0[2], B0[0]), SR[1], R0[1]);
    R1[3] = R1[2]; R1[2] = R1[1]; R1[1] = R1[0]; R1[0] = r1;
    const double b1 = relax(nb(f[1], side, R1[1], R1[2], R1[0]), SB[2], B0[2]);
    B1[2] = B1[1]; B1[1] = B1[0]; B1[0] = b1;
    double vr = R1[1], vb = b1;
    if constexpr (S == 4) {
      const double r2 = relax(nb(f[2], side, B1[1], B1[2], B1[0]), SR[3], R1[2]);
      R2[3] = R2[2]; R2[2] = R2[1]; R2[1] = R2[0]; R2[0] = r2;
      vb = relax(nb(f[3], side, R2[1], R2[2], R2[0]), SB[4], B1[2]);
      vr = R2[1];
      B2[2] = B2[1]; B2[1] = B2[0]; B2[0] = vb;
    }
    const int q = z - S;
    if (mine && q >= k0 && q < k1) {
      const long long p = q * plane + col;
      out[p] = vr;
      out[half + p] = vb;
    }
    if constexpr (NORM) {  // plane z-3
      const double dr = defect(nb(f[2], side, B1[1], B1[2], B1[0]), SR[3], R1[2]);
      const double db = defect(nb(f[3], other, R1[2], R1[3], R1[1]), SB[3], B1[1]);
      if (mine && z - 3 >= k0 && z - 3 < k1) sum += dr * dr + db * db;
    }
    if constexpr (REST) {
      // plane z-6, whose rows' sums are in LDS: the children of one coarse cell
      // are a pair in two rows and two planes
      if (mine && (row & 1)) {
        const double(*p)[kMgSmoothThreads] = rows[(z & 1) ^ 1];
        const double fs = p[0][t] + p[0][t + kMgEdge], ds = p[1][t] + p[1][t + kMgEdge];
        const int k = z - 6;
        if (k & 1) {
          if (k > k0 && k < k1) {
            const int cj = pj >> 1, ck = k >> 1;
            const long long q = ((pi + cj + ck) & 1) * (ncell(C) >> 1) + (((long long)ck * C.ny + cj) * C.nx + pi >> 1);
            const double r = 0.125 * (f0 + fs);
            C.phi[q] = r;
            C.rphi[q] = r;
            C.src[q] = 0.125 * (d0 + ds);
          }
        } else {
          f0 = fs;
          d0 = ds;
        }
      }
      // plane z-5
      const double dr = defect(nb(f[5], side, B2[1], B2[2], B2[0]), SR[5], R2[2]);
      const double db = defect(nb(f[4], other, R2[2], R2[3], R2[1]), SB[5], B2[1]);
      rows[z & 1][0][t] = R2[2] + B2[1];
      rows[z & 1][1][t] = dr + db;
      g[4][t] = R2[1];
      g[5][t] = B2[0];
    }
    g[0][t] = B0[0];
    g[1][t] = R1[0];
    g[2][t] = B1[0];
    g[3][t] = NORM ? R1[1] : R2[0];
    __syncthreads();
  }
  if constexpr (NORM) {
    double *red = sh[0][0];
    red[t] = sum;
    __syncthreads();
    for (int w = kMgSmoothThreads / 2; w > 0; w >>= 1) {
      if (t < w) red[t] += red[t + w];
      __syncthreads();
    }
    if (t == 0) part[id] = red[0];
  }
}

// coarse start R phi (also kept in rphi) and the restricted defect, the
// children's defects computed here (the same values and order of summation
// as a stored defect averaged over the eight children)
__global__ __launch_bounds__(kMgThreads) void mg_restrict_kernel(MgLevel F, MgLevel C) {
  const long long n = ncell(C);
  for (long long q = blockIdx.x * (long long)kMgThreads + threadIdx.x; q < n; q += (long long)gridDim.x * kMgThreads) {
    int i, j, k;
    cell_of(C, q, i, j, k);
    const double r = child_mean(F, F.phi, i, j, k);
    C.phi[q] = r;
    C.rphi[q] = r;
    const int I = 2 * i, J = 2 * j, K = 2 * k;
    double dm;
    {
#pragma clang fp contract(off)
      const double a = defect_at(F, I, J, K) + defect_at(F, I + 1, J, K);
      const double b = defect_at(F, I, J + 1, K) + defect_at(F, I + 1, J + 1, K);
      const double c = defect_at(F, I, J, K + 1) + defect_at(F, I + 1, J, K + 1);
      const double d = defect_at(F, I, J + 1, K + 1) + defect_at(F, I + 1, J + 1, K + 1);
      dm = 0.125 * ((a + b) + (c + d));
    }
    C.src[q] = dm;
  }
}

// coarse source R d + A_c R phi
__global__ __launch_bounds__(kMgThreads) void mg_coarse_source_kernel(MgLevel C) {
  const long long n = ncell(C);
  for (long long q = blockIdx.x * (long long)kMgThreads + threadIdx.x; q < n; q += (long long)gridDim.x * kMgThreads) {
    int i, j, k;
    cell_of(C, q, i, j, k);
    C.src[q] = C.src[q] + apply_A(C, C.phi, i, j, k);
  }
}

// ---------------------------------------------------------------------------
// The V-cycle from the first level of at most kMgLdsTop cells down, in one
// workgroup's LDS: its sweeps, restrictions, coarse sources, the coarsest
// level's sweeps, prolongations and post-sweeps, with the values and the order
// of operations of the level-by-level kernels.  Those levels are too small to
// fill the chip, and as kernels of their own each of their passes costs a launch
// of 2 to 5 us (37 launches for 16^3 down to 2^3, 48 of the 64 x 16 x 16 solve's
// 65 launches per cycle).  A serial chain bounds it: one workgroup, a barrier per
// colour.  Measured per solve: 64 x 16 x 16 995 -> 664 us, 256^3 9.62 -> 9.20 ms.
// ---------------------------------------------------------------------------
constexpr int kMgCoarseMax = 2048;
constexpr int kMgLdsTop = 8192;
constexpr int kMgLdsDoubles = 20480;  // all 160 KB: potential and source of the top, three arrays below it
constexpr int kMgLdsLevels = 12;
constexpr int kMgLdsThreads = 1024;

// A level of the LDS cycle: offsets (in doubles) of its arrays; mx, my: rounded-
// up 2^32 / hx and 2^32 / ny (row and plane of a cell by one multiplication).
struct MgLdsLevel {
  int nx, ny, nz, hx, half;
  unsigned mx, my;
  int phi, src, rphi;
  double hx2, wy, wz, c0, r0;  // r0 = 1 / c0
};
struct MgLdsCycle {
  int n;
  MgLdsLevel lv[kMgLdsLevels];
  double *phi;        // the top level's arrays in global memory
  const double *src;
};

struct LdsCell {
  int i, j, k;
};
__device__ __forceinline__ LdsCell lds_cell(const MgLdsLevel &L, int r, int color) {
  const int row = L.hx == 1 ? r : (int)__umulhi((unsigned)r, L.mx);
  const int k = L.ny == 1 ? row : (int)__umulhi((unsigned)row, L.my);
  LdsCell c;
  c.k = k;
  c.j = row - k * L.ny;
  c.i = 2 * (r - row * L.hx) + ((c.j + k + color) & 1);
  return c;
}
__device__ __forceinline__ int lds_at(const MgLdsLevel &L, int i, int j, int k) {
  i = pwrap(i, L.nx);
  j = pwrap(j, L.ny);
  k = pwrap(k, L.nz);
  return ((i + j + k) & 1) * L.half + (((k * L.ny + j) * L.nx + i) >> 1);
}
// The six neighbours of cell (i, j, k) are in the other colour's half: along y
// and z at the same place of their rows, along x one at the cell's own place of
// the row and the other beside it.
struct LdsNeighbours {
  int xm, xp, ym, yp, zm, zp;
};
__device__ __forceinline__ LdsNeighbours lds_neighbours(const MgLdsLevel &L, int i, int j, int k) {
  const int o = ((i + j + k) & 1) ? 0 : L.half;
  const int ih = i >> 1, row = (k * L.ny + j) * L.hx + o;
  const int il = (i & 1) ? ih : (ih == 0 ? L.hx - 1 : ih - 1);
  const int ir = (i & 1) ? (ih == L.hx - 1 ? 0 : ih + 1) : ih;
  const int sy = L.hx, sz = L.hx * L.ny;
  LdsNeighbours n;
  n.xm = row + il;
  n.xp = row + ir;
  n.ym = row + ih + (j == 0 ? (L.ny - 1) * sy : -sy);
  n.yp = row + ih + (j == L.ny - 1 ? -(L.ny - 1) * sy : sy);
  n.zm = row + ih + (k == 0 ? (L.nz - 1) * sz : -sz);
  n.zp = row + ih + (k == L.nz - 1 ? -(L.nz - 1) * sz : sz);
  return n;
}
__device__ __forceinline__ double lds_nbsum(const MgLdsLevel &L, const double *f, const LdsNeighbours &n) {
#pragma clang fp contract(off)
  const double sx = f[n.xm] + f[n.xp];
  const double sy = f[n.ym] + f[n.yp];
  const double sz = f[n.zm] + f[n.zp];
  return (sx + L.wy * sy) + L.wz * sz;
}
__device__ __forceinline__ double lds_nbsum(const MgLdsLevel &L, const double *f, int i, int j, int k) {
  return lds_nbsum(L, f, lds_neighbours(L, i, j, k));
}
__device__ __forceinline__ double lds_apply(const MgLdsLevel &L, const double *f, int i, int j, int k) {
#pragma clang fp contract(off)
  return (L.c0 * f[lds_at(L, i, j, k)] - lds_nbsum(L, f, i, j, k)) / L.hx2;
}

__device__ __forceinline__ void lds_sweep(const MgLdsLevel &L, double *lds) {
  double *phi = lds + L.phi;
  const double *src = lds + L.src;
  for (int color = 0; color < 2; ++color) {
    for (int r = threadIdx.x; r < L.half; r += kMgLdsThreads) {
#pragma clang fp contract(off)
      const LdsCell c = lds_cell(L, r, color);
      const int q = color * L.half + r;
      const double gs = over_c0(L.c0, L.r0, lds_nbsum(L, phi, c.i, c.j, c.k) + L.hx2 * src[q]);
      phi[q] = (1.0 - kOmegaGS) * phi[q] + kOmegaGS * gs;
    }
    __syncthreads();
  }
}

// Restriction of level L to C (as mg_restrict_kernel, then mg_coarse_source_kernel).
__device__ __forceinline__ void lds_restrict(const MgLdsLevel &L, const MgLdsLevel &C, double *lds) {
#pragma clang fp contract(off)
  const double *f = lds + L.phi, *src = lds + L.src;
  auto defect = [&](int i, int j, int k) { return src[lds_at(L, i, j, k)] - lds_apply(L, f, i, j, k); };
  for (int q = threadIdx.x; q < 2 * C.half; q += kMgLdsThreads) {
    const LdsCell c = lds_cell(C, q >= C.half ? q - C.half : q, q >= C.half);
    const int I = 2 * c.i, J = 2 * c.j, K = 2 * c.k;
    double m[2][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = J + (e & 1), k = K + (e >> 1);
      m[0][e] = f[lds_at(L, I, j, k)] + f[lds_at(L, I + 1, j, k)];
      m[1][e] = defect(I, j, k) + defect(I + 1, j, k);
    }
    const double r = 0.125 * ((m[0][0] + m[0][1]) + (m[0][2] + m[0][3]));
    lds[C.phi + q] = r;
    lds[C.rphi + q] = r;
    lds[C.src + q] = 0.125 * ((m[1][0] + m[1][1]) + (m[1][2] + m[1][3]));
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 2 * C.half; q += kMgLdsThreads) {
    const LdsCell c = lds_cell(C, q >= C.half ? q - C.half : q, q >= C.half);
    lds[C.src + q] = lds[C.src + q] + lds_apply(C, lds + C.phi, c.i, c.j, c.k);
  }
  __syncthreads();
}

// Tricubic prolongation of the correction of C onto L (as mg_prolong_kernel).
__device__ __forceinline__ void lds_prolong(const MgLdsLevel &L, const MgLdsLevel &C, double *lds) {
  const double w[2][4] = {{-5.0 / 128.0, 35.0 / 128.0, 105.0 / 128.0, -7.0 / 128.0},
                          {-7.0 / 128.0, 105.0 / 128.0, 35.0 / 128.0, -5.0 / 128.0}};
  for (int q = threadIdx.x; q < 2 * C.half; q += kMgLdsThreads) lds[C.rphi + q] = lds[C.phi + q] - lds[C.rphi + q];
  __syncthreads();
  const double *e = lds + C.rphi;
  double *phi = lds + L.phi;
  for (int q = threadIdx.x; q < 4 * C.half; q += kMgLdsThreads) {
    // a coarse cell and the z side of its children
    const int cz = q >= 2 * C.half, p = q - (cz ? 2 * C.half : 0);
    const LdsCell c = lds_cell(C, p >= C.half ? p - C.half : p, p >= C.half);
    int xs[5];
#pragma unroll
    for (int ox = 0; ox < 5; ++ox) xs[ox] = pwrap(c.i + ox - 2, C.nx);
    double Z[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll 1
    for (int oz = 0; oz < 4; ++oz) {
      double Y[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
      for (int oy = 0; oy < 5; ++oy) {
        const int j = pwrap(c.j + oy - 2, C.ny), k = pwrap(c.k + oz + cz - 2, C.nz);
        const int row = (k * C.ny + j) * C.hx, par = j + k;
        double v[5];
#pragma unroll
        for (int ox = 0; ox < 5; ++ox) {
          const int i = xs[ox];
          v[ox] = e[((i + par) & 1) * C.half + row + (i >> 1)];
        }
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) {
          double sx = 0.0;
#pragma unroll
          for (int a = 0; a < 4; ++a) sx += w[cx][a] * v[cx + a];
#pragma unroll
          for (int cy = 0; cy < 2; ++cy) {
            const int b = oy - cy;
            if (b >= 0 && b <= 3) Y[cy][cx] += w[cy][b] * sx;
          }
        }
      }
      const double wz = cz ? (oz == 0 ? w[1][0] : (oz == 1 ? w[1][1] : (oz == 2 ? w[1][2] : w[1][3])))
                           : (oz == 0 ? w[0][0] : (oz == 1 ? w[0][1] : (oz == 2 ? w[0][2] : w[0][3])));
#pragma unroll
      for (int cy = 0; cy < 2; ++cy)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) Z[cy][cx] += wz * Y[cy][cx];
    }
#pragma unroll
    for (int cy = 0; cy < 2; ++cy)
#pragma unroll
      for (int cx = 0; cx < 2; ++cx) phi[lds_at(L, 2 * c.i + cx, 2 * c.j + cy, 2 * c.k + cz)] += Z[cy][cx];
  }
  __syncthreads();
}

// The coarsest level's sweeps: at most 2048 cells, so every thread owns at most
// one cell of each colour, whose neighbour slots it finds once.  Up to 64 cells
// of a colour one wave sweeps alone, without barriers (kMgOneWave); where some
// waves have no cell (kMgSomeWaves) those only wait, since their idle passes
// through LDS hold up the others': a cycle of 256 x 256 x 32 (512 coarsest
// cells) takes 930 us, 1234 with every wave at work.  Where every wave has a cell
// (kMgAllWaves) the check would only cost: 16 x 256 x 256 (2048 cells) 3.85 ms
// per cycle, 4.61 with it.
enum { kMgOneWave, kMgSomeWaves, kMgAllWaves };
template <int WAVES>
__device__ __forceinline__ void lds_coarse_sweeps(const MgLdsLevel &C, int sweeps, double *lds) {
#pragma clang fp contract(off)
  double *phi = lds + C.phi;
  const int half = C.half;
  const bool own = (int)threadIdx.x < half;
  const bool busy = WAVES != kMgSomeWaves || 64 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < half;
  const int t = own ? (int)threadIdx.x : 0;
  LdsNeighbours nb[2];
  double hs[2], old[2];
#pragma unroll
  for (int color = 0; color < 2; ++color) {
    const LdsCell c = lds_cell(C, t, color);
    nb[color] = lds_neighbours(C, c.i, c.j, c.k);
    hs[color] = C.hx2 * lds[C.src + color * half + t];
    old[color] = phi[color * half + t];
  }
  for (int s = 0; s < sweeps; ++s) {
#pragma unroll
    for (int color = 0; color < 2; ++color) {
      if (busy) {
        const double gs = over_c0(C.c0, C.r0, lds_nbsum(C, phi, nb[color]) + hs[color]);
        old[color] = (1.0 - kOmegaGS) * old[color] + kOmegaGS * gs;
        if (own) phi[color * half + t] = old[color];
      }
      if (WAVES == kMgOneWave) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      else __syncthreads();
    }
  }
}
__device__ __forceinline__ void lds_coarse_solve(const MgLdsLevel &C, int sweeps, double *lds) {
  if (C.half <= 64) {
    if (threadIdx.x < 64) lds_coarse_sweeps<kMgOneWave>(C, sweeps, lds);
  } else if (C.half <= kMgLdsThreads - 64) {
    lds_coarse_sweeps<kMgSomeWaves>(C, sweeps, lds);
  } else {
    lds_coarse_sweeps<kMgAllWaves>(C, sweeps, lds);
  }
  __syncthreads();
}

// The coarsest level's sweeps are one linear map of its potential and source,
// but each sweep is a chain of two dependent passes (0.23 us; 2 x 2 x 2 cells
// take 72 of them, 8 x 2 x 2 cells 288).  Up to kMgMatCells cells the map's
// matrix is found once per solve, each column by the sweeps of a unit vector on
// its own compute unit, and a cycle multiplies by it: 55 us per solve and 27 us
// per cycle where the sweeps take 90 us per cycle (64 x 16 x 16; with 2 x 2 x 2
// cells 62 and 48 us).  128 cells and more would need 4 times the matrix and
// gain less, each sweep spreading over more threads.
//   mat: [2 n] columns of n (potential, then source)
constexpr int kMgMatCells = 64;
constexpr int kMgMatThreads = 512;  // that multiply; 2 n columns over 512 / n groups of threads: at most 16 each
__global__ __launch_bounds__(64) void mg_coarse_matrix_kernel(MgLdsLevel C, int sweeps, double *mat) {
  __shared__ double lds[2 * kMgMatCells];
  const int n = 2 * C.half;
  for (int q = threadIdx.x; q < 2 * n; q += 64) lds[q] = q == (int)blockIdx.x ? 1.0 : 0.0;
  __syncthreads();
  C.phi = 0;
  C.src = n;
  lds_coarse_solve(C, sweeps, lds);
  for (int q = threadIdx.x; q < n; q += 64) mat[(long long)blockIdx.x * n + q] = lds[q];
}

// phi = mat (phi, src): the 2 n columns are shared among kMgMatThreads threads
// (n of them per group of columns) and the groups' sums added in order; red:
// kMgMatThreads doubles of LDS.
__device__ __forceinline__ void lds_coarse_apply(const MgLdsLevel &C, const double *m, double *lds, double *red) {
  const int n = 2 * C.half, groups = kMgMatThreads / n;
  const int q = (int)threadIdx.x % n, g = (int)threadIdx.x / n;
  if (g < groups) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kMgMatCells / 4; ++k) {
      const int c = g + k * groups;
      if (c < 2 * n) s = fma(m[k], lds[(c < n ? C.phi : C.src - n) + c], s);
    }
    red[threadIdx.x] = s;
  }
  __syncthreads();
  if ((int)threadIdx.x < n) {
    double s = red[threadIdx.x];
    for (int k = 1; k < groups; ++k) s += red[k * n + threadIdx.x];
    lds[C.phi + threadIdx.x] = s;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kMgLdsThreads) void mg_lds_cycle_kernel(MgLdsCycle P, int sweeps, const double *mat) {
  __shared__ double lds[kMgLdsDoubles];
  const MgLdsLevel &B = P.lv[P.n - 1];
  const int nb = 2 * B.half;
  // this thread's share of the coarsest level's matrix, on its way from the start
  double m[kMgMatCells / 4];
  if (mat) {
    const int groups = kMgMatThreads / nb, q = (int)threadIdx.x % nb, g = (int)threadIdx.x / nb;
#pragma unroll
    for (int k = 0; k < kMgMatCells / 4; ++k) {
      const int c = g + k * groups;
      m[k] = g < groups && c < 2 * nb ? mat[c * nb + q] : 0.0;
    }
  }
  const int n0 = 2 * P.lv[0].half;
  for (int q = threadIdx.x; q < n0; q += kMgLdsThreads) {
    lds[P.lv[0].phi + q] = P.phi[q];
    lds[P.lv[0].src + q] = P.src[q];
  }
  __syncthreads();
  for (int l = 0; l + 1 < P.n; ++l) {
    lds_sweep(P.lv[l], lds);
    lds_sweep(P.lv[l], lds);
    lds_restrict(P.lv[l], P.lv[l + 1], lds);
  }
  if (mat) lds_coarse_apply(B, m, lds, lds + kMgLdsDoubles - kMgMatThreads);
  else lds_coarse_solve(B, sweeps, lds);
  for (int l = P.n - 2; l >= 0; --l) {
    lds_prolong(P.lv[l], P.lv[l + 1], lds);
    lds_sweep(P.lv[l], lds);
    lds_sweep(P.lv[l], lds);
  }
  for (int q = threadIdx.x; q < n0; q += kMgLdsThreads) P.phi[q] = lds[P.lv[0].phi + q];
}

// fine phi += tricubic interpolation of the coarse correction (coarse result -
// R phi, formed where it is read): per axis the
// cubic through the four nearest coarse centres, weights (-5, 35, 105, -7)/128
// for the child at -1/4 of its parent (centres parent-2 .. parent+1) and
// (-7, 105, 35, -5)/128 for the child at +1/4 (parent-1 .. parent+2), summed
// along x, then y, then z.  One thread per coarse cell makes its eight
// children from the 5 x 5 x 5 coarse neighbourhood they share (125 loads
// instead of 512), keeping that order of summation for each child.
__global__ __launch_bounds__(kMgThreads) void mg_prolong_kernel(MgLevel F, MgLevel C, double *out) {
  const double w[2][4] = {{-5.0 / 128.0, 35.0 / 128.0, 105.0 / 128.0, -7.0 / 128.0},
                          {-7.0 / 128.0, 105.0 / 128.0, 35.0 / 128.0, -5.0 / 128.0}};
  const long long n = ncell(C);
  for (long long q = blockIdx.x * (long long)kMgThreads + threadIdx.x; q < n; q += (long long)gridDim.x * kMgThreads) {
    int i, j, k;
    cell_of(C, q, i, j, k);
    double Z[2][2][2] = {{{0.0, 0.0}, {0.0, 0.0}}, {{0.0, 0.0}, {0.0, 0.0}}};  // [cz][cy][cx]
    // coarse offsets -2..2 along each axis; child c (0 left, 1 right) uses offsets c-2 .. c+1
#pragma unroll
    for (int oz = 0; oz < 5; ++oz) {
      double Y[2][2] = {{0.0, 0.0}, {0.0, 0.0}};  // [cy][cx] at this z offset
#pragma unroll
      for (int oy = 0; oy < 5; ++oy) {
        double e[5];
#pragma unroll
        for (int ox = 0; ox < 5; ++ox) {
          const long long c = at(C, i + ox - 2, j + oy - 2, k + oz - 2);
          e[ox] = C.phi[c] - C.rphi[c];
        }
        double X[2];
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) {
          double sx = 0.0;
#pragma unroll
          for (int a = 0; a < 4; ++a) sx += w[cx][a] * e[cx + a];
          X[cx] = sx;
        }
#pragma unroll
        for (int cy = 0; cy < 2; ++cy) {
          const int b = oy - cy;  // this row's place in child cy's stencil
          if (b < 0 || b > 3) continue;
#pragma unroll
          for (int cx = 0; cx < 2; ++cx) Y[cy][cx] += w[cy][b] * X[cx];
        }
      }
#pragma unroll
      for (int cz = 0; cz < 2; ++cz) {
        const int c = oz - cz;
        if (c < 0 || c > 3) continue;
#pragma unroll
        for (int cy = 0; cy < 2; ++cy)
#pragma unroll
          for (int cx = 0; cx < 2; ++cx) Z[cz][cy][cx] += w[cz][c] * Y[cy][cx];
      }
    }
#pragma unroll
    for (int cz = 0; cz < 2; ++cz)
#pragma unroll
      for (int cy = 0; cy < 2; ++cy)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) {
          const long long q = at(F, 2 * i + cx, 2 * j + cy, 2 * k + cz);
          out[q] = F.phi[q] + Z[cz][cy][cx];
        }
  }
}

// The same prolongation by tiles: a workgroup stages the correction of a tile of
// coarse cells with a two-cell halo in LDS, then interpolates along x, y and z
// in turn, each value once (one thread per coarse cell repeats the x sums of its
// 25 rows that its neighbours form too, four times the arithmetic in all); every
// sum has mg_prolong_kernel's terms in its order (the same bits).  Reading and
// writing the fine potential bounds it; 16 coarse cells along x make 128-byte
// rows of each colour.  All levels of a 256^3 cycle 136 us, one thread per coarse
// cell 174.  Levels whose edges are multiples of the tile's.
constexpr int kPtx = 16, kPty = 4, kPtz = 4;

__global__ __launch_bounds__(kMgThreads) void mg_prolong_tiled_kernel(MgLevel F, MgLevel C, double *out) {
  constexpr int HX = kPtx + 4, HY = kPty + 4, HZ = kPtz + 4, FX = 2 * kPtx, FY = 2 * kPty, FZ = 2 * kPtz;
  constexpr int kA = HX * HY * HZ, kY = FX * FY * HZ;
  __shared__ double sx[HZ * HY * FX];
  __shared__ double sa[kA > kY ? kA : kY];  // the correction, then the sums along y
  const double w[2][4] = {{-5.0 / 128.0, 35.0 / 128.0, 105.0 / 128.0, -7.0 / 128.0},
                          {-7.0 / 128.0, 105.0 / 128.0, 35.0 / 128.0, -5.0 / 128.0}};
  // four values at a stride, from the child's side on
  auto cubic = [&](const double *v, int stride, int side) {
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a) s += (side ? w[1][a] : w[0][a]) * v[a * stride];
    return s;
  };
  const int tx = C.nx / kPtx, ty = C.ny / kPty, tz = C.nz / kPtz;
  const long long half = ncell(F) >> 1;
  const int hx = F.nx >> 1;
  for (int tile = blockIdx.x; tile < tx * ty * tz; tile += gridDim.x) {
    const int i0 = (tile % tx) * kPtx, j0 = ((tile / tx) % ty) * kPty, k0 = (tile / (tx * ty)) * kPtz;
    __syncthreads();  // the previous tile's reads are done
    for (int v = threadIdx.x; v < kA; v += kMgThreads) {
      const int a = v % HX, b = (v / HX) % HY, c = v / (HX * HY);
      const long long q = at(C, i0 + a - 2, j0 + b - 2, k0 + c - 2);
      sa[v] = C.phi[q] - C.rphi[q];
    }
    __syncthreads();
    for (int v = threadIdx.x; v < HZ * HY * FX; v += kMgThreads) {
      const int i = v % FX, r = v / FX;
      sx[v] = cubic(sa + r * HX + (i >> 1) + (i & 1), 1, i & 1);
    }
    __syncthreads();
    for (int v = threadIdx.x; v < kY; v += kMgThreads) {
      const int i = v % FX, j = (v / FX) % FY, k = v / (FX * FY);
      sa[v] = cubic(sx + (k * HY + (j >> 1) + (j & 1)) * FX + i, FX, j & 1);
    }
    __syncthreads();
    for (int v = threadIdx.x; v < FX * FY * FZ; v += kMgThreads) {
      // in the order of storage: a row's cells of one colour, then of the other
      const int h = v % kPtx, color = (v / kPtx) & 1, j = (v / FX) % FY, k = v / (FX * FY);
      const int i = 2 * h + ((j + k + color) & 1);  // the tile's first cell is red
      const long long q = color * half + ((long long)(2 * k0 + k) * F.ny + 2 * j0 + j) * hx + i0 + h;
      out[q] = F.phi[q] + cubic(sa + (((k >> 1) + (k & 1)) * FY + j) * FX + i, FX * FY, k & 1);
    }
  }
}

// the per-block stored potential with one periodic ghost layer; blockIdx.y = block
__global__ __launch_bounds__(kMgThreads) void mg_scatter_kernel(MeshDev m, MgLevel F, double *phib) {
  const BlockInfo B = m.blocks[blockIdx.y];
  const int np = B.n + 2;
  const int tot = np * np * np;
  for (int e = blockIdx.x * kMgThreads + threadIdx.x; e < tot; e += gridDim.x * kMgThreads) {
    const int i = e % np - 1, j = (e / np) % np - 1, k = e / (np * np) - 1;
    phib[B.poff + e] = F.phi[at(F, B.ox + i, B.oy + j, B.oz + k)];
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int grid_for(long long n) {
  const long long g = (n + kMgThreads - 1) / kMgThreads;
  return (int)(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

hipError_t mg_launch_gather(const MeshDev &m, const int *par, const double *Qa, const double *Qb, const MgLevel &F,
                            hipStream_t s) {
  hipLaunchKernelGGL(mg_gather_kernel, dim3(grid_for((long long)m.nx * m.ny * m.nz)), dim3(kMgThreads), 0, s, m, par,
                     Qa, Qb, F);
  return hipGetLastError();
}

hipError_t mg_launch_sum(const double *x, long long n, int square, double scale, int op, double *part, double *out,
                         hipStream_t s) {
  hipLaunchKernelGGL(mg_partial_sum_kernel, dim3(kMgSumParts), dim3(kMgThreads), 0, s, x, n, square, part);
  hipLaunchKernelGGL(mg_final_sum_kernel, dim3(1), dim3(kMgThreads), 0, s, part, kMgSumParts, scale, op, out);
  return hipGetLastError();
}

hipError_t mg_launch_source(double *src, const double *mean, double four_pi_G, long long n, hipStream_t s) {
  hipLaunchKernelGGL(mg_source_kernel, dim3(grid_for(n)), dim3(kMgThreads), 0, s, src, mean, four_pi_G, n);
  return hipGetLastError();
}

hipError_t mg_launch_affine(double *x, const double *shift, double fill, long long n, hipStream_t s) {
  hipLaunchKernelGGL(mg_affine_kernel, dim3(grid_for(n)), dim3(kMgThreads), 0, s, x, shift, fill, n);
  return hipGetLastError();
}

hipError_t mg_launch_sweep(const MgLevel &L, hipStream_t s) {
  const long long half = ((long long)L.nx * L.ny * L.nz) >> 1;
  for (int color = 0; color < 2; ++color)
    hipLaunchKernelGGL(mg_rbgs_kernel, dim3(grid_for(half)), dim3(kMgThreads), 0, s, L, color);
  return hipGetLastError();
}

// z chunks of a level's fused sweeps: the count that gives the fewest planes per
// compute unit (rounds of workgroups times planes of a chunk with its ends)
template <int S, int TAIL>
static hipError_t launch_smooth(const MgLevel &L, double *out, double *part, const MgLevel &C, int cus, int *parts,
                                hipStream_t s) {
  using G = MgSmooth<S, TAIL>;
  const long long tx = (L.nx / 2 + G::OX - 1) / G::OX, ty = (L.ny + G::OY - 1) / G::OY;
  int nc = 1;
  long long best = 0;
  for (int c = 1; c <= L.nz / 2 && tx * ty * c <= kMgSumParts; ++c) {
    const long long cost = (tx * ty * c + cus - 1) / cus * (2 * ((L.nz / 2 + c - 1) / c) + 2 * G::H);
    if (c == 1 || cost < best) {
      best = cost;
      nc = c;
    }
  }
  const int g = (int)(tx * ty * nc);
  if (parts) *parts = g;
  hipLaunchKernelGGL((mg_smooth_kernel<S, TAIL>), dim3((g + 7) / 8 * 8), dim3(kMgSmoothThreads), 0, s, L, out, (int)tx,
                     (int)ty, nc, part, C);
  return hipGetLastError();
}

// Two sweeps, then the restriction: with it from 2^22 cells on (ten cycles of 256^3
// 8.95 -> 8.1 ms, 256 x 256 x 128 4.58 -> 4.40); on smaller levels the wider edge
// costs more than the pass (128^3 2.68 -> 2.73, 128 x 128 x 64 2.19 -> 2.30).
constexpr long long kMgRestrictCells = 1 << 22;

bool mg_smooth_fits(const MgLevel &L) {
  using G = MgSmooth<4, kMgRestrict>;
  const long long tiles = ((L.nx / 2 + G::OX - 1) / G::OX) * (long long)((L.ny + G::OY - 1) / G::OY);
  return (long long)L.nx * L.ny * L.nz >= kMgSmoothCells && tiles <= kMgSumParts;
}

hipError_t mg_launch_smooth(const MgLevel &L, double *out, int cus, hipStream_t s) {
  return launch_smooth<4, kMgPlain>(L, out, nullptr, L, cus, nullptr, s);
}

hipError_t mg_launch_smooth_restrict(const MgLevel &L, double *out, const MgLevel &C, int cus, hipStream_t s) {
  if ((long long)L.nx * L.ny * L.nz < kMgRestrictCells) {
    const hipError_t e = mg_launch_smooth(L, out, cus, s);
    if (e != hipSuccess) return e;
    MgLevel A = L;
    A.phi = out;
    return mg_launch_restrict(A, C, s);
  }
  const hipError_t e = launch_smooth<4, kMgRestrict>(L, out, nullptr, C, cus, nullptr, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mg_coarse_source_kernel, dim3(grid_for((long long)C.nx * C.ny * C.nz)), dim3(kMgThreads), 0, s, C);
  return hipGetLastError();
}

hipError_t mg_launch_smooth_norm(const MgLevel &L, double *out, double *part, double *norm, int cus, hipStream_t s) {
  const long long n = (long long)L.nx * L.ny * L.nz;
  int parts = 0;
  const hipError_t e = launch_smooth<2, kMgNorm>(L, out, part, L, cus, &parts, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mg_final_sum_kernel, dim3(1), dim3(kMgThreads), 0, s, part, parts, 1.0 / (double)n, 1, norm);
  return hipGetLastError();
}

hipError_t mg_launch_defect_norm(const MgLevel &L, double *part, double *out, hipStream_t s) {
  const long long n = (long long)L.nx * L.ny * L.nz;
  hipLaunchKernelGGL(mg_defect_sq_partial_kernel, dim3(kMgSumParts), dim3(kMgThreads), 0, s, L, part);
  hipLaunchKernelGGL(mg_final_sum_kernel, dim3(1), dim3(kMgThreads), 0, s, part, kMgSumParts, 1.0 / (double)n, 1,
                     out);
  return hipGetLastError();
}

hipError_t mg_launch_restrict(const MgLevel &F, const MgLevel &C, hipStream_t s) {
  const long long n = (long long)C.nx * C.ny * C.nz;
  hipLaunchKernelGGL(mg_restrict_kernel, dim3(grid_for(n)), dim3(kMgThreads), 0, s, F, C);
  hipLaunchKernelGGL(mg_coarse_source_kernel, dim3(grid_for(n)), dim3(kMgThreads), 0, s, C);
  return hipGetLastError();
}

static MgLdsLevel lds_level(const MgLevel &g) {
  MgLdsLevel L{};
  L.nx = g.nx; L.ny = g.ny; L.nz = g.nz;
  L.hx = L.nx / 2;
  L.half = g.nx * g.ny * g.nz / 2;
  L.mx = (unsigned)(((1ULL << 32) + L.hx - 1) / L.hx);
  L.my = (unsigned)(((1ULL << 32) + L.ny - 1) / L.ny);
  L.hx2 = g.hx2; L.wy = g.wy; L.wz = g.wz; L.c0 = g.c0; L.r0 = 1.0 / L.c0;
  return L;
}

// doubles of LDS the V-cycle from level lv[0] down takes (the coarsest level's
// product adds one per multiplying thread)
static long long lds_doubles(const MgLevel *lv, int n) {
  long long d = kMgMatThreads;
  for (int k = 0; k < n; ++k) d += (k ? 3 : 2) * ((long long)lv[k].nx * lv[k].ny * lv[k].nz);
  return d;
}

// the first of levels 0 .. nlev-1 from which the rest of the V-cycle fits the LDS kernel
int mg_lds_top(const MgLevel *lv, int nlev) {
  for (int l = 0; l < nlev; ++l)
    if ((long long)lv[l].nx * lv[l].ny * lv[l].nz <= kMgLdsTop && lds_doubles(lv + l, nlev - l) <= kMgLdsDoubles &&
        nlev - l <= kMgLdsLevels)
      return l;
  return nlev - 1;
}

// doubles of the coarsest level's matrix (0: its sweeps run in every cycle)
int mg_coarse_matrix_doubles(const MgLevel &C) {
  const long long n = (long long)C.nx * C.ny * C.nz;
  return n <= kMgMatCells ? (int)(2 * n * n) : 0;
}

hipError_t mg_launch_coarse_matrix(const MgLevel &C, int sweeps, double *mat, hipStream_t s) {
  const int n = C.nx * C.ny * C.nz;
  if (n > kMgMatCells) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mg_coarse_matrix_kernel, dim3(2 * n), dim3(64), 0, s, lds_level(C), sweeps, mat);
  return hipGetLastError();
}

hipError_t mg_launch_lds_cycle(const MgLevel *lv, int n, int sweeps, const double *mat, hipStream_t s) {
  const MgLevel &C = lv[n - 1];
  if (n < 1 || n > kMgLdsLevels || (long long)C.nx * C.ny * C.nz > kMgCoarseMax || lds_doubles(lv, n) > kMgLdsDoubles)
    return hipErrorInvalidValue;
  MgLdsCycle P{};
  P.n = n;
  P.phi = lv[0].phi;
  P.src = lv[0].src;
  int off = 0;
  for (int l = 0; l < n; ++l) {
    MgLdsLevel &L = P.lv[l];
    L = lds_level(lv[l]);
    const int cells = 2 * L.half;
    L.phi = off;
    L.src = off + cells;
    L.rphi = l ? off + 2 * cells : 0;
    off += (l ? 3 : 2) * cells;
  }
  hipLaunchKernelGGL(mg_lds_cycle_kernel, dim3(1), dim3(kMgLdsThreads), 0, s, P, sweeps, mat);
  return hipGetLastError();
}

hipError_t mg_launch_prolong(const MgLevel &F, const MgLevel &C, double *out, hipStream_t s) {
  if (C.nx % kPtx == 0 && C.ny % kPty == 0 && C.nz % kPtz == 0) {
    const int tiles = (C.nx / kPtx) * (C.ny / kPty) * (C.nz / kPtz);
    hipLaunchKernelGGL(mg_prolong_tiled_kernel, dim3(tiles < 4096 ? tiles : 4096), dim3(kMgThreads), 0, s, F, C,
                       out);
  } else {
    hipLaunchKernelGGL(mg_prolong_kernel, dim3(grid_for((long long)C.nx * C.ny * C.nz)), dim3(kMgThreads), 0, s, F,
                       C, out);
  }
  return hipGetLastError();
}

hipError_t mg_launch_scatter(const MeshDev &m, int nblocks, int nmax, const MgLevel &F, double *phib, hipStream_t s) {
  const int np = nmax + 2;
  const int gx = (np * np * np + kMgThreads - 1) / kMgThreads;
  hipLaunchKernelGGL(mg_scatter_kernel, dim3(gx, nblocks), dim3(kMgThreads), 0, s, m, F, phib);
  return hipGetLastError();
}

int mg_coarse_max() { return kMgCoarseMax; }

}  // namespace tdh
