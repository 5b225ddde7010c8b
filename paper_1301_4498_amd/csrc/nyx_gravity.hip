// nyx_gravity.hip -- the mesh side of the gravity input of the gas step
// (Sec. 2.4 and Sec. 3.4 Self-gravity): cloud-in-cell deposit of particle
// mass, the periodic Poisson equation lap(phi) = coef (rho - mean(rho))
// discretised with the 7-point stencil and solved by geometric multigrid
// V-cycles with red-black Gauss-Seidel relaxation, and g = -grad(phi) by
// centred differences, written in the step's padded gravity layout.
//
// Fields of the periodic domain are stored x fastest without ghost cells.
// Every kernel is a plain stencil over HBM-resident arrays, one lane per
// cell (or per cell of one colour); reductions are deterministic (fixed
// block partials, then one block), so a solve gives the same bits on every
// run.  The deposit adds with hardware FP64 atomics and is therefore exact
// only up to the order of the additions.  Built without contraction.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "nyx_internal.h"

namespace nyx {
namespace grav {

constexpr int kRedBlocks = 4096;  // block partials of a reduction
constexpr int kResidBlocks = 2048;

__device__ __forceinline__ unsigned wrap_dec(unsigned i, unsigned n) { return i == 0 ? n - 1 : i - 1; }
__device__ __forceinline__ unsigned wrap_inc(unsigned i, unsigned n) { return i + 1 == n ? 0 : i + 1; }

struct Grid {
  unsigned nx, ny, nz;
};

// natural order (the caller's mesh fields): x fastest
__device__ __forceinline__ unsigned nat(const Grid& g, unsigned i, unsigned j, unsigned k) {
  return (k * g.ny + j) * g.nx + i;
}

// the solver's own arrays keep the two colours of the red-black ordering
// apart: colour (i + j + k) & 1 holds its cells x fastest with half-length
// rows, so a half sweep reads the other colour's neighbours, its own rhs
// and writes its own cells, each contiguous across the lanes of a row
__device__ __forceinline__ unsigned at(const Grid& g, unsigned i, unsigned j, unsigned k) {
  const unsigned half = g.nx >> 1;
  return ((i + j + k) & 1) * (half * g.ny * g.nz) + (k * g.ny + j) * half + (i >> 1);
}

__device__ __forceinline__ void coords(const Grid& g, unsigned c, unsigned* i, unsigned* j,
                                       unsigned* k) {
  *i = c % g.nx;
  *j = (c / g.nx) % g.ny;
  *k = c / (g.nx * g.ny);
}

// the six-neighbour sum of the 7-point stencil, (x pair + y pair) + z pair
__device__ __forceinline__ double nb_sum(const double* p, const Grid& g, unsigned i, unsigned j,
                                         unsigned k) {
  const double sx = p[at(g, wrap_dec(i, g.nx), j, k)] + p[at(g, wrap_inc(i, g.nx), j, k)];
  const double sy = p[at(g, i, wrap_dec(j, g.ny), k)] + p[at(g, i, wrap_inc(j, g.ny), k)];
  const double sz = p[at(g, i, j, wrap_dec(k, g.nz))] + p[at(g, i, j, wrap_inc(k, g.nz))];
  return (sx + sy) + sz;
}

// ---- cloud-in-cell deposit: one lane per particle, 8 adds ----
// Atomic adds to memory are carried out beyond the L2, one request per touched
// 64-byte piece, and bound a deposit that sends each particle's eight adds
// there: neighbouring particles differ in their y and z cells, so a request
// holds two adds in the mean (70M requests, 3.07 ms for 256^3 particles near
// their lattice points, 23 requests per ns).  A workgroup therefore collects
// its NT particles in LDS where they lie close together, as particles kept in
// any spatial order do: the box of cells they touch, at most CELLS, is
// accumulated with LDS atomics and added to memory row by row, full requests
// and each cell once.  Particles that lie further apart go to memory directly, a
// wavefront whose own 64 do so at once, before the workgroup's box is formed
// (waiting for it, 2^18 scattered particles took 100 us).
// Sizes: 1024 particles and 80 KB keep two workgroups (32 waves) on a CU, so
// that the direct path loses little; below kCicWide particles, where these
// would leave CUs idle, 256 particles and 48 KB.
// Measured (us, particles added one by one, and this): 256^3 particles near
// their lattice points 3440 and 478, 64^3 53 and 13.5, 2^18 clustered 1070 and
// 20; scattered over the domain, where every wavefront takes the direct path,
// 2^18 on 128^3 93 and 94.5, 2^22 on 256^3 1432 and 1431, 2^24 on 512^3 5950 and
// 6200; every second one of 256^3 scattered 5230 and 4890.
constexpr int kCicBlock = 1024, kCicCells = 10000;
constexpr int kCicSmallBlock = 256, kCicSmallCells = 6144;
constexpr long long kCicWide = 1 << 18;

__device__ __forceinline__ unsigned wrap_mod(long long u, unsigned n) {
  const long long r = u % (long long)n;
  return (unsigned)(r < 0 ? r + n : r);
}

template <int NT, int CELLS>
__global__ __launch_bounds__(NT) void k_cic(const double* __restrict__ pos,
                                                   const double* __restrict__ mass, long long np,
                                                   Grid g, double dx, double inv_vol,
                                                   double* __restrict__ rho) {
  __shared__ double acc[CELLS];
  __shared__ int first, lo_sh[3], hi_sh[3];
  __shared__ long long ref[3];
  // consecutive workgroups on one XCD: neighbouring particles' cells are in its L2
  const long long p = (long long)xcd_linear_block(true) * NT + threadIdx.x;
  const unsigned n[3] = {g.nx, g.ny, g.nz};
  bool on = p < np;
  long long u[3] = {0, 0, 0};  // the lower cell of each axis, not wrapped
  double f[3] = {0.0, 0.0, 0.0}, m = 0.0;
  if (on) {
    m = mass[p] * inv_vol;
    for (int d = 0; d < 3; ++d) {
      const double s = pos[d * np + p] / dx - 0.5;
      if (!(fabs(s) < 1e15)) on = false;  // non-finite or absurd position: the particle is skipped
      const double fl = floor(s);
      f[d] = s - fl;
      u[d] = on ? (long long)fl : 0;
    }
  }
  auto weight = [&](int q) {
    double w = 1.0;
    w = w * (q & 1 ? f[0] : 1.0 - f[0]);
    w = w * (q & 2 ? f[1] : 1.0 - f[1]);
    w = w * (q & 4 ? f[2] : 1.0 - f[2]);
    return m * w;
  };
  // extents of the box between the lower cells lo and hi, the upper cells
  // included; an axis it spans whole is indexed by the wrapped cell itself
  auto extents = [&](const int* lo, const int* hi, long long* ext, bool* whole) {
    for (int d = 0; d < 3; ++d) {
      ext[d] = (long long)hi[d] - lo[d] + 2;
      whole[d] = ext[d] >= (long long)n[d];
      if (whole[d]) ext[d] = n[d];
    }
    return ext[0] * ext[1] <= CELLS && ext[0] * ext[1] * ext[2] <= CELLS;
  };
  auto add_direct = [&]() {
    unsigned a[3], b[3];  // lower and upper cell in the domain
    for (int d = 0; d < 3; ++d) {
      a[d] = wrap_mod(u[d], n[d]);
      b[d] = a[d] + 1 == n[d] ? 0 : a[d] + 1;
    }
    for (int q = 0; q < 8; ++q)
      unsafeAtomicAdd(rho + nat(g, q & 1 ? b[0] : a[0], q & 2 ? b[1] : a[1], q & 4 ? b[2] : a[2]),
                      weight(q));
  };
  auto clamped = [](long long v) {
    return v > (1 << 24) ? 1 << 24 : (v < -(1 << 24) ? -(1 << 24) : (int)v);
  };
  if (threadIdx.x == 0) first = NT;
  if (threadIdx.x < 3) {
    lo_sh[threadIdx.x] = 1 << 30;
    hi_sh[threadIdx.x] = -(1 << 30);
  }
  // the box of a wavefront's cells, relative to its first particle's
  const unsigned long long lanes = __ballot(on);
  long long wref[3];
  int wlo[3], whi[3];
  long long ext[3];
  bool whole[3];
  for (int d = 0; d < 3; ++d) {
    wref[d] = __shfl(u[d], lanes ? __ffsll((long long)lanes) - 1 : 0, 64);
    const int r = clamped(u[d] - wref[d]);
    int a = on ? r : 1 << 24, b = on ? r : -(1 << 24);
    for (int o = 32; o > 0; o >>= 1) {
      a = min(a, __shfl_xor(a, o, 64));
      b = max(b, __shfl_xor(b, o, 64));
    }
    wlo[d] = a;
    whi[d] = b;
  }
  // particles that lie apart already in a wavefront go to memory without
  // waiting for the rest of the workgroup
  bool apart = lanes != 0 && !extents(wlo, whi, ext, whole);
  if (apart) {
    if (on) add_direct();
    on = false;
  }
  __syncthreads();
  // the workgroup's box, relative to its first particle's
  const bool lead = lanes != 0 && !apart && (threadIdx.x & 63) == 0;
  if (lead) atomicMin(&first, (int)threadIdx.x);
  __syncthreads();
  if (first == NT) return;  // no particle left (uniform)
  if ((int)threadIdx.x == first)
    for (int d = 0; d < 3; ++d) ref[d] = wref[d];
  __syncthreads();
  if (lead)
    for (int d = 0; d < 3; ++d) {
      atomicMin(&lo_sh[d], clamped(wref[d] - ref[d] + wlo[d]));
      atomicMax(&hi_sh[d], clamped(wref[d] - ref[d] + whi[d]));
    }
  __syncthreads();
  int lo[3], hi[3];
  for (int d = 0; d < 3; ++d) {
    lo[d] = lo_sh[d];
    hi[d] = hi_sh[d];
  }
  if (!extents(lo, hi, ext, whole)) {
    if (on) add_direct();
    return;
  }
  unsigned c0[3], c1[3];  // lower and upper cell in the box
  for (int d = 0; d < 3; ++d) {
    if (!whole[d]) {
      c0[d] = (unsigned)(clamped(u[d] - ref[d]) - lo[d]);
      c1[d] = c0[d] + 1;
    } else {
      c0[d] = wrap_mod(u[d], n[d]);
      c1[d] = c0[d] + 1 == n[d] ? 0 : c0[d] + 1;
    }
  }
  const int e0 = (int)ext[0], e01 = e0 * (int)ext[1], vol = e01 * (int)ext[2];
  for (int i = threadIdx.x; i < vol; i += NT) acc[i] = 0.0;
  __syncthreads();
  if (on)
    for (int q = 0; q < 8; ++q)
      __hip_atomic_fetch_add(acc + (q & 4 ? c1[2] : c0[2]) * e01 + (q & 2 ? c1[1] : c0[1]) * e0 +
                                 (q & 1 ? c1[0] : c0[0]),
                             weight(q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __syncthreads();
  // the domain cell of the box's first cell, then row by row
  unsigned base[3];
  for (int d = 0; d < 3; ++d) base[d] = whole[d] ? 0u : wrap_mod(ref[d] + lo[d], n[d]);
  for (int i = threadIdx.x; i < vol; i += NT) {
    const double v = acc[i];
    if (v == 0.0) continue;
    const unsigned z = (unsigned)(i / e01), t = (unsigned)(i - (int)z * e01);
    const unsigned y = t / (unsigned)e0, x = t - y * (unsigned)e0;
    unsigned X = base[0] + x, Y = base[1] + y, Z = base[2] + z;
    X = X >= n[0] ? X - n[0] : X;
    Y = Y >= n[1] ? Y - n[1] : Y;
    Z = Z >= n[2] ? Z - n[2] : Z;
    unsafeAtomicAdd(rho + nat(g, X, Y, Z), v);
  }
}

// total density of a cell: the deposited field plus, when given, the gas
// density of the state (component 0 of a padded box covering the domain)
struct RhoSrc {
  const double* rho;
  const double* state;  // or nullptr
  long long soff;
  unsigned px, py, ng;
};

__device__ __forceinline__ double rho_total(const RhoSrc& R, const Grid& g, unsigned c) {
  double r = R.rho[c];
  if (R.state) {
    const unsigned i = c % g.nx, j = (c / g.nx) % g.ny, k = c / (g.nx * g.ny);
    r = r + R.state[R.soff + ((long long)(k + R.ng) * R.py + (j + R.ng)) * R.px + (i + R.ng)];
  }
  return r;
}

// ---- deterministic reductions: fixed block partials, then one block ----
template <int OP>  // 0: sum, 1: max
__device__ __forceinline__ double combine(double a, double b) {
  return OP == 0 ? a + b : fmax(a, b);
}

template <int OP>
__device__ double block_reduce(double v) {
  __shared__ double sh[kBlock];
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] = combine<OP>(sh[threadIdx.x], sh[threadIdx.x + s]);
    __syncthreads();
  }
  return sh[0];
}

// MODE 0: sum of rho_total (natural order); 2: max |f|; 3: sum of phi
// (solver order)
template <int MODE>
__global__ __launch_bounds__(kBlock) void k_partial(RhoSrc R, const double* __restrict__ phi,
                                                    const double* __restrict__ f, Grid g,
                                                    double* __restrict__ part) {
  constexpr int OP = (MODE == 0 || MODE == 3) ? 0 : 1;
  const unsigned n = g.nx * g.ny * g.nz;
  double acc = 0.0;
  for (unsigned c = blockIdx.x * kBlock + threadIdx.x; c < n; c += gridDim.x * kBlock) {
    double v;
    if (MODE == 0) {
      v = rho_total(R, g, c);
    } else if (MODE == 2) {
      v = fabs(f[c]);
    } else {
      v = phi[c];
    }
    acc = combine<OP>(acc, v);
  }
  const double b = block_reduce<OP>(acc);
  if (threadIdx.x == 0) part[blockIdx.x] = b;
}

template <int OP>
__global__ __launch_bounds__(kBlock) void k_final(const double* __restrict__ part, int nb,
                                                  double* __restrict__ out) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < nb; i += kBlock) acc = combine<OP>(acc, part[i]);
  const double b = block_reduce<OP>(acc);
  if (threadIdx.x == 0) *out = b;
}

// f = coef (rho_total - sum / n) in the solver's order; the initial guess
// copied into it
__global__ __launch_bounds__(kBlock) void k_rhs(RhoSrc R, Grid g, double coef,
                                                const double* __restrict__ sum,
                                                double* __restrict__ f,
                                                const double* __restrict__ phi_in,
                                                double* __restrict__ phi) {
  const unsigned n = g.nx * g.ny * g.nz;
  const unsigned c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= n) return;
  unsigned i, j, k;
  coords(g, c, &i, &j, &k);
  const unsigned a = at(g, i, j, k);
  const double mean = *sum / (double)n;
  f[a] = coef * (rho_total(R, g, c) - mean);
  phi[a] = phi_in[c];
}

// the caller's phi (natural order) = the solution minus sum / n
__global__ __launch_bounds__(kBlock) void k_sub_mean(const double* __restrict__ phi, Grid g,
                                                     const double* __restrict__ sum,
                                                     double* __restrict__ out) {
  const unsigned n = g.nx * g.ny * g.nz;
  const unsigned c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= n) return;
  unsigned i, j, k;
  coords(g, c, &i, &j, &k);
  out[c] = phi[at(g, i, j, k)] - *sum / (double)n;
}

// ---- multigrid kernels ----
// x / 6, correctly rounded, by a product and one correction instead of the
// range-scaled division: y = RN(1/6) is within 2^-54 of 1/6, so x y rounded is
// within one unit in the last place of x / 6, the remainder x - 6 q is exact,
// and adding its quotient to q rounds to the correctly rounded x / 6
// (Markstein's theorem).  For finite x with a normal quotient, or 0: below
// 2^-1019 the last bit may differ, and an infinite x gives NaN, which the next
// sweep's differences of infinities give anyway.
__device__ __forceinline__ double div6(double x) {
  constexpr double y = 1.0 / 6.0;
  const double q = x * y;
  return fma(fma(-6.0, q, x), y, q);
}

// one Gauss-Seidel half sweep: cells with (i + j + k) % 2 == color.  Bound by
// memory (12 bytes a cell: 41 us at 256^3, 4.9 TB/s).  Workgroups are numbered
// XCD by XCD, here and in the kernels below: the rows and planes beside a cell
// are then read through the L2 that holds them (256^3 in place: 42 us in launch
// order, the residual's maximum 89 and 79, a solve 8045 and 7720).
__global__ __launch_bounds__(kBlock) void k_rbgs(double* __restrict__ phi,
                                                 const double* __restrict__ f, Grid g, double h2,
                                                 unsigned color) {
  const unsigned half = g.nx >> 1;
  const unsigned t = xcd_linear_block() * kBlock + threadIdx.x;
  if (t >= half * g.ny * g.nz) return;
  const unsigned ih = t % half, r = t / half;
  const unsigned j = r % g.ny, k = r / g.ny;
  const unsigned i = 2 * ih + ((j + k + color) & 1);
  const unsigned c = at(g, i, j, k);
  phi[c] = div6(nb_sum(phi, g, i, j, k) - h2 * f[c]);
}

// One pair of cells (2 ih, 2 ih + 1) of a row and what its stencils read: in
// the solver's order a cell's x neighbours are entries ih and ih -+ 1 of the
// other colour's row, its y and z neighbours the entries ih of the rows beside.
struct Pair {
  unsigned row, rs, rn, rb, rt;  // row starts: own, y below and above, z below and above
  unsigned ih, im, ip;           // half index and its periodic neighbours
  unsigned par;                  // (j + k) & 1
};
__device__ __forceinline__ Pair pair_at(unsigned half, unsigned ny, unsigned nz, unsigned ih,
                                        unsigned j, unsigned k) {
  Pair p;
  p.row = (k * ny + j) * half;
  p.rs = (k * ny + wrap_dec(j, ny)) * half;
  p.rn = (k * ny + wrap_inc(j, ny)) * half;
  p.rb = (wrap_dec(k, nz) * ny + j) * half;
  p.rt = (wrap_inc(k, nz) * ny + j) * half;
  p.ih = ih;
  p.im = wrap_dec(ih, half);
  p.ip = wrap_inc(ih, half);
  p.par = (j + k) & 1;
  return p;
}
// nb_sum of the pair's cell of colour `color`; other: the other colour's array
__device__ __forceinline__ double pair_sum(const double* other, const Pair& p, unsigned color) {
  const bool odd = ((p.par + color) & 1) != 0;
  const double sx = other[p.row + (odd ? p.ih : p.im)] + other[p.row + (odd ? p.ip : p.ih)];
  const double sy = other[p.rs + p.ih] + other[p.rn + p.ih];
  const double sz = other[p.rb + p.ih] + other[p.rt + p.ih];
  return (sx + sy) + sz;
}

// max |f - L phi|: one lane per pair of cells.  Bound by memory (16 bytes a
// cell): 97 us at 256^3 with a lane per cell, its coordinates divided out, 89
// with pairs, 79 with the workgroups numbered XCD by XCD, 92 behind the marching
// smoother, which passes over more memory than the chip's last cache holds.
__global__ __launch_bounds__(kBlock) void k_resid_max(const double* __restrict__ phi,
                                                      const double* __restrict__ f, Grid g,
                                                      FastDiv dh, FastDiv dy, double inv_h2,
                                                      double* __restrict__ part) {
  const unsigned half = g.nx >> 1, hn = half * g.ny * g.nz;
  double acc = 0.0;
  for (unsigned t = xcd_linear_block() * kBlock + threadIdx.x; t < hn; t += gridDim.x * kBlock) {
    const unsigned r = fast_div(t, dh), ih = t - r * half;
    const unsigned k = fast_div(r, dy), j = r - k * g.ny;
    const Pair p = pair_at(half, g.ny, g.nz, ih, j, k);
    for (unsigned color = 0; color < 2; ++color) {
      const unsigned c = color * hn + t;
      const double lap = (pair_sum(phi + (1 - color) * hn, p, color) - 6.0 * phi[c]) * inv_h2;
      acc = fmax(acc, fabs(f[c] - lap));
    }
  }
  const double b = block_reduce<1>(acc);
  if (threadIdx.x == 0) part[blockIdx.x] = b;
}

// The V-cycle from a level of at most kSmallCells cells down, in one launch:
// one workgroup keeps phi and f of these levels in LDS and carries out the
// same sweeps, restrictions and prolongations, in the same order, as the
// kernels of the larger levels do.  Bound by latency: the chain of half sweeps
// (88 from 16^3 down), each an LDS read, seven operations and a barrier.  As
// 13 launches on arrays in memory a cycle took about 115 us here; in one 54 us;
// with the pairs' places and right-hand sides kept in registers and div6 33 us.
constexpr int kCoarseThreads = 512;
constexpr int kMaxCoarse = 8;  // levels of at most 4096 cells, halved down to 8 cells
constexpr size_t kSmallCells = 4096;
struct CoarseArgs {
  int nlev;
  Grid g[kMaxCoarse];
  double h2[kMaxCoarse], inv_h2[kMaxCoarse];
  double* phi;  // of the finest of these levels
  const double* f;
};

// The half sweeps of one of these levels: NP pairs per thread, whose places
// and right-hand sides stay in registers over the sweeps.
template <int NP>
__device__ __forceinline__ void lds_sweeps(double* phi, const double* f, const Grid& g, double h2,
                                           int sweeps) {
  const unsigned half = g.nx >> 1, hn = half * g.ny * g.nz;
  // a level of one wavefront's pairs is swept by the first one alone, whose
  // LDS accesses keep their order without a barrier
  const bool one = NP == 1 && hn <= 64;
  if (one && threadIdx.x >= 64) return;
  Pair p[NP];
  double hf[NP][2];
  for (int q = 0; q < NP; ++q) {
    const unsigned t = threadIdx.x + q * kCoarseThreads;
    if (t >= hn) continue;
    const unsigned r = t / half, ih = t - r * half, k = r / g.ny, j = r - k * g.ny;
    p[q] = pair_at(half, g.ny, g.nz, ih, j, k);
    hf[q][0] = h2 * f[t];
    hf[q][1] = h2 * f[hn + t];
  }
  for (int it = 0; it < sweeps; ++it)
#pragma unroll
    for (unsigned color = 0; color < 2; ++color) {
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const unsigned t = threadIdx.x + q * kCoarseThreads;
        if (t < hn)
          phi[color * hn + t] = div6(pair_sum(phi + (1 - color) * hn, p[q], color) - hf[q][color]);
      }
      if (one) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      } else {
        __syncthreads();
      }
    }
}
__device__ __forceinline__ void lds_smooth(double* phi, const double* f, const Grid& g, double h2,
                                           int sweeps) {
  const unsigned hn = (g.nx >> 1) * g.ny * g.nz;
  if (hn > kCoarseThreads) lds_sweeps<kSmallCells / 2 / kCoarseThreads>(phi, f, g, h2, sweeps);
  else lds_sweeps<1>(phi, f, g, h2, sweeps);
  __syncthreads();
}

// Two sweeps (four half sweeps) of a level in one launch, from `src` to `dst`:
// a workgroup loads a tile of 8^3 cells with a halo of four, one cell per half
// sweep, relaxes the whole 16^3 block in LDS and stores the tile.  Every cell
// gets the operations of the half sweeps above on the same values.
// For levels of at most kTileCells cells, where the four launches it replaces
// are latency: two sweeps of 64^3 18.8 -> 10.0 us, of 32^3 18.4 -> 5.9 us.  A
// larger level is bound by its traffic, which the halo multiplies by eight
// (128^3 takes 28 us in place, and its tiles alone would load 268 MB).
constexpr int kTileThreads = 512;
constexpr int kTB = 16, kTBHalf = 8, kTileOwn = 8, kTileHalo = 4;
constexpr size_t kTileCells = 1 << 18, kTileBlocks = 768;
__global__ __launch_bounds__(kTileThreads) void k_smooth_tile(const double* __restrict__ src,
                                                              double* __restrict__ dst,
                                                              const double* __restrict__ f, Grid g,
                                                              unsigned tx, unsigned ty,
                                                              double h2) {
  constexpr unsigned hn = kTBHalf * kTB * kTB;      // pairs of the block
  constexpr int NP = hn / kTileThreads;             // per thread
  constexpr int SJ = kTBHalf, SK = kTBHalf * kTB;   // LDS strides of a row and a plane
  __shared__ double u[2 * hn];
  const unsigned half = g.nx >> 1, gn = half * g.ny * g.nz;
  const unsigned b = blockIdx.x, bz = b / (tx * ty), by = (b - bz * tx * ty) / tx;
  const unsigned bx = b - bz * tx * ty - by * tx;
  auto wrap = [](int x, unsigned n) { return (unsigned)(((x % (int)n) + (int)n) % (int)n); };
  unsigned at_[NP];        // the pair's place in the level's colour arrays
  int li[NP];              // and in the block
  double hf[NP][2];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int t = (int)threadIdx.x + q * kTileThreads;
    const int lh = t % kTBHalf, lj = t / SJ % kTB, lk = t / SK;
    const unsigned ih = wrap((int)(bx * (kTileOwn / 2)) + lh - kTileHalo / 2, half);
    const unsigned j = wrap((int)(by * kTileOwn) + lj - kTileHalo, g.ny);
    const unsigned k = wrap((int)(bz * kTileOwn) + lk - kTileHalo, g.nz);
    at_[q] = (k * g.ny + j) * half + ih;
    li[q] = t;
    u[t] = src[at_[q]];
    u[hn + t] = src[gn + at_[q]];
    hf[q][0] = h2 * f[at_[q]];
    hf[q][1] = h2 * f[gn + at_[q]];
  }
  __syncthreads();
#pragma unroll
  for (int stage = 0; stage < 4; ++stage) {
    const int color = stage & 1;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int t = li[q], lh = t % kTBHalf, lj = t / SJ % kTB, lk = t / SK;
      // block origins are even, so the block's parity is the level's
      const bool odd = ((lj + lk + color) & 1) != 0;
      const int i = 2 * lh + (odd ? 1 : 0);
      if (i >= 1 && i < kTB - 1 && lj >= 1 && lj < kTB - 1 && lk >= 1 && lk < kTB - 1) {
        const double* o = u + (1 - color) * hn;
        const double sx = o[odd ? t : t - 1] + o[odd ? t + 1 : t];
        const double sy = o[t - SJ] + o[t + SJ];
        const double sz = o[t - SK] + o[t + SK];
        u[color * hn + t] = div6(((sx + sy) + sz) - hf[q][color]);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int t = li[q], lh = t % kTBHalf, lj = t / SJ % kTB, lk = t / SK;
    const bool own = lh >= kTileHalo / 2 && lh < (kTileHalo + kTileOwn) / 2 && lj >= kTileHalo &&
                     lj < kTileHalo + kTileOwn && lk >= kTileHalo && lk < kTileHalo + kTileOwn &&
                     bx * (kTileOwn / 2) + lh - kTileHalo / 2 < half &&
                     by * kTileOwn + lj - kTileHalo < g.ny && bz * kTileOwn + lk - kTileHalo < g.nz;
    if (own) {
      dst[at_[q]] = u[t];
      dst[gn + at_[q]] = u[hn + t];
    }
  }
}

// Two sweeps of a large level in one pass over its arrays.  A workgroup takes a
// tile of 64 x 16 cell columns with a halo of four cells and marches up a chunk
// of planes; a thread keeps one column of pairs.  With plane K the newest one
// loaded, the four half sweeps work on planes K - 1, K - 3, K - 5 and K - 7: each
// then needs only what earlier steps have finished, so that a step takes one
// barrier (the planes that the four read across columns alternate between two
// LDS buffers).  Along z the neighbours are in the thread's registers.
// The first half sweep reads black cells only, so red is written in place and
// black from one array to another: 20 bytes a cell instead of the four
// launches' 48.  Every cell gets the operations of the half sweeps above on the
// same values.
// Bound by a step's chain of LDS accesses, arithmetic and barrier (75 steps of
// 1.2 us for 256^3; loads two steps ahead change nothing), with the halo's work
// on top (1.7 x): two sweeps of 256^3 164 -> 92 us.  Blocks of 16 rows, two a
// CU, take 152.
constexpr int kMarchX = 36, kMarchY = 24;  // block: pairs in x, rows in y
constexpr int kMarchOwnX = 32, kMarchOwnY = 16;
constexpr int kMarchThreads = kMarchX * kMarchY;
// one workgroup per CU, whose chunk is at least kMarchPlanes planes
constexpr unsigned kMarchBlocks = 256, kMarchPlanes = 8;
__global__ __launch_bounds__(kMarchThreads) void k_smooth_march(
    const double* __restrict__ bsrc, const double* __restrict__ f, double* __restrict__ red,
    double* __restrict__ bdst, Grid g, unsigned tx, unsigned ty, unsigned chunk, double h2) {
  __shared__ double sh[2][4][kMarchThreads];
  const unsigned half = g.nx >> 1, ps = half * g.ny, hn = ps * g.nz;
  const unsigned b = xcd_linear_block(), bz = b / (tx * ty), by = (b - bz * tx * ty) / tx;
  const unsigned bx = b - bz * tx * ty - by * tx;
  auto wrap = [](int x, unsigned n) { return (unsigned)(((x % (int)n) + (int)n) % (int)n); };
  const int t = (int)threadIdx.x, lj = t / kMarchX, lh = t - lj * kMarchX;
  const int oi = (int)(bx * kMarchOwnX) + lh - 2, oj = (int)(by * kMarchOwnY) + lj - 4;
  const unsigned j = wrap(oj, g.ny), col = j * half + wrap(oi, half);
  const int z0 = (int)(bz * chunk);
  const int z1 = z0 + (int)chunk < (int)g.nz ? z0 + (int)chunk : (int)g.nz;
  const bool own = lh >= 2 && lh < 2 + kMarchOwnX && lj >= 4 && lj < 4 + kMarchOwnY &&
                   oi < (int)half && oj < (int)g.ny;
  // neighbours in the block; at its rim any entry, whose values never reach
  // the tile
  const int im = lh > 0 ? t - 1 : t, ip = lh < kMarchX - 1 ? t + 1 : t;
  const int jm = lj > 0 ? t - kMarchX : t, jp = lj < kMarchY - 1 ? t + kMarchX : t;
  // planes of the next loads: black K + 1, f of red K, f of black K - 2
  unsigned kb = wrap(z0 - 3, g.nz), kr = wrap(z0 - 4, g.nz), kf = wrap(z0 - 6, g.nz);
  double b0 = bsrc[kr * ps + col], b1 = 0.0, b2 = 0.0;       // black as loaded, planes K ..
  double r1 = 0.0, r2 = 0.0, r3 = 0.0;                       // red after 1, planes K - 2 ..
  double c1 = 0.0, c2 = 0.0, c3 = 0.0;                       // black after 2, planes K - 4 ..
  double d1 = 0.0, d2 = 0.0, d3 = 0.0;                       // red after 3, planes K - 6 ..
  double fr[5] = {}, fb[5] = {};  // h2 f of red, planes K - 1 .., of black, K - 3 ..
  // five steps an iteration, so that the values' moves from plane to plane are
  // renamings (the steps past the last plane store nothing)
  for (int K0 = z0 - 4; K0 < z1 + 7; K0 += 5) {
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const int K = K0 + q;
      double(*L)[kMarchThreads] = sh[K & 1];
      L[0][t] = b1;
      L[1][t] = r2;
      L[2][t] = c2;
      L[3][t] = d2;
      __syncthreads();
      const double nb = (bsrc + (size_t)kb * ps)[col];
      const double nr = h2 * (f + (size_t)kr * ps)[col];
      const double nf = h2 * (f + ((size_t)kf * ps + hn))[col];
      kb = wrap_inc(kb, g.nz);
      kr = wrap_inc(kr, g.nz);
      kf = wrap_inc(kf, g.nz);
      // the four planes have one parity; a red cell of odd column has its
      // other neighbour in the next pair, a black one's pair the other way round
      const bool odd = ((j + (unsigned)(K - 1)) & 1u) != 0;
      const int xr = odd ? ip : im, xb = odd ? im : ip;
      const double rn = div6((((b1 + L[0][xr]) + (L[0][jm] + L[0][jp])) + (b2 + b0)) - fr[0]);
      const double cn = div6((((r2 + L[1][xb]) + (L[1][jm] + L[1][jp])) + (r3 + r1)) - fb[0]);
      const double dn = div6((((c2 + L[2][xr]) + (L[2][jm] + L[2][jp])) + (c3 + c1)) - fr[4]);
      const double on = div6((((d2 + L[3][xb]) + (L[3][jm] + L[3][jp])) + (d3 + d1)) - fb[4]);
      if (own && K >= z0 + 7 && K < z1 + 7) {
        (red + (size_t)(K - 7) * ps)[col] = d2;
        (bdst + (size_t)(K - 7) * ps)[col] = on;
      }
      b2 = b1; b1 = b0; b0 = nb;
      r3 = r2; r2 = r1; r1 = rn;
      c3 = c2; c2 = c1; c1 = cn;
      d3 = d2; d2 = d1; d1 = dn;
      for (int m = 4; m > 0; --m) {
        fr[m] = fr[m - 1];
        fb[m] = fb[m - 1];
      }
      fr[0] = nr;
      fb[0] = nf;
    }
  }
}

// coarse f = mean of the eight children's residuals f - L phi; coarse phi = 0.
// Red and black cells may lie in different arrays (both indexed by at()).
__device__ __forceinline__ void restrict_cell(unsigned C, const double* red,
                                              const double* black, const double* f,
                                              const Grid& g, double inv_h2, const Grid& gc,
                                              double* fc, double* phic) {
  const unsigned I = C % gc.nx, J = (C / gc.nx) % gc.ny, K = C / (gc.nx * gc.ny);
  double s = 0.0;
  for (int q = 0; q < 8; ++q) {
    const unsigned i = 2 * I + (q & 1), j = 2 * J + ((q >> 1) & 1), k = 2 * K + (q >> 2);
    const unsigned c = at(g, i, j, k);
    const bool odd = ((q ^ (q >> 1) ^ (q >> 2)) & 1) != 0;  // the child's colour
    const double lap = nb_sum(odd ? red : black, g, i, j, k) - 6.0 * (odd ? black : red)[c];
    const double r = f[c] - lap * inv_h2;
    s = q == 0 ? r : s + r;
  }
  const unsigned a = at(gc, I, J, K);
  fc[a] = 0.125 * s;
  phic[a] = 0.0;
}
__global__ __launch_bounds__(kBlock) void k_restrict(const double* __restrict__ red,
                                                     const double* __restrict__ black,
                                                     const double* __restrict__ f, Grid g,
                                                     double inv_h2, Grid gc,
                                                     double* __restrict__ fc,
                                                     double* __restrict__ phic) {
  const unsigned C = xcd_linear_block() * kBlock + threadIdx.x;
  if (C < gc.nx * gc.ny * gc.nz) restrict_cell(C, red, black, f, g, inv_h2, gc, fc, phic);
}

// fine phi += trilinear (cell-centred) interpolation of the coarse
// correction: one lane per coarse cell reads its 3 x 3 x 3 neighbourhood
// once and corrects its eight children; child (a, b, c) takes the parent
// with weight 27/64, the three face neighbours on its side 9/64, the three
// edge neighbours 3/64 and the corner 1/64
__device__ __forceinline__ void prolong_cell(unsigned C, double* red, double* black,
                                             const Grid& g,
                                             const double* ec, const Grid& gc) {
  unsigned I, J, K;
  coords(gc, C, &I, &J, &K);
  const unsigned xs[3] = {wrap_dec(I, gc.nx), I, wrap_inc(I, gc.nx)};
  const unsigned ys[3] = {wrap_dec(J, gc.ny), J, wrap_inc(J, gc.ny)};
  const unsigned zs[3] = {wrap_dec(K, gc.nz), K, wrap_inc(K, gc.nz)};
  double e[3][3][3];
  for (int z = 0; z < 3; ++z)
    for (int y = 0; y < 3; ++y)
      for (int x = 0; x < 3; ++x) e[z][y][x] = ec[at(gc, xs[x], ys[y], zs[z])];
  for (int q = 0; q < 8; ++q) {
    const int a = q & 1, b = (q >> 1) & 1, c = q >> 2;
    const int X = a ? 2 : 0, Y = b ? 2 : 0, Z = c ? 2 : 0;  // the neighbour on the child's side
    const double c000 = e[1][1][1];
    const double c100 = e[1][1][X], c010 = e[1][Y][1], c001 = e[Z][1][1];
    const double c110 = e[1][Y][X], c101 = e[Z][1][X], c011 = e[Z][Y][1];
    const double c111 = e[Z][Y][X];
    const double v = (27.0 * c000 + 9.0 * ((c100 + c010) + c001) + 3.0 * ((c110 + c101) + c011) +
                      c111) *
                     (1.0 / 64.0);
    const unsigned f = at(g, 2 * I + a, 2 * J + b, 2 * K + c);
    double* phi = ((a ^ b ^ c) & 1) != 0 ? black : red;
    phi[f] = phi[f] + v;
  }
}
__global__ __launch_bounds__(kBlock) void k_prolong(double* red, double* black, Grid g,
                                                    const double* __restrict__ ec, Grid gc) {
  const unsigned C = xcd_linear_block() * kBlock + threadIdx.x;
  if (C < gc.nx * gc.ny * gc.nz) prolong_cell(C, red, black, g, ec, gc);
}

constexpr int kPre = 2, kPost = 2, kCoarseSweeps = 32;

__global__ __launch_bounds__(kCoarseThreads) void k_coarse(CoarseArgs A) {
  // every level an eighth of the one above: at most 4096 (1 + 1/8 + 1/64 + ...)
  // cells in all
  __shared__ double sphi[kSmallCells + kSmallCells / 7 + 8], sf[kSmallCells + kSmallCells / 7 + 8];
  const unsigned n0 = A.g[0].nx * A.g[0].ny * A.g[0].nz;
  for (unsigned i = threadIdx.x; i < n0; i += kCoarseThreads) {
    sphi[i] = A.phi[i];
    sf[i] = A.f[i];
  }
  __syncthreads();
  unsigned o = 0;  // offset of the level's cells
  int l = 0;
  for (; l + 1 < A.nlev; ++l) {
    const Grid g = A.g[l], gc = A.g[l + 1];
    const unsigned n = g.nx * g.ny * g.nz, nc = gc.nx * gc.ny * gc.nz;
    lds_smooth(sphi + o, sf + o, g, A.h2[l], kPre);
    for (unsigned C = threadIdx.x; C < nc; C += kCoarseThreads)
      restrict_cell(C, sphi + o, sphi + o, sf + o, g, A.inv_h2[l], gc, sf + o + n, sphi + o + n);
    __syncthreads();
    o += n;
  }
  lds_smooth(sphi + o, sf + o, A.g[l], A.h2[l], kCoarseSweeps);
  for (--l; l >= 0; --l) {
    const Grid g = A.g[l], gc = A.g[l + 1];
    const unsigned nc = gc.nx * gc.ny * gc.nz, oc = o;
    o -= g.nx * g.ny * g.nz;
    for (unsigned C = threadIdx.x; C < nc; C += kCoarseThreads)
      prolong_cell(C, sphi + o, sphi + o, g, sphi + oc, gc);
    __syncthreads();
    lds_smooth(sphi + o, sf + o, g, A.h2[l], kPost);
  }
  for (unsigned i = threadIdx.x; i < n0; i += kCoarseThreads) A.phi[i] = sphi[i];
}

// ---- g = -grad(phi) into the padded layout of a box covering the domain ----
template <class T>
__global__ __launch_bounds__(kBlock) void k_gradient(const double* __restrict__ phi, Grid g,
                                                     double two_dx, BoxDev b,
                                                     T* __restrict__ grav) {
  const unsigned c = xcd_linear_block() * kBlock + threadIdx.x;
  if (c >= (unsigned)b.P) return;
  const unsigned px = (unsigned)b.px, py = (unsigned)b.py;
  const int pi = (int)(c % px), pj = (int)((c / px) % py), pk = (int)(c / (px * py));
  // the periodic image of the padded cell in the domain
  auto wrapc = [](int x, unsigned n) { return (unsigned)(((x % (int)n) + (int)n) % (int)n); };
  const unsigned i = wrapc(pi - b.ng, g.nx), j = wrapc(pj - b.ng, g.ny), k = wrapc(pk - b.ng, g.nz);
  const double gx = -(phi[nat(g, wrap_inc(i, g.nx), j, k)] - phi[nat(g, wrap_dec(i, g.nx), j, k)]) / two_dx;
  const double gy = -(phi[nat(g, i, wrap_inc(j, g.ny), k)] - phi[nat(g, i, wrap_dec(j, g.ny), k)]) / two_dx;
  const double gz = -(phi[nat(g, i, j, wrap_inc(k, g.nz))] - phi[nat(g, i, j, wrap_dec(k, g.nz))]) / two_dx;
  T* out = grav + b.goff;
  out[c] = (T)gx;
  out[b.gstride + c] = (T)gy;
  out[2 * b.gstride + c] = (T)gz;
}

static unsigned blocks_for(unsigned long long n) { return (unsigned)((n + kBlock - 1) / kBlock); }

struct Level {
  Grid g;
  double h2, inv_h2;
  double* phi;
  double* f;
  double* alt;  // a second phi array, free while the level is worked on
};

static int check_dom(const int32_t* dom) {
  if (!dom) return NYX_E_NULL;
  unsigned long long n = 1;
  for (int d = 0; d < 3; ++d) {
    if (dom[d] < 2 || (dom[d] & 1) || dom[d] > (1 << 16)) return NYX_E_SHAPE;
    n *= (unsigned long long)dom[d];
  }
  if (n > (1ull << 31) - 1) return NYX_E_SHAPE;
  return NYX_OK;
}

// level sizes: halve while every extent stays even (red-black sweeps pair
// the cells of a row), down to extents of 2
static std::vector<Grid> levels_of(const int32_t* dom) {
  std::vector<Grid> L;
  Grid g{(unsigned)dom[0], (unsigned)dom[1], (unsigned)dom[2]};
  L.push_back(g);
  while (g.nx % 4 == 0 && g.ny % 4 == 0 && g.nz % 4 == 0) {
    g = Grid{g.nx / 2, g.ny / 2, g.nz / 2};
    L.push_back(g);
  }
  return L;
}

static size_t cells(const Grid& g) { return (size_t)g.nx * g.ny * g.nz; }
static size_t r256(size_t x) { return (x + 255) / 256 * 256; }

// workspace: block partials, 8 scalars, then phi and f of every level in the
// solver's colour-split order, each 256-byte aligned
constexpr size_t kOffScalars = (size_t)kRedBlocks * sizeof(double);
constexpr size_t kOffLevels = kOffScalars + 256;

static size_t mg_bytes(const int32_t* dom) {
  const auto L = levels_of(dom);
  size_t b = kOffLevels;
  for (size_t l = 0; l < L.size(); ++l) b += 2 * r256(cells(L[l]) * sizeof(double));
  return b;
}

template <int MODE, int OP>
static void reduce(const RhoSrc& R, const double* phi, const double* f, const Grid& g,
                   unsigned nb, double* part, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_partial<MODE>, dim3(nb), dim3(kBlock), 0, s, R, phi, f, g, part);
  hipLaunchKernelGGL(k_final<OP>, dim3(1), dim3(kBlock), 0, s, part, (int)nb, out);
}

// `iters` sweeps of a level's phi in place
static hipError_t smooth(const Level& v, int iters, hipStream_t s) {
  const unsigned nb = blocks_for((unsigned long long)(v.g.nx / 2) * v.g.ny * v.g.nz);
  for (int it = 0; it < iters; ++it)
    for (unsigned color = 0; color < 2; ++color)
      hipLaunchKernelGGL(k_rbgs, dim3(nb), dim3(kBlock), 0, s, v.phi, v.f, v.g, v.h2, color);
  return hipGetLastError();
}
// Tiled sweeps: levels of at most kTileCells cells, unless they are so thin that
// most of a block is halo (a V-cycle, tiled and in place: 12 x 20 x 1088, 816
// blocks, 176 and 156 us; 4 x 4 x 8192, 1024 blocks, 160 and 154).
static bool tiled(const Grid& g) {
  const size_t b = (size_t)((g.nx + kTileOwn - 1) / kTileOwn) * ((g.ny + kTileOwn - 1) / kTileOwn) *
                   ((g.nz + kTileOwn - 1) / kTileOwn);
  return cells(g) <= kTileCells && b <= kTileBlocks;
}
// The marching sweep's tiles, and chunks of equal length, as many as give the
// chip a workgroup per CU.
struct March {
  unsigned tx, ty, chunk, blocks;
};
static March march_of(const Grid& g) {
  March m;
  m.tx = (g.nx / 2 + kMarchOwnX - 1) / kMarchOwnX;
  m.ty = (g.ny + kMarchOwnY - 1) / kMarchOwnY;
  const unsigned want = std::max(1u, kMarchBlocks / std::max(1u, m.tx * m.ty));
  const unsigned nz = std::min(want, std::max(1u, g.nz / kMarchPlanes));
  m.chunk = (g.nz + nz - 1) / nz;
  m.blocks = m.tx * m.ty * ((g.nz + m.chunk - 1) / m.chunk);
  return m;
}
// Marching sweeps where their steps of 1.2 us, chunk + 11 for each round of
// workgroups, take less time than two sweeps in place, 15.4 us and 10 us per
// million cells.  V-cycles in place and marching (us): 80^3 106 and 111, 96^3
// 125 and 120, 128^3 171 and 152, 192^3 309 and 253, 256^3 673 and 546, 320^3
// 1410 and 1010; of thin domains, whose tiles are mostly halo, 8 x 16 x 8192 219
// and 245, 264 x 4 x 1024 217 and 227, 16 x 256 x 512 161 and 171.
static bool marching(const Grid& g) {
  if (tiled(g)) return false;
  const March m = march_of(g);
  const size_t rounds = (m.blocks + kMarchBlocks - 1) / kMarchBlocks;
  return 1.2 * (double)(rounds * (m.chunk + 11)) < 15.4 + 1e-5 * (double)cells(g);
}

// two sweeps from src to dst
static hipError_t smooth_tile(const Level& v, const double* src, double* dst, hipStream_t s) {
  const unsigned tx = (v.g.nx + kTileOwn - 1) / kTileOwn, ty = (v.g.ny + kTileOwn - 1) / kTileOwn,
                 tz = (v.g.nz + kTileOwn - 1) / kTileOwn;
  hipLaunchKernelGGL(k_smooth_tile, dim3(tx * ty * tz), dim3(kTileThreads), 0, s, src, dst, v.f, v.g,
                     tx, ty, v.h2);
  return hipGetLastError();
}

// two sweeps in one pass, black cells from one array to another
static hipError_t smooth_march(const Level& v, const double* src, double* dst, hipStream_t s) {
  const unsigned hn = v.g.nx / 2 * v.g.ny * v.g.nz;
  const March m = march_of(v.g);
  hipLaunchKernelGGL(k_smooth_march, dim3(m.blocks), dim3(kMarchThreads), 0, s, src + hn, v.f, v.phi,
                     dst + hn, v.g, m.tx, m.ty, m.chunk, v.h2);
  return hipGetLastError();
}

static hipError_t vcycle(std::vector<Level>& L, size_t l, hipStream_t s) {
  if (cells(L[l].g) <= kSmallCells) {
    CoarseArgs A{};
    A.nlev = (int)(L.size() - l);
    for (int i = 0; i < A.nlev; ++i) {
      A.g[i] = L[l + i].g;
      A.h2[i] = L[l + i].h2;
      A.inv_h2[i] = L[l + i].inv_h2;
    }
    A.phi = L[l].phi;
    A.f = L[l].f;
    hipLaunchKernelGGL(k_coarse, dim3(1), dim3(kCoarseThreads), 0, s, A);
    return hipGetLastError();
  }
  if (l + 1 == L.size()) return smooth(L[l], kCoarseSweeps, s);
  static_assert(kPre == 2 && kPost == 2, "the tiled smoother does two sweeps");
  const Level& f = L[l];
  Level& c = L[l + 1];
  const bool tile = tiled(f.g), march = marching(f.g);
  double* u = tile ? f.alt : f.phi;  // phi during the coarse correction
  double* ub = march ? f.alt : u;       // its black cells
  hipError_t e = tile ? smooth_tile(f, f.phi, u, s)
                      : (march ? smooth_march(f, f.phi, ub, s) : smooth(f, kPre, s));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_restrict, dim3(blocks_for(cells(c.g))), dim3(kBlock), 0, s, u, ub, f.f, f.g,
                     f.inv_h2, c.g, c.f, c.phi);
  if ((e = vcycle(L, l + 1, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_prolong, dim3(blocks_for(cells(c.g))), dim3(kBlock), 0, s, u, ub, f.g, c.phi,
                     c.g);
  return tile ? smooth_tile(f, u, f.phi, s)
              : (march ? smooth_march(f, ub, f.phi, s) : smooth(f, kPost, s));
}

// max |f - L phi| of a level into *out
static void resid_max(const Level& v, double* part, double* out, hipStream_t s) {
  const unsigned half = v.g.nx / 2;
  const unsigned nb = std::min<unsigned>(kResidBlocks, blocks_for(cells(v.g) / 2));
  hipLaunchKernelGGL(k_resid_max, dim3(nb), dim3(kBlock), 0, s, v.phi, v.f, v.g, make_fastdiv(half),
                     make_fastdiv(v.g.ny), v.inv_h2, part);
  hipLaunchKernelGGL(k_final<1>, dim3(1), dim3(kBlock), 0, s, part, (int)nb, out);
}

}  // namespace grav
}  // namespace nyx

using namespace nyx;
using namespace nyx::grav;

extern "C" {

int nyx_cic_deposit(const double* pos, const double* mass, long long np, const int32_t* dom,
                    double dx, double* rho, void* stream) {
  int rc = check_dom(dom);
  if (rc) return rc;
  if (!rho) return NYX_E_NULL;
  if (np < 0 || !(dx > 0.0) || !std::isfinite(dx)) return NYX_E_PARAM;
  if (np == 0) return NYX_OK;
  if (!pos || !mass) return NYX_E_NULL;
  Grid g{(unsigned)dom[0], (unsigned)dom[1], (unsigned)dom[2]};
  const double inv_vol = 1.0 / ((dx * dx) * dx);
  hipStream_t s = (hipStream_t)stream;
  if (np >= kCicWide)
    hipLaunchKernelGGL((k_cic<kCicBlock, kCicCells>), dim3((unsigned)((np + kCicBlock - 1) / kCicBlock)),
                       dim3(kCicBlock), 0, s, pos, mass, np, g, dx, inv_vol, rho);
  else
    hipLaunchKernelGGL((k_cic<kCicSmallBlock, kCicSmallCells>),
                       dim3((unsigned)((np + kCicSmallBlock - 1) / kCicSmallBlock)),
                       dim3(kCicSmallBlock), 0, s, pos, mass, np, g, dx, inv_vol, rho);
  return hipGetLastError() == hipSuccess ? NYX_OK : NYX_E_HIP;
}

int nyx_poisson_workspace_bytes(const int32_t* dom, size_t* bytes) {
  int rc = check_dom(dom);
  if (rc) return rc;
  if (!bytes) return NYX_E_NULL;
  *bytes = mg_bytes(dom);
  return NYX_OK;
}

int nyx_poisson_solve(const int32_t* dom, double dx, double coef, const double* rho,
                      const double* state, const nyx_box* box, double* phi, double tol,
                      int max_vcycles, void* workspace, size_t ws_bytes, void* stream,
                      int* vcycles, double* rel_resid) {
  int rc = check_dom(dom);
  if (rc) return rc;
  if (!rho || !phi || !workspace) return NYX_E_NULL;
  if (!(dx > 0.0) || !std::isfinite(dx) || !std::isfinite(coef) || !(tol >= 0.0) ||
      max_vcycles < 1 || max_vcycles > 1000)
    return NYX_E_PARAM;
  if ((uintptr_t)workspace & 255) return NYX_E_WORKSPACE;
  if (ws_bytes < mg_bytes(dom)) return NYX_E_WORKSPACE;
  RhoSrc R{rho, nullptr, 0, 0, 0, 0};
  if (state) {
    if (!box) return NYX_E_NULL;
    if ((rc = validate_box(box))) return rc;
    for (int d = 0; d < 3; ++d)
      if (box->n[d] != dom[d]) return NYX_E_SHAPE;
    R.state = state;
    R.soff = box->state_off;
    R.ng = (unsigned)box->ng;
    R.px = (unsigned)(box->n[0] + 2 * box->ng);
    R.py = (unsigned)(box->n[1] + 2 * box->ng);
  }
  hipStream_t s = (hipStream_t)stream;
  const auto G = levels_of(dom);
  double* part = (double*)workspace;
  double* scal = (double*)((char*)workspace + kOffScalars);  // sum rho, max|f|, max|r|, sum phi
  char* w = (char*)workspace + kOffLevels;
  std::vector<Level> L(G.size());
  double h = dx;
  for (size_t l = 0; l < G.size(); ++l) {
    L[l].g = G[l];
    L[l].h2 = h * h;
    L[l].inv_h2 = 1.0 / (h * h);
    L[l].phi = (double*)w;
    w += r256(cells(G[l]) * sizeof(double));
    L[l].f = (double*)w;
    w += r256(cells(G[l]) * sizeof(double));
    h *= 2.0;
  }
  // Second phi arrays for the smoothers that need one: on the finest level the
  // caller's phi, which after the right-hand side has been set up is not read
  // before the end; the coarser levels' (together a seventh of its cells) lie in
  // whichever of the finest level's two arrays is free while they are worked on
  // (the marching smoother uses only the second half of its level's, so the
  // finest level's black cells and the coarser levels do not meet).
  L[0].alt = phi;
  double* spare = tiled(L[0].g) ? L[0].phi : phi;
  for (size_t l = 1; l < L.size(); ++l) {
    L[l].alt = spare;
    spare += cells(L[l].g);
  }
  const Level& F = L[0];
  const unsigned nb = std::min<unsigned>(kRedBlocks, blocks_for(cells(F.g)));
  // right-hand side and its size
  reduce<0, 0>(R, F.phi, F.f, F.g, nb, part, scal + 0, s);
  hipLaunchKernelGGL(k_rhs, dim3(blocks_for(cells(F.g))), dim3(kBlock), 0, s, R, F.g, coef,
                     scal + 0, F.f, phi, F.phi);
  if (hipGetLastError() != hipSuccess) return NYX_E_HIP;
  // with tol > 0 or a residual requested the stream is synchronised (once,
  // then once per V-cycle); otherwise only kernels are enqueued
  const bool check = tol > 0.0 || rel_resid;
  auto read = [&](const double* src, double* dst) {
    return hipMemcpyAsync(dst, src, sizeof(double), hipMemcpyDeviceToHost, s) == hipSuccess &&
           hipStreamSynchronize(s) == hipSuccess;
  };
  double fnorm = 0.0, rmax = 0.0, rel = 0.0;
  if (check) {
    reduce<2, 1>(R, F.phi, F.f, F.g, nb, part, scal + 1, s);
    if (!read(scal + 1, &fnorm)) return NYX_E_HIP;
  }
  int done = 0;
  for (int cyc = 0; cyc < max_vcycles; ++cyc) {
    if (vcycle(L, 0, s) != hipSuccess) return NYX_E_HIP;
    ++done;
    if (tol > 0.0 || (check && cyc + 1 == max_vcycles)) {
      resid_max(F, part, scal + 2, s);
      if (!read(scal + 2, &rmax)) return NYX_E_HIP;
      rel = fnorm > 0.0 ? rmax / fnorm : rmax;
      if (tol > 0.0 && rel <= tol) break;
    }
  }
  // the periodic problem fixes phi up to a constant: remove its mean
  reduce<3, 0>(R, F.phi, F.f, F.g, nb, part, scal + 3, s);
  hipLaunchKernelGGL(k_sub_mean, dim3(blocks_for(cells(F.g))), dim3(kBlock), 0, s, F.phi, F.g,
                     scal + 3, phi);
  if (hipGetLastError() != hipSuccess) return NYX_E_HIP;
  if (vcycles) *vcycles = done;
  if (rel_resid) *rel_resid = rel;
  return NYX_OK;
}

int nyx_gravity_from_phi(const int32_t* dom, double dx, const double* phi, const nyx_box* box,
                         void* grav, int precision, void* stream) {
  int rc = check_dom(dom);
  if (rc) return rc;
  if (!phi || !box || !grav) return NYX_E_NULL;
  if ((rc = validate_box(box))) return rc;
  for (int d = 0; d < 3; ++d)
    if (box->n[d] != dom[d]) return NYX_E_SHAPE;
  if (!(dx > 0.0) || !std::isfinite(dx)) return NYX_E_PARAM;
  if (precision != NYX_FP64 && precision != NYX_MIXED) return NYX_E_PARAM;
  BoxDev b;
  box_layout(*box, 0, 0, &b);
  Grid g{(unsigned)dom[0], (unsigned)dom[1], (unsigned)dom[2]};
  const double two_dx = 2.0 * dx;
  hipStream_t s = (hipStream_t)stream;
  if (precision == NYX_FP64)
    hipLaunchKernelGGL(k_gradient<double>, dim3(blocks_for(b.P)), dim3(kBlock), 0, s, phi, g,
                       two_dx, b, (double*)grav);
  else
    hipLaunchKernelGGL(k_gradient<float>, dim3(blocks_for(b.P)), dim3(kBlock), 0, s, phi, g,
                       two_dx, b, (float*)grav);
  return hipGetLastError() == hipSuccess ? NYX_OK : NYX_E_HIP;
}

}  // extern "C"
