// diag.hip -- in-situ diagnostics on the GPU: PDFs (histograms) of cell
// quantities and slab profiles with mixing measures.
//
// Large runs need their analysis done where the data is (the paper's
// discussion of the capabilities needed at the exascale); it fixes no
// diagnostic, so these are standard ones of stratified and shear-layer
// flows.  Each is one HBM-bound pass over the interior cells.
//
// Cell quantities are evaluated in FP64 with IEEE operations (no contraction:
// the library is built with -ffp-contract=off; FP64 division and square
// root are correctly rounded), in a fixed order:
//   m2 = mx mx + my my + mz mz,  ke = (0.5 m2) / rho,  p = (gamma-1)(E - ke),
//   speed = sqrt(m2) / rho,      mach = speed / sqrt((gamma p) / rho).
// An FP32 state is widened first (exact), so a quantity's bin is a pure
// function of the stored bits.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fft.hpp"
#include "launch.hpp"

namespace hydro {

constexpr int kDiagBlock = 256;
constexpr int kDiagCells = 4;   // cells per thread in flight (loads before arithmetic)

template <class T, int Q>
__device__ __forceinline__ double diag_quantity(const T* p0, int64_t plane, int64_t o,
                                                double gamma) {
  const double r = double(p0[o]);
  if constexpr (Q == kQRho) {
    return r;
  } else {
    const double mx = double(p0[o + plane]), my = double(p0[o + 2 * plane]);
    const double mz = double(p0[o + 3 * plane]);
    const double m2 = mx * mx + my * my + mz * mz;
    if constexpr (Q == kQSpeed) {
      return __builtin_sqrt(m2) / r;
    } else {
      const double e = double(p0[o + 4 * plane]);
      const double p = (gamma - 1.0) * (e - (0.5 * m2) / r);
      if constexpr (Q == kQPressure) return p;
      // |v| / c = sqrt(|m|^2 / (gamma p rho)): one division and one root
      return __builtin_sqrt(m2 / ((gamma * p) * r));
    }
  }
}

// Bin of value v: 0 below lo (or NaN), 1 + floor((v - lo) w) inside,
// nbins + 1 at or above hi.
__device__ __forceinline__ int diag_bin(double v, double lo, double w, int nbins) {
  if (!(v >= lo)) return 0;
  const double t = (v - lo) * w;
  return t < double(nbins) ? 1 + int(t) : nbins + 1;
}

// Adds one to counter b (b < 0: nothing) for every lane of the wave.  Lanes
// that share the bin of the first lane still pending add together with one
// atomic, twice over (a flow with few distinct values, like a two-density
// layer, puts most of a wave in one or two bins); the lanes left add one
// by one.  Integer adds commute, so the counts do not depend on the grouping.
template <class C>
__device__ __forceinline__ void count_bin(C* ctr, int b) {
  bool todo = b >= 0;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const unsigned long long m = __ballot(todo);
    if (m == 0ull) return;  // wave-uniform
    const int lead = __builtin_amdgcn_readlane(b, int(__builtin_ctzll(m)));
    const bool mine = todo && b == lead;
    const unsigned long long same = __ballot(mine);
    if (mine) {
      if ((threadIdx.x & 63) == unsigned(__builtin_ctzll(same)))
        atomicAdd(&ctr[lead], C(__builtin_popcountll(same)));
      todo = false;
    }
  }
  if (todo) atomicAdd(&ctr[b], C(1));
}

__global__ void __launch_bounds__(kDiagBlock) zero_u64_kernel(unsigned long long* p, int n) {
  for (int i = blockIdx.x * kDiagBlock + threadIdx.x; i < n; i += gridDim.x * kDiagBlock)
    p[i] = 0ull;
}

template <class T>
struct DiagArgs {
  const T* pool;
  const PatchDev* patches;  // null: single grid
  PatchDev single;
  double gamma;
  int nbins;
  double lo, w;
  unsigned long long* counts;
  bool lds;                 // per-workgroup LDS counters (pdf_lds)
  int axis, chunks;
  FastDiv dnx, dny;         // single grid: division by nx and ny
  double rho_lo, drho, dx_axis;
  double* partials;
  double* out;
};

// Histogram of quantity Q over the interior cells of one grid (y = 0) or of
// patch blockIdx.y: workgroups stride over the flattened cells (x fastest,
// coalesced), count into LDS, then add their nonzero counters to the global
// 64-bit counters (exact: integer adds commute).
//
// A workgroup ends by adding its counters to the global ones: with 1000 bins
// and 4096 workgroups on 256^3 cells that was half the time (100 us for the
// density, 57 us so).  Up to 8192 counters take workgroups of 256 threads;
// up to kPdfLdsBins, where one or two workgroups fill the LDS of a CU,
// workgroups of 1024.  Counting straight into memory instead took 11.2 ms
// for 20000 bins (0.10 ms so) and is left for more, and for few cells (pdf_lds).
template <class T, int Q, int BLOCK>
__global__ void __launch_bounds__(BLOCK) pdf_kernel(DiagArgs<T> a) {
  extern __shared__ unsigned int hist[];
  const bool batch = a.patches != nullptr;
  const PatchDev P = batch ? a.patches[blockIdx.y] : a.single;
  const int nb2 = a.nbins + 2;
  const unsigned nx = unsigned(P.n[0]), ny = unsigned(P.n[1]);
  const unsigned cells = nx * ny * unsigned(P.n[2]);
  // wide counters of a batch: a workgroup of the patch for 12 cells per counter
  unsigned nwg = gridDim.x;
  if (BLOCK > kDiagBlock && batch) nwg = max(1u, min(nwg, cells / (12u * unsigned(nb2))));
  if (blockIdx.x >= nwg) return;
  if (a.lds) {
    for (int i = threadIdx.x; i < nb2; i += BLOCK) hist[i] = 0u;
    __syncthreads();
  }
  const FastDiv dnx = batch ? FastDiv(nx) : a.dnx, dny = batch ? FastDiv(ny) : a.dny;
  const T* p0 = a.pool + P.base0;
  constexpr int U = kDiagCells;
  const unsigned stride = nwg * BLOCK * U;
  for (unsigned i0 = blockIdx.x * BLOCK * U + threadIdx.x; i0 < cells; i0 += stride) {
    // the U cells' offsets, then their quantities (all loads issued first)
    int64_t o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned i = min(i0 + unsigned(u) * BLOCK, cells - 1);
      const unsigned row = dnx.div(i), x = i - row * nx;
      const unsigned z = dny.div(row), y = row - z * ny;
      o[u] = int64_t(x) + int64_t(y) * P.sy + int64_t(z) * P.sz;
    }
    double q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = diag_quantity<T, Q>(p0, P.plane, o[u], a.gamma);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool valid = i0 + unsigned(u) * BLOCK < cells;
      const int b = valid ? diag_bin(q[u], a.lo, a.w, a.nbins) : -1;
      if (a.lds)
        count_bin(hist, b);
      else
        count_bin(a.counts, b);
    }
  }
  if (a.lds) {
    __syncthreads();
    for (int i = threadIdx.x; i < nb2; i += BLOCK)
      if (hist[i]) atomicAdd(&a.counts[i], (unsigned long long)hist[i]);
  }
}

// The five conserved values of one cell, widened to FP64.
template <class T>
__device__ __forceinline__ void load_cell(const T* p0, int64_t plane, int64_t o, double (&c)[5]) {
#pragma unroll
  for (int v = 0; v < 5; ++v) c[v] = double(p0[o + v * plane]);
}

// Adds the five profile fields of one cell: rho, p, ke, f, f (1 - f).
template <class T>
__device__ __forceinline__ void profile_add(const double (&c)[5], const DiagArgs<T>& a,
                                            double (&acc)[5]) {
  const double r = c[0];
  const double m2 = c[1] * c[1] + c[2] * c[2] + c[3] * c[3];
  const double ke = (0.5 * m2) / r;
  const double p = (a.gamma - 1.0) * (c[4] - ke);
  const double f = __builtin_fmin(__builtin_fmax((r - a.rho_lo) / a.drho, 0.0), 1.0);
  acc[0] += r;
  acc[1] += p;
  acc[2] += ke;
  acc[3] += f;
  acc[4] += f * (1.0 - f);
}

// Slabs normal to y (axis 1) or z (axis 2): workgroup (c, s) sums the cells
// j = c 256 U + t + u 256 (u < U), then the same plus C 256 U, ... of slab s
// (x fastest), then reduces its threads in a fixed order into
// partials[s][c][5].
template <class T>
__global__ void __launch_bounds__(kDiagBlock) profile_slab_kernel(DiagArgs<T> a) {
  __shared__ double red[kDiagBlock / 64][5];
  const PatchDev& P = a.single;
  const int s = blockIdx.y, c = blockIdx.x;
  const unsigned nx = unsigned(P.n[0]);
  const unsigned rows = unsigned(a.axis == 2 ? P.n[1] : P.n[2]);
  const unsigned cells = nx * rows;
  const T* p0 = a.pool + P.base0;
  const int64_t srow = a.axis == 2 ? P.sy : P.sz;          // stride between the slab's rows
  const int64_t sbase = int64_t(s) * (a.axis == 2 ? P.sz : P.sy);
  constexpr int U = kDiagCells;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (unsigned j0 = unsigned(c) * kDiagBlock * U + threadIdx.x; j0 < cells;
       j0 += unsigned(a.chunks) * kDiagBlock * U) {
    double cv[U][5];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned j = min(j0 + unsigned(u) * kDiagBlock, cells - 1);
      const unsigned r = a.dnx.div(j), x = j - r * nx;
      load_cell<T>(p0, P.plane, sbase + int64_t(x) + int64_t(r) * srow, cv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + unsigned(u) * kDiagBlock < cells) profile_add<T>(cv[u], a, acc);
  }
#pragma unroll
  for (int v = 0; v < 5; ++v)
    for (int off = 32; off > 0; off >>= 1) acc[v] += __shfl_xor(acc[v], off);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int v = 0; v < 5; ++v) red[wave][v] = acc[v];
  __syncthreads();
  if (threadIdx.x < 5) {
    double t = red[0][threadIdx.x];
    for (int w = 1; w < kDiagBlock / 64; ++w) t += red[w][threadIdx.x];
    a.partials[(int64_t(s) * a.chunks + c) * 5 + threadIdx.x] = t;
  }
}

// Slabs normal to x (axis 0): a workgroup (c, xb) of 1024 threads holds R
// rows of w = min(nx, 256) neighbouring x each; thread (x, r) sums the rows
// c R + r, (c + C) R + r, ... (U of them in flight) at its own x, then the
// threads of an x add their sums in the order of r into partials[x][c][5].
// One row per workgroup of 256 threads left a quarter of the waves: 155
// against 116 us on 256^3 FP32.
constexpr int kXslabBlock = 1024;
constexpr int kXslabWidth = 256;
__host__ __device__ inline int xslab_width(int nx) { return nx < kXslabWidth ? nx : kXslabWidth; }
__host__ __device__ inline int xslab_rows(int nx) { return kXslabBlock / xslab_width(nx); }
template <class T>
__global__ void __launch_bounds__(kXslabBlock) profile_xslab_kernel(DiagArgs<T> a) {
  __shared__ double red[5][kXslabBlock];
  const PatchDev& P = a.single;
  const int c = blockIdx.x, w = xslab_width(P.n[0]), R = xslab_rows(P.n[0]);
  const int rg = threadIdx.x / w, xi = threadIdx.x - rg * w, x = blockIdx.y * w + xi;
  const unsigned ny = unsigned(P.n[1]), rows = ny * unsigned(P.n[2]);
  const T* p0 = a.pool + P.base0;
  constexpr int U = kDiagCells;
  const unsigned C = unsigned(a.chunks) * R;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (rg < R && x < P.n[0]) {
    for (unsigned r0 = unsigned(c * R + rg); r0 < rows; r0 += C * U) {
      double cv[U][5];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const unsigned r = min(r0 + unsigned(u) * C, rows - 1);
        const unsigned z = a.dny.div(r), y = r - z * ny;
        load_cell<T>(p0, P.plane, int64_t(x) + int64_t(y) * P.sy + int64_t(z) * P.sz, cv[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (r0 + unsigned(u) * C < rows) profile_add<T>(cv[u], a, acc);
    }
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) red[v][threadIdx.x] = acc[v];
  __syncthreads();
  // sum i = (x, v) of the tile, over the row groups that had a row (the others
  // hold zeros: a grid of 2 x 1 x 1 cells has one of 512)
  const int used = max(1, min(R, int(rows) - c * R));
  for (int i = threadIdx.x; i < 5 * w; i += kXslabBlock) {
    const int xo = i / 5, v = i - 5 * xo, xg = blockIdx.y * w + xo;
    if (xg >= P.n[0]) continue;
    double t = red[v][xo];
    for (int q = 1; q < used; ++q) t += red[v][q * w + xo];
    a.partials[(int64_t(xg) * a.chunks + c) * 5 + v] = t;
  }
}

// Sum of v over the workgroup in a fixed order (wave shuffles, then the
// waves in order); the result is returned to every thread.
__device__ __forceinline__ double block_sum(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();  // red is free
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = red[0];
  for (int w = 1; w < kDiagBlock / 64; ++w) t += red[w];
  return t;
}

// Slab means out[s][v] = sum_c partials[s][c][v] / cells per slab, then the
// mixing width and mixedness from per-thread sums over slabs t, t + 1024, ...
// reduced in a fixed order (one workgroup: 15 us with a thread per slab and
// one partial at a time, 3 us so; 256 slabs of 16 partials).
constexpr int kFinalBlock = 1024;
__global__ void __launch_bounds__(kFinalBlock) profile_final_kernel(const double* partials,
                                                                     int nslab, int chunks,
                                                                     double cells_per_slab,
                                                                     double dx_axis, double* out) {
  constexpr int NW = kFinalBlock / 64;
  __shared__ double red[3][NW];
  double w = 0.0, num = 0.0, den = 0.0;
  // the means: a thread per slab and field, eight partials in flight
  for (int i = threadIdx.x; i < 5 * nslab; i += kFinalBlock) {
    const int s = i / 5, v = i - 5 * s;
    const double* p = partials + int64_t(s) * chunks * 5 + v;
    double t = 0.0;
    int c = 0;
    for (; c + 8 <= chunks; c += 8) {
      double x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = p[(c + q) * 5];
#pragma unroll
      for (int q = 0; q < 8; ++q) t += x[q];
    }
    for (; c < chunks; ++c) t += p[c * 5];
    out[i] = t / cells_per_slab;
  }
  __syncthreads();  // the means are visible to the workgroup
  for (int s = threadIdx.x; s < nslab; s += kFinalBlock) {
    const double f = out[s * 5 + 3];
    w += 4.0 * f * (1.0 - f);
    den += f * (1.0 - f);
    num += out[s * 5 + 4];
  }
  // the three sums together: wave shuffles, then the waves in order
  for (int off = 32; off > 0; off >>= 1) {
    w += __shfl_xor(w, off);
    den += __shfl_xor(den, off);
    num += __shfl_xor(num, off);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = w;
    red[1][threadIdx.x >> 6] = den;
    red[2][threadIdx.x >> 6] = num;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    w = red[0][0];
    den = red[1][0];
    num = red[2][0];
    for (int q = 1; q < NW; ++q) {
      w += red[0][q];
      den += red[1][q];
      num += red[2][q];
    }
    out[nslab * 5] = w * dx_axis;
    out[nslab * 5 + 1] = den > 0.0 ? num / den : 0.0;
  }
}

// --------------------------------------------------------------------------
// One-dimensional kinetic-energy spectrum along x
// --------------------------------------------------------------------------
//
// A workgroup owns groups of P (even) whole x-lines (y, z): groups
// blockIdx.x, blockIdx.x + gridDim.x, ...  For each line it widens rho and m
// to FP64 and forms u = m / rho (IEEE division); it packs the complex lines
// ux + i uy of every x-line and uz + i uz' of every pair of x-lines (3P/2
// lines, no line of zeros), and transforms them in LDS with the in-place
// mixed-radix Stockham FFT of fft.hpp (radices 16, 4, 2, 3; output in
// natural order).  For a real pair packed as a + i b,
// |A(k)|^2 + |B(k)|^2 = (|Z(k)|^2 + |Z(N-k)|^2) / 2, so the power summed over
// the components and lines needs no unpacking: the threads sum |Z(k)|^2 over
// their lines (each k by 256 / n threads, each over every (256 / n)-th line;
// or 256 values of k at a time), and the workgroup folds k and N - k once, at
// its end, into its partial spectrum.  One workgroup a wavenumber sums the
// partials in a fixed order.
//
// Bound by the phases of a pass (loads, FFT stages, sums, with barriers
// between): two workgroups of 256 threads share a CU's LDS and overlap them,
// and a pass takes as many lines as fill 4096 complex values, so that a
// radix-16 stage has a butterfly for nearly every thread.  With one workgroup
// of 512 threads on a CU, 192 of them in a stage, 129 in the sums, three
// divisions a cell and the general stages: 256^3 FP32 200 instead of 117 us,
// FP64 309 instead of 140, 512^3 1830 instead of 1085, 768 x 384 x 768 2350
// instead of 2140, 64^3 15.7 instead of 12.

// the 3/2 complex lines of every x-line of a pass fill at most kSpecElems
// complex values of LDS
constexpr int kSpecElems = 4096;
constexpr int kSpecBlock = 256;  // threads of the spectrum kernel

template <class T>
__global__ void __launch_bounds__(kSpecBlock, 2)
    spectrum_kernel(DiagArgs<T> a, FftPlan sp, int P, FastDiv dn, FastDiv dny) {
  extern __shared__ double2 sbuf[];
  const PatchDev& Pd = a.single;
  const int n = sp.n, nl = P + P / 2;
  double2* W = sbuf;       // W[t] = exp(-2 pi i t / n)
  double2* buf = sbuf + n;  // 3P/2 complex lines (fft_pad slots), transformed in place
  for (int t = threadIdx.x; t < n; t += kSpecBlock) {
    double sn, cs;
    sincospi(-2.0 * double(t) / double(n), &sn, &cs);
    W[t] = make_double2(cs, sn);
  }
  // |Z(k)|^2 of k = k0 + 256 i over the lines g, g + ng, ... of every pass
  constexpr int KPT = (kSpecMaxLen + kSpecBlock - 1) / kSpecBlock;
  const int ng = n <= kSpecBlock ? kSpecBlock / n : 1;
  const int g = n <= kSpecBlock ? int(dn.div(threadIdx.x)) : 0, k0 = int(threadIdx.x) - g * n;
  double acc[KPT];
#pragma unroll
  for (int i = 0; i < KPT; ++i) acc[i] = 0.0;
  const int ny = Pd.n[1], lines = Pd.n[1] * Pd.n[2];
  const int groups = (lines + P - 1) / P;
  const T* p0 = a.pool + Pd.base0;
  // this thread's cells c = t + 256 i of the pass (line c / n of the group,
  // x = c mod n), fetched one pass ahead so that the next pass's loads are
  // in flight during the current transform
  constexpr int XPT = (kSpecElems * 2 / 3 + kSpecBlock - 1) / kSpecBlock;
  T fr[XPT], fm[XPT][3];
  auto fetch = [&](int grp) {
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
      const int c = threadIdx.x + i * kSpecBlock;
      const int lp = int(dn.div(uint32_t(c)));
      const int x = c - lp * n, line = grp * P + lp;
      if (lp < P && line < lines) {
        const int z = int(dny.div(uint32_t(line))), y = line - z * ny;
        const int64_t o = int64_t(y) * Pd.sy + int64_t(z) * Pd.sz + x;
        fr[i] = p0[o];
#pragma unroll
        for (int v = 0; v < 3; ++v) fm[i][v] = p0[o + (v + 1) * Pd.plane];
      }
    }
  };
  if (int(blockIdx.x) < groups) fetch(blockIdx.x);
  for (int grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    __syncthreads();  // the previous pass's buffer and the twiddles
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
      const int c = threadIdx.x + i * kSpecBlock;
      const int lp = int(dn.div(uint32_t(c)));
      const int x = c - lp * n;
      if (lp < P) {
        double u[3] = {0.0, 0.0, 0.0};  // lines past the end: zeros
        if (grp * P + lp < lines) velocity(fr[i], fm[i], u);
        buf[fft_pad(lp * n + x)] = make_double2(u[0], u[1]);
        // the real (even lp) or imaginary (odd lp) part of the pair's uz line
        double* zp = reinterpret_cast<double*>(&buf[fft_pad((P + (lp >> 1)) * n + x)]);
        zp[lp & 1] = u[2];
      }
    }
    if (grp + int(gridDim.x) < groups) fetch(grp + gridDim.x);
    __syncthreads();
    fft_lines_inplace<kSpecElems, kSpecBlock>(buf, nl, n, sp, W);
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const int k = k0 + i * kSpecBlock;
      if (k < n && g < ng)
        for (int q = g; q < nl; q += ng) {
          const double2 z = buf[fft_pad(q * n + k)];
          acc[i] += __builtin_fma(z.x, z.x, z.y * z.y);
        }
    }
  }
  __syncthreads();
  double* pw = reinterpret_cast<double*>(buf);  // [g][k]
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const int k = k0 + i * kSpecBlock;
    if (k < n && g < ng) pw[g * n + k] = acc[i];
  }
  __syncthreads();
  const int nk = n / 2 + 1;
  for (int k = threadIdx.x; k < nk; k += kSpecBlock) {
    const int km = k == 0 ? 0 : n - k;
    double s = 0.0;
    // (groups past the lines of a pass hold zeros)
    for (int h = 0; h < min(ng, nl); ++h) s += pw[h * n + k] + pw[h * n + km];
    a.partials[int64_t(blockIdx.x) * nk + k] = 0.5 * s;
  }
}

// E[k] = sum over workgroups of the partials / (lines n^2), halved at k = 0
// and at the Nyquist wavenumber of an even n.  Workgroup k: thread t sums
// partials t, t + 256, ..., then a fixed-order workgroup sum.
__global__ void __launch_bounds__(kDiagBlock) spectrum_final_kernel(const double* partials,
                                                                      int blocks, int n,
                                                                      double lines, double* out) {
  __shared__ double red[kDiagBlock / 64];
  const int nk = n / 2 + 1, k = blockIdx.x;
  double t = 0.0;
  for (int b = threadIdx.x; b < blocks; b += kDiagBlock) t += partials[int64_t(b) * nk + k];
  t = block_sum(t, red);
  if (threadIdx.x == 0) {
    double e = t / lines / (double(n) * double(n));
    if (k == 0 || (2 * k == n)) e *= 0.5;
    out[k] = e;
  }
}

// Whether a PDF counts in LDS: always up to kPdfNarrowBins counters, never above
// kPdfLdsBins.  Between them a workgroup of 1024 threads clears and adds 9 to 40
// counters a thread, which pays from 12 cells per counter on (grids, memory
// against LDS: 64^3 cells and 39000 bins 17 against 20 us, 20000 bins 16.3 and
// 16.4, 9000 bins 20 and 11; 16^3 and 39000 bins 9 and 14; batches: 64 patches of
// 16^3 and 39000 bins 17 and 21, 9000 bins 20 and 11.5).  In a batch it also does
// where one patch has a cell per counter, since four workgroups are all that a
// patch has with counters in memory (one of 32^3 cells and 20000 bins 28 and 26,
// 39000 bins 28 and 30).
static bool pdf_lds(const LaunchDiag& L) {
  const int64_t nb2 = int64_t(L.nbins) + 2;
  if (nb2 <= kPdfNarrowBins) return true;
  if (nb2 > kPdfLdsBins) return false;
  return L.cells >= 12 * nb2 || (L.patches && L.most >= nb2);
}

template <class T>
static DiagArgs<T> to_dargs(const LaunchDiag& L) {
  DiagArgs<T> a;
  a.pool = static_cast<const T*>(L.pool);
  a.patches = L.patches;
  a.single = L.single;
  a.gamma = L.gamma;
  a.nbins = L.nbins;
  a.lo = L.lo;
  a.w = L.w;
  a.counts = L.counts;
  a.lds = pdf_lds(L);
  a.axis = L.axis;
  a.chunks = L.chunks;
  a.dnx = FastDiv(uint32_t(L.single.n[0]));
  a.dny = FastDiv(uint32_t(L.single.n[1]));
  a.rho_lo = L.rho_lo;
  a.drho = L.drho;
  a.dx_axis = L.dx_axis;
  a.partials = L.partials;
  a.out = L.out;
  return a;
}

template <class T>
static hipError_t launch_pdf_t(const LaunchDiag& L, hipStream_t st) {
  const DiagArgs<T> a = to_dargs<T>(L);
  const int nb2 = L.nbins + 2;
  hipLaunchKernelGGL(zero_u64_kernel, dim3(unsigned(std::min(1024, (nb2 + kDiagBlock - 1) / kDiagBlock))),
                     dim3(kDiagBlock), 0, st, L.counts, nb2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = a.lds ? size_t(nb2) * sizeof(unsigned int) : 0;
  const bool wide = a.lds && nb2 > kPdfNarrowBins;
  dim3 grid;
  if (L.patches) {
    // wide counters: as many workgroups as the largest patch takes (smaller
    // ones leave theirs at once), at most kPdfWideBlocks and 64 K in all.  With
    // one a patch, 9000 bins: a patch of 256^3 FP32 cells 9170 instead of 76 us,
    // beside 1000 of 16^3 9200 instead of 160, 300 of 64^3 257 instead of 200
    const int64_t w = std::min<int64_t>({L.most / (12 * nb2), kPdfWideBlocks, 65536 / L.npatch});
    grid = dim3(wide ? unsigned(std::max<int64_t>(1, w)) : kPdfPatchBlocks, unsigned(L.npatch));
  } else {
    // up to one workgroup for 8192 cells and for 12 cells per counter (256^3
    // cells: 16 bins 64 -> 45 us with half the workgroups of 4096 cells, 1000
    // bins 100 -> 55 us), or one per CU if that is more (256 of them; all of
    // the wide counters').  In any case 1024 cells to a workgroup, the only
    // bound with counters in memory
    int64_t b = kPdfMaxBlocks;
    if (wide)
      b = kPdfWideBlocks;
    else if (a.lds)
      b = std::max<int64_t>(std::min(L.cells / (12 * nb2), L.cells / 8192), kPdfWideBlocks);
    b = std::min<int64_t>({b, kPdfMaxBlocks, (L.cells + 4 * kDiagBlock - 1) / (4 * kDiagBlock)});
    grid = dim3(unsigned(std::max<int64_t>(1, b)));
  }
  auto run = [&](auto narrow_kernel, auto wide_kernel) {
    if (wide)
      hipLaunchKernelGGL(wide_kernel, grid, dim3(1024), lds, st, a);
    else
      hipLaunchKernelGGL(narrow_kernel, grid, dim3(kDiagBlock), lds, st, a);
  };
  switch (L.quantity) {
    case kQRho: run(pdf_kernel<T, kQRho, kDiagBlock>, pdf_kernel<T, kQRho, 1024>); break;
    case kQPressure: run(pdf_kernel<T, kQPressure, kDiagBlock>, pdf_kernel<T, kQPressure, 1024>); break;
    case kQSpeed: run(pdf_kernel<T, kQSpeed, kDiagBlock>, pdf_kernel<T, kQSpeed, 1024>); break;
    case kQMach: run(pdf_kernel<T, kQMach, kDiagBlock>, pdf_kernel<T, kQMach, 1024>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_diag_pdf(const LaunchDiag& L, hipStream_t st) {
  if (L.nbins < 1 || L.nbins > kPdfMaxBins) return hipErrorInvalidValue;
  return L.fp64 ? launch_pdf_t<double>(L, st) : launch_pdf_t<float>(L, st);
}

template <class T>
static hipError_t launch_profile_t(const LaunchDiag& L, hipStream_t st) {
  const DiagArgs<T> a = to_dargs<T>(L);
  const int ns = L.single.n[L.axis];
  if (L.axis == 0)
    hipLaunchKernelGGL(profile_xslab_kernel<T>,
                       dim3(unsigned(L.chunks), unsigned((ns + xslab_width(ns) - 1) / xslab_width(ns))),
                       dim3(kXslabBlock), 0, st, a);
  else
    hipLaunchKernelGGL(profile_slab_kernel<T>, dim3(unsigned(L.chunks), unsigned(ns)),
                       dim3(kDiagBlock), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const double cells = double(L.single.n[0]) * L.single.n[1] * L.single.n[2];
  hipLaunchKernelGGL(profile_final_kernel, dim3(1), dim3(kFinalBlock), 0, st, L.partials, ns,
                     L.chunks, cells / ns, L.dx_axis, L.out);
  return hipGetLastError();
}

template <class T>
static hipError_t launch_spectrum_t(const LaunchDiag& L, hipStream_t st) {
  const DiagArgs<T> a = to_dargs<T>(L);
  FftPlan sp;
  if (!make_fft_plan(L.single.n[0], sp)) return hipErrorInvalidValue;
  // x-lines per pass: as many pairs as fill the buffer, but no fewer than 512
  // groups where there are lines for them (two workgroups per CU)
  const int n = sp.n;
  const int64_t nlines = int64_t(L.single.n[1]) * L.single.n[2];
  const int P = 2 * int(std::max<int64_t>(
                        1, std::min<int64_t>(kSpecElems / (3 * n), (nlines + 1023) / 1024)));
  // workgroups: about 16 passes each (a workgroup forms the twiddles and ends
  // in a partial spectrum), 512 to kSpecBlocks of them (L.chunks)
  const int64_t groups = (nlines + P - 1) / P;
  const int blocks = int(std::min<int64_t>(std::min<int64_t>(groups, L.chunks),
                                           std::max<int64_t>(512, groups / 16)));
  // (the lines, or at the end kSpecBlock sums)
  const size_t lds = size_t(n + std::max(fft_lds(3 * P / 2 * n), kSpecBlock / 2)) * sizeof(double2);
  hipLaunchKernelGGL((spectrum_kernel<T>), dim3(unsigned(blocks)), dim3(kSpecBlock), lds, st, a,
                     sp, P, FastDiv(uint32_t(n)), FastDiv(uint32_t(L.single.n[1])));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const double lines = double(L.single.n[1]) * L.single.n[2];
  hipLaunchKernelGGL(spectrum_final_kernel, dim3(unsigned(sp.n / 2 + 1)), dim3(kDiagBlock), 0,
                     st, L.partials, blocks, sp.n, lines, L.out);
  return hipGetLastError();
}

hipError_t launch_diag_spectrum(const LaunchDiag& L, hipStream_t st) {
  const int n = L.single.n[0];
  if (L.patches || n < 2 || n > kSpecMaxLen || L.chunks < 1) return hipErrorInvalidValue;
  return L.fp64 ? launch_spectrum_t<double>(L, st) : launch_spectrum_t<float>(L, st);
}

hipError_t launch_diag_profile(const LaunchDiag& L, hipStream_t st) {
  if (L.axis < 0 || L.axis > 2 || L.chunks < 1 || L.patches) return hipErrorInvalidValue;
  return L.fp64 ? launch_profile_t<double>(L, st) : launch_profile_t<float>(L, st);
}

}  // namespace hydro
