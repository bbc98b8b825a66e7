// amr.hip -- operators around the batched patches for adaptive refinement
// (ratio 2): the stored ghost layers, conservative restriction and
// MC-limited conservative prolongation.
//
// The paper's codes run the hydrodynamics on adaptively refined grids (its
// description of their capabilities) without fixing these operators; they
// are the standard conservative ones.  The sweep kernels apply the physical
// boundary conditions on the fly and never read stored ghosts, so these are
// for the layers around the step: regridding, coarse-fine data exchange,
// output and checkpoints.  Every operator is one HBM-bound pass over the
// cells it writes, and each reproduces its definition's floating-point
// operations in order, so results are bitwise those of a plain evaluation:
//   * ghosts: stored index i of an axis maps to interior i (inside), to
//     i mod n (periodic), to the edge cell (outflow) or to the mirror image
//     with period 2n (reflect: ghost -k copies cell k-1), axis by axis; the
//     momentum normal to a reflecting side is negated;
//   * restriction: coarse = (sum of the 8 children in (dz, dy, dx) order)/8;
//   * prolongation: child = ((U_c + s_x D_x) + s_y D_y) + s_z D_z with
//     s = -1/4 or +1/4 and D the monotonised-central slope from the two
//     coarse neighbours along each axis; for the ghosts of a subcycled fine
//     step, U_c is first interpolated in time, U_old + theta (U - U_old);
//   * flux registers: the flux of a sweep through the coarse-fine faces,
//     evaluated from the cells the sweep reads with the sweep's own
//     arithmetic (euler.hpp), so a coarse register holds the very flux the
//     coarse update applied; fine fluxes are averaged over the 2 x 2 fine
//     faces of a coarse face in (t2, t1) order;
//   * refluxing: the uncovered coarse cell across a coarse-fine face trades
//     the coarse flux for the fine one, U += (R_c - R_f)/dx on a patch's low
//     side and (R_f - R_c)/dx on its high side (Berger & Colella 1989).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "euler.hpp"
#include "launch.hpp"

namespace hydro {

constexpr int kAmrBlock = 256;

// Interior source of stored index i (interior 0..n-1) along one axis.
__device__ __forceinline__ int ghost_src(int i, int n, int bclo, int bchi, bool& flip) {
  if (i >= 0 && i < n) return i;
  const int bc = i < 0 ? bclo : bchi;
  if (bc == kBcPeriodic) {
    const int w = i < 0 ? i + n : i - n;
    if (w >= 0 && w < n) return w;  // at most one period away: no division
    const int m = i % n;
    return m < 0 ? m + n : m;
  }
  if (bc == kBcOutflow) return i < 0 ? 0 : n - 1;
  flip = true;
  const int k = i < 0 ? -i - 1 : i - n;  // distance beyond the edge
  const int m = k % (2 * n);
  const int d = m < n ? m : 2 * n - 1 - m;
  return i < 0 ? d : n - 1 - d;
}

template <class T>
struct AmrArgs {
  T* pool;
  const PatchDev* patches;  // null: single grid
  PatchDev single;
  int ng;                   // single grid: stored ghost layers
  int bc[6];
  AmrLink links[kAmrLinksPerLaunch];
  T* fpool;                 // fine side of the links
  const PatchDev* fpatches;
  int finset;
  const T* cold;            // prolongation: coarse data at the start of the step
  int margin;               // snapshot: coarse cells around each covered box
  double theta;
  double* reg;
  int64_t nreg;
  int link0, maxface;
  int axis, side, fine;
  double dt, weight, gamma, grav;
  const T* face;
  int nface;
  const AmrLink* dlinks;
};

// Link l of a launch.
template <class T>
__device__ __forceinline__ AmrLink link_of(const AmrArgs<T>& a, int l) {
  return a.dlinks ? a.dlinks[l] : a.links[l];
}

// Fine patch of a link: the table entry, or the patch inside a ghost-free
// stored box whose outer `inset` layers are its ghost shell.
__device__ __forceinline__ PatchDev fine_patch(const PatchDev* t, int i, int inset) {
  PatchDev F = t[i];
  if (inset) {
    F.base0 += int64_t(inset) * (1 + int64_t(F.sy) + int64_t(F.sz));
    for (int a = 0; a < 3; ++a) F.n[a] -= 2 * inset;
    F.ng = inset;
  }
  return F;
}

// Element stride of an axis, and the two transverse axes of a sweep along
// `axis` in ascending order.
__device__ __forceinline__ int64_t axis_stride(const PatchDev& P, int a) {
  return a == 0 ? 1 : a == 1 ? int64_t(P.sy) : int64_t(P.sz);
}
// Component a of a 3-vector by selects (a runtime index into a local array
// would put the array in scratch memory).
template <class U>
__device__ __forceinline__ U sel3(int a, U x, U y, U z) {
  return a == 0 ? x : a == 1 ? y : z;
}
__device__ __forceinline__ int ext(const PatchDev& P, int a) {
  return sel3(a, P.n[0], P.n[1], P.n[2]);
}
__device__ __forceinline__ double width(const PatchDev& P, int a) {
  return sel3(a, P.dx[0], P.dx[1], P.dx[2]);
}
__device__ __forceinline__ int t1_of(int axis) { return axis == 0 ? 1 : 0; }
__device__ __forceinline__ int t2_of(int axis) { return axis == 2 ? 1 : 2; }

// Every stored ghost cell of the grid (y = 0) or of patch blockIdx.y, from
// the interior, in the order of memory: the slabs below the interior along z;
// per interior slab its rows below along y, the g cells at either end of
// each interior row, and its rows above; the slabs above.  Only ghost cells
// are visited, one per thread and trip (five independent loads, then five
// stores) at 32-bit offsets from the stored corner.
//
// What bounds the fill are the row ends: runs of g cells, often in lines of
// their own, written in parts of a 64-byte sector.  Such writes of 16 or 32
// bytes take 2.6 to 3.9 times those of a whole sector, about 0.044 ns each over
// the chip; the fill below of padded rows makes 7.4e7 of them (3.2 of its
// 5.2 ms), 3.0e7 of whole sectors (0.5 ms) and reads 8.1 GB.  The stores go past the caches: nothing here reads them again.
// 1024 64^3 and 1024 32^3 patches, against a walk over every stored cell
// with plain stores and 64-bit offsets: 4 FP32 layers, rows back to back
// 3.44 -> 2.07 ms, padded to 128-byte lines 5.1 -> 5.2 ms (4.7 to 5.4 with
// where the pool lies); FP64, padded, 5.8 -> 5.7 ms.
template <class T>
__global__ void __launch_bounds__(kAmrBlock) fill_ghosts_kernel(AmrArgs<T> a) {
  const PatchDev P = a.patches ? a.patches[blockIdx.y] : a.single;
  const int g = a.patches ? P.ng : a.ng;
  const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
  const unsigned g2 = 2u * unsigned(g), sx = unsigned(nx) + g2, sy = unsigned(ny) + g2;
  const unsigned below = unsigned(g) * sy * sx;        // cells of g whole slabs
  const unsigned edge = unsigned(g) * sx, ends = unsigned(ny) * g2;
  const unsigned slab = 2u * edge + ends;              // ghost cells of an interior slab
  const unsigned total = 2u * below + unsigned(nz) * slab;  // a stored patch holds < 2^32 cells
  T* p0 = a.pool + P.base0 - int64_t(g) * (1 + int64_t(P.sy) + int64_t(P.sz));
  for (unsigned c = blockIdx.x * kAmrBlock + threadIdx.x; c < total;
       c += gridDim.x * kAmrBlock) {
    int i, j, k;
    const unsigned m = c - below;
    if (c < below || m >= unsigned(nz) * slab) {
      const unsigned e = c < below ? c : m - unsigned(nz) * slab;
      const unsigned row = e / sx, kk = row / sy;
      i = int(e - row * sx) - g;
      j = int(row - kk * sy) - g;
      k = c < below ? int(kk) - g : nz + int(kk);
    } else {
      const unsigned kk = m / slab, r = m - kk * slab;
      k = int(kk);
      if (r < edge || r >= edge + ends) {
        const unsigned e = r < edge ? r : r - edge - ends;
        const unsigned row = e / sx;
        i = int(e - row * sx) - g;
        j = r < edge ? int(row) - g : ny + int(row);
      } else {
        const unsigned row = (r - edge) / g2, q = r - edge - row * g2;
        i = int(q) < g ? int(q) - g : nx + int(q) - g;
        j = int(row);
      }
    }
    bool fx = false, fy = false, fz = false;
    const int si = ghost_src(i, nx, a.bc[0], a.bc[1], fx);
    const int sj = ghost_src(j, ny, a.bc[2], a.bc[3], fy);
    const int sk = ghost_src(k, nz, a.bc[4], a.bc[5], fz);
    // a plane is below 4 GiB: element offsets from its corner fit 32 bits
    const unsigned src = unsigned(si + g) + unsigned(sj + g) * unsigned(P.sy) +
                         unsigned(sk + g) * unsigned(P.sz);
    const unsigned dst = unsigned(i + g) + unsigned(j + g) * unsigned(P.sy) +
                         unsigned(k + g) * unsigned(P.sz);
    T v[5];
#pragma unroll
    for (int w = 0; w < 5; ++w) v[w] = (p0 + w * P.plane)[src];
    if (fx) v[1] = -v[1];
    if (fy) v[2] = -v[2];
    if (fz) v[3] = -v[3];
#pragma unroll
    for (int w = 0; w < 5; ++w) __builtin_nontemporal_store(v[w], p0 + w * P.plane + dst);
  }
}

// Coarse cells covered by the fine patch of link blockIdx.y.
template <class T>
__global__ void __launch_bounds__(kAmrBlock) restrict_kernel(AmrArgs<T> a) {
  const AmrLink L = link_of(a, int(blockIdx.y));
  const PatchDev F = fine_patch(a.fpatches, L.fine, a.finset), C = a.patches[L.coarse];
  const unsigned cx = unsigned(F.n[0] / 2), cxy = cx * unsigned(F.n[1] / 2);
  const unsigned total = cxy * unsigned(F.n[2] / 2);
  const T* f0 = a.fpool + F.base0;
  T* c0 = a.pool + C.base0;
  if (blockIdx.x * kAmrBlock >= total) return;
  for (unsigned c = blockIdx.x * kAmrBlock + threadIdx.x; c < total;
       c += gridDim.x * kAmrBlock) {
    const unsigned k = c / cxy, rem = c - k * cxy;
    const unsigned j = rem / cx, i = rem - j * cx;
    const int64_t fb = int64_t(2 * i) + int64_t(2 * j) * F.sy + int64_t(2 * k) * F.sz;
    const int64_t cb = int64_t(L.ox + int(i)) + int64_t(L.oy + int(j)) * C.sy +
                       int64_t(L.oz + int(k)) * C.sz;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const T* f = f0 + fb + v * F.plane;
      double s = 0.0;
      bool first = true;
#pragma unroll
      for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
          for (int dx = 0; dx < 2; ++dx) {
            const double x = double(f[dx + dy * F.sy + dz * F.sz]);
            s = first ? x : s + x;
            first = false;
          }
      c0[cb + v * C.plane] = T(s * 0.125);
    }
  }
}

// Monotonised-central slope from one-sided differences a and b: zero unless
// both are strictly positive or both strictly negative (a sign test: a
// product of two tiny differences could underflow to zero).
__device__ __forceinline__ double mc_slope(double a, double b) {
  const double m = fmin(fmin(2.0 * fabs(a), 2.0 * fabs(b)), 0.5 * fabs(a + b));
  const bool same = (a > 0.0 && b > 0.0) || (a < 0.0 && b < 0.0);
  return same ? copysign(m, a) : 0.0;
}

// Two x-neighbours at p (element pair; PAIR: aligned to it, one access).
template <class T>
struct alignas(2 * sizeof(T)) Pair {
  T a, b;
};
template <bool PAIR, class T>
__device__ __forceinline__ void store_pair(T* p, T a, T b) {
  if (PAIR) {
    *reinterpret_cast<Pair<T>*>(p) = Pair<T>{a, b};
  } else {
    p[0] = a;
    p[1] = b;
  }
}

// Whether the x pairs (2i, 2i + 1) of a patch start on pairs of elements in
// every row and plane (the pool is 16-byte aligned).
__device__ __forceinline__ bool pairs_aligned(const PatchDev& F) {
  return ((F.base0 | F.plane | F.sy | F.sz) & 1) == 0;
}

// Link and workgroup of a link launch: with a grid of (bx, n) workgroups,
// dispatched round robin over the eight XCDs, the workgroups of one link are
// given to one XCD, whose L2 then holds the coarse lines they share (the
// level step on 338 patches 2.97 -> 2.86 ms).  Workgroups past the last
// multiple of eight links keep their place.
__device__ __forceinline__ void link_block(int& link, unsigned& bx) {
  const unsigned G = gridDim.x, n8 = gridDim.y & ~7u, b = blockIdx.y * G + blockIdx.x;
  if (b < n8 * G) {
    const unsigned r = b >> 3, q = r / G;
    link = int(q * 8 + (b & 7));
    bx = r - q * G;
  } else {
    link = int(blockIdx.y);
    bx = blockIdx.x;
  }
}

// Fine cells (interior, or with SHELL the stored ghost shell) of a link, one
// coarse parent per thread, of variable blockIdx.z (SHELL) or of all five: per
// variable the parent's value and its three limited slopes are formed once and
// give its children, written as x pairs (PAIR: one access each).  Fine extents are even, so a parent's children are all
// inside or all outside the interior, and only with an odd number of ghost
// layers (ODD) can some of them lie beyond the stored shell.
//
// The interior's parents are a box.  The shell's are walked as three parts:
// whole planes of parents below and above the interior's along z; within its
// z range whole rows below and above it along y; within both the parents
// below and above it along x (rows of ceil(g/2) + ceil(g/2)).
//
// The interior is bound by instruction issue (FP64 slopes in the definition's
// order), the shell by its x ends (parts of 64-byte sectors, as the ghost
// fill).  Against one test and one 64-bit offset per child over the whole box
// of parents (2047 instructions a thread, now about 850): 128 FP32 links of
// 32^3 cells, interior 51 -> 31 us, 4 ghost layers 137 -> 104 us; the level
// step's 338 shells of 4 layers 209 -> 167 us, interpolated 272 -> 245 us (now, a
// variable to a thread, 146 and 175).
//
// A shell has few parents; with a variable to a thread it has five times the
// waves, each of fewer registers.  FP32 links of 64^3 cells, 2 layers: one link
// 7.9 -> 4.6 us, 16 22.4 -> 14.5, 64 87 -> 76 (4 layers 111 -> 102).  The interior
// of 64 links takes 155 us with all five, 163 with one.
template <class T, bool COLD, bool PAIR, bool ODD, bool SHELL>
__device__ void prolong_link(const AmrArgs<T>& a, const AmrLink& L, const PatchDev& F,
                             const PatchDev& C, unsigned bx) {
  const int g = SHELL ? F.ng : 0;  // a shell without stored ghosts has no cells
  const int h = (g + 1) >> 1;  // parents beyond the interior's on each side
  const unsigned ix = unsigned(F.n[0]) >> 1, iy = unsigned(F.n[1]) >> 1,
                 iz = unsigned(F.n[2]) >> 1;  // the interior's parents
  const unsigned o = 2u * unsigned(h), px = ix + o, py = iy + o;
  const unsigned zpart = o * py * px, ypart = iz * o * px;
  const unsigned total = SHELL ? zpart + ypart + iz * iy * o : iz * iy * ix;
  // t-th parent outside [0, I) along an axis: -h .. -1, then I ..
  auto outside = [&](unsigned t, unsigned I) {
    return int(t) < h ? int(t) - h : int(I) + int(t) - h;
  };
  // wave-uniform bases and one 32-bit byte offset per cell (a plane is below
  // 4 GiB): the coarse base is the lowest neighbour of the lowest parent, the
  // fine base the first cell written.  With an odd number of layers the lowest
  // parents' first children lie before it: their offsets wrap, and those of the
  // cells that are written come out right modulo 2^32
  const int64_t corner = C.base0 + (L.ox - h - 1) + int64_t(L.oy - h - 1) * C.sy +
                         int64_t(L.oz - h - 1) * C.sz;
  const T* c0 = a.pool + corner;
  const T* o0 = COLD ? a.cold + corner : nullptr;
  T* f0 = a.fpool + F.base0 - g * (1 + int64_t(F.sy) + int64_t(F.sz));
  const unsigned csy = unsigned(C.sy) * sizeof(T), csz = unsigned(C.sz) * sizeof(T);
  const unsigned fsy = unsigned(F.sy) * sizeof(T), fsz = unsigned(F.sz) * sizeof(T);
  auto at = [](const T* p, unsigned b) {
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + b);
  };
  const double th = a.theta;
  for (unsigned c = bx * kAmrBlock + threadIdx.x; c < total; c += gridDim.x * kAmrBlock) {
    int pi, pj, pk;
    if (!SHELL) {
      const unsigned row = c / ix, kk = row / iy;
      pi = int(c - row * ix);
      pj = int(row - kk * iy);
      pk = int(kk);
    } else if (c < zpart) {
      const unsigned row = c / px, kk = row / py;
      pi = int(c - row * px) - h;
      pj = int(row - kk * py) - h;
      pk = outside(kk, iz);
    } else if (c < zpart + ypart) {
      const unsigned d = c - zpart, row = d / px, kk = row / o;
      pi = int(d - row * px) - h;
      pj = outside(row - kk * o, iy);
      pk = int(kk);
    } else {
      const unsigned d = c - zpart - ypart, row = d / o, kk = row / iy;
      pi = outside(d - row * o, ix);
      pj = int(row - kk * iy);
      pk = int(kk);
    }
    const unsigned pc = unsigned(pi + h + 1) * unsigned(sizeof(T)) + unsigned(pj + h + 1) * csy +
                        unsigned(pk + h + 1) * csz;
    const unsigned fc = unsigned(2 * pi + g) * unsigned(sizeof(T)) + unsigned(2 * pj + g) * fsy +
                        unsigned(2 * pk + g) * fsz;
    constexpr int NV = SHELL ? 1 : 5;  // variables v0 .. v0 + NV - 1
    const int v0 = SHELL ? int(blockIdx.z) : 0;
    double u[NV][7];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const T* q = c0 + (v0 + v) * C.plane;
      const T* qo = COLD ? o0 + (v0 + v) * C.plane : nullptr;
      // coarse value at byte offset b, interpolated in time when a start copy is given
      auto cv = [&](unsigned b) {
        if constexpr (!COLD) {
          return double(*at(q, b));
        } else {
          const double w = double(*at(qo, b));
          return w + th * (double(*at(q, b)) - w);
        }
      };
      u[v][0] = cv(pc);
      u[v][1] = cv(pc - unsigned(sizeof(T)));
      u[v][2] = cv(pc + unsigned(sizeof(T)));
      u[v][3] = cv(pc - csy);
      u[v][4] = cv(pc + csy);
      u[v][5] = cv(pc - csz);
      u[v][6] = cv(pc + csz);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double w = u[v][0];
      const double dx = mc_slope(w - u[v][1], u[v][2] - w);
      const double dy = mc_slope(w - u[v][3], u[v][4] - w);
      const double dz = mc_slope(w - u[v][5], u[v][6] - w);
      T* fv = f0 + (v0 + v) * F.plane;
      const double x0 = w + -0.25 * dx, x1 = w + 0.25 * dx;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double oy = (r & 1) ? 0.25 : -0.25, oz = (r >> 1) ? 0.25 : -0.25;
        const T y0 = T((x0 + oy * dy) + oz * dz), y1 = T((x1 + oy * dy) + oz * dz);
        const unsigned fr = fc + (r & 1) * fsy + (r >> 1) * fsz;
        auto cell = [&](unsigned b) { return const_cast<T*>(at(fv, b)); };
        if (!ODD) {
          store_pair<PAIR>(cell(fr), y0, y1);
        } else {
          const int i = 2 * pi, j = 2 * pj + (r & 1), k = 2 * pk + (r >> 1);
          if (j < -g || j >= F.n[1] + g || k < -g || k >= F.n[2] + g) continue;
          if (i >= -g) *cell(fr) = y0;
          if (i + 1 < F.n[0] + g) *cell(fr + unsigned(sizeof(T))) = y1;
        }
      }
    }
  }
}

template <class T, bool COLD, bool SHELL>
__global__ void __launch_bounds__(kAmrBlock) prolong_kernel(AmrArgs<T> a) {
  int l;
  unsigned bx;
  link_block(l, bx);
  const AmrLink L = link_of(a, l);
  const PatchDev F = fine_patch(a.fpatches, L.fine, a.finset), C = a.patches[L.coarse];
  if (SHELL && (F.ng & 1))
    prolong_link<T, COLD, false, SHELL, SHELL>(a, L, F, C, bx);
  else if (pairs_aligned(F))
    prolong_link<T, COLD, true, false, SHELL>(a, L, F, C, bx);
  else
    prolong_link<T, COLD, false, false, SHELL>(a, L, F, C, bx);
}

// Copy of the coarse cells within a.margin of the box link blockIdx.y
// covers (every cell its ghost prolongation reads), into a.cold at the
// pool's offsets.  Boxes of neighbouring links may overlap; they copy the
// same values.
template <class T>
__global__ void __launch_bounds__(kAmrBlock) snapshot_kernel(AmrArgs<T> a) {
  const AmrLink L = link_of(a, int(blockIdx.y));
  const PatchDev F = fine_patch(a.fpatches, L.fine, a.finset), C = a.patches[L.coarse];
  const int m = a.margin;
  const unsigned bx = unsigned(F.n[0] / 2 + 2 * m), bxy = bx * unsigned(F.n[1] / 2 + 2 * m);
  const unsigned total = bxy * unsigned(F.n[2] / 2 + 2 * m);
  const T* c0 = a.pool + C.base0;
  T* o0 = const_cast<T*>(a.cold) + C.base0;
  for (unsigned c = blockIdx.x * kAmrBlock + threadIdx.x; c < total;
       c += gridDim.x * kAmrBlock) {
    const unsigned kk = c / bxy, rem = c - kk * bxy;
    const unsigned jj = rem / bx;
    const int64_t cell = int64_t(L.ox - m + int(rem - jj * bx)) +
                         int64_t(L.oy - m + int(jj)) * C.sy + int64_t(L.oz - m + int(kk)) * C.sz;
#pragma unroll
    for (int v = 0; v < 5; ++v) o0[cell + v * C.plane] = c0[cell + v * C.plane];
  }
}

// Flux through the face between cells f - 1 and f along `axis` at
// transverse indices (i1, i2), from the four cells f - 2 .. f + 1 exactly as
// a sweep computes it (interior cells: the full gravity half kick).
// Returned in the sweep frame (rho, m_n, m_t1, m_t2, E); lab_var maps a
// sweep-frame component to its lab index (kept out of the local array so
// that it stays in registers).
__device__ __forceinline__ int lab_var(int axis, int v) {
  return v == 1 ? 1 + axis : v == 2 ? 1 + t1_of(axis) : v == 3 ? 1 + t2_of(axis) : v;
}

template <class T>
__device__ __forceinline__ void face_flux(const T* p0, const PatchDev& P, int axis, int f,
                                          int i1, int i2, const SweepConst<T>& k,
                                          double out[5]) {
  const int a1 = t1_of(axis), a2 = t2_of(axis);
  const int64_t sd = axis_stride(P, axis);
  const int64_t c0 = int64_t(f) * sd + int64_t(i1) * axis_stride(P, a1) +
                     int64_t(i2) * axis_stride(P, a2);
  Prim<T> W[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const T* q = p0 + c0 + (m - 2) * sd;
    Cons<T> U;
    U.r = q[0];
    U.mn = q[(1 + axis) * P.plane];
    U.mt1 = q[(1 + a1) * P.plane];
    U.mt2 = q[(1 + a2) * P.plane];
    U.e = q[4 * P.plane];
    W[m] = to_prim(U, k);
  }
  Prim<T> Wm0, Wp0, Wm1, Wp1;
  face_states(W[0], W[1], W[2], k, k.gk, Wm0, Wp0);  // cell f - 1
  face_states(W[1], W[2], W[3], k, k.gk, Wm1, Wp1);  // cell f
  const Cons<T> F = hllc(Wp0, Wm1, k);
  out[0] = double(F.r);
  out[1] = double(F.mn);
  out[2] = double(F.mt1);
  out[3] = double(F.mt2);
  out[4] = double(F.e);
}

// Flux registers of link blockIdx.y, side blockIdx.z, along a.axis: coarse
// faces (a.fine = 0) or the means of the fine faces (a.fine = 1), times
// a.weight, added to the register.
template <class T>
__global__ void __launch_bounds__(kAmrBlock) flux_reg_kernel(AmrArgs<T> a) {
  const AmrLink L = link_of(a, int(blockIdx.y));
  const int side = int(blockIdx.z);
  const PatchDev F = fine_patch(a.fpatches, L.fine, a.finset);
  const int axis = a.axis, a1 = t1_of(axis), a2 = t2_of(axis);
  const int m1 = ext(F, a1) / 2, m2 = ext(F, a2) / 2;
  const int nface = m1 * m2;
  double* reg = a.reg + (a.fine ? a.nreg : 0) +
                (((int64_t(a.link0) + blockIdx.y) * 3 + axis) * 2 + side) * a.maxface * 5;
  const PatchDev C = a.patches[L.coarse];
  const SweepConst<T> k = make_const<T>(a.dt, a.fine ? width(F, axis) : width(C, axis),
                                        a.gamma, a.grav);
  double acc[5];
  if (!a.fine) {
    const int f = sel3(axis, L.ox, L.oy, L.oz) + (side ? ext(F, axis) / 2 : 0);
    const int c1 = sel3(a1, L.ox, L.oy, L.oz), c2 = sel3(a2, L.ox, L.oy, L.oz);
    for (int fc = blockIdx.x * kAmrBlock + threadIdx.x; fc < nface;
         fc += gridDim.x * kAmrBlock) {
      const int j1 = fc % m1, j2 = fc / m1;
      face_flux(a.pool + C.base0, C, axis, f, c1 + j1, c2 + j2, k, acc);
#pragma unroll
      for (int v = 0; v < 5; ++v) reg[int64_t(fc) * 5 + lab_var(axis, v)] += a.weight * acc[v];
    }
  } else if (axis == 0) {
    // x faces: sixteen lanes per coarse face, lane 4q + m on cell m of the
    // 4-cell stencil of fine face q (t2, t1 offsets (q >> 1, q & 1)), so the
    // four lanes of a stencil read one contiguous run.  Each lane forms its
    // cell's primitives; the face states of cells f - 1 (m = 1) and f (m = 2)
    // take their neighbours' primitives by shuffle, and lane m = 2 forms the
    // flux from exactly the operands a sweep uses.  The segment's first lane
    // sums the four fine fluxes in the order (0,0), (0,1), (1,0), (1,1).
    const int f = side ? ext(F, 0) : 0;
    const int l = threadIdx.x & 15, q = l >> 2, m = l & 3;
    for (int t = blockIdx.x * kAmrBlock + threadIdx.x; t < 16 * nface;
         t += gridDim.x * kAmrBlock) {
      const int fc = t >> 4;
      const int j1 = fc % m1, j2 = fc / m1;
      const int64_t cell = int64_t(f - 2 + m) + int64_t(2 * j1 + (q & 1)) * F.sy +
                           int64_t(2 * j2 + (q >> 1)) * F.sz;
      const T* c = a.fpool + F.base0 + cell;
      Cons<T> U;
      U.r = c[0];
      U.mn = c[F.plane];
      U.mt1 = c[2 * F.plane];
      U.mt2 = c[3 * F.plane];
      U.e = c[4 * F.plane];
      const Prim<T> W = to_prim(U, k);
      // neighbours m - 1 and m + 1 within the stencil (the ends take
      // unused values)
      Prim<T> Wl, Wr;
      Wl.r = __shfl(W.r, l - 1, 16);
      Wl.u = __shfl(W.u, l - 1, 16);
      Wl.t1 = __shfl(W.t1, l - 1, 16);
      Wl.t2 = __shfl(W.t2, l - 1, 16);
      Wl.p = __shfl(W.p, l - 1, 16);
      Wl.ri = T(0);
      Wr.r = __shfl(W.r, l + 1, 16);
      Wr.u = __shfl(W.u, l + 1, 16);
      Wr.t1 = __shfl(W.t1, l + 1, 16);
      Wr.t2 = __shfl(W.t2, l + 1, 16);
      Wr.p = __shfl(W.p, l + 1, 16);
      Wr.ri = T(0);
      Prim<T> Wm, Wp;
      face_states(Wl, W, Wr, k, k.gk, Wm, Wp);
      // lane m = 2 takes W+ of cell f - 1 from lane m = 1
      Prim<T> L1;
      L1.r = __shfl(Wp.r, l - 1, 16);
      L1.u = __shfl(Wp.u, l - 1, 16);
      L1.t1 = __shfl(Wp.t1, l - 1, 16);
      L1.t2 = __shfl(Wp.t2, l - 1, 16);
      L1.p = __shfl(Wp.p, l - 1, 16);
      L1.ri = T(0);
      const Cons<T> Fx = hllc(L1, Wm, k);
      const double fl[5] = {double(Fx.r), double(Fx.mn), double(Fx.mt1), double(Fx.mt2),
                            double(Fx.e)};
      double s5[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const double x0 = __shfl(fl[v], 2, 16), x1 = __shfl(fl[v], 6, 16);
        const double x2 = __shfl(fl[v], 10, 16), x3 = __shfl(fl[v], 14, 16);
        s5[v] = ((x0 + x1) + x2) + x3;
      }
      if (l == 0) {
#pragma unroll
        for (int v = 0; v < 5; ++v)
          reg[int64_t(fc) * 5 + lab_var(0, v)] += a.weight * (0.25 * s5[v]);
      }
    }
  } else {
    // four consecutive lanes per coarse face, lane q on the fine face with
    // (t2, t1) offsets (q >> 1, q & 1); the group's first lane sums the four
    // in the order (0,0), (0,1), (1,0), (1,1).  Groups are whole: the block
    // size and the trip bound are multiples of 4.
    const int f = side ? ext(F, axis) : 0;
    const int q = threadIdx.x & 3;
    for (int t = blockIdx.x * kAmrBlock + threadIdx.x; t < 4 * nface;
         t += gridDim.x * kAmrBlock) {
      const int fc = t >> 2;
      const int j1 = fc % m1, j2 = fc / m1;
      face_flux(a.fpool + F.base0, F, axis, f, 2 * j1 + (q & 1), 2 * j2 + (q >> 1), k, acc);
      double s[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const double x0 = __shfl(acc[v], 0, 4), x1 = __shfl(acc[v], 1, 4);
        const double x2 = __shfl(acc[v], 2, 4), x3 = __shfl(acc[v], 3, 4);
        s[v] = ((x0 + x1) + x2) + x3;
      }
      if (q == 0) {
#pragma unroll
        for (int v = 0; v < 5; ++v)
          reg[int64_t(fc) * 5 + lab_var(axis, v)] += a.weight * (0.25 * s[v]);
      }
    }
  }
}
static_assert(kAmrBlock % 16 == 0, "whole lane groups per workgroup");

// Fine flux registers of link blockIdx.y, axis blockIdx.z / 2, side
// blockIdx.z mod 2, from the fine face fluxes that the sweeps wrote (sweep
// frame, a.face): one coarse face per thread, the mean of its four fine faces
// summed in (t2, t1) order, times a.weight.
template <class T>
__global__ void __launch_bounds__(kAmrBlock) flux_gather_kernel(AmrArgs<T> a) {
  const AmrLink L = link_of(a, int(blockIdx.y));
  const int axis = int(blockIdx.z >> 1), side = int(blockIdx.z & 1);
  const PatchDev F = fine_patch(a.fpatches, L.fine, a.finset);
  const int n1 = ext(F, t1_of(axis)), m1 = n1 / 2, nface = m1 * (ext(F, t2_of(axis)) / 2);
  double* reg = a.reg + a.nreg +
                (((int64_t(a.link0) + blockIdx.y) * 3 + axis) * 2 + side) * a.maxface * 5;
  const T* f = a.face + int64_t((L.fine * 3 + axis) * 2 + side) * 5 * a.nface;
  for (int fc = blockIdx.x * kAmrBlock + threadIdx.x; fc < nface; fc += gridDim.x * kAmrBlock) {
    const int j2 = fc / m1, j1 = fc - j2 * m1;
    const T* q = f + int64_t(2 * j2) * n1 + 2 * j1;
    double x[5][4];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const T* p = q + int64_t(v) * a.nface;
      x[v][0] = double(p[0]);
      x[v][1] = double(p[1]);
      x[v][2] = double(p[n1]);
      x[v][3] = double(p[n1 + 1]);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double s = ((x[v][0] + x[v][1]) + x[v][2]) + x[v][3];
      reg[int64_t(fc) * 5 + lab_var(axis, v)] += a.weight * (0.25 * s);
    }
  }
}

// Refluxing of link blockIdx.y across its a.side faces along a.axis.
template <class T>
__global__ void __launch_bounds__(kAmrBlock) reflux_kernel(AmrArgs<T> a) {
  const AmrLink L = link_of(a, int(blockIdx.y));
  const PatchDev F = fine_patch(a.fpatches, L.fine, a.finset);
  const PatchDev C = a.patches[L.coarse];
  const int axis = a.axis, a1 = t1_of(axis), a2 = t2_of(axis), side = a.side;
  const int m1 = ext(F, a1) / 2, m2 = ext(F, a2) / 2;
  const int nface = m1 * m2;
  const int od = sel3(axis, L.ox, L.oy, L.oz);
  const int c1 = sel3(a1, L.ox, L.oy, L.oz), c2 = sel3(a2, L.ox, L.oy, L.oz);
  const int64_t ro = (((int64_t(a.link0) + blockIdx.y) * 3 + axis) * 2 + side) * a.maxface * 5;
  const double* rc = a.reg + ro;
  const double* rf = a.reg + a.nreg + ro;
  const int c = side ? od + ext(F, axis) / 2 : od - 1;  // the uncovered coarse cell
  const double dx = width(C, axis);
  T* c0 = a.pool + C.base0;
  for (int fc = blockIdx.x * kAmrBlock + threadIdx.x; fc < nface; fc += gridDim.x * kAmrBlock) {
    const int j1 = fc % m1, j2 = fc / m1;
    const int64_t cell = int64_t(c) * axis_stride(C, axis) +
                         int64_t(c1 + j1) * axis_stride(C, a1) +
                         int64_t(c2 + j2) * axis_stride(C, a2);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double rcv = rc[int64_t(fc) * 5 + v], rfv = rf[int64_t(fc) * 5 + v];
      const double delta = side ? rfv - rcv : rcv - rfv;
      T* u = c0 + cell + v * C.plane;
      *u = T(double(*u) + delta / dx);
    }
  }
}

template <class T>
static AmrArgs<T> to_aargs(const LaunchAmr& L) {
  AmrArgs<T> a{};
  a.pool = static_cast<T*>(L.pool);
  a.patches = L.patches;
  a.single = L.single;
  a.ng = L.ng;
  for (int i = 0; i < 6; ++i) a.bc[i] = L.bc[i];
  // by-value links only without a device table (launch_amr caps them at
  // kAmrLinksPerLaunch); with one, nlinks may exceed the array
  if (!L.dlinks) {
    const int m = std::min<int32_t>(L.nlinks, kAmrLinksPerLaunch);
    for (int i = 0; i < m; ++i) a.links[i] = L.links[i];
  }
  a.fpool = L.fpool ? static_cast<T*>(L.fpool) : a.pool;
  a.fpatches = L.fpatches ? L.fpatches : L.patches;
  a.finset = L.finset;
  a.cold = static_cast<const T*>(L.cold);
  a.margin = L.margin;
  a.theta = L.theta;
  a.reg = L.reg;
  a.nreg = L.nreg;
  a.link0 = L.link0;
  a.maxface = L.maxface;
  a.axis = L.axis;
  a.side = L.side;
  a.fine = L.fine;
  a.dt = L.dt;
  a.weight = L.weight;
  a.gamma = L.gamma;
  a.grav = L.grav;
  a.face = static_cast<const T*>(L.face);
  a.nface = L.nface;
  a.dlinks = L.dlinks;
  return a;
}

struct LinkChunk {
  AmrLink l[kAmrLinksPerLaunch];
};

__global__ void upload_links_kernel(AmrLink* dst, LinkChunk src, int n) {
  const int i = int(threadIdx.x);
  if (i < n) dst[i] = src.l[i];
}

hipError_t launch_amr_upload(AmrLink* dst, const AmrLink* src, int32_t n, hipStream_t st) {
  for (int32_t b = 0; b < n; b += kAmrLinksPerLaunch) {
    LinkChunk c{};
    const int m = std::min<int32_t>(kAmrLinksPerLaunch, n - b);
    for (int i = 0; i < m; ++i) c.l[i] = src[b + i];
    hipLaunchKernelGGL(upload_links_kernel, dim3(1), dim3(kAmrLinksPerLaunch), 0, st, dst + b,
                       c, m);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

static_assert(sizeof(AmrArgs<double>) <= 4096, "AMR kernel arguments exceed 4 KiB");

static unsigned amr_blocks(int64_t cells) {
  return unsigned(std::max<int64_t>(1, std::min<int64_t>((cells + kAmrBlock - 1) / kAmrBlock,
                                                         kAmrMaxBlocks)));
}

template <class T>
static hipError_t launch_amr_t(const LaunchAmr& L, hipStream_t st) {
  const AmrArgs<T> a = to_aargs<T>(L);
  if (L.op == kAmrFill) {
    // four ghost cells per thread of the patch with the most; one in a launch of
    // few workgroups, which takes as long as one thread's trips (a patch of 16^3
    // FP32 cells and 2 layers 5.5 -> 3.4 us, 100 of 16^3 and 1 layer 7.3 -> 6.0;
    // above it 1000 of 16^3 and 2 layers 57 us with four, 65 with one)
    const unsigned ny = L.patches ? unsigned(L.npatch) : 1u;
    const int64_t wgs = (L.cells + kAmrBlock - 1) / kAmrBlock * ny;  // a cell per thread
    const int64_t trips = wgs <= 1500 ? 1 : 4;
    const unsigned nx = amr_blocks((L.cells + trips - 1) / trips);
    hipLaunchKernelGGL(fill_ghosts_kernel<T>, dim3(nx, ny), dim3(kAmrBlock), 0, st, a);
  } else if (L.op == kAmrRestrict) {
    hipLaunchKernelGGL(restrict_kernel<T>, dim3(amr_blocks(L.cells), unsigned(L.nlinks)),
                       dim3(kAmrBlock), 0, st, a);
  } else if (L.op == kAmrProlong) {
    const dim3 grid(amr_blocks(L.cells), unsigned(L.nlinks), L.ghosts_only ? 5u : 1u);
    if (!L.ghosts_only)
      hipLaunchKernelGGL((prolong_kernel<T, false, false>), grid, dim3(kAmrBlock), 0, st, a);
    else if (L.cold)
      hipLaunchKernelGGL((prolong_kernel<T, true, true>), grid, dim3(kAmrBlock), 0, st, a);
    else
      hipLaunchKernelGGL((prolong_kernel<T, false, true>), grid, dim3(kAmrBlock), 0, st, a);
  } else if (L.op == kAmrSnapshot) {
    hipLaunchKernelGGL(snapshot_kernel<T>, dim3(amr_blocks(L.cells), unsigned(L.nlinks)),
                       dim3(kAmrBlock), 0, st, a);
  } else if (L.op == kAmrFlux) {
    hipLaunchKernelGGL(flux_reg_kernel<T>, dim3(amr_blocks(L.cells), unsigned(L.nlinks), 2u),
                       dim3(kAmrBlock), 0, st, a);
  } else if (L.op == kAmrGather) {
    hipLaunchKernelGGL(flux_gather_kernel<T>, dim3(amr_blocks(L.cells), unsigned(L.nlinks), 6u),
                       dim3(kAmrBlock), 0, st, a);
  } else {
    hipLaunchKernelGGL(reflux_kernel<T>, dim3(amr_blocks(L.cells), unsigned(L.nlinks)),
                       dim3(kAmrBlock), 0, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_amr(const LaunchAmr& L, hipStream_t st) {
  if (L.op < kAmrFill || L.op > kAmrGather) return hipErrorInvalidValue;
  if (L.op == kAmrSnapshot && (!L.cold || L.margin < 0)) return hipErrorInvalidValue;
  if (L.op == kAmrProlong && L.cold && !L.ghosts_only) return hipErrorInvalidValue;
  if (L.op != kAmrFill &&
      (!L.patches || L.nlinks < 1 || (!L.dlinks && L.nlinks > kAmrLinksPerLaunch) ||
       L.nlinks > 65535))
    return hipErrorInvalidValue;
  if (L.op == kAmrGather && (!L.reg || !L.face || L.maxface < 1)) return hipErrorInvalidValue;
  if ((L.op == kAmrFlux || L.op == kAmrReflux) &&
      (!L.reg || L.maxface < 1 || L.axis < 0 || L.axis > 2 || L.side < 0 || L.side > 1))
    return hipErrorInvalidValue;
  return L.fp64 ? launch_amr_t<double>(L, st) : launch_amr_t<float>(L, st);
}

}  // namespace hydro
