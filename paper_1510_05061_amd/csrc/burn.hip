// burn.hip -- operator-split reactive source: a toy chain network per zone.
//
// The paper's explosion models carry nuclear networks of 10-20 nuclei in
// the hydrodynamics (its discussion of the physics the simulations need)
// without rates; this is a self-contained stand-in with the same shape of
// work, a stiff ODE per zone:
//   species 0 -> 1 -> ... -> M-1 (the last stable); link i at
//   k_i = A_i exp(-Ta_i / T), T = p / rho (code units, frozen over the step),
//   releasing q_i per unit mass converted.
// Integration: nsub backward-Euler substeps of h = dt / nsub.  The system is
// lower bidiagonal, so each substep is exact forward substitution,
//   X_0 <- X_0 d_0,  X_s <- (X_s + c_s X_{s-1}) d_s,
// with c_s = h k_{s-1} and d_s = 1 / (1 + h k_s) (d_{M-1} = 1) formed once
// per zone.  Backward Euler is L-stable (a link with h k >> 1 empties in one
// substep) and conserves sum_s X_s.  The energy density then rises by
// rho sum_s B_s (X_s - X_s^0), B_s = q_0 + ... + q_{s-1}.
//
// One thread per zone (FP64 arithmetic whatever the storage precision); the
// species live in registers, so the kernel is instantiated per species
// count.  Composition planes X are laid out like the state's planes (same
// plane size, pitches and interior origin).
#include <hip/hip_runtime.h>

#include "euler.hpp"
#include "fastdiv.hpp"
#include "launch.hpp"

namespace hydro {

constexpr int kBurnBlock = 256;

template <class T>
struct BurnArgs {
  T* pool;
  T* X;
  PatchDev single;
  double gamma;
  double h;
  int nsub;
  unsigned cells;
  FastDiv dnx, dny;  // division by nx and ny
  double A[kBurnMaxSpecies - 1];
  double Ta[kBurnMaxSpecies - 1];
  double B[kBurnMaxSpecies];
};

// One wavefront pass of J substeps over the chain: at time t substep j
// updates species t - j, so J independent chains are in flight.  Each update
// reads the same values as in sequential order (substep j's species s-1 is
// written at time t-1, and substep j+1 overwrites it only after substep j,
// later in the same time step), so the bits are those of the plain loop.
template <int M, int J, class First, class Next>
__device__ __forceinline__ void substeps(First first, Next next) {
#pragma unroll
  for (int t = 0; t < M + J - 1; ++t) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int s = t - j;
      if (s == 0) first();
      else if (s > 0 && s < M) next(s);
    }
  }
}
template <int M, class First, class Next>
__device__ __forceinline__ void all_substeps(int nsub, First first, Next next) {
  int n = 0;
  for (; n + 4 <= nsub; n += 4) substeps<M, 4>(first, next);
  for (; n < nsub; ++n) substeps<M, 1>(first, next);
}

// From kScaledSubsteps substeps on, the chain is stepped in scaled species
// W_s = X_s / a_s with a_s = e_1 .. e_s, e_s = c_s d_s: the update
// X_s <- d_s X_s + e_s X_{s-1} becomes W_s <- d_s W_s + W_{s-1}, one FMA (and
// one rounding) per species and substep instead of two.  The scaling costs
// about 14 instructions per species and saves one an update.  192^3 FP32 zones,
// 13 species, scaled and plain: 8 substeps 225 and 217 us, 12 236 and 236, 16
// 247 and 262 (20 species 347 and 337, 363 and 370, 388 and 398).  A zone whose a_s leave [2^-400, 2^64] (a frozen link) or,
// in FP64, with a species above 2^600 is stepped as it stands: the bounds keep W
// within range and X / a_s from underflow.
constexpr int kScaledSubsteps = 12;

// 1 / x: the estimate after two Newton steps whose residuals are exact is
// rounded as the quotient is, in half the instructions of a division (the same
// bits in every burn measured);
// div_fixup keeps 0, infinity and NaN as a division has them.
__device__ __forceinline__ double recip(double x) {
  return __builtin_amdgcn_div_fixup(rcp(x), x, 1.0);
}

// The kernel is bound by FP64 issue: 1563 VALU instructions a zone with 13
// species and 64 substeps (832 the substeps), 92 % of the cycles that a SIMD is
// busy, at a clock that falls to 1.9 GHz.  13 species and 64 substeps on 256^3
// FP32 zones: with (X_s + c_s X_{s-1}) d_s as three operations, a division
// per link for Ta / T and the network's constants hoisted out of a
// grid-stride loop into spilled scalars 1.72 ms; with divisions 1 / (1 + h k)
// 0.974 ms; without 0.950 ms (held to 128 registers it spills: 1.32 ms); with a
// branch a zone for exponents out of range in place of selects 0.940 -> 0.920 ms.
template <class T, int M>
__global__ void __launch_bounds__(kBurnBlock) burn_kernel(BurnArgs<T> a) {
  const PatchDev& P = a.single;
  const unsigned i = blockIdx.x * kBurnBlock + threadIdx.x;
  if (i >= a.cells) return;
  const unsigned row = a.dnx.div(i), x = i - row * a.dnx.d;
  const unsigned z = a.dny.div(row), y = row - z * a.dny.d;
  const int64_t o = int64_t(x) + int64_t(y) * P.sy + int64_t(z) * P.sz;
  T* p0 = a.pool + P.base0 + o;
  T* x0 = a.X + P.base0 + o;
  const double r = double(p0[0]);
  const double mx = double(p0[P.plane]), my = double(p0[2 * P.plane]);
  const double mz = double(p0[3 * P.plane]), e = double(p0[4 * P.plane]);
  double X[M], c[M], d[M];
#pragma unroll
  for (int s = 0; s < M; ++s) X[s] = double(x0[s * P.plane]);
  const double m2 = mx * mx + my * my + mz * mz;
  const double temp = ((a.gamma - 1.0) * (e - (0.5 * m2) / r)) / r;
  // Ta / T for every link from one reciprocal: the residual of the product
  // corrects it to the quotient (a rounding error of the exponent would be
  // carried through all substeps).  Where a product or 1 / T overflows, or T is
  // no finite number, the correction is NaN and the quotients are divided out,
  // behind one branch (with one a link the exponentials no longer overlap:
  // 19 species, 18 substeps on 72 x 114 x 31 zones 18.3 instead of 16.6 us).
  const double itemp = 1.0 / temp;
  bool exact = true;
#pragma unroll
  for (int s = 0; s < M - 1; ++s) {
    const double q = a.Ta[s] * itemp;
    d[s] = fma(fma(-q, temp, a.Ta[s]), itemp, q);
    exact = exact && d[s] == d[s];
  }
  if (__builtin_expect(!exact, 0)) {
#pragma unroll
    for (int s = 0; s < M - 1; ++s) d[s] = a.Ta[s] / temp;
  }
  double e0 = 0.0;
#pragma unroll
  for (int s = 0; s < M; ++s) e0 += a.B[s] * X[s];
  c[0] = 0.0;
  d[M - 1] = 1.0;
#pragma unroll
  for (int s = 0; s < M - 1; ++s) {
    c[s + 1] = a.h * (a.A[s] * exp(-d[s]));
    d[s] = recip(1.0 + c[s + 1]);
  }
  bool scaled = a.nsub >= kScaledSubsteps;
  if (scaled) {
    double g = 1.0;
#pragma unroll
    for (int s = 1; s < M; ++s) {
      g *= c[s] * d[s];
      scaled = scaled && g >= 0x1p-400 && g <= 0x1p64;
    }
    if (sizeof(T) == 8) {  // |X| below 2^600, by the largest upper word
      unsigned top = 0;
#pragma unroll
      for (int s = 0; s < M; ++s)
        top = max(top, unsigned(__double2hiint(X[s])) & 0x7fffffffu);
      scaled = scaled && top < (1023u + 600u) << 20;
    }
  }
  if (scaled) {
    double g = 1.0;
#pragma unroll
    for (int s = 1; s < M; ++s) {
      g *= c[s] * d[s];
      c[s] = g;  // a_s
      X[s] *= rcp(g);
    }
    all_substeps<M>(a.nsub, [&] { X[0] *= d[0]; },
                    [&](int s) { X[s] = s < M - 1 ? fma(d[s], X[s], X[s - 1]) : X[s] + X[s - 1]; });
#pragma unroll
    for (int s = 1; s < M; ++s) X[s] *= c[s];
  } else {
    all_substeps<M>(a.nsub, [&] { X[0] *= d[0]; },
                    [&](int s) { X[s] = fma(c[s], X[s - 1], X[s]) * d[s]; });
  }
  double e1 = 0.0;
#pragma unroll
  for (int s = 0; s < M; ++s) {
    e1 += a.B[s] * X[s];
    x0[s * P.plane] = T(X[s]);
  }
  p0[4 * P.plane] = T(e + r * (e1 - e0));
}

template <class T, int M>
static hipError_t launch_burn_m(const LaunchBurn& L, const BurnArgs<T>& a, dim3 grid,
                                hipStream_t st) {
  if constexpr (M > kBurnMaxSpecies) {
    return hipErrorInvalidValue;
  } else {
    if (L.nspec != M) return launch_burn_m<T, M + 1>(L, a, grid, st);
    hipLaunchKernelGGL((burn_kernel<T, M>), grid, dim3(kBurnBlock), 0, st, a);
    return hipGetLastError();
  }
}

template <class T>
static hipError_t launch_burn_t(const LaunchBurn& L, hipStream_t st) {
  BurnArgs<T> a{};
  a.pool = static_cast<T*>(L.pool);
  a.X = static_cast<T*>(L.X);
  a.single = L.single;
  a.gamma = L.gamma;
  a.h = L.h;
  a.nsub = L.nsub;
  for (int i = 0; i < L.nspec - 1; ++i) {
    a.A[i] = L.A[i];
    a.Ta[i] = L.Ta[i];
  }
  for (int s = 0; s < L.nspec; ++s) a.B[s] = L.B[s];
  // a plane is below 4 GiB: the cells and the workgroups fit 32 bits
  a.cells = unsigned(L.single.n[0]) * unsigned(L.single.n[1]) * unsigned(L.single.n[2]);
  a.dnx = FastDiv(uint32_t(L.single.n[0]));
  a.dny = FastDiv(uint32_t(L.single.n[1]));
  const dim3 grid((a.cells + kBurnBlock - 1) / kBurnBlock);
  return launch_burn_m<T, 2>(L, a, grid, st);
}

hipError_t launch_burn(const LaunchBurn& L, hipStream_t st) {
  if (L.nspec < 2 || L.nspec > kBurnMaxSpecies || L.nsub < 1) return hipErrorInvalidValue;
  return L.fp64 ? launch_burn_t<double>(L, st) : launch_burn_t<float>(L, st);
}

}  // namespace hydro
