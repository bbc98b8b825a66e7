// fft.hpp -- device helpers shared by the spectra (diag.hip, spec3.hip):
// complex arithmetic in FP64, and an in-place mixed-radix (4, 2, 3) Stockham
// FFT of complex lines held in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fastdiv.hpp"

namespace hydro {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// -i a
__device__ __forceinline__ double2 cmi(double2 a) { return make_double2(a.y, -a.x); }
__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }

// W_16^e = exp(-2 pi i e / 16) times a, for the internal twiddles of the
// 16-point DFT (e = b c, b and c in 0..3)
template <int E>
__device__ __forceinline__ double2 w16(double2 a) {
  constexpr double C1 = 0.92387953251128675613;  // cos(pi/8)
  constexpr double S1 = 0.38268343236508977173;  // sin(pi/8)
  constexpr double H = 0.70710678118654752440;   // cos(pi/4)
  if constexpr (E == 0) return a;
  else if constexpr (E == 1) return cmul(a, make_double2(C1, -S1));
  else if constexpr (E == 2) return cmul(a, make_double2(H, -H));
  else if constexpr (E == 3) return cmul(a, make_double2(S1, -C1));
  else if constexpr (E == 4) return cmi(a);
  else if constexpr (E == 6) return cmul(a, make_double2(-H, -H));
  else return cmul(a, make_double2(-C1, S1));  // E == 9
}

// Forward R-point DFT (R = 2, 3, 4, 16) of v in place, W_R = exp(-2 pi i / R).
// R = 16 as 4 x 4: with r = 4a + b and k = c + 4d,
// X[c + 4d] = sum_b W_4^(bd) W_16^(bc) sum_a x[4a + b] W_4^(ac).
template <int R>
__device__ __forceinline__ void dft_small(double2 (&v)[R]) {
  if constexpr (R == 16) {
    double2 y[4][4];  // y[b][c]
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      double2 t[4] = {v[b], v[4 + b], v[8 + b], v[12 + b]};
      dft_small<4>(t);
#pragma unroll
      for (int c = 0; c < 4; ++c) y[b][c] = t[c];
    }
    y[1][1] = w16<1>(y[1][1]); y[1][2] = w16<2>(y[1][2]); y[1][3] = w16<3>(y[1][3]);
    y[2][1] = w16<2>(y[2][1]); y[2][2] = w16<4>(y[2][2]); y[2][3] = w16<6>(y[2][3]);
    y[3][1] = w16<3>(y[3][1]); y[3][2] = w16<6>(y[3][2]); y[3][3] = w16<9>(y[3][3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      double2 t[4] = {y[0][c], y[1][c], y[2][c], y[3][c]};
      dft_small<4>(t);
#pragma unroll
      for (int d = 0; d < 4; ++d) v[c + 4 * d] = t[d];
    }
  } else if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    const double2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    const double2 s13 = cadd(v[1], v[3]), d13 = cmi(csub(v[1], v[3]));  // -i (v1 - v3)
    v[0] = cadd(s02, s13);
    v[1] = cadd(d02, d13);
    v[2] = csub(s02, s13);
    v[3] = csub(d02, d13);
  } else {  // R == 3: W_3 = -1/2 - i sqrt(3)/2
    const double h = 0.86602540378443864676;  // sqrt(3) / 2
    const double2 t1 = cadd(v[1], v[2]);
    const double2 t2 = make_double2(v[0].x - 0.5 * t1.x, v[0].y - 0.5 * t1.y);
    const double2 dd = csub(v[1], v[2]);
    const double2 t3 = make_double2(h * dd.y, -h * dd.x);  // -i h (v1 - v2)
    v[0] = cadd(v[0], t1);
    v[1] = cadd(t2, t3);
    v[2] = csub(t2, t3);
  }
}

// Stages of an FFT of length n = 16^a 4^b 2^c 3^d (radix 16 first, then 4,
// 2, 3: fewer stages mean fewer LDS round trips and barriers), built on the
// host.  Stage s has radix rad[s], span ns[s] (product of
// the earlier radices) and twiddle step tw[s] = n / (ns R).
constexpr int kFftMaxStages = 12;
struct FftPlan {
  int n;
  int nst;
  int rad[kFftMaxStages];
  int ns[kFftMaxStages];
  int tw[kFftMaxStages];
  FastDiv nsd[kFftMaxStages];  // division by ns
  FastDiv md[kFftMaxStages];   // division by n / R (butterflies per line)
};

// false if n is not 2^a 3^b (1 <= n)
inline bool make_fft_plan(int n, FftPlan& p) {
  p = FftPlan{};
  p.n = n;
  if (n < 1) return false;
  int m = n;
  while (m % 16 == 0 && p.nst < kFftMaxStages) { p.rad[p.nst++] = 16; m /= 16; }
  while (m % 4 == 0 && p.nst < kFftMaxStages) { p.rad[p.nst++] = 4; m /= 4; }
  while (m % 2 == 0 && p.nst < kFftMaxStages) { p.rad[p.nst++] = 2; m /= 2; }
  while (m % 3 == 0 && p.nst < kFftMaxStages) { p.rad[p.nst++] = 3; m /= 3; }
  if (m != 1) return false;
  for (int s = 0, ns = 1; s < p.nst; ns *= p.rad[s], ++s) {
    p.ns[s] = ns;
    p.tw[s] = n / (ns * p.rad[s]);
    p.nsd[s] = FastDiv(uint32_t(ns));
    p.md[s] = FastDiv(uint32_t(n / p.rad[s]));
  }
  return true;
}

// LDS slot of complex element o of an FFT buffer: one pad slot after every
// 16 elements.  A radix-16 stage writes its outputs 16 elements apart (256
// bytes, the same banks for every lane); with the pad they land 272 bytes
// apart, on different banks.  A buffer of n elements takes fft_lds(n) slots.
__host__ __device__ __forceinline__ int fft_pad(int o) { return o + (o >> 4); }
__host__ __device__ __forceinline__ int fft_lds(int n) { return n + (n >> 4) + 1; }

// One radix-R stage of the Stockham autosort FFT (Govindaraju et al., SC
// 2008) over nl complex lines in LDS (line l at buf + l ls), in place:
// butterfly j of a line takes the elements j + r n/R, twiddled by
// W^(r (j mod ns) tw), through an R-point DFT to (j div ns) ns R +
// (j mod ns) + r ns.  Every thread first holds the inputs of its
// butterflies (j = t, t + B, ... over the nl n/R of the stage, at most MAXB)
// in registers; after a barrier it writes the outputs; a second barrier
// ends the stage.  Element o of the buffer sits at slot fft_pad(o).
// W[t] = exp(-2 pi i t / n) in LDS.  B = blockDim.x.
//  * FIRST: the first stage (ns = 1), whose twiddles are all 1.
//  * LIN: n/R is a multiple of 16, and so is ns (FIRST: R and ls are), so an
//    element r steps on sits r (step + step / 16) slots on: one add instead
//    of four integer operations an access.
// With a general stage throughout (and products without FMA) the shell spectrum
// of 256^3 FP32 cells took 575 instead of 532 us.
template <int R, int MAXB, bool FIRST, bool LIN>
__device__ __forceinline__ void fft_stage_inplace(double2* buf, int nl, int ls, int n, int ns,
                                                  int tw, const FastDiv& md, const FastDiv& nsd,
                                                  const double2* W) {
  const int m = n / R, nb = nl * m;
  const int mp = m + (m >> 4), np = FIRST ? 1 : ns + (ns >> 4);  // LIN: slots per step
  double2 v[MAXB][R];
  int dst[MAXB];
#pragma unroll
  for (int b = 0; b < MAXB; ++b) {
    const int j = int(threadIdx.x) + b * int(blockDim.x);
    dst[b] = -1;
    if (j < nb) {
      const int l = int(md.div(uint32_t(j))), jj = j - l * m;
      const int q = FIRST ? jj : int(nsd.div(uint32_t(jj))), k = FIRST ? 0 : jj - q * ns;
      const int s = l * ls + jj;
      const double2* in = buf + fft_pad(s);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double2 x = LIN ? in[r * mp] : buf[fft_pad(s + r * m)];
        v[b][r] = FIRST || r == 0 ? x : cmul(x, W[r * k * tw]);
      }
      dst[b] = l * ls + q * ns * R + k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < MAXB; ++b) {
    if (dst[b] >= 0) {
      dft_small<R>(v[b]);
      double2* out = buf + fft_pad(dst[b]);
#pragma unroll
      for (int r = 0; r < R; ++r)
        (LIN ? out[r * np] : buf[fft_pad(dst[b] + r * ns)]) = v[b][r];
    }
  }
  __syncthreads();
}

// A stage of the radix R in the form its sizes allow (wave-uniform).
template <int R, int EMAX, int BLOCK>
__device__ __forceinline__ void fft_stage(double2* buf, int nl, int ls, const FftPlan& p, int s,
                                          const double2* W) {
  constexpr int MAXB = (EMAX + R * BLOCK - 1) / (R * BLOCK);
  const int n = p.n, ns = p.ns[s];
  const bool lin = (n / R) % 16 == 0;
  if (R == 16 && s == 0 && lin && ls % 16 == 0)
    fft_stage_inplace<R, MAXB, true, true>(buf, nl, ls, n, ns, p.tw[s], p.md[s], p.nsd[s], W);
  else if (s > 0 && lin && ns % 16 == 0)
    fft_stage_inplace<R, MAXB, false, true>(buf, nl, ls, n, ns, p.tw[s], p.md[s], p.nsd[s], W);
  else if (s == 0)
    fft_stage_inplace<R, MAXB, true, false>(buf, nl, ls, n, ns, p.tw[s], p.md[s], p.nsd[s], W);
  else
    fft_stage_inplace<R, MAXB, false, false>(buf, nl, ls, n, ns, p.tw[s], p.md[s], p.nsd[s], W);
}

// The whole FFT of nl lines of length p.n (nl p.n <= EMAX elements) with a
// workgroup of BLOCK threads; the caller has made the input visible
// (barrier) and the output is visible to every thread on return.
template <int EMAX, int BLOCK>
__device__ void fft_lines_inplace(double2* buf, int nl, int ls, const FftPlan& p, const double2* W) {
  for (int s = 0; s < p.nst; ++s) {
    const int R = p.rad[s];
    if (R == 16) fft_stage<16, EMAX, BLOCK>(buf, nl, ls, p, s, W);
    else if (R == 4) fft_stage<4, EMAX, BLOCK>(buf, nl, ls, p, s, W);
    else if (R == 2) fft_stage<2, EMAX, BLOCK>(buf, nl, ls, p, s, W);
    else fft_stage<3, EMAX, BLOCK>(buf, nl, ls, p, s, W);
  }
}

// The velocity of a cell in FP64, correctly rounded quotients m / r.  FP64
// cells divide.  Widened FP32 cells lie far inside the range of FP64, so the
// three quotients share one reciprocal (two Newton steps) and take one exact
// residual step each, which rounds them as a division does (Markstein, IBM J.
// Res. Dev. 1990); div_fixup keeps 0, infinity and NaN as a division has them.
template <class T>
__device__ __forceinline__ void velocity(T rho, const T (&mom)[3], double (&u)[3]) {
  const double r = double(rho);
  if constexpr (sizeof(T) == 8) {
#pragma unroll
    for (int v = 0; v < 3; ++v) u[v] = mom[v] / r;
  } else {
    double y = __builtin_amdgcn_rcp(r);
    y = __builtin_fma(y, __builtin_fma(-r, y, 1.0), y);
    y = __builtin_fma(y, __builtin_fma(-r, y, 1.0), y);
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      const double m = double(mom[v]), q = m * y;
      u[v] = __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-q, r, m), y, q), r, m);
    }
  }
}

}  // namespace hydro
