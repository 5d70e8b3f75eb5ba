// tables.hip -- per-parameter-row tables of the frequency-summed propagator
// product (Sec. 2: the frequency integral done in closed form per scale).
//
// For every parameter row the odd function
//   S(z) = T sum_{n in Z} W(w_n) / (i w_n - z) = -2 z T sum_{n >= 0} W(w_n) / (w_n^2 + z^2)
// with W = d/dOmega theta^2 = -4 Omega w^4/(w^2+Omega^2)^3 (or theta^2 for the
// non-differentiated bubble) is sampled on circles in the complex plane and
// turned into Taylor coefficients on real intervals (Cauchy's formula with a
// trapezoid rule in the angle, exponentially accurate).  The Matsubara sum
// is done directly for the first `nmats` frequencies; the rest is expanded
// in v = 1/w^2 (w_N^2 exceeds |z|^2 and Omega^2 sixteenfold, so the expansion
// converges geometrically) and summed with
//   sum_{n >= N} w_n^{-2k} = (2 pi T)^{-2k} zeta(2k, N + 1/2)  (Hurwitz zeta).
#include <math.h>

#include <algorithm>

#include "launch.h"

namespace paid {

namespace {

constexpr double kPi = 3.14159265358979323846;

// Hurwitz zeta sum_{j >= 0} (q + j)^-s by Euler-Maclaurin after shifting q.
__device__ double hurwitz_zeta(double s, double q) {
  const double B2[10] = {1.0 / 6,   -1.0 / 30,        1.0 / 42,     -1.0 / 30,      5.0 / 66,
                         -691.0 / 2730, 7.0 / 6, -3617.0 / 510, 43867.0 / 798, -174611.0 / 330};
  int J = (int)ceil(s + 25.0 - q);
  if (J < 0) J = 0;
  double head = 0.0;
  for (int j = J - 1; j >= 0; --j) head += pow(q + j, -s);
  double a = q + J, as = pow(a, -s);
  double tail = a * as / (s - 1.0) + 0.5 * as;
  double term = s * as / a;  // s a^{-s-1}
  double fac = 2.0;          // (2i)!
  for (int i = 1; i <= 10; ++i) {
    tail += B2[i - 1] / fac * term;
    term *= (s + 2 * i - 1) * (s + 2 * i) / (a * a);
    fac *= (2.0 * i + 1) * (2.0 * i + 2);
  }
  return head + tail;
}

__global__ void k_zeta(const Entry *entries, int n, double *zeta) {
  int e = blockIdx.x, k = threadIdx.x;
  if (e >= n || k > kTabKTail) return;
  const Entry E = entries[e];
  double z = 0.0;
  if (k >= 1) z = pow(2.0 * kPi * E.T, -2.0 * k) * hurwitz_zeta(2.0 * k, E.nmats + 0.5);
  zeta[e * (kTabKTail + 1) + k] = z;
}


constexpr int kTabLanes = 8;  // lanes sharing a point's sum

// S(z) at one complex point: lane `part` of kTabLanes neighbouring lanes sums
// every kTabLanes-th Matsubara term, and the lanes' sums are added pairwise
// (a + b = b + a: every lane holds the same total)
__device__ double2 S_complex(const Entry &E, const double *zeta, double zr, double zi, int part) {
  const double T = E.T, Om = E.Om, O2 = Om * Om;
  const double z2r = zr * zr - zi * zi, z2i = 2.0 * zr * zi;  // z^2
  double sr = 0.0, si = 0.0;
  for (int n = E.nmats - 1 - part; n >= 0; n -= kTabLanes) {  // small terms first
    double w = (2.0 * n + 1.0) * kPi * T, u = w * w, d = u + O2;
    double W = (E.kind == 0) ? -4.0 * Om * u * u / (d * d * d) : u * u / (d * d);
    double dr = u + z2r, di = z2i, inv = W / (dr * dr + di * di);
    sr += dr * inv;
    si -= di * inv;
  }
  for (int o = 1; o < kTabLanes; o <<= 1) {
    sr += __shfl_xor(sr, o, 64);
    si += __shfl_xor(si, o, 64);
  }
  // tail: series in v = 1/w^2 of W(w)/(w^2+z^2)
  double cr[kTabKTail + 1], ci[kTabKTail + 1];
  for (int k = 0; k <= kTabKTail; ++k) cr[k] = ci[k] = 0.0;
  int nom;
  if (E.kind == 0) { cr[2] = -4.0 * Om; nom = 3; }   // -4 Omega v^2 (1+O2 v)^-3 (1+z^2 v)^-1
  else { cr[1] = 1.0; nom = 2; }                      // v (1+O2 v)^-2 (1+z^2 v)^-1
  for (int k = 1; k <= kTabKTail; ++k) {              // divide by (1 + z^2 v)
    double pr = cr[k - 1], pi_ = ci[k - 1];
    cr[k] -= z2r * pr - z2i * pi_;
    ci[k] -= z2r * pi_ + z2i * pr;
  }
  for (int r = 0; r < nom; ++r)                       // divide by (1 + Omega^2 v)
    for (int k = 1; k <= kTabKTail; ++k) {
      cr[k] -= O2 * cr[k - 1];
      ci[k] -= O2 * ci[k - 1];
    }
  for (int k = kTabKTail; k >= 1; --k) {
    sr += cr[k] * zeta[k];
    si += ci[k] * zeta[k];
  }
  // S = -2 z T (sum)
  double f = -2.0 * T;
  return make_double2(f * (zr * sr - zi * si), f * (zr * si + zi * sr));
}

// S at the points of the circles of radius kTabRho half-widths around every
// interval, upper half only (S(conj z) = conj S(z)): kValHalf points of the
// value intervals, then kTabHalf of the close ones.  Eight lanes share a
// point's Matsubara sum (every eighth term each, smallest first, added in a
// fixed order): hundreds of terms with a division each, on a few thousand
// points, are a chain of dependent divisions too long for one thread to walk
// (110 us of a 12 ms call at T = 0.01, 208 us at 0.005).
__global__ void __launch_bounds__(256) k_tab_points(TabArgs a, int blocks) {
  const int e = blockIdx.x / blocks;  // `blocks` workgroups per parameter row
  const Entry E = a.entries[e];
  if (E.kind > 1) return;
  const long gid = (long)(blockIdx.x - e * blocks) * blockDim.x + threadIdx.x;
  const long pt = gid / kTabLanes;
  const int part = (int)(gid % kTabLanes);
  const long nv = (long)E.JV * kValHalf, nc = (long)E.J * kTabHalf;
  if (pt >= nv + nc) return;  // whole groups of kTabLanes lanes
  const bool val = pt < nv;
  const long r = val ? pt : pt - nv;
  const int half = val ? kValHalf : kTabHalf, j = (int)(r / half), p = (int)(r % half);
  double c, h;
  if (val) val_interval(j, E.w, c, h);
  else tab_interval(j, E.w, c, h);
  double sn, cs;
  sincos(2.0 * kPi * p / (val ? kValPts : kTabPts), &sn, &cs);
  const double zr = c + kTabRho * h * cs, zi = kTabRho * h * sn;
  const double2 s = S_complex(E, a.zeta + (long)e * (kTabKTail + 1), zr, zi, part);
  if (part == 0) a.svals[(long)e * a.max_points + pt] = s;
}

// Sixteen threads per row (value rows first).  Thread k forms Taylor coefficient
// k of S/w around the interval's centre in units of its half-width, from the
// circle's points (Cauchy's formula, the trapezoid rule in the angle; the lower
// half by symmetry).  A value row is the Taylor series to degree kTabDeg
// economised to degree kValDeg (its Chebyshev coefficients beyond that
// dropped), then written in tau = (1 + t)/32, t in [-1, 1].
constexpr int kRowThreads = 16;
static_assert(kTabDeg < kRowThreads, "a thread per Taylor coefficient");

__global__ void __launch_bounds__(256) k_tab_coef(TabArgs a, int blocks) {
  __shared__ double C[256];
  const int e = blockIdx.x / blocks;
  const Entry E = a.entries[e];
  const int gid = (blockIdx.x - e * blocks) * blockDim.x + threadIdx.x;
  const int j = gid / kRowThreads, k = gid % kRowThreads;
  const bool val = j < E.JV, close = !val && j < E.JV + E.J;
  const int jc = j - E.JV;
  double coef = 0.0;
  // (S is odd: the even terms of close row 0 vanish)
  if (E.kind <= 1 && (val || close) && k <= kTabDeg && !(close && jc == 0 && (k & 1) == 0)) {
    const int n = val ? kValPts : kTabPts, st = kTabPts / n;
    const double2 *sv = a.svals + (long)e * a.max_points +
                        (val ? (long)j * kValHalf : (long)E.JV * kValHalf + (long)jc * kTabHalf);
    double s = 0.0;
    for (int p = n / 2; p >= 0; --p) {
      const int m = (st * k * p) % kTabPts;  // angle 2 pi m / kTabPts
      const double v = sv[p].x * a.cosine[m] + sv[p].y * a.cosine[(m + 3 * kTabPts / 4) % kTabPts];  // Re(S e^{-i k th})
      s += (p == 0 || 2 * p == n) ? v : 2.0 * v;
    }
    coef = E.inv_w * s / n * ldexp(1.0, -k);  // kTabRho = 2
  }
  C[threadIdx.x] = coef;
  __syncthreads();
  if (val && k <= kValDeg) {
    const double *c = &C[threadIdx.x - k];
    double d = 0.0;
    for (int i = kValDeg; i >= k; --i) {  // coefficient of t^i, times binomial(i, k) (-1)^(i-k) 32^k
      double b = c[i];
      for (int m = kValDeg + 1; m <= kTabDeg; ++m) b += a.econ[m - kValDeg - 1][i] * c[m];
      double bin = 1.0;
      for (int q = 1; q <= k; ++q) bin = bin * (i - k + q) / q;
      d += (((i - k) & 1) ? -b : b) * bin;
    }
    a.tab[E.tab_off + (long)j * kValStride + k] = d * ldexp(1.0, 5 * k);
  }
  if (close && k <= kTabDeg) {
    double *row = a.tab + E.tab_off + (long)E.JV * kValStride + (long)jc * kTabStride;
    if (k == 0) {
      double c, h;
      tab_interval(jc, 1.0, c, h);
      // -c/h, exact: 2j for a central interval, 2P + 1 + 2m for interval m of an octave
      row[0] = -(double)(jc < kTabCentral ? 2 * jc
                                          : 2 * kTabPerOct + 1 + 2 * ((jc - kTabCentral) % kTabPerOct));
      row[1] = 1.0 / h;
      row[kTabStride - 1] = 0.0;
    }
    row[kTabCoef + k] = coef;
  }
}

}  // namespace

// Economisation t^m = sum_{i <= kValDeg} econ[m][i] t^i + (Chebyshev terms of
// degree > kValDeg), m = kValDeg + 1 .. kTabDeg: t^m in Chebyshev polynomials
// (t T_n = (T_{n+1} + T_{|n-1|})/2), truncated, back in powers
static void econ_matrix(double econ[kTabDeg - kValDeg][kValDeg + 1]) {
  double T[kTabDeg + 1][kTabDeg + 1] = {};  // T_n in powers
  T[0][0] = 1.0;
  T[1][1] = 1.0;
  for (int n = 2; n <= kTabDeg; ++n)
    for (int i = 0; i <= n; ++i) T[n][i] = (i ? 2.0 * T[n - 1][i - 1] : 0.0) - T[n - 2][i];
  double c[kTabDeg + 2] = {1.0};  // t^m in Chebyshev polynomials, m = 0
  for (int m = 1; m <= kTabDeg; ++m) {
    double q[kTabDeg + 2] = {};
    for (int n = 0; n < m; ++n) {
      q[n + 1] += (n ? 0.5 : 1.0) * c[n];
      if (n) q[n - 1] += 0.5 * c[n];
    }
    for (int n = 0; n <= m; ++n) c[n] = q[n];
    if (m > kValDeg)
      for (int i = 0; i <= kValDeg; ++i) {
        double s = 0.0;
        for (int n = i; n <= kValDeg; ++n) s += c[n] * T[n][i];
        econ[m - kValDeg - 1][i] = s;
      }
  }
}

hipError_t launch_tables(TabArgs a, hipStream_t s) {
  if (a.n_entries == 0) return hipSuccess;
  econ_matrix(a.econ);
  for (int m = 0; m < kTabPts; ++m) a.cosine[m] = cos(2.0 * kPi * m / kTabPts);
  a.cosine[kTabPts / 4] = a.cosine[3 * kTabPts / 4] = 0.0;
  const int b1 = (int)((a.max_points * kTabLanes + 255) / 256);
  const int b2 = (a.max_rows * kRowThreads + 255) / 256;
  // A launch may have 2^32 threads, which 200,000 rows of 84 workgroups (T = 0.01)
  // reach: as many rows a launch as stay below half of that.
  const int most = (int)std::max(1L, (1L << 23) / std::max(b1, b2));
  for (int left = a.n_entries; left > 0; left -= most) {
    const int n = std::min(left, most);
    hipLaunchKernelGGL(k_zeta, dim3(n), dim3(64), 0, s, a.entries, n, a.zeta);
    hipLaunchKernelGGL(k_tab_points, dim3((unsigned)(n * b1)), dim3(256), 0, s, a, b1);
    hipLaunchKernelGGL(k_tab_coef, dim3((unsigned)(n * b2)), dim3(256), 0, s, a, b2);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.entries += n;
    a.zeta += (long)n * (kTabKTail + 1);
    a.svals += (long)n * a.max_points;
  }
  return hipSuccess;
}

// container constants: parameter row, channel, cos/sin of l/2 per axis
namespace {
__global__ void k_container_setup(Ctr *ctr, int n_ctr, const double *q, int n_q, int n_ch,
                                  int ch_first) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_ctr) return;
  int ich = c % n_ch, iq = (c / n_ch) % n_q, ip = c / (n_ch * n_q);
  Ctr r;
  r.entry = ip;
  r.ch = (n_ch == 2) ? ich : ch_first;
  sincos(0.5 * q[2 * iq], &r.sLx, &r.cLx);
  sincos(0.5 * q[2 * iq + 1], &r.sLy, &r.cLy);
  ctr[c] = r;
}
}  // namespace

hipError_t launch_container_setup(Ctr *ctr, int n_ctr, const double *q, int n_q, int n_ch,
                                  int ch_first, hipStream_t s) {
  if (n_ctr == 0) return hipSuccess;
  hipLaunchKernelGGL(k_container_setup, dim3((n_ctr + 255) / 256), dim3(256), 0, s, ctr, n_ctr, q,
                     n_q, n_ch, ch_first);
  return hipGetLastError();
}

}  // namespace paid
