// paid_device.h -- data layout and device helpers shared by the libpaid
// kernels (gfx950).  Library-internal: not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace paid {

// ---------------------------------------------------------------------------
// Rule pair (Sec. 3): N = 4 intervals per axis for Q_N, 2N = 8 for Q_2N.
// A parent's four children share 17 coordinates per axis (9 + 9 - 1).
constexpr int kNF = 9;    // fine-rule nodes per axis of one rectangle
constexpr int kNCo = 5;   // coarse-rule nodes per axis
constexpr int kNX = 17;   // distinct coordinates per axis over 4 children
constexpr int kMaxL = 2;  // box basis order: up to 5 harmonics per axis
constexpr int kMaxNB = 2 * kMaxL + 1;
constexpr int kMaxMB = kMaxNB * kMaxNB;       // 25 box functions
constexpr int kMaxMU = kMaxMB * (kMaxMB + 1) / 2;

// ---------------------------------------------------------------------------
// Frequency-sum tables.  For one parameter row the scalar integrand depends
// on the energies only through the odd function
//   S(x) = T sum_{n in Z} hdot(w_n) / (i w_n - x),   hdot = d/dOmega theta^2
// (theta^2 itself for the non-differentiated bubble), because partial
// fractions give K_ph(a,b) = S[a,b] = (S(a)-S(b))/(a-b) and
// K_pp(a,b) = -S[a,-b].  S is analytic except at x = +-i w_n, so on short
// intervals of x >= 0 it is a short polynomial.  Energies are taken in units
// of w = pi T, the distance of the nearest singularity from the real axis
// (v = |x|/w), and the tables hold S/w, so that divided differences in v are
// K itself.  Two tables per row:
//
// Value rows (far pairs: two values and a division).  Intervals follow from
// the bits of u = v + 1/4: 16 per octave of u from u = 1/4 on, so the row is
// the high word's exponent and top four mantissa bits, and the low mantissa
// bits with the exponent of 1 are 1 + tau with tau in [0, 1/16), exactly: no
// compare, conversion or stored centre and width.  An interval's half-width
// is at most 1/31 of the distance from its centre to the nearest singularity
// (1/4 is the offset that keeps the first octaves' ratio as large as the
// later ones'), so the Chebyshev series falls by 62 per degree and degree 8
// is exact to rounding: truncation at most 9e-17 of S over the workloads'
// temperatures and scales.  9 doubles a row (odd: the rows that the lanes of
// a wave read at one coefficient spread over the LDS banks) instead of the 16
// that a degree-13 Taylor row with its centre and width takes.  The node loop
// of the region evaluation is bound by LDS bandwidth and instruction issue
// together, and both fall (72 instead of 128 bytes an energy, 8 FMAs and 7
// other instructions instead of 13 and 12).
//
// Close rows (pairs with |x - y| < 0.02 sqrt(x^2 + w^2)).  The divided
// difference is formed on the polynomial of x's interval, also up to 1.5
// half-widths from its centre and with its derivative's accuracy, which a
// truncated series does not have: Taylor series of degree 13 on P + 1 central
// intervals centred at 0, 1/P, ..., 1 with half-width 1/(2P), then P per
// octave of v, [2^e (1 + m/P), 2^e (1 + (m+1)/P)), m = 0..P-1.  Every
// half-width is at most 1/(2P) of the distance from its centre to the nearest
// singularity.  Row layout: -c/h, 1/h, coef[deg + 1] of P(t) = S(c + h t)/w,
// padded to an odd number of doubles; c/h is an integer (2j in the centre,
// 2P + 1 + 2m in an octave), so t = v/h - c/h is one fused multiply-add.
constexpr int kValDeg = 8;
constexpr int kValLogOct = 4;                     // log2 of the intervals per octave of u
constexpr int kValPerOct = 1 << kValLogOct;
constexpr double kValOff = 0.25;                  // u = v + kValOff
constexpr int kValBase = (1023 - 2) * kValPerOct;  // index bits of u = kValOff
constexpr int kValStride = kValDeg + 1;
constexpr int kValPts = 16;                       // Cauchy points per interval (9 by symmetry)
constexpr int kValHalf = kValPts / 2 + 1;

constexpr int kTabDeg = 13;
constexpr int kTabLogOct = 3;                  // log2 of the intervals per octave
constexpr int kTabPerOct = 1 << kTabLogOct;    // intervals per octave above |x| = w
constexpr int kTabCentral = kTabPerOct + 1;    // central intervals
constexpr int kTabStride = (kTabDeg + 3) | 1;  // -c/h, 1/h, coef[deg + 1], odd
constexpr int kTabCoef = 2;                    // offset of the coefficients in a row
constexpr int kTabPts = 32;                    // Cauchy points per interval (17 by symmetry)
constexpr int kTabHalf = kTabPts / 2 + 1;
constexpr double kTabRho = 2.0;                // Cauchy radius in half-widths
constexpr int kTabKTail = 24;                  // tail expansion terms
constexpr double kDdSwitch2 = 0.0004;          // (0.02)^2: close-pair switch

// close interval j in units of w: centre c and half-width h (j >= 0)
__host__ __device__ inline void tab_interval(int j, double w, double &c, double &h) {
  constexpr double inv_p = 1.0 / kTabPerOct;
  if (j < kTabCentral) {
    c = w * (inv_p * j);
    h = w * (0.5 * inv_p);
  } else {
    const int k = j - kTabCentral, e = k / kTabPerOct, m = k - e * kTabPerOct;
    const double s = ldexp(w, e);
    c = s * (1.0 + inv_p * (m + 0.5));
    h = s * (0.5 * inv_p);
  }
}

// value interval j: centre c and half-width h
__host__ __device__ inline void val_interval(int j, double w, double &c, double &h) {
  constexpr double inv_p = 1.0 / kValPerOct;
  const int e = j >> kValLogOct, m = j & (kValPerOct - 1);
  c = w * (ldexp(kValOff, e) * (1.0 + inv_p * (m + 0.5)) - kValOff);
  h = w * (ldexp(kValOff, e) * (0.5 * inv_p));
}

// close rows needed to cover |x| <= top
__host__ __device__ inline int tab_rows(double top, double w) {
  if (top < w) return kTabCentral;
  int E = 0;
  (void)frexp(top / w, &E);  // top/w in [2^(E-1), 2^E)
  return kTabCentral + kTabPerOct * E;
}

// value rows needed to cover |x| <= top (whole octaves)
__host__ __device__ inline int val_rows(double top, double w) {
  int E = 0;
  (void)frexp(top / w + kValOff, &E);  // u in [2^(E-1), 2^E), u >= 1/4
  return kValPerOct * (E + 2);
}

struct Entry {        // one parameter row
  double t, tp, mu, T, Om;
  double emax;        // bound of |eps| over the zone
  double w, inv_w;    // pi T and its inverse
  int J;              // close rows
  int JV;             // value rows
  int nmats;          // Matsubara head terms used to build the table
  int kind;           // PAID_BUBBLE_DOT / PAID_BUBBLE / ...
  long tab_off;       // offset of this row's tables (in doubles): value rows, then close rows
};

// doubles of one parameter row's tables
__host__ __device__ inline int close_doubles(const Entry &e) { return e.J * kTabStride; }
__host__ __device__ inline int tab_doubles(const Entry &e) { return e.JV * kValStride + close_doubles(e); }

struct Ctr {          // one container (parameter row, transfer momentum, channel)
  int entry, ch;      // ch: 0 = pp, 1 = ph
  double cLx, sLx, cLy, sLy;  // cos/sin of l/2 per axis
};

// ---------------------------------------------------------------------------
// Products of the 9-function box basis.  The products of two box harmonics
// u_a u_c (u_0 = 1, u_1 = sqrt2 cos, u_2 = sqrt2 sin) lie in the span of five
// functions phi = {1, sqrt2 cos, sqrt2 sin, cos 2x, sin 2x} (2 cos^2 = 1 +
// cos 2x, 2 cos sin = sin 2x, 2 sin^2 = 1 - cos 2x), so every pair of box
// functions of a rectangle is a signed sum of one to four of the 25 integrals
// I_jk = int g phi_j(x) phi_k(y), and every pair of form factors over the
// 9-function box (or its first function) a combination of them.
constexpr int kPhi = 5, kProd = kPhi * kPhi;
constexpr int kPairs9 = 45;  // pairs of the 9 box functions

// product integral kPhi j + k: whether phi_j(x) phi_k(y) is odd under p -> -p
// (phi_2 and phi_4 are sines)
__host__ __device__ constexpr bool product_odd(int i) {
  return ((i / kPhi) == 2 || (i / kPhi) == 4) != ((i % kPhi) == 2 || (i % kPhi) == 4);
}

// phi index and sign of the terms of the product u_a u_c (a <= c)
struct Terms {
  int n, j0, s0, j1, s1;
};
__host__ __device__ constexpr Terms prod_terms(int a, int c) {
  return (a == 0 && c == 0) ? Terms{1, 0, 1, 0, 0}
       : (a == 0 && c == 1) ? Terms{1, 1, 1, 0, 0}
       : (a == 0 && c == 2) ? Terms{1, 2, 1, 0, 0}
       : (a == 1 && c == 1) ? Terms{2, 0, 1, 3, 1}
       : (a == 1 && c == 2) ? Terms{1, 4, 1, 0, 0}
                            : Terms{2, 0, 1, 3, -1};  // (2, 2)
}

// the 45 box pairs (m, n), m <= n, m = 3 a + b: x terms of u_am u_an
// (phi index j0, optional j1 with sign) and y terms of u_bm u_bn; -1 = none
struct PairTab {
  signed char t[kPairs9][6];  // jx0, jx1, sx1, ky0, ky1, sy1
};
__host__ __device__ constexpr PairTab make_pair_tab() {
  PairTab T{};
  int p = 0;
  for (int m = 0; m < 9; ++m)
    for (int n = m; n < 9; ++n) {
      const int am = m / 3, bm = m % 3, an = n / 3, bn = n % 3;
      const Terms tx = prod_terms(am < an ? am : an, am < an ? an : am);
      const Terms ty = prod_terms(bm < bn ? bm : bn, bm < bn ? bn : bm);
      T.t[p][0] = (signed char)tx.j0;
      T.t[p][1] = (signed char)(tx.n == 2 ? tx.j1 : -1);
      T.t[p][2] = (signed char)tx.s1;
      T.t[p][3] = (signed char)ty.j0;
      T.t[p][4] = (signed char)(ty.n == 2 ? ty.j1 : -1);
      T.t[p][5] = (signed char)ty.s1;
      ++p;
    }
  return T;
}

// box pair (m, n) from the 25 product integrals
template <class T>
__host__ __device__ inline double pair_of_products(const T &I, int m, int n) {
  const int am = m / 3, bm = m % 3, an = n / 3, bn = n % 3;
  const Terms tx = prod_terms(am < an ? am : an, am < an ? an : am);
  const Terms ty = prod_terms(bm < bn ? bm : bn, bm < bn ? bn : bm);
  double v = I[kPhi * tx.j0 + ty.j0];
  if (ty.n == 2) v += ty.s1 * I[kPhi * tx.j0 + ty.j1];
  if (tx.n == 2) {
    double u = I[kPhi * tx.j1 + ty.j0];
    if (ty.n == 2) u += ty.s1 * I[kPhi * tx.j1 + ty.j1];
    v += tx.s1 * u;
  }
  return v;
}

// ---------------------------------------------------------------------------
// Region codes: depth in bits 56..63, ix in 28..55, iy in 0..27.
__host__ __device__ inline uint64_t make_code(int d, uint64_t ix, uint64_t iy) {
  return ((uint64_t)d << 56) | (ix << 28) | iy;
}
__host__ __device__ inline int code_depth(uint64_t c) { return (int)(c >> 56); }
__host__ __device__ inline uint64_t code_ix(uint64_t c) { return (c >> 28) & 0xFFFFFFFull; }
__host__ __device__ inline uint64_t code_iy(uint64_t c) { return c & 0xFFFFFFFull; }

// ---------------------------------------------------------------------------
// Frequency-sum table evaluation.
// close interval of v = |x|/w (no transcendental: exponent and top mantissa
// bits).  Central intervals: jc = round(P v), at most P; octave intervals from
// the high word of v, whose bits above the top log2(P) mantissa bits are
// (exponent << log2(P) | m).  For v < 1 the octave index is at most jc and for
// v >= 1 at least P + 1 > jc, so the larger of the two is the interval: no
// compare or select.
__device__ inline int tab_index(int J, double v) {
  const int jc = min((int)fma(v, (double)kTabPerOct, 0.5), kTabPerOct);
  const unsigned hi = (unsigned)(__double_as_longlong(v) >> 32);
  const int jo = kTabCentral - 1023 * kTabPerOct + (int)(hi >> (20 - kTabLogOct));
  const int j = max(jc, jo);
  return j < J - 1 ? j : J - 1;
}

// FP32 copy of a per-pair error estimate (the stored E and the running sums
// built from it): rounded to nearest, except that a positive estimate below
// the smallest normal float is kept as that float, an upper bound, instead of
// flushing towards zero and passing a tolerance it does not meet.
__device__ inline float err_f32(double e) {
  const float f = (float)e;
  return (e > 0.0 && f < 1.17549435e-38f) ? 1.17549435e-38f : f;
}

// n / d for a normal, non-zero d: the hardware reciprocal estimate (2^-24 or
// better) refined by one Newton-Raphson step (2^-48), then one residual
// correction of the quotient (Markstein's scheme: the error left is that of
// the reciprocal times that of the uncorrected quotient, below 2^-90, so a
// second step changes no quotient); no scaling for extreme exponents, which
// the far pairs (|d| >= 0.02 w) never reach.
__device__ inline double div_nr(double n, double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  const double q = n * r;
  return fma(fma(-d, q, n), r, q);
}

// S[x,y] with x = a and y = b (sgn_ch = 0: ph, K itself) or -b (sgn_ch the
// sign bit: pp, -K), a and b in units of w.  S is odd and S[x,y] = S[-x,-y], so
// both are flipped to x >= 0 (XORs of sign bits).  Far pairs take two values,
// S[x,y] = (S(x) - sign(y) S(|y|))/(x - y); close pairs, |x - y| < 0.02
// sqrt(x^2 + 1), are left to pair_close (a few per cent of the nodes at most
// transfer momenta).
__device__ inline double flip_y(unsigned sgn_ch, double a, double b) {
  const unsigned ha = (unsigned)(__double_as_longlong(a) >> 32) & 0x80000000u;
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  return __longlong_as_double((long long)(((unsigned long long)((unsigned)(y >> 32) ^ ha ^ sgn_ch) << 32) |
                                          (unsigned)y));
}

__device__ inline double with_sign_of(double v, double y) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned sy = (unsigned)(__double_as_longlong(y) >> 32) & 0x80000000u;
  return __longlong_as_double((long long)(((unsigned long long)((unsigned)(b >> 32) ^ sy) << 32) | (unsigned)b));
}

__device__ inline bool pair_is_close(double x, double d) { return d * d < fma(kDdSwitch2 * x, x, kDdSwitch2); }

// The row of v and the argument in it
__device__ inline const double *val_row(int JV, const double *tab, double v, double &tau) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(v) + kValOff);
  const unsigned hi = (unsigned)(b >> 32);
  const unsigned j = min((hi >> (20 - kValLogOct)) - (unsigned)kValBase, (unsigned)(JV - 1));
  const unsigned hf = (hi & ((1u << (20 - kValLogOct)) - 1u)) | 0x3FF00000u;
  tau = __longlong_as_double((long long)(((unsigned long long)hf << 32) | (unsigned)b)) - 1.0;
  // row offset by a 24-bit multiply (full rate; the 32-bit one is not)
  return tab + __umul24(j, kValStride);
}

struct PairNode {
  double s;    // S[x,y] of a far pair
  bool close;  // (s is not a value)
};

// A far pair.  cn and sn: values that the caller has loaded for its next node;
// the empty asm takes them and both rows as operands, so that every load is
// issued before the first of them is waited for.
__device__ inline PairNode pair_node(const Entry &e, const double *tab, unsigned sgn_ch, double a, double b,
                                     double &cn, double &sn) {
  static_assert(kValDeg == 8, "the operand list holds nine coefficients");
  const double y = flip_y(sgn_ch, a, b), d = fabs(a) - y;
  double tx, ty, p[9], q[9];
  const double *rx = val_row(e.JV, tab, a, tx), *ry = val_row(e.JV, tab, b, ty);
#pragma unroll
  for (int k = kValDeg; k >= 0; --k) p[k] = rx[k];
#pragma unroll
  for (int k = kValDeg; k >= 0; --k) q[k] = ry[k];
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]), "+v"(p[4]), "+v"(p[5]), "+v"(p[6]),
                    "+v"(p[7]), "+v"(p[8]), "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(q[4]),
                    "+v"(q[5]), "+v"(q[6]), "+v"(q[7]), "+v"(q[8]), "+v"(cn), "+v"(sn));
#endif
  double sx = p[kValDeg], sy = q[kValDeg];
#pragma unroll
  for (int k = kValDeg - 1; k >= 0; --k) {
    sx = fma(sx, tx, p[k]);
    sy = fma(sy, ty, q[k]);
  }
  PairNode n;
  n.s = div_nr(sx - with_sign_of(sy, y), d);
  n.close = pair_is_close(fabs(a), d);
  return n;
}

// A close pair: the divided difference on the polynomial of x's interval.
// Horner at tx carries the quotient coefficients, Horner of those at ty is the
// divided difference (no subtraction of values; there |ty| <= 1.5, a tenth of
// the radius of convergence in units of the half-width).
__device__ inline double pair_close(const Entry &e, const double *tab, unsigned sgn_ch, double a, double b) {
  const double x = fabs(a), y = flip_y(sgn_ch, a, b);
  const double *rx = tab + e.JV * kValStride + __umul24(tab_index(e.J, x), kTabStride);
  const double tx = fma(x, rx[1], rx[0]), ty = fma(y, rx[1], rx[0]);
  const double *c = rx + kTabCoef;
  double q = c[kTabDeg], r = 0.0;
#pragma unroll
  for (int k = kTabDeg - 1; k >= 0; --k) {
    r = fma(r, ty, q);
    q = fma(q, tx, c[k]);
  }
  return r * rx[1];
}

// kernel K_j(a, b) of two energies from both tables: ph = S[a,b], pp = -S[a,-b]
// (the two-lanes kernel's form as one function, for the diagnostic)
__device__ inline double K_eval(const Entry &e, const double *tab, int ch, double a, double b) {
  double cn = 0.0, sn = 0.0;
  const unsigned sg = ch ? 0u : 0x80000000u;
  a *= e.inv_w;
  b *= e.inv_w;
  const PairNode n = pair_node(e, tab, sg, a, b, cn, sn);
  const double s = n.close ? pair_close(e, tab, sg, a, b) : n.s;
  return ch ? s : -s;
}

// The same from the close rows alone (tab: the first of them), for the kernels
// that hold one node per lane and whose waves mix far and close pairs of one
// parent: the far pair's two values and the close pair's divided difference
// are written as one loop with the second row and argument chosen per lane
// (the compiler moves the chain that a lane's form does not use into a branch).
__device__ inline double K_taylor(const Entry &e, const double *tab, int ch, double a, double b) {
  const unsigned sg = ch ? 0u : 0x80000000u;
  a *= e.inv_w;
  b *= e.inv_w;
  const double x = fabs(a), y = flip_y(sg, a, b), ay = fabs(y), d = x - y;
  const bool close = pair_is_close(x, d);
  const double *rx = tab + __umul24(tab_index(e.J, x), kTabStride);
  const double *ry = close ? rx : tab + __umul24(tab_index(e.J, ay), kTabStride);
  const double tx = fma(x, rx[1], rx[0]);
  const double ty = fma(close ? y : ay, ry[1], ry[0]);
  const double *cx = rx + kTabCoef, *cy = ry + kTabCoef;
  double q = cx[kTabDeg], py = cy[kTabDeg], r = 0.0;
#pragma unroll
  for (int k = kTabDeg - 1; k >= 0; --k) {
    r = fma(r, ty, q);
    q = fma(q, tx, cx[k]);
    py = fma(py, ty, cy[k]);
  }
  const double s = close ? r * rx[1] : div_nr(q - with_sign_of(py, y), d);
  return ch ? s : -s;
}

}  // namespace paid
