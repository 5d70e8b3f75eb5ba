// region_eval.hip -- the hot kernel: evaluation of rectangles with the nested
// Clenshaw-Curtis pair (Sec. 3) for all form-factor pairs at once.
//
// Two kernels compute the same rule sums.  k_children_lpc (second half of the
// file) serves form factors over the 9-function box in the separable FP64 form
// over the full zone; k_children everything else: the 25-function box, the dense
// Gram, the half-zone mode and the Gaussian test integrand.  In k_children one
// wavefront owns one work item: a parent rectangle and its four children (Alg.
// 2: split into 4, evaluate Q_N and Q_2N on each).  The children share
// 17 x 17 node coordinates, so the integrand g is evaluated 289 times instead
// of 324.  Per child the projection onto the box basis U[node][m] is the
// weighted Gram contraction
//     Q_2N = U^T diag(w_2N g) U,    Q_N = U^T diag(w_N g) U,   E = Q_2N - Q_N,
// and err of a child is sum_pq |E_pq| (the paper's error summed over pairs).
// Two ways to form it:
//   - separable (default): U[node][(a,b)] = u_a(x) u_b(y) and the weights are
//     tensor products, so the sum runs first over y for every x and every
//     product u_b u_d, then over x for every product u_a u_c; for 9 form
//     factors this is ~4.4k FMAs per parent instead of a 16x16x84 tile pair;
//   - dense Gram on the FP64 matrix cores (16x16x4 tiles; a 9-function basis
//     fills one tile, 25 functions 2x2 tiles of which the lower-left one is
//     skipped by symmetry).
// The frequency-sum table of the parameter row is staged in LDS once per
// workgroup and shared by its waves.
#include <math.h>

#include <type_traits>

#include "launch.h"
#include "share.h"

namespace paid {

__constant__ RuleConst c_rule;

hipError_t set_rule_constants(const RuleConst &rc) {
  return hipMemcpyToSymbol(HIP_SYMBOL(c_rule), &rc, sizeof(RuleConst));
}

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr double kTwoPi = 6.28318530717958647692;
constexpr double kSqrt2 = 1.41421356237309504880;

typedef double d4 __attribute__((ext_vector_type(4)));

template <int L>
struct Dims {
  static constexpr int NB = 2 * L + 1;          // harmonics per axis
  static constexpr int MB = NB * NB;            // box functions
  static constexpr int NP = NB * (NB + 1) / 2;  // products u_a u_c, a <= c
  static constexpr int MU = MB * (MB + 1) / 2;  // pairs of box functions
  // the four children's x-sums fit in the storage of the integrand values
  static constexpr bool XALL = 4 * 2 * NP * NP <= kNX * kNX;
};

// per-wave scratch in LDS.  Buffers of different phases share storage: the
// integrand g is dead once the y-sums are formed (separable path), the
// per-axis cosines once g is, and the separable path never uses the box
// harmonics of the dense Gram.
template <int L>
struct WaveLds {
  static constexpr int NB = Dims<L>::NB, MB = Dims<L>::MB, NP = Dims<L>::NP, MU = Dims<L>::MU;
  double pp[2][kNX][NP];           // products u_a u_c of the box harmonics per axis
  union {
    double g[kNX * kNX];           // integrand at the shared nodes
    struct {
      double g2[NP * NP], g1[NP * NP];  // x-sums of one child (separable path)
    };
    struct {  // x-sums of all four children (where XALL)
      double g2b[Dims<L>::XALL ? 4 : 1][NP * NP], g1b[Dims<L>::XALL ? 4 : 1][NP * NP];
    };
  };
  union {
    struct {
      double cp[2][kNX], cm[2][kNX];    // cos(l/2 + p), cos(l/2 - p) per axis
      double pos[2][kNX];               // coordinates
    };
    double h1[2][kNCo * 2 - 1][NP];     // y-sums with the coarse weights (even x)
  };
  union {
    double h2[2][kNX][NP];         // y-sums with the fine weights, per child row
    double u[2][kNX][NB];          // box harmonics per axis (dense Gram)
  };
  // one child's Q_2N and E over form-factor pairs: not for the box basis itself
  // in the separable form, whose pairs go straight to memory (the root's too
  // are staged)
  double cq[MU], ce[MU];
  // general form-factor sets only (dropped from the allocation otherwise)
  double tq[MB * MB], ts[MB * MB], tr[MB * MB];
};

template <int L>
constexpr size_t wave_lds_doubles(bool identity, bool direct = false) {
  return sizeof(WaveLds<L>) / sizeof(double) - (identity ? 3 * Dims<L>::MB * Dims<L>::MB : 0) -
         (identity && direct ? 2 * Dims<L>::MU : 0);
}

// wave-local synchronisation for LDS traffic between lanes of one wave
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline int lane_id() { return threadIdx.x & 63; }

__device__ inline int pair_index(int p, int q, int M) { return p * M - p * (p - 1) / 2 + (q - p); }

template <int NB>
__device__ inline int prod_index(int a, int c) {  // (a, c) -> index of u_a u_c
  if (a > c) { int t = a; a = c; c = t; }
  return a * NB - a * (a - 1) / 2 + (c - a);
}

// parity of box function m = a NB + b under p -> -p: 1 if it has one sine
// factor (u_{2k} = sqrt2 sin kx is odd, 1 and the cosines are even)
template <int NB>
__device__ inline int box_odd(int m) {
  const int a = m / NB, b = m - a * NB;
  return ((a > 0 && !(a & 1)) ? 1 : 0) ^ ((b > 0 && !(b & 1)) ? 1 : 0);
}

// weight of a box pair in the half-zone mode: 0 for odd joint parity (the
// full-zone integral vanishes), else 2 (the two halves are equal)
template <int NB>
__device__ inline double half_zone_factor(int m, int n) {
  return (box_odd<NB>(m) ^ box_odd<NB>(n)) ? 0.0 : 2.0;
}

// sin and cos of |x| <= pi (+ rounding): reduction by pi/2 in two parts
// (Cody-Waite; q*pi/2 is exact for |q| <= 2) to |r| <= pi/4, then the Taylor
// series of sin and cos to degree 17/18 (truncation below 1e-19 there).  The
// coefficients come by scalar loads through a pointer that the compiler cannot
// follow: as literals in a loop they are hoisted out of it into registers that
// the loop has not got, and reloaded from scratch memory.
__device__ inline void sincos_zone(double x, double *s, double *c) {
  typedef const __attribute__((address_space(4))) RuleConst CR;
  CR *cr = (CR *)&c_rule;
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+s"(cr));
#endif
  const double pio2_hi = 1.5707963267948966, pio2_lo = 6.123233995736766e-17;
  const double q = rint(x * 0.63661977236758134);
  const double r = (x - q * pio2_hi) - q * pio2_lo, r2 = r * r;
  double ps = cr->sin_c[0], pc = cr->cos_c[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) ps = fma(ps, r2, cr->sin_c[i]);
#pragma unroll
  for (int i = 1; i < 9; ++i) pc = fma(pc, r2, cr->cos_c[i]);
  const double sr = fma(ps * r2, r, r), cr1 = fma(-pc, r2, 1.0);
  const int k = ((int)q) & 3;
  *s = (k == 0) ? sr : (k == 1) ? cr1 : (k == 2) ? -sr : -cr1;
  *c = (k == 0) ? cr1 : (k == 1) ? -sr : (k == 2) ? -cr1 : sr;
}

// Coordinates of one axis: nco = 17 (four children of a rectangle of width
// wdt starting at x0) or 9 (a single rectangle).
__device__ inline double axis_coord(int j, int nco, double x0, double wdt) {
  if (nco == kNF) return x0 + 0.5 * wdt + 0.5 * wdt * c_rule.xi[j];
  if (j <= 8) return x0 + 0.25 * wdt + 0.25 * wdt * c_rule.xi[j];
  return x0 + 0.75 * wdt + 0.25 * wdt * c_rule.xi[j - 8];
}

// Per-axis data and the integrand on the nco x nco node grid.  `tab` is the
// parameter row's close rows (LDS or global memory).
template <int L>
__device__ void fill_nodes(WaveLds<L> &S, const Problem &P, const Ctr &C, const Entry &E,
                           const double *tab, int nco, double x0, double y0, double wdt) {
  constexpr int NB = Dims<L>::NB;
  const int lane = lane_id();
  if (lane < 2 * nco) {
    int ax = lane >= nco, j = lane - ax * nco;
    double p = axis_coord(j, nco, ax ? y0 : x0, wdt);
    double sp, cpp;
    sincos_zone(p, &sp, &cpp);
    double cL = ax ? C.cLy : C.cLx, sL = ax ? C.sLy : C.sLx;
    S.pos[ax][j] = p;
    S.cp[ax][j] = cL * cpp - sL * sp;  // cos(l/2 + p)
    S.cm[ax][j] = cL * cpp + sL * sp;  // cos(l/2 - p)
    double u[NB];
    u[0] = 1.0;
    if (L >= 1) {
      u[1] = kSqrt2 * cpp;
      u[2] = kSqrt2 * sp;
    }
    if (L >= 2) {
      u[3] = kSqrt2 * (cpp - sp) * (cpp + sp);
      u[4] = kSqrt2 * 2.0 * sp * cpp;
    }
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      S.u[ax][j][a] = u[a];
#pragma unroll
      for (int c = a; c < NB; ++c) S.pp[ax][j][prod_index<NB>(a, c)] = u[a] * u[c];
    }
  }
  wave_sync();
  const int nn = nco * nco;
#pragma unroll 1
  for (int v = lane; v < nn; v += 64) {
    int ix = v / nco, iy = v - ix * nco;
    double g;
    if (P.kind <= 1) {
      double px = S.cp[0][ix], py = S.cp[1][iy], mx = S.cm[0][ix], my = S.cm[1][iy];
      double a = -2.0 * E.t * (px + py) - 4.0 * E.tp * px * py - E.mu;
      double b = -2.0 * E.t * (mx + my) - 4.0 * E.tp * mx * my - E.mu;
      g = K_taylor(E, tab, C.ch, a, b);
    } else if (P.kind == 2) {
      g = 1.0;
    } else {
      double dx = S.pos[0][ix] - P.gauss_x, dy = S.pos[1][iy] - P.gauss_y;
      g = exp(-(dx * dx + dy * dy) / (2.0 * P.gauss_s * P.gauss_s));
    }
    S.g[v] = g;
  }
  wave_sync();
}

// ------------------------------------------------------------- separable
// Stage 1: for every x of the grid and each child row cy, the y-sums
//   h2[cy][x][k] = sum_b w2_b g(x, y_b) P_k(y_b),  h1 likewise with w1 on even b.
template <int L>
__device__ void sep_stage1(WaveLds<L> &S, int nco, int nrow) {
  constexpr int NP = Dims<L>::NP;
  const int lane = lane_id();
  for (int idx = lane; idx < nrow * nco * NP; idx += 64) {
    int cy = idx / (nco * NP), rem = idx - cy * nco * NP, x = rem / NP, k = rem - x * NP;
    const double *gr = &S.g[x * nco + 8 * cy];
    double s2 = 0.0, s1 = 0.0;
#pragma unroll
    for (int b = 0; b < kNF; ++b) {
      double v = gr[b] * S.pp[1][8 * cy + b][k];
      s2 = fma(c_rule.w2[b], v, s2);
      if (!(b & 1)) s1 = fma(c_rule.w1[b >> 1], v, s1);
    }
    S.h2[cy][x][k] = s2;
    if (!(x & 1)) S.h1[cy][x >> 1][k] = s1;
  }
  wave_sync();
}

// Stage 2 for child (cx, cy), then the form-factor pairs (identity basis) or
// the full box Gram (general sets) scaled by the area factor fa.
// the four children's x-sums in one pass over the lanes (where they fit:
// 144 tasks in 3 passes instead of 36 in each of 4)
template <int L>
constexpr bool kXsumsAll = Dims<L>::XALL;

template <int L>
__device__ void sep_xsums_all(WaveLds<L> &S) {
  constexpr int NP = Dims<L>::NP;
  const int lane = lane_id();
  for (int idx = lane; idx < 4 * NP * NP; idx += 64) {
    const int ch = idx / (NP * NP), r = idx - ch * (NP * NP), cx = ch & 1, cy = ch >> 1;
    const int j = r / NP, k = r - j * NP;
    double s2 = 0.0, s1 = 0.0;
#pragma unroll
    for (int a = 0; a < kNF; ++a) {
      int x = 8 * cx + a;
      double pj = S.pp[0][x][j];
      s2 = fma(c_rule.w2[a] * pj, S.h2[cy][x][k], s2);
      if (!(a & 1)) s1 = fma(c_rule.w1[a >> 1] * pj, S.h1[cy][x >> 1][k], s1);
    }
    S.g2b[ch][r] = s2;
    S.g1b[ch][r] = s1;
  }
  wave_sync();
}

// x-sums of one child
template <int L>
__device__ void sep_xsums(WaveLds<L> &S, int cx, int cy) {
  constexpr int NP = Dims<L>::NP;
  const int lane = lane_id();
  for (int idx = lane; idx < NP * NP; idx += 64) {
    int j = idx / NP, k = idx - j * NP;
    double s2 = 0.0, s1 = 0.0;
#pragma unroll
    for (int a = 0; a < kNF; ++a) {
      int x = 8 * cx + a;
      double pj = S.pp[0][x][j];
      s2 = fma(c_rule.w2[a] * pj, S.h2[cy][x][k], s2);
      if (!(a & 1)) s1 = fma(c_rule.w1[a >> 1] * pj, S.h1[cy][x >> 1][k], s1);
    }
    S.g2[idx] = s2;
    S.g1[idx] = s1;
  }
  wave_sync();
}

template <int L>
__device__ void sep_stage2(WaveLds<L> &S, const Problem &P, const int *pidmap, const int *podd,
                           int cx, int cy, double fa, bool xsums_done) {
  constexpr int NB = Dims<L>::NB, NP = Dims<L>::NP, MB = Dims<L>::MB, MU = Dims<L>::MU;
  const int lane = lane_id();
  const double *G2 = S.g2, *G1 = S.g1;
  bool done = false;
  if constexpr (kXsumsAll<L>) {
    if (xsums_done) {
      G2 = S.g2b[2 * cy + cx];
      G1 = S.g1b[2 * cy + cx];
      done = true;
    }
  }
  if (!done) {
    sep_xsums<L>(S, cx, cy);
  }
  if (P.ff_identity) {
    for (int pid = lane; pid < MU; pid += 64) {
      int jk = pidmap[pid];
      double q2 = G2[jk], f = fa, fe = fa;
      if (P.sym || P.mirror) f = podd[pid] ? 0.0 : 2.0 * fa;
      if (P.sym || P.mirror) fe = P.mirror ? 2.0 * fa : f;
      S.cq[pid] = f * q2;
      S.ce[pid] = fe * (q2 - G1[jk]);
    }
  } else {
    for (int idx = lane; idx < MB * MB; idx += 64) {
      int m = idx / MB, n = idx - m * MB;
      int jk = prod_index<NB>(m / NB, n / NB) * NP + prod_index<NB>(m % NB, n % NB);
      double q2 = G2[jk], f = fa, fe = fa;
      if (P.sym || P.mirror) f = half_zone_factor<NB>(m, n) * fa;
      if (P.sym || P.mirror) fe = P.mirror ? 2.0 * fa : f;
      S.tq[idx] = f * q2;
      S.ts[idx] = fe * (q2 - G1[jk]);
    }
  }
  wave_sync();
}

// ------------------------------------------------------------- dense MFMA
// Weighted Gram of one rectangle on the matrix cores.  Its 9 x 9 nodes are
// rows offx.. and columns offy.. of the nco x nco grid.  A row of A is a box
// function times w g (fine weights for Q_2N, w_2N - w_N for E, which keeps the
// error estimate free of a rounding floor in reduced precision), B is the box
// function; results are scaled by fa and widened to FP64.

// one product term of the Gram at a node: values for this lane's A and B
struct GramVals {
  double aq0, ae0, b0, aq1, ae1, b1;
};

template <int L>
__device__ inline GramVals gram_node_vals(const WaveLds<L> &S, int nu, int nco, int offx, int offy,
                                         bool v0, bool v1, int a0, int b0, int a1, int b1) {
  GramVals r = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (nu < kNF * kNF) {
    int a = nu / kNF, b = nu - a * kNF;
    int gx = offx + a, gy = offy + b;
    double g = S.g[gx * nco + gy];
    double w2 = c_rule.w2[a] * c_rule.w2[b];
    double wn = ((a | b) & 1) ? 0.0 : c_rule.w1[a >> 1] * c_rule.w1[b >> 1];
    double gq = g * w2, ge = g * (w2 - wn);
    if (v0) {
      r.b0 = S.u[0][gx][a0] * S.u[1][gy][b0];
      r.aq0 = r.b0 * gq;
      r.ae0 = r.b0 * ge;
    }
    if (v1) {
      r.b1 = S.u[0][gx][a1] * S.u[1][gy][b1];
      r.aq1 = r.b1 * gq;
      r.ae1 = r.b1 * ge;
    }
  }
  return r;
}

// store the accumulated tiles: element (i, j) of tile t
template <int L>
__device__ inline void gram_put(WaveLds<L> &S, const Problem &P, int i, int j, double q, double e) {
  constexpr int MB = Dims<L>::MB;
  if (i < MB && j < MB && i <= j) {
    if (P.sym) {
      const double f = half_zone_factor<Dims<L>::NB>(i, j);
      q *= f;
      e *= f;
    }
    if (P.ff_identity) {
      int pid = pair_index(i, j, MB);
      S.cq[pid] = q;
      S.ce[pid] = e;
    } else {
      S.tq[i * MB + j] = q;
      S.tq[j * MB + i] = q;
      S.ts[i * MB + j] = e;
      S.ts[j * MB + i] = e;
    }
  }
}

typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

// three-term bf16 split x = hi + mid + lo (8 significant bits each)
__device__ inline void split3(double x, __bf16 &hi, __bf16 &mid, __bf16 &lo) {
  float f = (float)x;
  hi = (__bf16)f;
  float r1 = f - (float)hi;
  mid = (__bf16)r1;
  lo = (__bf16)(r1 - (float)mid);
}

template <int L, int PREC>
__device__ void gram_mfma(WaveLds<L> &S, const Problem &P, int nco, int offx, int offy, double fa) {
  constexpr int NB = Dims<L>::NB, MB = Dims<L>::MB, NT = MB > 16 ? 2 : 1;
  constexpr int NACC = NT * (NT + 1) / 2;
  const int lane = lane_id(), m = lane & 15, kk = lane >> 4;
  const bool v0 = m < MB, v1 = (NT == 2) && (m + 16 < MB);
  const int a0 = v0 ? m / NB : 0, b0 = v0 ? m % NB : 0;
  const int a1 = v1 ? (m + 16) / NB : 0, b1 = v1 ? (m + 16) % NB : 0;
  if (PREC == PAID_FP64) {
    d4 aq[NACC], ae[NACC];
#pragma unroll
    for (int t = 0; t < NACC; ++t) {
      aq[t] = d4{0.0, 0.0, 0.0, 0.0};
      ae[t] = d4{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll 3
    for (int kb = 0; kb < 21; ++kb) {
      GramVals v = gram_node_vals<L>(S, 4 * kb + kk, nco, offx, offy, v0, v1, a0, b0, a1, b1);
      aq[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.aq0, v.b0, aq[0], 0, 0, 0);
      ae[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.ae0, v.b0, ae[0], 0, 0, 0);
      if (NT == 2) {
        aq[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.aq0, v.b1, aq[1], 0, 0, 0);
        ae[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.ae0, v.b1, ae[1], 0, 0, 0);
        aq[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.aq1, v.b1, aq[2], 0, 0, 0);
        ae[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.ae1, v.b1, ae[2], 0, 0, 0);
      }
    }
    // f64 16x16x4 result: row = 4 r + lane >> 4, col = lane & 15
#pragma unroll
    for (int t = 0; t < NACC; ++t) {
      int tr = (NT == 2 && t == 2) ? 1 : 0, tc = (NT == 2 && t >= 1) ? 1 : 0;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        gram_put<L>(S, P, 16 * tr + 4 * r + kk, 16 * tc + m, fa * aq[t][r], fa * ae[t][r]);
    }
  } else if (PREC == PAID_FP32) {
    f4v aq[NACC], ae[NACC];
#pragma unroll
    for (int t = 0; t < NACC; ++t) {
      aq[t] = f4v{0.f, 0.f, 0.f, 0.f};
      ae[t] = f4v{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll 3
    for (int kb = 0; kb < 21; ++kb) {
      GramVals v = gram_node_vals<L>(S, 4 * kb + kk, nco, offx, offy, v0, v1, a0, b0, a1, b1);
      aq[0] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)v.aq0, (float)v.b0, aq[0], 0, 0, 0);
      ae[0] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)v.ae0, (float)v.b0, ae[0], 0, 0, 0);
      if (NT == 2) {
        aq[1] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)v.aq0, (float)v.b1, aq[1], 0, 0, 0);
        ae[1] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)v.ae0, (float)v.b1, ae[1], 0, 0, 0);
        aq[2] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)v.aq1, (float)v.b1, aq[2], 0, 0, 0);
        ae[2] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)v.ae1, (float)v.b1, ae[2], 0, 0, 0);
      }
    }
    // f32 16x16x4 result: row = 4 (lane >> 4) + r, col = lane & 15
#pragma unroll
    for (int t = 0; t < NACC; ++t) {
      int tr = (NT == 2 && t == 2) ? 1 : 0, tc = (NT == 2 && t >= 1) ? 1 : 0;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        gram_put<L>(S, P, 16 * tr + 4 * kk + r, 16 * tc + m, fa * (double)aq[t][r],
                    fa * (double)ae[t][r]);
    }
  } else {  // three-term bf16 split, 16x16x32 tiles, FP32 accumulation
    f4v aq[NACC], ae[NACC];
#pragma unroll
    for (int t = 0; t < NACC; ++t) {
      aq[t] = f4v{0.f, 0.f, 0.f, 0.f};
      ae[t] = f4v{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll 1
    for (int kb = 0; kb < 3; ++kb) {
      // this lane: row/col m, nodes 32 kb + 8 kk + e, e = 0..7
      bf8v q0[3], e0[3], c0[3], q1[3], e1[3], c1[3];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        GramVals v = gram_node_vals<L>(S, 32 * kb + 8 * kk + e, nco, offx, offy, v0, v1, a0, b0,
                                       a1, b1);
        __bf16 h, md, lo;
        split3(v.aq0, h, md, lo); q0[0][e] = h; q0[1][e] = md; q0[2][e] = lo;
        split3(v.ae0, h, md, lo); e0[0][e] = h; e0[1][e] = md; e0[2][e] = lo;
        split3(v.b0, h, md, lo); c0[0][e] = h; c0[1][e] = md; c0[2][e] = lo;
        if (NT == 2) {
          split3(v.aq1, h, md, lo); q1[0][e] = h; q1[1][e] = md; q1[2][e] = lo;
          split3(v.ae1, h, md, lo); e1[0][e] = h; e1[1][e] = md; e1[2][e] = lo;
          split3(v.b1, h, md, lo); c1[0][e] = h; c1[1][e] = md; c1[2][e] = lo;
        }
      }
      // A B ~ hi hi + hi mid + mid hi + hi lo + lo hi + mid mid (terms >= 2^-16)
      const int ia[6] = {0, 0, 1, 0, 2, 1}, ib[6] = {0, 1, 0, 2, 0, 1};
#pragma unroll
      for (int t6 = 0; t6 < 6; ++t6) {
        const int x = ia[t6], y = ib[t6];
        aq[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q0[x], c0[y], aq[0], 0, 0, 0);
        ae[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e0[x], c0[y], ae[0], 0, 0, 0);
        if (NT == 2) {
          aq[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q0[x], c1[y], aq[1], 0, 0, 0);
          ae[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e0[x], c1[y], ae[1], 0, 0, 0);
          aq[2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q1[x], c1[y], aq[2], 0, 0, 0);
          ae[2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e1[x], c1[y], ae[2], 0, 0, 0);
        }
      }
    }
    // bf16 16x16x32 result: row = 4 (lane >> 4) + r, col = lane & 15
#pragma unroll
    for (int t = 0; t < NACC; ++t) {
      int tr = (NT == 2 && t == 2) ? 1 : 0, tc = (NT == 2 && t >= 1) ? 1 : 0;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        gram_put<L>(S, P, 16 * tr + 4 * kk + r, 16 * tc + m, fa * (double)aq[t][r],
                    fa * (double)ae[t][r]);
    }
  }
  wave_sync();
}

// General form-factor sets: C G C^T of a box matrix G.  IMAGE: of the mirror
// image's E (odd box pairs with the other sign), and dst becomes the mean
// magnitude of the two.
template <int L, bool IMAGE>
__device__ inline void transform_pairs(WaveLds<L> &S, const Problem &P, const double *G, double *dst) {
  constexpr int MB = Dims<L>::MB, NB = Dims<L>::NB;
  const int lane = lane_id(), M = P.M;
  double *R = S.tr;
  for (int idx = lane; idx < MB * M; idx += 64) {  // R[a][q] = sum_b G[a][b] C[q][b]
    int a = idx / M, q = idx - a * M;
    double s = 0.0;
    for (int b = 0; b < MB; ++b) {
      const double g = G[a * MB + b];
      s = fma(IMAGE && box_odd<NB>(a) != box_odd<NB>(b) ? -g : g, P.ffc[q * MB + b], s);
    }
    R[idx] = s;
  }
  wave_sync();
  for (int pid = lane; pid < P.MU; pid += 64) {
    int p = 0, k = pid;
    while (k >= M - p) { k -= M - p; ++p; }
    int q = p + k;
    double s = 0.0;
    for (int a = 0; a < MB; ++a) s = fma(P.ffc[p * MB + a], R[a * M + q], s);
    dst[pid] = IMAGE ? 0.5 * (fabs(dst[pid]) + fabs(s)) : s;
  }
  wave_sync();
}

template <int L>
__device__ void transform_ff(WaveLds<L> &S, const Problem &P) {
  for (int which = 0; which < 2; ++which)
    transform_pairs<L, false>(S, P, which ? S.ts : S.tq, which ? S.ce : S.cq);
  if (P.mixed) transform_pairs<L, true>(S, P, S.ts, S.ce);
}

// a double moved between lanes by a DPP pattern (both halves; VALU, no LDS)
// v from another lane of the same row (CTRL: a quad permutation or a row
// mirror, which every lane reads within its row, so no lane keeps an old
// value and none need be set up)
template <int CTRL>
__device__ inline double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ inline double lane_value(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// sum over the 64 lanes in a fixed order, the same in every lane: within
// each row of 16 lanes by DPP exchanges (partners lane ^ 1, lane ^ 2, then
// the mirror images within 8 and within 16 lanes; a + b = b + a exactly, so
// partners agree), then the four row sums as (r0 + r1) + (r2 + r3)
__device__ inline double wave_sum(double v) {
  v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);  // row_half_mirror
  v += dpp_move<0x140>(v);  // row_mirror
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Store one evaluated rectangle (S.cq, S.ce) into pool slot `ri` of slot s,
// return its key.
template <int L>
__device__ double store_region(WaveLds<L> &S, const Problem &P, int s, long ri, uint64_t code) {
  const int lane = lane_id();
  const long base = slot_base(P, s) + ri;
  double part = 0.0;
  for (int pid = lane; pid < P.MU; pid += 64) {
    double q = S.cq[pid], e = fabs(S.ce[pid]);
    if (!P.products) P.Q[base * P.MQ + pid] = q;
    if (P.E) P.E[base * P.MU + pid] = err_f32(e);
    part += (P.err_mode != 0) ? e * (double)P.itau[(long)s * P.MU + pid] : e;
  }
  double key = wave_sum(part);
  if (lane == 0) {
    P.key[base] = key;
    P.code[base] = code;
  }
  return key;
}

// One rectangle of the grid (child (cx, cy) of the 17-grid, or the 9-grid
// root with cx = cy = 0): fills S.cq / S.ce.
// GRAM: 0..2 = dense Gram on the matrix cores in FP64 / FP32 / bf16x3,
// 3 = separable FP64
constexpr int kSep = 3;

template <int L, int GRAM>
__device__ void eval_rect(WaveLds<L> &S, const Problem &P, const int *pidmap, const int *podd,
                          int nco, int cx, int cy, double fa, bool xsums_done = false) {
  if (GRAM == kSep) {
    sep_stage2<L>(S, P, pidmap, podd, cx, cy, fa, xsums_done);
  } else {
    gram_mfma<L, GRAM>(S, P, nco, 8 * cx, 8 * cy, fa);
  }
  if (!P.ff_identity) transform_ff<L>(S, P);
}

// pair index -> index into the x-sum matrix of the separable form
// and whether the pair has odd joint parity (half-zone mode)
template <int L>
__device__ void build_pidmap(int *map, int *odd, int tid, int nthr) {
  constexpr int NB = Dims<L>::NB, MB = Dims<L>::MB, NP = Dims<L>::NP, MU = Dims<L>::MU;
  for (int pid = tid; pid < MU; pid += nthr) {
    int m = 0, k = pid;
    while (k >= MB - m) { k -= MB - m; ++m; }
    int n = m + k;
    map[pid] = prod_index<NB>(m / NB, n / NB) * NP + prod_index<NB>(m % NB, n % NB);
    odd[pid] = box_odd<NB>(m) ^ box_odd<NB>(n);
  }
}

// ---------------------------------------------------------------- root
// A region that the seed tree splits is stored as a placeholder: zero value,
// error and key.  It is split in a later round of the seed phase before any
// termination test runs, so the running sums never miss it.
template <int L>
__device__ void store_zero(const Problem &P, int s, long ri, uint64_t code) {
  const int lane = lane_id();
  const long base = slot_base(P, s) + ri;
  for (int i = lane; i < P.MQ; i += 64) P.Q[base * P.MQ + i] = 0.0;
  if (P.E)
    for (int pid = lane; pid < P.MU; pid += 64) P.E[base * P.MU + pid] = 0.0f;
  if (lane == 0) {
    P.key[base] = 0.0;
    P.code[base] = code;
  }
}

// Seed admission (one wave): pyramid of predicted leaf counts in the
// container's frame, n = max(0, 2^y - 1) per cell and 2 x 2 sums upwards,
// and the depth bound D, lowered from seed_dmax until the seed tree has at
// most seed_limit leaves.  Returns D.
__device__ int seed_admit(const Problem &P, int s, int c, double *spyr) {
  const int t = threadIdx.x;
  const float *y = P.seed_y + (long)c * (kSeedG * kSeedG);
  const int fold = P.seed_fold[c];
  for (int cell = t; cell < kSeedG * kSeedG; cell += 64) {
    double n = exp2((double)y[seed_model_cell(fold, cell & 15, cell >> 4)]) - 1.0;
    spyr[pyr_off(4) + cell] = n > 0.0 ? n : 0.0;
  }
  __syncthreads();
  for (int d = 3; d >= 0; --d) {
    const int w = 1 << d, o = pyr_off(d), o1 = pyr_off(d + 1);
    for (int k = t; k < w * w; k += 64) {
      int i = k % w, j = k / w;
      const double *ch = spyr + o1;
      const int w1 = 2 * w;
      spyr[o + k] = ((ch[(2 * j) * w1 + 2 * i] + ch[(2 * j) * w1 + 2 * i + 1]) +
                     ch[(2 * j + 1) * w1 + 2 * i]) + ch[(2 * j + 1) * w1 + 2 * i + 1];
    }
    __syncthreads();
  }
  double *py = P.pyr + (long)s * kPyr;
  for (int k = t; k < kPyr; k += 64) py[k] = spyr[k];
  const double th = P.seed_thresh;
  int D = P.seed_dmax;
  for (; D > 0; --D) {
    long long leaves = 0;
    for (int k = t; k < kPyr; k += 64) {
      int d = 0;
      while (k >= pyr_off(d + 1)) ++d;
      if (d > D) continue;
      const int w = 1 << d, i = (k - pyr_off(d)) % w, j = (k - pyr_off(d)) / w;
      bool exists = true;
      for (int a = 0; a < d; ++a) {
        int sh = d - a;
        double ca = spyr[pyr_off(a) + ((j >> sh) << a) + (i >> sh)];
        exists = exists && (a < D) && (ca >= th);
      }
      if (!exists) continue;
      const double cn = spyr[k];
      if (d < 4) {
        if (!(d < D && cn >= th)) leaves += 1;
      } else {  // uniform subtree below a cell: levels split while the share >= th
        int lev = 0;
        double v = cn;
        while (4 + lev < D && v >= th) {
          ++lev;
          v *= 0.25;
        }
        leaves += 1LL << (2 * lev);
      }
    }
    for (int off = 32; off >= 1; off >>= 1) leaves += __shfl_xor(leaves, off, 64);
    if (leaves <= P.seed_limit) break;
  }
  return D;
}

template <int L, int GRAM>
__global__ void __launch_bounds__(64) k_root(Problem P) {
  extern __shared__ double lds_raw[];
  __shared__ int pidmap[Dims<L>::MU], podd[Dims<L>::MU];
  __shared__ double spyr[kPyr];
  WaveLds<L> &S = *reinterpret_cast<WaveLds<L> *>(lds_raw);
  const int s = blockIdx.x;
  if (s >= P.W || P.state[s] != SLOT_NEW) return;
  build_pidmap<L>(pidmap, podd, threadIdx.x, 64);
  const int c = P.cid[s];
  if (threadIdx.x == 0) P.sctr[s] = P.ctr[c];
  // key weights: the pair weights in the weighted mode, else one (the
  // per-integral mode refreshes them with 1/tau every round)
  for (int pid = threadIdx.x; pid < P.MU; pid += 64) {
    float w = 1.0f;
    if (P.err_mode == 2) {
      const int M = P.M;
      int p = 0, k = pid;
      while (k >= M - p) { k -= M - p; ++p; }
      const int q = p + k;
      const double *W = P.pair_w + (long)c * M * M;
      w = (float)((p == q) ? W[p * M + p] : W[p * M + q] + W[q * M + p]);
    }
    P.itau[(long)s * P.MU + pid] = w;
  }
  __syncthreads();
  int D = 0;
  bool placeholder = false;
  if (P.seed_y) {
    D = seed_admit(P, s, c, spyr);
    placeholder = D > 0 && spyr[0] >= P.seed_thresh;
  }
  double key = 0.0;
  // leaves the container starts from: the zone, or its two quadrants with p_y >= 0
  const bool half = P.sym || P.mirror;
  const int nroot = half ? 2 : 1;
  int filled = 0;
  if (placeholder && !half) {
    store_zero<L>(P, s, 0, make_code(0, 0, 0));
    for (int i = threadIdx.x; i < P.MQ; i += 64) P.val[(long)s * P.MQ + i] = 0.0;
    if (P.errp)
      for (int pid = threadIdx.x; pid < P.MU; pid += 64) P.errp[(long)s * P.MU + pid] = 0.0;
  } else {
    const Ctr C = P.ctr[c];
    const Entry E = P.entries[C.entry];
    const double *tab = P.tab + E.tab_off + (long)E.JV * kValStride;  // close rows
    const double wr = half ? kPi : kTwoPi;
    if (half) {  // the sums below add up the quadrants
      for (int i = threadIdx.x; i < P.MQ; i += 64) P.val[(long)s * P.MQ + i] = 0.0;
      if (P.errp)
        for (int pid = threadIdx.x; pid < P.MU; pid += 64) P.errp[(long)s * P.MU + pid] = 0.0;
    }
    for (int h = 0; h < nroot; ++h) {
      // a quadrant that the seed tree splits again (the root is split then)
      if (placeholder && D > 1 && spyr[pyr_off(1) + 2 + h] >= P.seed_thresh) {
        store_zero<L>(P, s, h, make_code(1, h, 1));
        continue;
      }
      ++filled;
      fill_nodes<L>(S, P, C, E, tab, kNF, -kPi + h * wr, half ? 0.0 : -kPi, wr);
      if (GRAM == kSep) sep_stage1<L>(S, kNF, 1);
      eval_rect<L, GRAM>(S, P, pidmap, podd, kNF, 0, 0, (0.5 * wr) * (0.5 * wr) / (4.0 * kPi * kPi));
      key += store_region<L>(S, P, s, h, half ? make_code(1, h, 1) : make_code(0, 0, 0));
      for (int pid = threadIdx.x; pid < P.MU; pid += 64) {
        const long o = (long)s * P.MU + pid;
        const double e = (double)err_f32(fabs(S.ce[pid]));
        if (!P.products) P.val[(long)s * P.MQ + pid] = half ? P.val[(long)s * P.MQ + pid] + S.cq[pid] : S.cq[pid];
        if (P.errp) P.errp[o] = half ? P.errp[o] + e : e;
      }
      if constexpr (L == 1 && GRAM == kSep)
        if (P.products && threadIdx.x < kProd) {
          // the product integrals from the x-sums over the harmonics' products
          // (phi_3 = u_1 u_1 - u_0 u_0; the others are products themselves)
          const int j = threadIdx.x / kPhi, k = threadIdx.x % kPhi;
          auto sum_y = [&](int x) { return k == 3 ? S.g2[x * 6 + 3] - S.g2[x * 6] : S.g2[x * 6 + k]; };
          double v = ((0.5 * wr) * (0.5 * wr) / (4.0 * kPi * kPi)) * (j == 3 ? sum_y(3) - sum_y(0) : sum_y(j));
          if (P.mirror) v *= product_odd(threadIdx.x) ? 0.0 : 2.0;
          P.Q[(slot_base(P, s) + h) * P.MQ + threadIdx.x] = v;
          P.val[(long)s * P.MQ + threadIdx.x] = half ? P.val[(long)s * P.MQ + threadIdx.x] + v : v;
        }
      wave_sync();
    }
  }
  if (threadIdx.x == 0) {
    P.err[s] = key;
    P.nleaf[s] = nroot;
    P.st_rounds[s] = 0;
    P.st_splits[s] = P.mirror ? 1 : 0;  // (the root's)
    P.st_evals[s] = (long)filled * images(P) * kNF * kNF;
    P.st_depth[s] = nroot - 1;
    if (P.born)
      for (int h = 0; h < nroot; ++h) P.born[slot_base(P, s) + h] = h;
    P.flags[s] = P.seed_y ? kFlagSeed : 0;
    if (P.seed_y) P.seed_d[s] = D;
    P.state[s] = SLOT_ACTIVE;
  }
}

// ---------------------------------------------------------------- children
// slot of a work item: woff is an exclusive prefix over slots
__device__ inline int item_slot(const Problem &P, int w) {
  int lo = 0, hi = P.W;  // woff[lo] <= w < woff[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (P.woff[mid] <= w) lo = mid; else hi = mid;
  }
  return lo;
}

// Work item r of slot s: split the selected leaf into its four children.
// tab: the table of the slot's parameter row (LDS or global memory).
template <int L, int GRAM>
__device__ void do_item(WaveLds<L> &S, const Problem &P, const int *pidmap, const int *podd, int s, int r,
                        const double *tab) {
  const Ctr C = P.sctr[s];
  const Entry E = P.entries[C.entry];
  // the pool and the deltas hold P.MU form-factor pairs (<= the box pairs)
  constexpr int KMAX = (Dims<L>::MU + 63) / 64;
  const int MU = P.MU;
  const int lane = lane_id();
  const long leaf = P.sel[(long)s * P.bmax + r];
  const long nold = P.nleaf[s];
  const long pbase = slot_base(P, s) + leaf;
  const uint64_t pc = P.code[pbase];
  const double pkey = P.key[pbase];
  // delta of the container sums: minus the parent, plus its children
  double dv[KMAX], dp[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    int pid = lane + 64 * k;
    dv[k] = (pid < MU) ? -P.Q[pbase * MU + pid] : 0.0;
    dp[k] = (pid < MU && P.E) ? -(double)P.E[pbase * MU + pid] : 0.0;
  }
  const int d = code_depth(pc);
  const uint64_t ix = code_ix(pc), iy = code_iy(pc);
  // children that the seed tree splits again become placeholders (uniform
  // in the wave); a parent with four of them needs no integrand values
  int skip = 0;
  if (P.seed_y && (P.flags[s] & kFlagSeed)) {
    for (int ch = 0; ch < 4; ++ch)
      if (seed_split(P, s, make_code(d + 1, 2 * ix + (ch & 1), 2 * iy + (ch >> 1)))) skip |= 1 << ch;
  }
  const double wdt = kTwoPi * ldexp(1.0, -d);
  const double x0 = -kPi + (double)ix * wdt, y0 = -kPi + (double)iy * wdt;
  if (skip != 15) {
    fill_nodes<L>(S, P, C, E, tab, kNX, x0, y0, wdt);
    if (GRAM == kSep) sep_stage1<L>(S, kNX, 2);
    if constexpr (GRAM == kSep && kXsumsAll<L>) sep_xsums_all<L>(S);
  }
  const double fa = (0.25 * wdt) * (0.25 * wdt) / (4.0 * kPi * kPi);
  double dkey = -pkey;
#pragma unroll 1
  for (int ch = 0; ch < 4; ++ch) {
    int cx = ch & 1, cy = ch >> 1;
    long ri = (ch == 0) ? leaf : nold + 3L * r + (ch - 1);
    const uint64_t cc = make_code(d + 1, 2 * ix + cx, 2 * iy + cy);
    if (P.born && lane == 0)  // the split is the container's st_splits-th (one per round)
      P.born[slot_base(P, s) + ri] = (unsigned int)(1 + 4 * P.st_splits[s] + ch);
    if ((skip >> ch) & 1) {
      store_zero<L>(P, s, ri, cc);
      wave_sync();
      continue;
    }
    if constexpr (GRAM == kSep) {
      if (P.ff_identity) {
        // Box-basis pairs straight from the x-sums into the child's record and
        // the parent's delta.  Staged in LDS, the 325 pairs of the 25-function
        // box took 5 KB of a wave's 19, and six waves a CU instead of ten.
        const double *G2, *G1;
        if constexpr (kXsumsAll<L>) {
          G2 = S.g2b[ch];
          G1 = S.g1b[ch];
        } else {
          sep_xsums<L>(S, cx, cy);
          G2 = S.g2;
          G1 = S.g1;
        }
        const long base = slot_base(P, s) + ri;
        double part = 0.0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
          const int pid = lane + 64 * k;
          if (pid < MU) {
            const int jk = pidmap[pid];
            double f = fa, fe = fa;
            if (P.sym || P.mirror) f = podd[pid] ? 0.0 : 2.0 * fa;
            if (P.sym || P.mirror) fe = P.mirror ? 2.0 * fa : f;
            const double q2 = G2[jk], q = f * q2, e = fabs(fe * (q2 - G1[jk]));
            P.Q[base * MU + pid] = q;
            if (P.E) P.E[base * MU + pid] = err_f32(e);
            part += (P.err_mode != 0) ? e * (double)P.itau[(long)s * MU + pid] : e;
            dv[k] += q;
            dp[k] += (double)err_f32(e);
          }
        }
        const double key = wave_sum(part);
        if (lane == 0) {
          P.key[base] = key;
          P.code[base] = cc;
        }
        dkey += key;
        wave_sync();
        continue;
      }
    }
    eval_rect<L, GRAM>(S, P, pidmap, podd, kNX, cx, cy, fa, true);
    dkey += store_region<L>(S, P, s, ri, cc);
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      int pid = lane + 64 * k;
      if (pid < MU) {
        dv[k] += S.cq[pid];
        // the same float-rounded value that is stored and later subtracted,
        // so the running per-pair error sums carry no rounding residue
        dp[k] += (double)err_f32(fabs(S.ce[pid]));
      }
    }
    wave_sync();
  }
  const long it = (long)s * P.bmax + r;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    int pid = lane + 64 * k;
    if (pid < MU) {
      P.dv[it * MU + pid] = dv[k];
      if (P.dep) P.dep[it * MU + pid] = dp[k];
    }
  }
  if (lane == 0) {
    P.de[it] = dkey;
    if (P.ifill) P.ifill[it] = skip != 15;
  }
}

// parameter row of slot s
__device__ inline int slot_entry(const Problem &P, int s) { return P.sctr[s].entry; }

// The problem description of a kernel whose only argument is a Problem, read
// through a pointer into the kernel-argument segment that the compiler cannot
// follow across loop iterations: its fields are then loaded (scalar loads
// from the constant cache) where an item uses them, instead of being held in
// scalar registers across the whole item loop, which overflowed them into
// vector-register lanes.
__device__ inline const Problem &kernarg_problem(const Problem &P) {
#ifdef __HIP_DEVICE_COMPILE__
  typedef const __attribute__((address_space(4))) Problem CP;
  CP *pk = (CP *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(pk));
  return *(const Problem *)pk;
#else
  return P;
#endif
}

// The next chunk (share.h), the same in every thread (two workgroup barriers).
// A counter rather than sixteen generations of workgroups with ranges shrinking
// by index: those paid the start of a workgroup - its table, its search for the
// first slot - sixteen times a round, 80 us a launch for rounds of 300 items.
__device__ inline Span next_chunk(const Problem &P, int *sh) {
  __syncthreads();  // every wave is done with the last chunk (and with sh)
  if (threadIdx.x == 0) {
    const int total = P.counters[2], waves = blockDim.x >> 6, grid = gridDim.x;
    const long base = chunk_base(total, waves, grid);
    Span k = {total, total};
    if (base < total) {
      const int seen = (int)base + __hip_atomic_load(&P.counters[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (seen < total) {
        const int c = chunk_items(total - seen, waves, grid);
        k = counted_span((int)base, total, atomicAdd(&P.counters[3], c), c);
      }
    }
    sh[0] = k.i0;
    sh[1] = k.i1;
  }
  __syncthreads();
  Span k;
  k.i0 = __builtin_amdgcn_readfirstlane(sh[0]);
  k.i1 = __builtin_amdgcn_readfirstlane(sh[1]);
  return k;
}

// Each workgroup takes contiguous chunks of work items; its waves take every
// nw-th item of one, so at any time they work on neighbouring parents, mostly
// of one container and parameter row.  A chunk is cut into segments of
// consecutive slots of one parameter row (usually a single one); at the
// start of a segment the workgroup stages that row's table in LDS (two
// barriers), and inside a segment there is no workgroup barrier: each wave
// runs through its items on its own.  The slot of an item is found by a
// search only when the wave's items leave the current slot's range.
template <int L, int GRAM>
__global__ void __launch_bounds__(GRAM == kSep ? 512 : 256) k_children(Problem P) {
  extern __shared__ double lds_raw[];
  __shared__ int pidmap[Dims<L>::MU], podd[Dims<L>::MU];
  double *tabl = lds_raw;
  // the wave index is uniform in a wave: keep it (and all per-item
  // bookkeeping derived from it) in scalar registers
  const int nw = blockDim.x >> 6, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  WaveLds<L> &S = *reinterpret_cast<WaveLds<L> *>(lds_raw + (size_t)P.close_doubles +
                                                  (size_t)wv * P.lds_wave_doubles);
  __shared__ int next[2];
  Span k = first_chunk(P.counters[2], nw, gridDim.x, blockIdx.x);
  if (k.i0 >= k.i1) return;  // uniform in the workgroup
  build_pidmap<L>(pidmap, podd, threadIdx.x, blockDim.x);
  int loaded = -1;
#pragma unroll 1
  for (; k.i0 < k.i1; k = next_chunk(P, next)) {
  const int i1 = k.i1;
  int s = item_slot(P, k.i0), lo = P.woff[s], hi = P.woff[s + 1];  // current slot, its items
  int w = k.i0 + wv, seg = k.i0;
#pragma unroll 1
  while (seg < i1) {
    // segment [seg, seg_hi): slots from s on while they hold items of row e
    // (slots without items are passed over)
    const int e = slot_entry(P, s);
    int t = s + 1;
    while (t < P.W && P.woff[t] < i1 && (P.woff[t + 1] == P.woff[t] || slot_entry(P, t) == e)) ++t;
    const int seg_hi = (t < P.W && P.woff[t] < i1) ? P.woff[t] : i1;
    if (e != loaded) {
      __syncthreads();  // every wave is done with the previous table
      const Entry E0 = P.entries[e];
      const double *src = P.tab + E0.tab_off + (long)E0.JV * kValStride;
      const int nt = close_doubles(E0);
      for (int i = threadIdx.x; i < nt; i += blockDim.x) tabl[i] = src[i];
      __syncthreads();
      loaded = e;
    }
#pragma unroll 1
    for (; w < seg_hi; w += nw) {
      if (w >= hi) {  // find the slot holding item w (woff is non-decreasing)
        int a = s + 1, b = P.W;  // woff[a] <= w < woff[b]
        while (b - a > 1) {
          const int mid = (a + b) >> 1;
          if (P.woff[mid] <= w) a = mid; else b = mid;
        }
        s = a;
        lo = P.woff[s];
        hi = P.woff[s + 1];
      }
      do_item<L, GRAM>(S, kernarg_problem(P), pidmap, podd, s, w - lo, tabl);
    }
    // the next segment starts at slot t (its first item is seg_hi)
    seg = seg_hi;
    if (seg < i1) {
      s = t;
      lo = P.woff[s];
      hi = P.woff[s + 1];
    }
  }
  }
}

// ---------------------------------------------------------------- two lanes per child
// Region evaluation for form factors over the 9-function box (L <= 1) with the
// separable FP64 projection, arranged so that every sum stays in registers: a
// wave holds 8 work items (parents); lane 8 it + 2 ch + h evaluates child ch of
// item it together with its partner lane (h = 0, 1).  Every pair of form
// factors of a rectangle is a combination of the 25 product integrals I_jk =
// int g phi_j(x) phi_k(y).  Lane h = 0 accumulates I for the fine rule (Q_2N);
// lane h = 1 accumulates the same sums with the weight difference of the two
// rules (E = Q_2N - Q_N, the error estimate), so the key of the child (sum over
// pairs of |E|) needs no lanes but its own.
// The two lanes of a child share its 81 nodes column by column: lane 0
// takes columns 0-3 and rows 0-4 of column 4, lane 1 columns 8-5 and rows
// 5-8 of column 4; after each column the partners swap their y-sums so
// that each adds both columns to its x-sums.  Nodes on the edges shared by
// neighbouring children are evaluated once per child (324 evaluations for
// the 289 distinct nodes of a parent).
// What bounds it: LDS bandwidth and the latency of a node's LDS round trip (two
// table rows of nine doubles and the row's cosine and sine), with three waves
// per SIMD to cover it.  Nine form factors at one scale on 24 x 24 momenta: 1.8
// ns a stored parent, with its mirror image 0.9 ns (2.8 ns with rows of degree
// 13, 45 pairs a record stored lane by lane, and no mirror images).
namespace lpc {

constexpr int kItems = 8;              // work items per wave
constexpr int kYRow = 2;               // doubles per node row: cos y, sin y
// the 9 node rows of one child row: 144 bytes, so that the 16-byte rows that
// the 16 child rows of a wave read at one time cover all 64 banks once
constexpr int kYBlock = kNF * kYRow;
constexpr int kYRows = kItems * 2 * kYBlock;  // per-wave LDS: rows of both child rows,
// then what a column starts from, per child: cos and sin of its centre in x and
// of l/2 (odd stride; read anew for each column rather than held in 12 registers)
constexpr int kCol = 7;
constexpr int kYDoubles = kYRows + 4 * kItems * kCol;
// records are staged in LDS, kStage values of each of the wave's 32 children at
// a time (an odd stride: the children's lanes write to distinct banks)
// a wide group holds its vectors behind its 18 node rows and behind the columns
constexpr int kWideOwn = 64, kWideSend = 512;
static_assert(kWideOwn >= 2 * kYBlock && kWideOwn + 200 <= kYRows && kWideSend >= kYDoubles, "wide groups' vectors");
constexpr int kChildren = 4 * kItems;
constexpr int kStage = kProd;
static_assert(kStage & 1, "bank spread of the staged records");
// per-wave LDS: the node rows while the sums run, then in the same space the
// staged records (errors of the box basis after its values; of a general set
// beside them); behind it the children's and items' places and the key weights
__host__ __device__ constexpr int area_doubles(bool with_e, bool general) {
  const int rec = kChildren * kStage + (with_e && general ? kChildren * kStage / 2 : 0);
  return rec > kYDoubles ? rec : kYDoubles;
}
__host__ __device__ constexpr int wave_doubles(bool with_e, bool with_w, bool general) {
  return area_doubles(with_e, general) + kChildren + kItems + (with_w ? kItems * kPairs9 / 2 : 0);
}
static_assert(kChildren * kPairs9 / 2 <= kChildren * kStage, "the box basis' errors fit in the area");

// sum of v over the four children of the item, the same in all lanes of the
// item with the same h: ((c0 + c1) + (c2 + c3)) with a + b = b + a exactly
__device__ inline double child_sum(double v) {
  v += dpp_move<0x4E>(v);                 // quad_perm [2,3,0,1]: child ch ^ 1, same h
  const double o = dpp_move<0x141>(dpp_move<0xB1>(v));  // lane ^ 1, then 7 - lane: other quad, same h
  return v + o;
}

__device__ inline double swap_h(double v) { return dpp_move<0xB1>(v); }  // partner lane (h ^ 1)

}  // namespace lpc

// What a group needs of its lane's item (items past the group's end repeat the
// last one and store nothing).
struct LpcItem {
  int s, r;       // slot, place in its selection
  uint64_t pc;    // parent's code
  int ch;         // channel
  double cLx, sLx, cLy, sLy;
};

// The slot holding item g (woff[s] <= g < woff[s + 1]; woff is non-decreasing),
// the same in every lane: each step splits the range in 64 by one load per
// lane, two or three dependent loads instead of the eleven of a binary search
// over a thousand slots (each one the latency of L2 or beyond).
__device__ inline int wave_slot(const Problem &P, int g) {
  const int lane = lane_id();
  int lo = 0, hi = P.W;
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6, i = lo + (lane + 1) * step;
    const int c = __popcll(__ballot(i < hi && P.woff[i] <= g));
    lo += c * step;
    hi = min(lo + step, hi);
  }
  return lo;
}

// The items of a group, one per eight lanes: w is the lane's item, g0 the first
// of the group.  The slots of the eight items follow from one load of the next
// 64 offsets.
__device__ inline LpcItem lpc_item(const Problem &P, int g0, int w) {
  const int lane = lane_id();
  int s = wave_slot(P, g0);
  const int next = min(s + 1 + lane, P.W);
  const int off = P.woff[next];
  int mine = 0;
#pragma unroll
  for (int i = 0; i < lpc::kItems; ++i) {  // offsets at or below each lane group's item
    const int c = __popcll(__ballot(off <= __shfl(w, 8 * i, 64)));
    if (i == lane >> 3) mine = c;
  }
  // (every lane takes part in the exchange: an idle lane's value reads as zero)
  const int first = P.woff[s], prev = __shfl(off, max(mine - 1, 0), 64);
  int lo = mine ? prev : first;
  s += mine;
  while (mine == 64 && P.woff[s + 1] <= w) lo = P.woff[++s];  // (more than 63 empty slots between two items)
  LpcItem q;
  q.s = s;
  q.r = w - lo;
  q.pc = P.selc[(long)s * P.bmax + q.r];
  const Ctr C = P.sctr[s];
  q.ch = C.ch;
  q.cLx = C.cLx;
  q.sLx = C.sLx;
  q.cLy = C.cLy;
  q.sLy = C.sLy;
  return q;
}

// End of the run of items from slot s on that belong to one parameter row e,
// at most i1, the same in every lane (slots without items are passed over)
__device__ inline int row_end(const Problem &P, int s, int e, int i1) {
  if (P.one_row) return i1;
  const int lane = lane_id();
  for (int t0 = s + 1; t0 < P.W; t0 += 64) {
    const int t = t0 + lane;
    const int lo = t < P.W ? P.woff[t] : i1, up = t < P.W ? P.woff[t + 1] : i1;
    const bool other = lo < i1 && up > lo && P.sctr[t].entry != e;
    const unsigned long long m = __ballot(other), past = __ballot(lo >= i1);
    if (m) return __shfl(lo, __ffsll((long long)m) - 1, 64);
    if (past) break;
  }
  return i1;
}

// How the items are shared out: a share of the XCD's items per workgroup, by
// index and then from the XCD's counter (share.h; the hardware places the
// workgroups b = x mod 8 on XCD x; one counter for all is a queue of thousands of
// atomics on one address: 50k cycles a wait); within a workgroup the waves take
// groups of eight items from its range, a run of one parameter row.  A wave that
// finds the range empty takes the next one for all (the lock), while the others
// finish their groups: no barrier until another row's table is needed or the
// items are gone.  (With a barrier at every chunk the waves of one flow scale's
// rounds spent 37% of their time waiting, 60% in the per-integral mode.)
struct LpcShare {
  unsigned long long range;  // range_word
  int lock;
  int mode;                  // 0: run, 1: another row's table, 2: no items left
  int row;                   // the next range and its row (mode 1)
  Span next;
  int rest, end;             // what is left of the chunk behind the range
  int base, total;           // the XCD's items behind the first chunks
  int group;                 // items per group
};

// Items per group: eight, or one where that leaves no wave a second group
// (P.wide_items: the waves of the grid).  A
// round of few items is bound by the latency of one group, 41 nodes one after
// the other in each lane; a wide group's lanes take one column each, 14 nodes
// (30k -> 13k clocks of a launch of 57k).  With twice as many items the eight
// lane groups of a common group are the better use of the wave: five form
// factors on 8x8 momenta take 666 us with this rule, 684 with twice and 742
// with four times as many items, 700 without wide groups.  (One momentum: 434
// -> 381 us.)
__device__ inline int group_items(const Problem &P, int total) { return total <= P.wide_items ? 1 : lpc::kItems; }

// the next range of this workgroup (one wave): of the present chunk, or of a
// new one from the counter
__device__ inline void next_range(const Problem &P, LpcShare &sh, int loaded) {
  const int lane = lane_id();
  Span k = {sh.rest, sh.end};
  if (k.i0 >= k.i1) {
    if (lane == 0 && sh.base < sh.total) {
      int *count = P.xcount + (blockIdx.x % min(kXcds, (int)gridDim.x)) * kXcdStride;
      const int seen = sh.base + __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (seen < sh.total) {
        const int c = share_items(sh.total - seen, sh.group, gridDim.x, kXcds);
        k = counted_span(sh.base, sh.total, atomicAdd(count, c), c);
      }
    }
    k.i0 = __builtin_amdgcn_readfirstlane(k.i0);
    k.i1 = __builtin_amdgcn_readfirstlane(k.i1);
  }
  if (k.i0 >= k.i1) {
    if (lane == 0) sh.mode = 2;
    return;
  }
  const int s = wave_slot(P, k.i0), e = __builtin_amdgcn_readfirstlane(P.sctr[s].entry);
  const int hi = row_end(P, s, e, k.i1);
  if (lane == 0) {
    sh.rest = hi;
    sh.end = k.i1;
    if (e == loaded) {
      atomicExch(&sh.range, range_word({k.i0, hi}));
    } else {
      sh.row = e;
      sh.next = {k.i0, hi};
      sh.mode = 1;
    }
  }
}

// a group of items for this wave: its first item (end: the one behind its last), or -1
// when the workgroup needs another table or has no items left
__device__ inline int take_group(const Problem &P, LpcShare &sh, int loaded, int &end) {
  const int lane = lane_id();
  for (;;) {
    unsigned long long r = 0;
    int mode = 0;
    if (lane == 0) {
      r = __hip_atomic_load(&sh.range, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (!range_empty(r)) r = atomicAdd(&sh.range, (unsigned long long)sh.group);
      mode = __hip_atomic_load(&sh.mode, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)r);
    const unsigned long long ru =
        ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)(r >> 32)) << 32) | lo;
    if (!range_empty(ru)) {
      const Span k = range_group(ru, __builtin_amdgcn_readfirstlane(sh.group));
      end = k.i1;
      return k.i0;
    }
    if (__builtin_amdgcn_readfirstlane(mode)) return -1;
    int mine = 0;
    if (lane == 0) mine = atomicCAS(&sh.lock, 0, 1) == 0;
    if (__builtin_amdgcn_readfirstlane(mine)) {
      // (another wave may have taken a range since)
      int empty = 0;
      if (lane == 0) {
        const unsigned long long q = __hip_atomic_load(&sh.range, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        empty = range_empty(q) &&
                __hip_atomic_load(&sh.mode, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      if (__builtin_amdgcn_readfirstlane(empty)) next_range(P, sh, loaded);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if (lane == 0) atomicExch(&sh.lock, 0);
    } else {
      __builtin_amdgcn_s_sleep(4);  // (the holder is a running wave and ends its turn)
    }
  }
}

// the rule in LDS: node offsets (cos, sin) of every depth, then the fine and the
// coarse weights of the nine nodes
constexpr int kDelWeights = kDelDepths * 10, kDelDoubles = kDelWeights + 2 * kNF;

__device__ inline double rule_value(int i) {
  if (i < kDelWeights) return i % 10 < 5 ? c_rule.cdel[i / 10][i % 10] : c_rule.sdel[i / 10][i % 10 - 5];
  i -= kDelWeights;
  return i < kNF ? c_rule.w2[i] : ((i - kNF) & 1) ? 0.0 : c_rule.w1[(i - kNF) >> 1];
}

// a parameter row's constants, in scalar registers (energies in units of w = pi T)
struct LpcRow {
  double mt2, mtp4, mmu;
  int J, JV;
};

// a value that is the same in every lane, held in scalar registers
__device__ inline double wave_uniform(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)b);
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// row of element e of a staged block [rows][n]: e / n (a constant for the box
// basis; e < 800 and n <= 25 otherwise, where the rounded product is exact)
template <bool GEN>
__device__ inline int stage_row(int e, int n, float inv_n) {
  return GEN ? (int)(((float)e + 0.5f) * inv_n) : e / kProd;
}

// One group of up to 8 work items of one parameter row (row R, its tables tab,
// the node offsets del and the pairs' coefficients co in LDS, the wave's LDS at
// Yw), first item g0; items g0 + it >= gend are inactive (their lanes repeat the
// last item and store nothing).  cur: the lane's item; on return g0, gend and
// cur are those of the wave's next group (take), g0 = -1 if there is none.  The
// next group's items, and the parents' values, are read before this group's records are stored: loads and stores of a wave complete
// in order, so a load behind the stores would wait until they have reached L2.
// Between its stores and the end of the next node loop a wave reads LDS only.
// BUB: the bubble integrands (kinds 0 and 1); otherwise the unit integrand.
// WE: per-pair errors are stored (FP32 records and deltas); otherwise the
// children's errors only form their keys.  WW: the keys weigh the pairs
// (per-integral and weighted modes); otherwise they are plain sums.  GEN:
// general form factors (pairs from P.pcoef); otherwise the box basis itself,
// whose leaves hold the product integrals.  MIX: P.mixed (a kernel of its own:
// as a branch of the pairs' loop it cost every general set 1 of 33 us a launch).
template <bool BUB, bool WE, bool WW, bool GEN, bool MIX>
__device__ void lpc_group(const Problem &P, const LpcRow &R, const double *tab, const double *del,
                          const double *co, double *Yw, LpcShare &share, int loaded, bool wide, int &g0, int &gend,
                          LpcItem &cur) {
  using namespace lpc;
  Entry E;
  E.J = R.J;
  E.JV = R.JV;
  const double mt2 = R.mt2, mtp4 = R.mtp4, mmu = R.mmu;
  // the lane's place, formed anew for every group rather than held in
  // registers across the kernel's loops
  int lane = lane_id();
  asm volatile("" : "+v"(lane));
  const int it = lane >> 3, ch = (lane >> 1) & 3, h = lane & 1;
  const int cx = ch & 1, cy = ch >> 1;
  const int MU = P.MU;

  // ---- the items: placeholders, node rows
  const int d = code_depth(cur.pc), chl = cur.ch;
  double *col = Yw + kYRows + (lane >> 1) * kCol;
  // slot, place and code of the items, for the records
  uint64_t *home = reinterpret_cast<uint64_t *>(Yw + lpc::area_doubles(WE, GEN));
  if ((lane & 7) == 0) {
    home[2 * it] = ((uint64_t)(unsigned)cur.s << 32) | (unsigned)cur.r;
    home[2 * it + 1] = cur.pc;
  }
  unsigned long long pm;
  bool wave_skip;
  {
    const uint64_t ix = code_ix(cur.pc), iy = code_iy(cur.pc);
    const uint64_t ccode = make_code(d + 1, 2 * ix + cx, 2 * iy + cy);
    // seed phase: children the seed tree splits again are placeholders
    const bool valid = g0 + it < gend;
    const bool phc = P.seed_y && (P.flags[cur.s] & kFlagSeed) && seed_split(P, cur.s, ccode);
    pm = __ballot(phc && valid);
    wave_skip = pm == __ballot(valid);  // every child of the group is one
    // trigonometric values of the nodes by angle addition: node a of a child
    // lies at offset delta_a (a table per depth) from the child's centre,
    // whose sine and cosine each lane pair forms once (lane 0 for x, lane 1
    // for y)
    if (!wave_skip) {
      const double wdt = kTwoPi * ldexp(1.0, -d);
      const double xm = -kPi + (double)ix * wdt + (0.25 + 0.5 * cx) * wdt;
      const double ym = -kPi + (double)iy * wdt + (0.25 + 0.5 * cy) * wdt;
      double c1, s1;
      sincos_zone(h ? ym : xm, &s1, &c1);
      if (h == 0) {
        col[0] = c1;
        col[1] = s1;
        col[2] = cur.cLx;
        col[3] = cur.sLx;
        col[4] = cur.cLy;
        col[5] = cur.sLy;
      }
      // rows of both child rows of every item
#pragma unroll 1
      for (int t0 = 0; t0 < (wide ? 1 : kItems * 2 * kNF); t0 += 64) {
        // every lane takes part in the exchanges; lanes past the last row idle after them
        const int t = t0 + lane, ti = min(t / (2 * kNF), kItems - 1);
        const int rem = t - ti * (2 * kNF), tcy = min(rem / kNF, 1), b = rem - tcy * kNF;
        const int src = 8 * ti + 4 * tcy + 1;  // lane 1 of child (0, tcy) of item ti
        const double cm = __shfl(c1, src, 64), sm = __shfl(s1, src, 64);
        const int td = __shfl(d, 8 * ti, 64);
        if (t >= (wide ? 2 * kNF : kItems * 2 * kNF)) continue;
        const int bb = b < 5 ? b : 8 - b;
        const double cd = del[td * 10 + bb];
        const double sd = b < 5 ? del[td * 10 + 5 + bb] : -del[td * 10 + 5 + bb];
        double *row = Yw + (ti * 2 + tcy) * kYBlock + b * kYRow;
        row[0] = cm * cd - sm * sd;  // cos y
        row[1] = sm * cd + cm * sd;  // sin y
      }
    }
  }
  wave_sync();

  // ---- the integrand and the sums
  const double *Yc = Yw + ((wide ? 0 : it) * 2 + cy) * kYBlock;
  const unsigned sgn_ch = chl ? 0u : 0x80000000u;  // pp takes -b
  double I[5][5];
#pragma unroll
  for (int j = 0; j < 5; ++j)
#pragma unroll
    for (int k = 0; k < 5; ++k) I[j][k] = 0.0;

  // cos and sin of column a of this lane's child
  auto column_trig = [&](int a, double &cxv, double &sx) {
    const int aa = a < 5 ? a : 8 - a;
    const double cd = del[d * 10 + aa], sd = a < 5 ? del[d * 10 + 5 + aa] : -del[d * 10 + 5 + aa];
    const double cxm = col[0], sxm = col[1];
    cxv = fma(cxm, cd, -(sxm * sd));  // (the same rounding wherever it is used)
    sx = fma(sxm, cd, cxm * sd);
  };
  // y-sums of column a over N nodes, of {1, c, s, c^2, c s} (c, s the node's
  // cosine and sine in y; the sums of phi follow from them, linearly, at the
  // end) with the fine (H2) and the coarse (H1) weights: rows i = 0..8 (N = 9),
  // or the lane's part of a column that both lanes share, rows 0..4 (h = 0) or
  // 8..5 (h = 1; the weights are symmetric) (N = 5).  The loop over the nodes
  // is unrolled: weights, row offsets and the rows without a coarse weight are
  // then known, and the loads of a node (both table rows and the next node's
  // cosine and sine) are issued together and waited for once; left to itself
  // the compiler loads a coefficient pair, waits, uses it and loads the next,
  // ten LDS round trips in a row per node.  What bounds the loop is LDS
  // bandwidth (160 bytes a node and lane at 128 bytes a clock, plus the bank
  // conflicts of the table rows), so a node's energies are formed from c and s
  // by two FMAs each instead of being read as cosines with phi_1..4 (48
  // bytes).  Close pairs are marked and summed after the loop.
  auto column = [&](int a, auto count, double (&H2)[5], double (&H1)[5]) {
    constexpr int N = decltype(count)::value;
    double cxv, sx;
    column_trig(a, cxv, sx);
    const double cLx = col[2], sLx = col[3], cLy = col[4], sLy = col[5];
    const double Cx = cLx * cxv - sLx * sx, Dx = cLx * cxv + sLx * sx;
    // the energies along the column are affine in the row's cosine
    // cos(l_y/2 +- y) = cLy c -+ sLy s:
    // -2t (Cx + py) - 4t' Cx py - mu = (-2t Cx - mu) + py (-2t - 4t' Cx)
    const double Aa = fma(mt2, Cx, mmu), Ba = fma(mtp4, Cx, mt2);
    const double Ab = fma(mt2, Dx, mmu), Bb = fma(mtp4, Dx, mt2);
    const double Pa = Ba * cLy, Qa = -Ba * sLy, Pb = Bb * cLy, Qb = Bb * sLy;
    const double *first = (N < kNF && h) ? Yc + 8 * kYRow : Yc;
    const int rstep = (N < kNF && h) ? -kYRow : kYRow;
    auto add = [](double (&H)[5], double g, double c, double s) {
      const double gc = g * c;
      H[0] += g;
      H[1] += gc;
      H[2] = fma(g, s, H[2]);
      H[3] = fma(gc, c, H[3]);
      H[4] = fma(gc, s, H[4]);
    };
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      H2[k] = 0.0;
      H1[k] = 0.0;
    }
    unsigned close = 0;
    double cn = first[0], sn = first[1];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const double c = cn, s = sn;
      double g = 1.0;  // PAID_UNIT
      if (i + 1 < N) {
        cn = first[(i + 1) * rstep];
        sn = first[(i + 1) * rstep + 1];
      }
      if constexpr (BUB) {
        const double ea = fma(c, Pa, fma(s, Qa, Aa)), eb = fma(c, Pb, fma(s, Qb, Ab));
        const PairNode n = pair_node(E, tab, sgn_ch, ea, eb, cn, sn);
        const bool cl = n.close;
        close |= cl ? 1u << i : 0u;
        g = cl ? 0.0 : n.s;
      }
      if (N < kNF && i == N - 1) g = h ? 0.0 : g;  // the middle row is lane 0's
      add(H2, c_rule.w2[i] * g, c, s);
      if (!(i & 1)) add(H1, c_rule.w1[i >> 1] * g, c, s);
    }
    if constexpr (BUB) {
      if (N < kNF && h) close &= (1u << (N - 1)) - 1u;
      while (close) {
        const int i = __ffs(close) - 1;
        close &= close - 1;
        const double c = first[i * rstep], s = first[i * rstep + 1];
        const double g = pair_close(E, tab, sgn_ch, fma(c, Pa, fma(s, Qa, Aa)), fma(c, Pb, fma(s, Qb, Ab)));
        add(H2, del[kDelWeights + i] * g, c, s);
        add(H1, del[kDelWeights + kNF + i] * g, c, s);
      }
    }
  };
  // phi_j at column a
  auto column_basis = [&](int a, double (&px)[5]) {
    double cxv, sx;
    column_trig(a, cxv, sx);
    px[0] = 1.0;
    px[1] = kSqrt2 * cxv;
    px[2] = kSqrt2 * sx;
    px[3] = (cxv - sx) * (cxv + sx);
    px[4] = 2.0 * sx * cxv;
  };
  // x-sums of one column from its y-sum vector dk: lane 0 adds the fine
  // rule's sums (wf H2), lane 1 fine minus coarse (wf H2 - wc H1)
  auto xsum = [&](const double (&dk)[5], const double (&px)[5]) {
#pragma unroll
    for (int k = 0; k < 5; ++k) I[0][k] += dk[k];
#pragma unroll
    for (int j = 1; j < 5; ++j)
#pragma unroll
      for (int k = 0; k < 5; ++k) I[j][k] = fma(px[j], dk[k], I[j][k]);
  };
  // the y-sum vectors of this lane's column a: its own (dk) and the one that
  // the partner needs (sk)
  auto sums = [&](int a, auto count, double wf, double wc, double (&dk)[5], double (&sk)[5]) {
    double H2[5], H1[5];
    column(a, count, H2, H1);
    if (decltype(count)::value < kNF) {  // both lanes hold part of the same column: add the parts
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        H2[k] += lpc::swap_h(H2[k]);
        H1[k] += lpc::swap_h(H1[k]);
      }
    }
    const double wown = h ? wc : 0.0, wsend = h ? 0.0 : wc;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      dk[k] = fma(wf, H2[k], -wown * H1[k]);
      sk[k] = fma(wf, H2[k], -wsend * H1[k]);
    }
  };

  if (!wave_skip) {
    // Columns s (lane 0) and 8 - s (lane 1), s = 0..3: the CC weights are
    // symmetric, so both columns of a step carry the same weights.  In a wide
    // group, whose one item every lane group repeats, lane group s takes step s
    // and its vectors go to LDS.
    double *Vd = Yw + kWideOwn, *Vs = Yw + kWideSend, *V4 = Vs + 160, *T = Vd;
#pragma unroll 1
    for (int st = 0; st < (wide ? 1 : 4); ++st) {
      const int u = wide ? min(it, 3) : st, a = h ? 8 - u : u;
      double dk[5], sk[5], px[5];
      sums(a, std::integral_constant<int, kNF>{}, del[kDelWeights + u], del[kDelWeights + kNF + u], dk, sk);
      if (wide) {
        if (it < 4)
#pragma unroll
          for (int k = 0; k < 5; ++k) {
            Vd[((lane & 7) * 4 + it) * 5 + k] = dk[k];
            Vs[((lane & 7) * 4 + it) * 5 + k] = sk[k];
          }
      } else {
        column_basis(a, px);
        xsum(dk, px);
#pragma unroll
        for (int k = 0; k < 5; ++k) sk[k] = lpc::swap_h(sk[k]);
#pragma unroll
        for (int j = 1; j < 5; ++j) px[j] = lpc::swap_h(px[j]);
        xsum(sk, px);
      }
    }
    {  // column 4: rows 0-4 on lane 0, rows 8-5 on lane 1
      double dk[5], sk[5], px[5];
      sums(4, std::integral_constant<int, 5>{}, c_rule.w2[4], c_rule.w1[2], dk, sk);
      if (wide) {
        if (it == 0)
#pragma unroll
          for (int k = 0; k < 5; ++k) V4[(lane & 7) * 5 + k] = dk[k];
      } else {
        column_basis(4, px);
        xsum(dk, px);
      }
    }
    if (wide) {
      // lane group k adds up the sums with index k, in the order of the steps
      const int k = min(it, 4), q = lane & 7;
      wave_sync();
      double acc[5], px[5];
#pragma unroll
      for (int j = 0; j < 5; ++j) acc[j] = 0.0;
      auto more = [&](double v, int a) {
        column_basis(a, px);
        acc[0] += v;
#pragma unroll
        for (int j = 1; j < 5; ++j) acc[j] = fma(px[j], v, acc[j]);
      };
#pragma unroll 1
      for (int st = 0; st < 4; ++st) {
        more(Vd[(q * 4 + st) * 5 + k], h ? 8 - st : st);
        more(Vs[((q ^ 1) * 4 + st) * 5 + k], h ? st : 8 - st);
      }
      more(V4[q * 5 + k], 4);
      wave_sync();
      if (it < 5)
#pragma unroll
        for (int j = 0; j < 5; ++j) T[q * 25 + 5 * j + k] = acc[j];
      wave_sync();
#pragma unroll
      for (int j = 0; j < 5; ++j)
#pragma unroll
        for (int k2 = 0; k2 < 5; ++k2) I[j][k2] = T[q * 25 + 5 * j + k2];
    }
    // from {1, c, s, c^2, c s} to phi in y
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      I[j][1] *= kSqrt2;
      I[j][2] *= kSqrt2;
      I[j][3] = fma(2.0, I[j][3], -I[j][0]);
      I[j][4] *= 2.0;
    }
  }
  // the item's bookkeeping is read again below rather than held in
  // registers across the loops above
  asm volatile("" ::: "memory");

  // ---- records.  Lane 0 of a child holds its Q_2N, lane 1 its E.  Values pass
  // through LDS, so that consecutive lanes store consecutive doubles of a
  // record (children of neighbouring items are neighbours in the pool) and the
  // items' deltas (children minus parent) are sums over the staged values.
  // Stored straight from the lanes, each value is a write of its own in L2 (32
  // lanes, 32 records): 236 requests a parent kept L2 busy 95% of the time.
  const bool valid = g0 + it < gend;
  const uint64_t place = home[2 * it], pc = home[2 * it + 1];
  const int item_s = (int)(place >> 32), item_r = (int)(unsigned)place;
  const long sbase = slot_base(P, item_s);
  const long itm = (long)item_s * P.bmax + item_r;
  const long leaf = P.sel[itm];
  const long nold = P.nleaf[item_s];
  double pkey = P.key[sbase + leaf];
  // the next group's items (cleared otherwise: the old ones are not kept
  // through the node loop)
  cur = LpcItem{};
  g0 = take_group(P, share, loaded, gend);
  if (g0 >= 0) cur = lpc_item(P, g0, min(g0 + it, gend - 1));
  const int dd = code_depth(pc);
  const uint64_t ix = code_ix(pc), iy = code_iy(pc);
  const uint64_t ccode = make_code(dd + 1, 2 * ix + cx, 2 * iy + cy);
  const bool phc = (pm >> lane) & 1ull;
  const bool item_skip = ((pm >> (8 * it)) & 0xFFull) == 0xFFull;
  const double wdt = kTwoPi * ldexp(1.0, -dd);
  const double fa = (0.25 * wdt) * (0.25 * wdt) / (4.0 * kPi * kPi);
  // the child and its mirror image; the node loop summed S[x,y], which is -K for pp
  const double fk = (BUB && !chl) ? -fa : fa, fm = P.mirror ? 2.0 * fk : fk;
  const double fx = phc ? 0.0 : fm;            // placeholders store zeros
  if (P.mirror && h == 0) {  // odd product integrals cancel between the images
#pragma unroll
    for (int j = 0; j < kPhi; ++j)
#pragma unroll
      for (int k = 0; k < kPhi; ++k)
        if (product_odd(kPhi * j + k)) I[j][k] = 0.0;
  }
  const long ri = (ch == 0) ? leaf : nold + 3L * item_r + (ch - 1);
  const long base = sbase + ri;
  const bool head = valid && ch == 0;
  const int child = lane >> 1;
  const long MQ = P.MQ;
  double *rec = Yw;  // [32][kStage]
  long *cbase = reinterpret_cast<long *>(Yw + lpc::area_doubles(WE, GEN));  // [32] region, -1: inactive
  long *ibase = cbase + kChildren;                                          // [8] item of the deltas
  [[maybe_unused]] float *wgt = reinterpret_cast<float *>(ibase + kItems);  // [8][45] key weights
  wave_sync();  // (cbase takes the place of home)
  if (h == 0) cbase[child] = valid ? base : -1;
  if ((lane & 7) == 0) ibase[it] = valid ? itm : -1;
  if constexpr (WW)
    for (int k = lane & 7; k < MU; k += 8) wgt[it * kPairs9 + k] = P.itau[(long)item_s * MU + k];
  wave_sync();
  // the parents' values of the first kProd columns, for the deltas
  constexpr int kPar = (kItems * kProd + 63) / 64;
  const int n1 = GEN ? min(MU, kStage) : kProd;  // (columns staged at a time)
  const float inv_n1 = 1.0f / (float)n1;
  double par[kPar];
#pragma unroll
  for (int i = 0; i < kPar; ++i) {
    const int e = lane + 64 * i, q = min(stage_row<GEN>(e, n1, inv_n1), kItems - 1), k = e - q * n1;
    const long b = cbase[4 * q];
    par[i] = (e < kItems * n1 && b >= 0) ? P.Q[b * MQ + k] : 0.0;
  }
  // and their errors
  constexpr int kPe = WE ? (kItems * (GEN ? kStage : kPairs9) + 63) / 64 : 1;
  const int ne1 = GEN ? n1 : kPairs9;
  const float inv_ne1 = GEN ? inv_n1 : 1.0f / kPairs9;
  [[maybe_unused]] float pe[kPe];
  if constexpr (WE) {
#pragma unroll
    for (int i = 0; i < kPe; ++i) {
      const int e = lane + 64 * i, q = min((int)(((float)e + 0.5f) * inv_ne1), kItems - 1), k = e - q * ne1;
      const long b = cbase[4 * q];
      pe[i] = (e < kItems * ne1 && b >= 0) ? P.E[b * MU + k] : 0.0f;
    }
  }
#ifdef __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_sched_barrier(0);  // (the loads above stay above the keys below)
#endif
  // staged values [32][n] of columns p0.. of the value records: deltas, then
  // the records (child 0's takes its parent's place, whose values the deltas
  // have read by then)
  auto put_values = [&](int n, float inv_n, int p0) {
#pragma unroll
    for (int i = 0; i < kPar; ++i) {
      const int e = lane + 64 * i, q = min(stage_row<GEN>(e, n, inv_n), kItems - 1), k = e - q * n;
      const long m = ibase[q];
      if (e < kItems * n && m >= 0) {
        const double *c = rec + q * 4 * kStage + k;
        const double sum = (c[0] + c[kStage]) + (c[2 * kStage] + c[3 * kStage]);
        P.dv[m * MQ + p0 + k] = sum - (p0 ? P.Q[cbase[4 * q] * MQ + p0 + k] : par[i]);
      }
    }
    wave_sync();
#pragma unroll 4
    for (int e = lane; e < kChildren * n; e += 64) {
      const int c = stage_row<GEN>(e, n, inv_n), k = e - c * n;
      const long b = cbase[c];
      if (b >= 0) P.Q[b * MQ + p0 + k] = rec[c * kStage + k];
    }
  };
  // the same for errors, staged as float [32][ld]; the deltas carry the
  // float-rounded errors that are stored and later subtracted
  [[maybe_unused]] auto put_errors = [&](const float *re, int ld, int n, float inv_n, int p0) {
#pragma unroll
    for (int i = 0; i < kPe; ++i) {
      const int e = lane + 64 * i, q = min((int)(((float)e + 0.5f) * inv_n), kItems - 1), k = e - q * n;
      const long m = ibase[q];
      if (e < kItems * n && m >= 0) {
        const float *c = re + q * 4 * ld + k;
        const double sum = ((double)c[0] + (double)c[ld]) + ((double)c[2 * ld] + (double)c[3 * ld]);
        P.dep[m * MU + p0 + k] = sum - (double)(p0 ? P.E[cbase[4 * q] * MU + p0 + k] : pe[i]);
      }
    }
    wave_sync();
#pragma unroll 4
    for (int e = lane; e < kChildren * n; e += 64) {
      const int c = (int)(((float)e + 0.5f) * inv_n), k = e - c * n;
      const long b = cbase[c];
      if (b >= 0) P.E[b * MU + p0 + k] = re[c * ld + k];
    }
  };
  // everything read has arrived, the next group's items too: no load is waited
  // for behind the stores
  auto loads_done = [&]() {
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+v"(pkey));
    if constexpr (WE)
#pragma unroll
      for (int i = 0; i < kPe; ++i) asm volatile("" : "+v"(pe[i]));
    asm volatile("" : "+v"(cur.s), "+v"(cur.r), "+v"(cur.pc), "+v"(cur.ch), "+v"(cur.cLx), "+v"(cur.sLx),
                      "+v"(cur.cLy), "+v"(cur.sLy));
#endif
  };
  double key = 0.0;
  if constexpr (!GEN) {
    // the key's pairs (and their errors for the records) from the registers
    [[maybe_unused]] float *re = reinterpret_cast<float *>(rec);
    auto pairs = [&]() {
      constexpr PairTab PT = make_pair_tab();
#pragma unroll
      for (int p = 0; p < kPairs9; ++p) {
        const signed char *tp = PT.t[p];
        double v = I[tp[0]][tp[3]];
        if (tp[4] >= 0) v = tp[5] > 0 ? v + I[tp[0]][tp[4]] : v - I[tp[0]][tp[4]];
        if (tp[1] >= 0) {
          double u = I[tp[1]][tp[3]];
          if (tp[4] >= 0) u = tp[5] > 0 ? u + I[tp[1]][tp[4]] : u - I[tp[1]][tp[4]];
          v = tp[2] > 0 ? v + u : v - u;
        }
        const double e = fabs(fx * v);  // lane 1: |E| of the pair
        if constexpr (WW)
          key += e * (double)wgt[it * kPairs9 + p];
        else
          key += e;
        if constexpr (WE)
          if (h == 1) re[child * kPairs9 + p] = err_f32(e);
      }
    };
    if constexpr (!WE) pairs();  // the loads above complete behind them
    if (h == 0) {
#pragma unroll
      for (int j = 0; j < kPhi; ++j)
#pragma unroll
        for (int k = 0; k < kPhi; ++k) rec[child * kStage + kPhi * j + k] = fx * I[j][k];
    }
    wave_sync();
    loads_done();
    put_values(kProd, 0.0f, 0);
    if constexpr (WE) {  // the errors take the values' place
      wave_sync();
      pairs();
      wave_sync();
      put_errors(re, kPairs9, kPairs9, 1.0f / kPairs9, 0);
    }
  } else {
    // pairs from the product integrals, kStage at a time.  Lane a of each half
    // wave reads coefficient a of a pair from LDS and hands it on through a
    // scalar register: read by every lane as they stand, the 25 coefficients
    // of a pair are thirteen LDS round trips in a row, and by scalar loads from
    // memory each pair of a cold launch waits for its own.
    [[maybe_unused]] float *re = reinterpret_cast<float *>(rec + kChildren * kStage);
    const int ca = min(lane & 31, kProd - 1);
#pragma unroll 1
    for (int p0 = 0; p0 < MU; p0 += kStage) {
      const int n = min(kStage, MU - p0);
      // two pairs at a time: one of each half wave's coefficients
      double cn = co[min(p0 + (lane >> 5), MU - 1) * kProd + ca];
#pragma unroll 1
      for (int j = 0; j < n; j += 2) {
        const long long cb = __double_as_longlong(cn);
        cn = co[min(p0 + j + 2 + (lane >> 5), MU - 1) * kProd + ca];
        const int clo = (int)cb, chi = (int)(cb >> 32);
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          double v = 0.0, u = 0.0;
#pragma unroll
          for (int a = 0; a < kProd; ++a) {
            const int lo = __builtin_amdgcn_readlane(clo, 32 * jj + a);
            const int hi = __builtin_amdgcn_readlane(chi, 32 * jj + a);
            const double c = __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
            double &t = (MIX ? product_odd(a) : (a & 1) != 0) ? u : v;
            t = fma(c, I[a / kPhi][a % kPhi], t);
          }
          if (j + jj < n) {  // (an odd last pair)
            // (MIX: the image's error is the even part minus the odd one)
            const double x = fx * (v + u), e = MIX ? 0.5 * (fabs(x) + fabs(fx * (v - u))) : fabs(x);
            if constexpr (WW)
              key += e * (double)wgt[it * kPairs9 + p0 + j + jj];
            else
              key += e;
            if (h == 0) rec[child * kStage + j + jj] = x;
            if constexpr (WE)
              if (h == 1) re[child * kStage + j + jj] = err_f32(e);
          }
        }
      }
      wave_sync();
      if (p0 == 0) loads_done();
      put_values(n, 1.0f / (float)n, p0);
      if constexpr (WE) put_errors(re, kStage, n, 1.0f / (float)n, p0);
      wave_sync();
    }
  }
  // child keys (lane 1) and the item's key delta
  const double kk = lpc::child_sum(h ? key : 0.0);
  if (valid) {
    if (h == 1) P.key[base] = key;
    else P.code[base] = ccode;
    if (P.born && h == 0) P.born[base] = (unsigned int)(1 + 4 * P.st_splits[item_s] + ch);
  }
  if (head && h == 1) P.de[itm] = kk - pkey;
  if (head && h == 0 && P.ifill) P.ifill[itm] = !item_skip;
  wave_sync();  // the next group's node rows take the records' place
}

// n doubles of a table to LDS by nt threads, t of them this one; four loads in
// flight each
__device__ inline void copy_table(double *dst, const double *src, int n, int t, int nt) {
  int i = t;
  for (; i + 3 * nt < n; i += 4 * nt) {
    const double a = src[i], b = src[i + nt], c = src[i + 2 * nt], d = src[i + 3 * nt];
    dst[i] = a;
    dst[i + nt] = b;
    dst[i + 2 * nt] = c;
    dst[i + 3 * nt] = d;
  }
  for (; i < n; i += nt) dst[i] = src[i];
}

// The grid is the workgroups resident at once; a workgroup stages a parameter
// row's tables and its waves take groups of 8 items (LpcShare).
template <bool BUB, bool WE, bool WW, bool GEN, bool MIX>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3))) k_children_lpc(Problem P) {
  extern __shared__ double lds_raw[];
  double *del = lds_raw, *co = lds_raw + kDelDoubles, *tabl = co + (GEN ? (P.MU * kProd + 1) / 2 * 2 : 0);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double *Yw = tabl + P.tab_doubles + wv * P.lds_wave_doubles;
  __shared__ LpcShare share;
  // (with one parameter row its table is staged before the items are known)
  bool staged = P.one_row && blockDim.x > 64;
  {  // the first share, by index among the XCD's workgroups
    const int total = P.counters[2], group = group_items(P, total);
    const XcdShare x = xcd_share(total, gridDim.x, blockIdx.x, kXcds);
    const int c = share_items(x.last - x.first, group, gridDim.x, kXcds);
    const Span k = first_share(x, c);
    if (k.i0 >= k.i1) return;  // uniform in the workgroup
    if (wv == 0) {
      if (threadIdx.x == 0) {
        share.base = share_base(x, c);
        share.total = x.last;
        share.group = group;
        share.lock = 0;
        share.mode = 0;
        share.range = 0;
        share.rest = k.i0;
        share.end = k.i1;
      }
      wave_sync();
      next_range(P, share, staged ? 0 : -1);
    } else if (staged) {  // the only row's table, while the first wave finds the range
      const Entry E0 = P.entries[0];
      copy_table(tabl, P.tab + E0.tab_off, tab_doubles(E0), threadIdx.x - 64, blockDim.x - 64);
    }
  }
  for (int i = threadIdx.x; i < kDelDoubles; i += blockDim.x) del[i] = rule_value(i);
  if constexpr (GEN)
    for (int i = threadIdx.x; i < P.MU * kProd; i += blockDim.x) co[i] = P.pcoef[i];
#pragma unroll 1
  for (;;) {
    __syncthreads();  // every wave is done with the previous row's table
    if (!staged && share.mode == 2) break;
    const int e = staged ? 0 : __builtin_amdgcn_readfirstlane(share.row);
    const Entry E0 = P.entries[e];
    if (!staged) {
      copy_table(tabl, P.tab + E0.tab_off, tab_doubles(E0), threadIdx.x, blockDim.x);
      __syncthreads();  // (and has read share.mode)
      if (threadIdx.x == 0) {
        atomicExch(&share.range, range_word(share.next));
        atomicExch(&share.mode, 0);
      }
      __syncthreads();
    }
    staged = false;
    LpcRow R;
    R.mt2 = wave_uniform(-2.0 * E0.t * E0.inv_w);
    R.mtp4 = wave_uniform(-4.0 * E0.tp * E0.inv_w);
    R.mmu = wave_uniform(-E0.mu * E0.inv_w);
    R.J = __builtin_amdgcn_readfirstlane(E0.J);
    R.JV = __builtin_amdgcn_readfirstlane(E0.JV);
    const bool wide = __builtin_amdgcn_readfirstlane(share.group) == 1;
    int gend, g = take_group(P, share, e, gend);
    if (g < 0) continue;
    LpcItem cur = lpc_item(P, g, min(g + (lane_id() >> 3), gend - 1));
#pragma unroll 1
    do lpc_group<BUB, WE, WW, GEN, MIX>(kernarg_problem(P), R, tabl, del, co, Yw, share, e, wide, g, gend, cur);
    while (g >= 0);
  }
}

// ---------------------------------------------------------------- diagnostics
// taylor: in the form of the one-wave kernel (k_children)
__global__ void k_kernel_eval(const Entry *e, const double *tab, int ch, const double *a,
                              const double *b, int n, double *out, bool taylor) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Entry E = *e;
  const double *t = tab + E.tab_off;
  out[i] = taylor ? K_taylor(E, t + (long)E.JV * kValStride, ch, a[i], b[i]) : K_eval(E, t, ch, a[i], b[i]);
}

template <int L, int GRAM>
hipError_t launch_root_t(const Problem &p, hipStream_t s) {
  size_t sh = sizeof(double) * wave_lds_doubles<L>(p.ff_identity);
  hipLaunchKernelGGL((k_root<L, GRAM>), dim3(p.W), dim3(64), sh, s, p);
  return hipGetLastError();
}

// projection/precision mode of a problem: separable FP64, or the dense Gram
// in the requested precision
int gram_mode(const Problem &p) { return p.gram == PAID_GRAM_SEPARABLE ? kSep : p.precision; }

// Dynamic LDS of the evaluation kernel: the largest table plus one WaveLds
// per wave, with the waves a workgroup that put the most of them on a CU (up to
// eight; four where the dense Gram needs the registers).  Returns 0 if not even
// one fits.
template <int L>
size_t eval_lds_t(const Problem &p, int *waves_out, int *wave_doubles_out) {
  const size_t wave_b = sizeof(double) * wave_lds_doubles<L>(p.ff_identity, gram_mode(p) == kSep);
  // fixed: the kernel's static LDS (two int tables over the form-factor pairs)
  const size_t tab_b = sizeof(double) * (size_t)p.close_doubles, fixed = 4096;
  const size_t limit = p.lds_limit > 0 ? (size_t)p.lds_limit : 65536;
  int waves = 0, best = 0;
  for (int w = 1; w <= (gram_mode(p) == kSep ? 8 : 4); ++w) {
    const int n = (int)(limit / (tab_b + fixed + w * wave_b)) * w;
    if (n > best || (n == best && n > 0 && w <= 4)) {  // (a table is staged per workgroup)
      best = n;
      waves = w;
    }
  }
  if (waves == 0) return 0;
  if (waves_out) *waves_out = waves;
  if (wave_doubles_out) *wave_doubles_out = (int)(wave_b / sizeof(double));
  return tab_b + (size_t)waves * wave_b;
}

template <int L, int GRAM>
int eval_occupancy_t(Problem p) {
  int waves = 0, wd = 0;
  const size_t sh = eval_lds_t<L>(p, &waves, &wd);
  if (sh == 0) return 1;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(&k_children<L, GRAM>),
                                                   64 * waves, sh) != hipSuccess || n < 1)
    n = 1;
  return n;
}

template <int L, int GRAM>
hipError_t launch_eval_t(Problem p, int grid, hipStream_t s) {
  int waves = 0, wd = 0;
  const size_t sh = eval_lds_t<L>(p, &waves, &wd);
  if (sh == 0) return hipErrorInvalidValue;
  p.lds_wave_doubles = wd;
  hipLaunchKernelGGL((k_children<L, GRAM>), dim3(grid), dim3(64 * waves), sh, s, p);
  return hipGetLastError();
}

// per-wave LDS of the two-lanes-per-child kernel (doubles)
int lpc_wave_doubles(const Problem &p) {
  return lpc::wave_doubles(p.E != nullptr, p.err_mode != 0, needs_pair_coefficients(p));
}

// the two-lanes-per-child kernel for the problem's integrand and form factors
template <bool BUB, bool GEN, bool MIX>
const void *lpc_kernel_t(bool we, bool ww) {
  return we ? (ww ? reinterpret_cast<const void *>(&k_children_lpc<BUB, true, true, GEN, MIX>)
                  : reinterpret_cast<const void *>(&k_children_lpc<BUB, true, false, GEN, MIX>))
            : (ww ? reinterpret_cast<const void *>(&k_children_lpc<BUB, false, true, GEN, MIX>)
                  : reinterpret_cast<const void *>(&k_children_lpc<BUB, false, false, GEN, MIX>));
}
template <bool BUB>
const void *lpc_kernel_b(const Problem &p) {
  const bool we = p.E != nullptr, ww = p.err_mode != 0;
  if (!needs_pair_coefficients(p)) return lpc_kernel_t<BUB, false, false>(we, ww);
  return p.mixed ? lpc_kernel_t<BUB, true, true>(we, ww) : lpc_kernel_t<BUB, true, false>(we, ww);
}
const void *lpc_kernel(const Problem &p) { return p.kind <= 1 ? lpc_kernel_b<true>(p) : lpc_kernel_b<false>(p); }

// Dynamic LDS of the two-lanes-per-child kernel: the table and each wave's
// node rows and records.  The table is staged once per workgroup, so the
// number of waves per workgroup (4, 6 or 8; fewer only if nothing else fits the
// device's per-workgroup limit) is the one that keeps the most waves resident
// per CU, by the runtime's occupancy calculator; the choice is remembered per
// table and wave size.
size_t lpc_lds(const Problem &p, int *waves_out) {
  const size_t wave_b = sizeof(double) * lpc_wave_doubles(p);
  const size_t tab_b = sizeof(double) * ((size_t)p.tab_doubles + kDelDoubles +
                                         (needs_pair_coefficients(p) ? (size_t)(p.MU * kProd + 1) / 2 * 2 : 0));
  const size_t limit = p.lds_limit > 0 ? (size_t)p.lds_limit : 65536;
  thread_local size_t memo_tab = 0, memo_wave = 0, memo_limit = 0;
  thread_local int memo_waves = 0;
  thread_local const void *memo_kern = nullptr;
  if (memo_waves == 0 || memo_tab != tab_b || memo_wave != wave_b || memo_limit != limit ||
      memo_kern != lpc_kernel(p)) {
    int best = 0, best_w = 0;
    for (int w : {4, 6, 8, 2, 1}) {
      const size_t sh = tab_b + (size_t)w * wave_b;
      if (sh > limit || (best > 0 && w < 4)) continue;
      int n = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, lpc_kernel(p), 64 * w, sh) != hipSuccess)
        n = 0;
      if (n < 1) n = (w < 4 && best == 0) ? 1 : 0;  // a last resort still runs
      if (n * w > best) {
        best = n * w;
        best_w = w;
      }
    }
    if (best_w == 0) return 0;
    memo_tab = tab_b;
    memo_kern = lpc_kernel(p);
    memo_wave = wave_b;
    memo_limit = limit;
    memo_waves = best_w;
  }
  if (waves_out) *waves_out = memo_waves;
  return tab_b + (size_t)memo_waves * wave_b;
}

}  // namespace

namespace {
// the two-lanes-per-child kernel serves form factors over the 9-function box
// (or its first function) with the separable FP64 projection over the full
// zone (bubble and unit integrands)
bool use_lpc(const Problem &p) {
  return p.eval_layout == 0 && p.L <= 1 && !p.sym && gram_mode(p) == kSep && p.kind != PAID_GAUSS;
}

template <int L>
hipError_t launch_root_l(const Problem &p, hipStream_t s) {
  switch (gram_mode(p)) {
    case kSep: return launch_root_t<L, kSep>(p, s);
    case PAID_FP32: return launch_root_t<L, PAID_FP32>(p, s);
    case PAID_BF16X3: return launch_root_t<L, PAID_BF16X3>(p, s);
    default: return launch_root_t<L, PAID_FP64>(p, s);
  }
}

template <int L>
int eval_occupancy_l(const Problem &p) {
  switch (gram_mode(p)) {
    case kSep: return eval_occupancy_t<L, kSep>(p);
    case PAID_FP32: return eval_occupancy_t<L, PAID_FP32>(p);
    case PAID_BF16X3: return eval_occupancy_t<L, PAID_BF16X3>(p);
    default: return eval_occupancy_t<L, PAID_FP64>(p);
  }
}

template <int L>
hipError_t launch_eval_l(const Problem &p, int grid, hipStream_t s) {
  switch (gram_mode(p)) {
    case kSep: return launch_eval_t<L, kSep>(p, grid, s);
    case PAID_FP32: return launch_eval_t<L, PAID_FP32>(p, grid, s);
    case PAID_BF16X3: return launch_eval_t<L, PAID_BF16X3>(p, grid, s);
    default: return launch_eval_t<L, PAID_FP64>(p, grid, s);
  }
}
}  // namespace

bool can_mirror(const Problem &p) { return !p.sym && gram_mode(p) == kSep && p.kind != PAID_GAUSS; }
bool leaves_hold_products(const Problem &p) { return use_lpc(p) && p.L == 1 && p.ff_identity; }
bool needs_pair_coefficients(const Problem &p) { return use_lpc(p) && !(p.L == 1 && p.ff_identity); }

hipError_t launch_root(const Problem &p, hipStream_t s) {
  switch (p.L) {
    case 0: return launch_root_l<0>(p, s);
    case 1: return launch_root_l<1>(p, s);
    default: return launch_root_l<2>(p, s);
  }
}

size_t eval_lds_bytes(const Problem &p) {
  if (use_lpc(p)) return lpc_lds(p, nullptr);
  switch (p.L) {
    case 0: return eval_lds_t<0>(p, nullptr, nullptr);
    case 1: return eval_lds_t<1>(p, nullptr, nullptr);
    default: return eval_lds_t<2>(p, nullptr, nullptr);
  }
}

int eval_occupancy(const Problem &p) {
  if (use_lpc(p)) {
    int waves = 0, n = 0;
    const size_t sh = lpc_lds(p, &waves);
    if (sh == 0) return 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, lpc_kernel(p), 64 * waves, sh) != hipSuccess || n < 1)
      n = 1;
    return n;
  }
  switch (p.L) {
    case 0: return eval_occupancy_l<0>(p);
    case 1: return eval_occupancy_l<1>(p);
    default: return eval_occupancy_l<2>(p);
  }
}

hipError_t launch_eval(const Problem &p, int grid, hipStream_t s) {
  if (use_lpc(p)) {
    int waves = 0;
    const size_t sh = lpc_lds(p, &waves);
    if (sh == 0) return hipErrorInvalidValue;
    Problem q = p;
    q.lds_wave_doubles = lpc_wave_doubles(p);
    if (q.wide_items == 0) q.wide_items = grid * waves;
    void *args[] = {&q};
    const hipError_t e = hipLaunchKernel(lpc_kernel(p), dim3(grid), dim3(64 * waves), args, sh, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  switch (p.L) {
    case 0: return launch_eval_l<0>(p, grid, s);
    case 1: return launch_eval_l<1>(p, grid, s);
    default: return launch_eval_l<2>(p, grid, s);
  }
}

hipError_t launch_kernel_eval(const Entry *e, const double *tab, int ch, const double *a,
                              const double *b, int n, double *out, bool taylor, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_kernel_eval, dim3((n + 255) / 256), dim3(256), 0, s, e, tab, ch, a, b, n,
                     out, taylor);
  return hipGetLastError();
}

}  // namespace paid
