// contract.hip -- the contraction beside the integration (Sec. 2, Eqs.
// matmul-P, matmul-C, matmul-D): per transfer momentum l, with the bubbles
// chi^pp(l), chi^ph(l) of the adaptive integration and the couplings
// V^P(l), V^C(l), V^D(l) (M x M over form factors),
//   dP = V^P chi^pp V^P,
//   dC = - V^C chi^ph V^C,
//   dD = 2 V^D chi^ph V^D - V^C chi^ph V^D - V^D chi^ph V^C,
// the last as (2 V^D - V^C) (chi^ph V^D) - V^D (chi^ph V^C), reusing chi^ph V^C.
//
// FP64 matrix cores, everything in registers.  A wave owns one l and one
// column tile (16 columns; M <= 16 has one, M <= 32 two): the columns of all
// products are independent.  In the 16 x 16 x 4 tiles, lane (kk, m) = (lane >> 4,
// lane & 15) holds A[m][4 kb + kk] and B[4 kb + kk][m] of k-step kb, and result
// register r of row tile t is row 16 t + 4 r + kk, column m: that is B of k-step
// 4 t + r, so chi V feeds the second product as it stands, with no exchange and
// no LDS.  The bound is memory (every matrix read and written once) and, at M
// > 16, the matrix cores; the operands come straight from global memory, a
// whole matrix's loads issued together, and many waves hide them.  Staging six
// zero-padded 32 x 32 matrices per wave in LDS (50.7 KB, three waves a compute
// unit) instead took 210 us for 11,520 momenta of order 9 and 77 us for 1,024
// of order 25; this takes 18 us each (33
// and 32 us a call with its synchronisation, 244 and 90 before).
#include "launch.h"

namespace paid {

namespace {

typedef double c4 __attribute__((ext_vector_type(4)));

// A[16 t + m][4 kb + kk] of X [M][M], zero outside
template <int NT>
__device__ inline void load_a(const double *X, int M, double (&a)[NT][4 * NT]) {
  const int lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int kb = 0; kb < 4 * NT; ++kb) {
      const int i = 16 * t + m, k = 4 * kb + kk;
      a[t][kb] = (i < M && k < M) ? X[i * M + k] : 0.0;
    }
}

// B[4 kb + kk][16 tc + m] of X, zero outside
template <int NT>
__device__ inline void load_b(const double *X, int M, int tc, double (&b)[4 * NT]) {
  const int lane = threadIdx.x & 63, j = 16 * tc + (lane & 15), kk = lane >> 4;
#pragma unroll
  for (int kb = 0; kb < 4 * NT; ++kb) {
    const int k = 4 * kb + kk;
    b[kb] = (k < M && j < M) ? X[k * M + j] : 0.0;
  }
}

// acc += A B over the k-steps that hold rows below M
template <int NT>
__device__ inline void mul(const double (&a)[NT][4 * NT], const double (&b)[4 * NT], int nk, c4 (&acc)[NT]) {
#pragma unroll
  for (int kb = 0; kb < 4 * NT; ++kb)
    if (kb < nk) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t][kb], b[kb], acc[t], 0, 0, 0);
    }
}

// a result as the right operand of the next product
template <int NT>
__device__ inline void as_b(const c4 (&acc)[NT], double (&b)[4 * NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) b[4 * t + r] = acc[t][r];
}

template <int NT>
__device__ inline void zero(c4 (&acc)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = c4{0.0, 0.0, 0.0, 0.0};
}

template <int NT>
__device__ inline void store(double *X, int M, int tc, const c4 (&acc)[NT], double f) {
  const int lane = threadIdx.x & 63, j = 16 * tc + (lane & 15), kk = lane >> 4;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * t + 4 * r + kk;
      if (i < M && j < M) X[i * M + j] = f * acc[t][r];
    }
}

// The work of one wave.  IN_PLACE: an output is the array of a coupling (dP =
// V^P, dC = V^C, dD = V^D).  Every load of a coupling stands before the first
// store that may overwrite it, and the two waves of one l (M > 16), each of which
// reads whole matrices and writes its half of the columns, meet before the stores.
template <int NT, bool IN_PLACE>
__device__ inline void contract(long l, int tc, int M, const double *chi, const double *VP, const double *VC,
                                const double *VD, double *dP, double *dC, double *dD) {
  const int nk = (M + 3) >> 2;
  const long mm2 = (long)M * M;
  const double *cpp = chi + (2 * l) * mm2, *cph = chi + (2 * l + 1) * mm2;
  double a[NT][4 * NT], v[NT][4 * NT], b[4 * NT], t1[4 * NT];
  c4 acc[NT], dp[NT];
  // V^P (chi^pp V^P)
  load_a<NT>(cpp, M, a);
  load_b<NT>(VP + l * mm2, M, tc, b);
  load_a<NT>(VP + l * mm2, M, v);
  zero<NT>(acc);
  mul<NT>(a, b, nk, acc);
  as_b<NT>(acc, t1);
  zero<NT>(dp);
  mul<NT>(v, t1, nk, dp);
  load_a<NT>(cph, M, a);
  load_b<NT>(VD + l * mm2, M, tc, t1);
  load_b<NT>(VC + l * mm2, M, tc, b);
  load_a<NT>(VC + l * mm2, M, v);
  if constexpr (IN_PLACE && NT > 1) __syncthreads();
  store<NT>(dP + l * mm2, M, tc, dp, 1.0);
  // t1 = chi^ph V^D, b = chi^ph V^C
  zero<NT>(acc);
  mul<NT>(a, t1, nk, acc);
  as_b<NT>(acc, t1);
  zero<NT>(acc);
  mul<NT>(a, b, nk, acc);
  as_b<NT>(acc, b);
  // dC = -V^C (chi^ph V^C)
  load_a<NT>(VD + l * mm2, M, a);
  zero<NT>(acc);
  mul<NT>(v, b, nk, acc);
  if constexpr (IN_PLACE && NT > 1) __syncthreads();
  store<NT>(dC + l * mm2, M, tc, acc, -1.0);
  // dD = (2 V^D - V^C) (chi^ph V^D) - V^D (chi^ph V^C)
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int kb = 0; kb < 4 * NT; ++kb) v[t][kb] = 2.0 * a[t][kb] - v[t][kb];
  zero<NT>(acc);
  mul<NT>(v, t1, nk, acc);
  // (sums of their own: one running through both products rounds at the larger
  // of the two all the way)
  c4 acc2[NT];
  zero<NT>(acc2);
  mul<NT>(a, b, nk, acc2);
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] -= acc2[t];
  store<NT>(dD + l * mm2, M, tc, acc, 1.0);
}

template <int NT>
__global__ void __launch_bounds__(256) k_contract(int n_l, int M, const double *__restrict__ chi,
                                                  const double *__restrict__ VP, const double *__restrict__ VC,
                                                  const double *__restrict__ VD, double *__restrict__ dP,
                                                  double *__restrict__ dC, double *__restrict__ dD) {
  const long unit = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (unit / NT >= n_l) return;  // whole waves only: nothing below synchronises the workgroup
  contract<NT, false>(unit / NT, (int)(unit % NT), M, chi, VP, VC, VD, dP, dC, dD);
}

// One l a workgroup.
template <int NT>
__global__ void __launch_bounds__(64 * NT) k_contract_in_place(int M, const double *chi, const double *VP,
                                                               const double *VC, const double *VD, double *dP,
                                                               double *dC, double *dD) {
  contract<NT, true>(blockIdx.x, threadIdx.x >> 6, M, chi, VP, VC, VD, dP, dC, dD);
}

// whether two blocks of doubles share memory
bool overlap(const double *a, size_t na, const double *b, size_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + 8 * nb && y < x + 8 * na;
}

}  // namespace

hipError_t launch_contract(int n_l, int M, const double *chi, const double *VP, const double *VC,
                           const double *VD, double *dP, double *dC, double *dD, hipStream_t s) {
  if (n_l <= 0) return hipSuccess;
  const int waves = 4, nt = M > 16 ? 2 : 1;
  const size_t n = (size_t)n_l * M * M;
  bool in_place = false;  // (stores and loads in order, and a barrier: 36.1 instead of 35.2 us for 1,024 of order 25)
  for (const double *out : {dP, dC, dD})
    for (const double *in : {VP, VC, VD}) in_place = in_place || overlap(out, n, in, n);
  if (in_place) {
    if (nt == 1)
      hipLaunchKernelGGL(k_contract_in_place<1>, dim3(n_l), dim3(64), 0, s, M, chi, VP, VC, VD, dP, dC, dD);
    else
      hipLaunchKernelGGL(k_contract_in_place<2>, dim3(n_l), dim3(128), 0, s, M, chi, VP, VC, VD, dP, dC, dD);
    return hipGetLastError();
  }
  const long units = (long)n_l * nt;
  const dim3 grid((unsigned)((units + waves - 1) / waves)), block(64 * waves);
  if (nt == 1)
    hipLaunchKernelGGL(k_contract<1>, grid, block, 0, s, n_l, M, chi, VP, VC, VD, dP, dC, dD);
  else
    hipLaunchKernelGGL(k_contract<2>, grid, block, 0, s, n_l, M, chi, VP, VC, VD, dP, dC, dD);
  return hipGetLastError();
}

}  // namespace paid
