// Moment-based form (Sec. II.A, moment-based implementation; Sec. III
// DOS-Concurrent-M): the per-order inner products (the recursion kernel's
// moment records, summed per column by k_cheb_mom_finish) are turned into
// the block moments mu_n = <psi0|T_n(H~) s_k> (directly, or with halving
// every moment above mu_1 from the self products of Eq. cheby_prod), and contracted
// with the expansion coefficients into correlations
//   C(t_{kb+j}) = sum_{n=0}^{N(j tau)} c_n(j tau) mu_n,   c_n = (-i)^n a_n.
// Everything here is FP64 and summed in a fixed order.
#include "csp_internal.h"

namespace csp {

// mu_n for n = 0..Nk of one instance.  dots row n holds the sums of the step
// that produced order n: [0] <psi0|phi_n>, [1] <psi0|phi_{n-1}>,
// [2] <phi_n|phi_n>, [3] <phi_n|phi_{n-1}>.  halving 2: no product with psi0
// was taken; mu_0 is C_0 = <psi0|psi0> (already in row 0 of corr) and mu_1 =
// <phi_1|phi_0>, both real.
__global__ void k_mom_assemble(const MomCorrInst* __restrict__ mc, int Nk, int halving) {
  const MomCorrInst& M = mc[blockIdx.y];
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (Nk + 1) * M.Rg) return;
  const int n = e / M.Rg, r = e - n * M.Rg;
  const int Rg = M.Rg;
  auto dot = [&](int row, int kind) {
    const double* p = M.dots + ((int64_t)row * 4 * Rg + kind * Rg + r) * 2;
    return make_double2(p[0], p[1]);
  };
  auto first = [&](int k) {               // mu_0, mu_1
    if (halving < 2) return dot(1, 1 - k);
    return k == 0 ? reinterpret_cast<const double2*>(M.corr)[M.col0 + r]
                  : make_double2(dot(1, 3).x, 0.0);
  };
  double2 mu;
  if (n == 0) {
    mu = first(0);                        // <psi0|s_k>
  } else if (!halving || n == 1) {
    mu = n == 1 ? first(1) : dot(n, 0);
  } else if ((n & 1) == 0) {              // mu_2k = 2 <phi_k|phi_k> - mu_0
    const double2 a = dot(n / 2, 2), m0 = first(0);
    mu = make_double2(2.0 * a.x - m0.x, 2.0 * a.y - m0.y);
  } else {                                // mu_2k+1 = 2 <phi_k+1|phi_k> - mu_1
    const double2 a = dot((n + 1) / 2, 3), m1 = first(1);
    mu = make_double2(2.0 * a.x - m1.x, 2.0 * a.y - m1.y);
  }
  reinterpret_cast<double2*>(M.mu)[(int64_t)n * Rg + r] = mu;
}

// corr[(t0 + 1 + j) * ldc + col0 + r] = sum_{n <= N((j+1) tau)} (-i)^n a[j][n] mu_n[r]
// A wave owns four times and four columns: its lanes take the orders n =
// lane, lane + 64, ... (coalesced coefficient rows; n mod 4 is the lane's, so
// (-i)^n is applied once at the end) and are summed by a fixed butterfly.
// One thread per time and column over all orders, each reading its own row,
// took 1.99 ms for 2048 times x 4 columns of up to 6547 orders.
constexpr int kMcT = 4, kMcC = 4;

__global__ __launch_bounds__(256) void k_mom_corr(const MomCorrInst* __restrict__ mc,
                                                  const double* __restrict__ a, int lda,
                                                  const int32_t* __restrict__ ntr, int bk,
                                                  int64_t t0, unsigned n_tb) {
  const MomCorrInst& M = mc[blockIdx.y];
  const int lane = threadIdx.x & 63;
  // blockIdx.x: n_tb blocks of times for every four columns
  const int j0 = ((blockIdx.x % n_tb) * 4 + (threadIdx.x >> 6)) * kMcT;
  const int r0 = (blockIdx.x / n_tb) * kMcC;
  const int Rg = M.Rg;
  if (j0 >= bk || r0 >= Rg) return;
  const double2* mu = reinterpret_cast<const double2*>(M.mu);
  // truncation orders of the four times (the last time again past the block's
  // end) and their rows of the table
  int nt[kMcT], nmin = INT32_MAX, nmax = 0;
  const double* row[kMcT];
#pragma unroll
  for (int q = 0; q < kMcT; ++q) {
    const int j = j0 + q < bk ? j0 + q : bk - 1;
    nt[q] = ntr[j];
    row[q] = a + (int64_t)j * lda;
    nmin = min(nmin, nt[q]);
    nmax = max(nmax, nt[q]);
  }
  double sx[kMcT][kMcC], sy[kMcT][kMcC];
#pragma unroll
  for (int q = 0; q < kMcT; ++q)
#pragma unroll
    for (int c = 0; c < kMcC; ++c) sx[q][c] = sy[q][c] = 0.0;
  auto moment = [&](int n, int c) {
    return r0 + c < Rg ? mu[(int64_t)n * Rg + r0 + c] : make_double2(0.0, 0.0);
  };
  int n = lane;
#pragma unroll 2
  for (; n <= nmin; n += 64) {
    double w[kMcT];
#pragma unroll
    for (int q = 0; q < kMcT; ++q) w[q] = row[q][n];
#pragma unroll
    for (int c = 0; c < kMcC; ++c) {
      const double2 m = moment(n, c);
#pragma unroll
      for (int q = 0; q < kMcT; ++q) {
        sx[q][c] = fma(w[q], m.x, sx[q][c]);
        sy[q][c] = fma(w[q], m.y, sy[q][c]);
      }
    }
  }
  // orders past a time's truncation are no part of its sum, whatever their
  // moments (with |H| below the spectrum they grow past the largest number)
  for (; n <= nmax; n += 64) {
#pragma unroll
    for (int q = 0; q < kMcT; ++q)
      if (n <= nt[q]) {
        const double w = row[q][n];
#pragma unroll
        for (int c = 0; c < kMcC; ++c) {
          const double2 m = moment(n, c);
          sx[q][c] = fma(w, m.x, sx[q][c]);
          sy[q][c] = fma(w, m.y, sy[q][c]);
        }
      }
  }
  double2* corr = reinterpret_cast<double2*>(M.corr);
#pragma unroll
  for (int q = 0; q < kMcT; ++q)
#pragma unroll
    for (int c = 0; c < kMcC; ++c) {
      double x = sx[q][c], y = sy[q][c];
      switch (lane & 3) {                   // (-i)^n (x + i y)
        case 0: break;
        case 1: { const double u = x; x = y; y = -u; break; }
        case 2: x = -x; y = -y; break;
        default: { const double u = x; x = -y; y = u; break; }
      }
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) {
        x += __shfl_xor(x, m);
        y += __shfl_xor(y, m);
      }
      if (lane == 0 && j0 + q < bk && r0 + c < Rg)
        corr[(t0 + 1 + j0 + q) * M.ldc + M.col0 + r0 + c] = make_double2(x, y);
    }
}

// (columns in x too: the conductivity has a column for every energy of every
// state, more than a grid's y or z hold)
static void launch_corr_sums(const MomCorrInst* d_mc, int n_inst, const double* d_a, int lda,
                             const int32_t* d_ntrunc, int bk, int64_t t0, int rg_max,
                             hipStream_t s) {
  const unsigned n_tb = (unsigned)ceil_div(bk, 4 * kMcT);
  const dim3 grid(n_tb * (unsigned)ceil_div(rg_max, kMcC), n_inst);
  hipLaunchKernelGGL(k_mom_corr, grid, dim3(256), 0, s, d_mc, d_a, lda, d_ntrunc, bk, t0, n_tb);
}

hipError_t launch_mom_corr(const MomCorrInst* d_mc, int n_inst, int Nk, int halving,
                           const double* d_a, int lda, const int32_t* d_ntrunc, int bk,
                           int64_t t0, int rg_max, hipStream_t s) {
  const int na = (Nk + 1) * rg_max;
  hipLaunchKernelGGL(k_mom_assemble, dim3((unsigned)ceil_div(na, 256), n_inst), dim3(256), 0, s,
                     d_mc, Nk, halving);
  launch_corr_sums(d_mc, n_inst, d_a, lda, d_ntrunc, bk, t0, rg_max, s);
  return hipGetLastError();
}

// Correlations from moments that are already assembled (M.mu filled by the
// caller): rows t0 + 1 .. t0 + bk of M.corr.
hipError_t launch_mom_corr_only(const MomCorrInst* d_mc, int n_inst, const double* d_a, int lda,
                                const int32_t* d_ntrunc, int bk, int64_t t0, int rg_max,
                                hipStream_t s) {
  launch_corr_sums(d_mc, n_inst, d_a, lda, d_ntrunc, bk, t0, rg_max, s);
  return hipGetLastError();
}

}  // namespace csp
