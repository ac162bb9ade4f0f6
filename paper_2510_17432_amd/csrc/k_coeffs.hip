// Chebyshev expansion coefficients of the propagator (App. B):
//   exp(-i x y) = sum_n c_n(x) T_n(y),  c_0 = J_0(x),  c_n = 2 (-i)^n J_n(x),
// in FP64 on the GPU, and the truncation order N(x) of Sec. II.A.
//
// J_n(x) by Miller's backward recurrence (J. C. P. Miller, 1952): start far
// above both the wanted orders and x with an arbitrary seed, run
// J_{k-1} = (2k/x) J_k - J_{k+1} down to k = 0 (the recurrence is stable in
// that direction for the decaying solution), and fix the overall factor with
// the Neumann identity J_0 + 2 (J_2 + J_4 + ...) = 1.  Growth in the
// evanescent region n > x is kept in range by rescaling by 2^-600 whenever a
// value exceeds 2^600, applied to the running sum and to every stored order.
#include "csp_internal.h"

namespace csp {

// A workgroup takes 64 arguments: wave 0 runs the recurrence, one argument
// per lane and all lanes on the same order, and wave 1 writes finished
// groups of 16 orders from an LDS tile (two, in turn) in 128-byte pieces of
// the rows.  The recurrence runs twice, once for the normalisation and once
// to store the finished orders, so no row is read again.  What bounds it is
// the serial chain of the largest argument, so a step has no branch (one
// that waits for a vector comparison costs more than the step): arguments
// start at a multiple of 16 orders (the recurrence of zeros stays zero
// before), and the range test multiplies by 1 or 2^-600 every EVERY steps.
// One thread per argument with branches in every step, scaling and
// zero-filling its own row, took 2.25 ms for 2048 arguments of up to 6547
// orders.
constexpr int kBesLanes = 64, kBesTile = 16;

struct BesRun {                                // the recurrence of one argument
  double cur, up, even, k2;                    // J_k, J_{k+1}, sum of even orders, 2 k
  int scaled;                                  // rescalings so far
};

// Orders 16 g + 16 .. 16 g + 1 of the recurrence; put(i) sees J_{16 g + i}
// in r.cur.
template <int EVERY, typename Put>
__device__ __forceinline__ void bes_group(BesRun& r, double inv_x, Put put) {
#pragma unroll
  for (int i = kBesTile; i >= 1; --i) {
    put(i);
    if ((i & 1) == 0) r.even += r.cur;
    const double down = (r.k2 * inv_x) * r.cur - r.up;
    r.up = r.cur;
    r.cur = down;
    r.k2 -= 2.0;
    if ((i - 1) % EVERY == 0) {
      const bool over = fabs(r.cur) > 0x1p600;
      const double f = over ? 0x1p-600 : 1.0;
      r.cur *= f;
      r.up *= f;
      r.even *= f;
      r.scaled += over ? 1 : 0;
    }
  }
}

// gM: group whose first order, 16 gM + 16, starts the lane's recurrence
// (-1: none); gW the workgroup's largest.  Returns N(x) of the lane.
template <int EVERY>
__device__ __forceinline__ int bes_rows(double (&tile)[2][kBesLanes][kBesTile + 1],
                                        const int (&tops)[kBesLanes], double inv_x, int gM,
                                        int gW, double eta, int first_above, int search_from,
                                        int nmax, double* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const bool writer = threadIdx.x >= 64;
  const double seed = 0x1p-300;                // J at the start order, arbitrary
  BesRun r{0.0, 0.0, 0.0, 2.0 * (double)(kBesTile * (gW + 1)), 0};
  if (!writer) {
#pragma unroll 1
    for (int g = gW; g >= 0; --g) {
      if (g == gM) r.cur = seed;
      bes_group<EVERY>(r, inv_x, [](int) {});
    }
  }
  // r.cur now holds J_0 (unnormalised).
  const double inv = 1.0 / (r.cur + 2.0 * r.even), inv2 = 2.0 * inv;
  const int total = r.scaled;
  r = BesRun{0.0, 0.0, 0.0, 2.0 * (double)(kBesTile * (gW + 1)), 0};
  int N = -1;
#pragma unroll 1
  for (int g = gW; g >= -1; --g) {
    double(&t)[kBesLanes][kBesTile + 1] = tile[g & 1];
    if (!writer) {
      if (g < 0) {
        t[lane][kBesTile - 1] = r.cur * inv;   // order 0, at 16 g + 16
      } else {
        if (g == gM) r.cur = seed;
        // orders stored before a rescaling take the ones still to come (the
        // power of two first: it underflows only with the coefficient)
        int e = 0;
        auto store = [&](int i) {
          if (i % EVERY == 0) e = 600 * (r.scaled - total);
          return t[lane][i - 1] = ldexp(r.cur, e) * inv2;
        };
        if (kBesTile * g + kBesTile >= search_from) {
          // truncation: the smallest order above x with |c_n| <= eta
          bes_group<EVERY>(r, inv_x, [&](int i) {
            const double v = store(i);
            const int k = kBesTile * g + i;
            if (k >= first_above && fabs(v) <= eta) N = k;
          });
        } else {
          bes_group<EVERY>(r, inv_x, store);
        }
      }
    }
    __syncthreads();
    if (writer) {
      const int col = lane & (kBesTile - 1);
      const int n = kBesTile * g + 1 + col;
#pragma unroll 4
      for (int q = lane / kBesTile; q < kBesLanes; q += 64 / kBesTile)
        if (n >= 0 && n <= tops[q])
          out[(size_t)(blockIdx.x * kBesLanes + q) * (nmax + 1) + n] = t[q][col];
    }
  }
  return N;
}

__global__ __launch_bounds__(128) void k_bessel(double tau, int nx, int nmax, double eta,
                                                int clip, double* __restrict__ out,
                                                int32_t* __restrict__ ntrunc) {
  __shared__ double tile[2][kBesLanes][kBesTile + 1];
  __shared__ int tops[kBesLanes];
  const int lane = threadIdx.x & 63;
  const bool writer = threadIdx.x >= 64;
  const int j = blockIdx.x * kBesLanes + lane;
  const double x = tau * (double)(j + 1);
  const bool run = j < nx && x > 0.0;
  if (j < nx && !run && !writer) {            // exp(0): c_0 = 1, the rest 0
    double* a = out + (size_t)j * (nmax + 1);
    a[0] = 1.0;
    for (int n = 1; n <= nmax; ++n) a[n] = 0.0;
    ntrunc[j] = 0;
  }
  // With clip, only the orders this argument needs are computed: past its
  // truncation order (bounded by x + 40 + 25 x^(1/3)) the coefficients are
  // below 1e-14 and are not stored.  Arguments far below the table's largest
  // then avoid a long, repeatedly rescaled recurrence.
  const int need = run ? (int)ceil(x + 40.0 + 25.0 * cbrt(x + 1.0)) : -1;
  const int top = run ? ((clip && need < nmax) ? need : nmax) : -1;   // highest order stored
  if (!writer) tops[lane] = top;
  // Start order: beyond the stored orders and the turning point x by a
  // margin that grows like x^(1/3) (the width of the transition region of
  // J_n near n = x), rounded up to the next multiple of 16 (even, so that
  // the Neumann sum ends on an even order).
  const double start = run ? (x > (double)top ? x : (double)top) + 24.0 + 18.0 * cbrt(x + 1.0) : 0.0;
  const int gM = run ? (int)(ceil(start) / kBesTile) : -1;
  const int first_above = run ? (int)floor(x) + 1 : INT32_MAX;
  // 2 k / x bounds the growth of a step: four steps between range tests are
  // safe below 2^100 (x above 1e-26)
  int slow = run && 2.0 * (start + kBesTile) > 0x1p100 * x ? 1 : 0;
  int gW = gM, from = first_above;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    gW = max(gW, __shfl_xor(gW, m));
    from = min(from, __shfl_xor(from, m));
    slow |= __shfl_xor(slow, m);
  }
  const double inv_x = run ? 1.0 / x : 0.0;
  const int N = slow ? bes_rows<1>(tile, tops, inv_x, gM, gW, eta, first_above, from, nmax, out)
                     : bes_rows<4>(tile, tops, inv_x, gM, gW, eta, first_above, from, nmax, out);
  if (run && !writer) ntrunc[j] = N <= top ? N : -1;
}

hipError_t launch_bessel(double tau, int nx, int nmax, double eta, bool clip, double* d_a,
                         int32_t* d_ntrunc, hipStream_t s) {
  hipLaunchKernelGGL(k_bessel, dim3((nx + kBesLanes - 1) / kBesLanes), dim3(128), 0, s, tau, nx, nmax, eta,
                     clip ? 1 : 0, d_a, d_ntrunc);
  return hipGetLastError();
}

__global__ void k_complex_coeffs(const double* __restrict__ a, int nmax, double2* __restrict__ c) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n > nmax) return;
  const double v = a[n];
  double2 o;
  switch (n & 3) {               // (-i)^n
    case 0: o = make_double2(v, 0.0); break;
    case 1: o = make_double2(0.0, -v); break;
    case 2: o = make_double2(-v, 0.0); break;
    default: o = make_double2(0.0, v); break;
  }
  c[n] = o;
}

hipError_t launch_complex_coeffs(const double* d_a, int nmax, double* d_c, hipStream_t s) {
  hipLaunchKernelGGL(k_complex_coeffs, dim3((nmax + 256) / 256), dim3(256), 0, s, d_a, nmax,
                     reinterpret_cast<double2*>(d_c));
  return hipGetLastError();
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
struct BopEntryP {
  bf16x8 hi;
  bf16x8 lo;
};

// One thread per (16-order step kb, time tile jt, lane): lane (j, h) holds
// a_{n, j+1} for n = n_lo + 16 kb + 8 h + v, v = 0..7, split into bf16 hi/lo.
__global__ void k_pack_bop(const double* __restrict__ a, int lda, const int32_t* __restrict__ ntr,
                           int bcols, int jtiles, int n_lo, int n_cnt, BopEntryP* __restrict__ bop,
                           float* __restrict__ ccarry) {
  const int n_kb = (n_cnt + 15) / 16;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n_kb * 16) {
    const int n = n_lo + e;
    float v = 0.f;
    if (e < n_cnt && n <= ntr[bcols - 1]) v = (float)a[(size_t)(bcols - 1) * lda + n];
    ccarry[e] = v;
  }
  if (e >= n_kb * jtiles * 64) return;
  const int lane = e & 63;
  const int jt = (e >> 6) % jtiles;
  const int kb = (e >> 6) / jtiles;
  const int j = jt * 32 + (lane & 31);
  BopEntryP out;
  for (int v = 0; v < 8; ++v) {
    const int rel = kb * 16 + (lane >> 5) * 8 + v;
    const int n = n_lo + rel;
    double val = 0.0;
    if (j < bcols && rel < n_cnt && n <= ntr[j]) val = a[(size_t)j * lda + n];
    const __bf16 hi = static_cast<__bf16>(static_cast<float>(val));
    const double rest = val - static_cast<double>(static_cast<float>(hi));
    out.hi[v] = hi;
    out.lo[v] = static_cast<__bf16>(static_cast<float>(rest));
  }
  bop[(kb * jtiles + jt) * 64 + lane] = out;
}

hipError_t launch_pack_bop(const double* d_a, int lda, const int32_t* d_ntrunc, int bcols,
                           int jtiles, int n_lo, int n_cnt, void* d_bop, float* d_ccarry,
                           hipStream_t s) {
  const int n_kb = (n_cnt + 15) / 16;
  const int total = n_kb * jtiles * 64 > n_kb * 16 ? n_kb * jtiles * 64 : n_kb * 16;
  hipLaunchKernelGGL(k_pack_bop, dim3((total + 255) / 256), dim3(256), 0, s, d_a, lda, d_ntrunc,
                     bcols, jtiles, n_lo, n_cnt, static_cast<BopEntryP*>(d_bop), d_ccarry);
  return hipGetLastError();
}

__global__ void k_pack_c64(const double* __restrict__ a, int lda, const int32_t* __restrict__ ntr,
                           int bcols, int n_lo, int n_cnt, double2* __restrict__ coef,
                           double2* __restrict__ ccarry) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_cnt * bcols) return;
  const int rel = e / bcols, j = e - rel * bcols;
  const int n = n_lo + rel;
  const double v = n <= ntr[j] ? a[(size_t)j * lda + n] : 0.0;
  double2 o;
  switch (n & 3) {
    case 0: o = make_double2(v, 0.0); break;
    case 1: o = make_double2(0.0, -v); break;
    case 2: o = make_double2(-v, 0.0); break;
    default: o = make_double2(0.0, v); break;
  }
  coef[e] = o;
  if (j == bcols - 1) ccarry[rel] = o;
}

hipError_t launch_pack_c64(const double* d_a, int lda, const int32_t* d_ntrunc, int bcols,
                           int n_lo, int n_cnt, double* d_coef, double* d_ccarry,
                           hipStream_t s) {
  const int total = n_cnt * bcols;
  hipLaunchKernelGGL(k_pack_c64, dim3((total + 255) / 256), dim3(256), 0, s, d_a, lda, d_ntrunc,
                     bcols, n_lo, n_cnt, reinterpret_cast<double2*>(d_coef),
                     reinterpret_cast<double2*>(d_ccarry));
  return hipGetLastError();
}

}  // namespace csp
