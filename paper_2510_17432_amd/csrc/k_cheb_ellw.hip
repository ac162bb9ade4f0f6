// Chebyshev step of an explicit matrix in the windowed layout (amxsy of
// Sec. II.B, for matrices of any density D_H):
//   phi_{n+1} = 2 H~ phi_n - phi_{n-1},
// one step per launch.  The layout (built at lattice creation,
// ell_windows.cpp) groups the rows into slices of 256 or 128 that are
// compact in the matrix graph and lists, per slice, its window: the distinct
// columns its entries name.  512^2 rows at D = 121, 5 columns, complex64
// moments: 93 -> 79 us a launch (190 MB of matrix, 2.4 TB/s) with 256-row
// slices, no ragged ones and narrower tiles; what bounds it is the latency of
// a slice (window, then 31 quads of entries) at 4 workgroups per CU.
//
// One workgroup, a thread per row, owns a slice and a tile of CT columns of a
// column group.  It stages the slice's window of phi_n for its columns in
// LDS (one plane of W complex values per column, coalesced where the
// window's columns run consecutively), then thread t accumulates row t of
// the slice over its D entries, reading the matrix once (16-bit
// window-local columns and values in quads of four entries per load,
// non-temporal: 6 B per entry in complex64 and 10 B in complex128, against
// 8 and 12 B in the slice layout) and gathering every phi_n value from LDS
// instead of the caches.
// A slice whose window exceeds the LDS budget gathers from global memory
// with the entries' global columns.  Rows keep their index in every vector:
// thread t reads and writes row rows[t] of phi_n, phi_{n-1}, phi_{n+1},
// psi0 and the carried state (scattered within the slice's ball of rows).
// Moment epilogue and carried state as the other recursion kernels: one
// record of 8 FP64 sums per (column, slice), the waves of the
// workgroup added in a fixed order.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "csp_internal.h"

#define CSP_GLOBAL __attribute__((address_space(1)))

namespace csp {
namespace ellw {

template <typename T> struct cplx {
  T x, y;
};
typedef float f32x2 __attribute__((ext_vector_type(2), aligned(8)));
typedef double f64x2 __attribute__((ext_vector_type(2), aligned(16)));
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(16)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4), aligned(8)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(16)));
template <typename T> struct vec2;
template <> struct vec2<float> { using type = f32x2; };
template <> struct vec2<double> { using type = f64x2; };

template <typename T>
__device__ __forceinline__ cplx<T> ld(const CSP_GLOBAL T* p) {
  const typename vec2<T>::type v = *reinterpret_cast<const CSP_GLOBAL typename vec2<T>::type*>(p);
  return {v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void st(CSP_GLOBAL T* p, cplx<T> c, bool nt) {
  typename vec2<T>::type v;
  v.x = c.x;
  v.y = c.y;
  CSP_GLOBAL typename vec2<T>::type* q = reinterpret_cast<CSP_GLOBAL typename vec2<T>::type*>(p);
  if (nt) __builtin_nontemporal_store(v, q);
  else *q = v;
}

template <typename T, int CT, bool MOM, bool CARRY>
__global__ __launch_bounds__(256) void k_cheb_ellw(const ChebInst* __restrict__ insts, int n_inst,
                                                   int64_t wg_lo, int64_t wg_hi, ChebStep sp) {
  using C = cplx<T>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nr = blockDim.x;                        // rows of a slice: 128 or 256
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int64_t L = wg_lo + xcd_remap(blockIdx.x, gridDim.x);
  if (L >= wg_hi) return;                           // the whole workgroup
  int ii = 0;
  while (ii + 1 < n_inst && L >= insts[ii + 1].wave0) ++ii;
  const ChebInst& I = insts[ii];
  const int64_t lw = L - I.wave0;
  // the group's columns in n_tiles tiles of as equal size as possible (the
  // first Rg mod n_tiles take one more): CT or CT - 1 columns each
  const int n_tiles = (I.Rg + CT - 1) / CT;
  const int64_t slice = lw / n_tiles;
  const int tile = static_cast<int>(lw - slice * n_tiles);
  const int tb = I.Rg / n_tiles, tr = I.Rg - tb * n_tiles;
  const int c0 = tile * tb + (tile < tr ? tile : tr);
  const int nc = tb + (tile < tr ? 1 : 0);          // columns of this tile
  const int64_t N = I.N;
  const int D = I.ell_D;
  const int32_t row = I.ellw_rows[slice * nr + t];
  const bool valid = row >= 0;
  const int64_t woff = I.ellw_off[slice];
  const int64_t W = I.ellw_off[slice + 1] - woff;
  const bool staged = W > 0 && W <= I.ellw_lds_cap;   // uniform over the workgroup

  const int64_t cofs = 2 * (int64_t)c0 * N;         // column c0 of the group, in T units
  CSP_GLOBAL T* base = (CSP_GLOBAL T*)(I.base);
  const CSP_GLOBAL T* cur =
      (sp.slot_cur < 0 ? (const CSP_GLOBAL T*)(I.src) : base + 2 * (int64_t)sp.slot_cur * I.slot_stride) +
      cofs;
  const CSP_GLOBAL T* prev =
      sp.first ? nullptr : base + 2 * (int64_t)sp.slot_prev * I.slot_stride + cofs;
  CSP_GLOBAL T* outv =
      sp.slot_out[0] >= 0 ? base + 2 * (int64_t)sp.slot_out[0] * I.slot_stride + cofs : nullptr;
  CSP_GLOBAL T* copyv =
      sp.copy_slot >= 0 ? base + 2 * (int64_t)sp.copy_slot * I.slot_stride + cofs : nullptr;

  // ---- the window of phi_n, one plane of W complex values per column
  // ([nc][W]).  Lanes gather window positions that are close together (the
  // rows of a slice ascend and most matrices name neighbouring columns from
  // neighbouring rows), so with 8-byte planes they hit distinct banks; an
  // interleaved [W][nc] layout put every position with the same residue of
  // 32 / nc on the same banks and serialised the gathers.
  // Each thread loads four window positions of every column before it
  // stores them, so the loads of a thread are in flight together.
  const int Wi = static_cast<int>(W);
  C* win = reinterpret_cast<C*>(smem);
  auto stage = [&](auto nc_tag) {
    constexpr int NC = decltype(nc_tag)::value;
    const CSP_GLOBAL int32_t* wi = (const CSP_GLOBAL int32_t*)(I.ellw_idx) + woff;
    int w = t;
    for (; w + 3 * nr < Wi; w += 4 * nr) {
      int64_t j[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) j[u] = wi[w + u * nr];
      C x[4][NC];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) x[u][c] = ld<T>(cur + 2 * ((int64_t)c * N + j[u]));
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) win[c * Wi + w + u * nr] = x[u][c];
    }
    for (; w < Wi; w += nr) {
      const int64_t j = wi[w];
      C x[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) x[c] = ld<T>(cur + 2 * ((int64_t)c * N + j));
#pragma unroll
      for (int c = 0; c < NC; ++c) win[c * Wi + w] = x[c];
    }
    __syncthreads();
  };

  // ---- sum_k H_{row,j_k} phi_n[j_k] for the tile's columns; the entries
  // come in quads (4 indices and 4 values per load), so a thread keeps
  // several quads of the matrix stream in flight.  The loop is compiled for
  // a fixed column count (tiles of a group hold CT or CT - 1 columns): a
  // run-time count would put a branch around every gather and keep the
  // gathers of one entry from being issued together.
  T ar[CT], ai[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) ar[c] = ai[c] = T(0);
  const int D4 = (D + 3) / 4;
  const int64_t qofs = (slice * D4 * nr + t) * 4;    // quad 0 of this row
  const CSP_GLOBAL T* vp = (const CSP_GLOBAL T*)(I.ellw_val) + qofs;
  auto ld_vals = [&](int q, T (&v)[4]) {
    if constexpr (sizeof(T) == 4) {
      const f32x4 a = __builtin_nontemporal_load(
          reinterpret_cast<const CSP_GLOBAL f32x4*>(vp + (int64_t)q * (4 * nr)));
      v[0] = a.x;
      v[1] = a.y;
      v[2] = a.z;
      v[3] = a.w;
    } else {
      const CSP_GLOBAL f64x2* p = reinterpret_cast<const CSP_GLOBAL f64x2*>(vp + (int64_t)q * (4 * nr));
      const f64x2 a = __builtin_nontemporal_load(p), b = __builtin_nontemporal_load(p + 1);
      v[0] = a.x;
      v[1] = a.y;
      v[2] = b.x;
      v[3] = b.y;
    }
  };
  // Entries of quads q .. q + NQ - 1 of the row: window-local indices (or
  // global columns) and values, loaded one group ahead of their use so the
  // matrix stream of the next group is in flight while the current one
  // gathers.  Quads past D4 are not loaded (they would belong to the next
  // slice, or lie past the matrix).
  constexpr int NQ = 2;
  auto accumulate = [&](auto nc_tag) {
    constexpr int NC = decltype(nc_tag)::value;
    if (staged) {
      stage(nc_tag);
      const CSP_GLOBAL u16x4* lp = reinterpret_cast<const CSP_GLOBAL u16x4*>(
          (const CSP_GLOBAL uint16_t*)(I.ellw_loc) + qofs);
      u16x4 la[NQ];
      T va[NQ][4];
#pragma unroll
      for (int p = 0; p < NQ; ++p)
        if (p < D4) {
          la[p] = __builtin_nontemporal_load(lp + (int64_t)p * nr);
          ld_vals(p, va[p]);
        }
#pragma unroll 1
      for (int q0 = 0; q0 < D4; q0 += NQ) {
        u16x4 lb[NQ];
        T vb[NQ][4];
#pragma unroll
        for (int p = 0; p < NQ; ++p)
          if (q0 + NQ + p < D4) {
            lb[p] = __builtin_nontemporal_load(lp + (int64_t)(q0 + NQ + p) * nr);
            ld_vals(q0 + NQ + p, vb[p]);
          }
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
          if (q0 + p < D4) {
            const int li[4] = {la[p].x, la[p].y, la[p].z, la[p].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              C x[NC];
#pragma unroll
              for (int c = 0; c < NC; ++c) x[c] = win[c * Wi + li[e]];
#pragma unroll
              for (int c = 0; c < NC; ++c) {
                ar[c] = fma(va[p][e], x[c].x, ar[c]);
                ai[c] = fma(va[p][e], x[c].y, ai[c]);
              }
            }
          }
        }
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
          la[p] = lb[p];
#pragma unroll
          for (int e = 0; e < 4; ++e) va[p][e] = vb[p][e];
        }
      }
    } else {
      // a window beyond the LDS budget: gather from the vectors, the NC x 4
      // values of a quad issued together; with few columns the next quad's
      // column numbers are loaded before them (64 steps: 400^2 rows, 1 column
      // 12.4 -> 10.2 ms; 512^2, 5 columns 10.2 -> 13.5 ms, so not there)
      constexpr bool AHEAD = NC <= 3;
      const CSP_GLOBAL i32x4* gp = reinterpret_cast<const CSP_GLOBAL i32x4*>(
          (const CSP_GLOBAL int32_t*)(I.ellw_col) + qofs);
      i32x4 jn = {0, 0, 0, 0};
      if constexpr (AHEAD) jn = __builtin_nontemporal_load(gp);
#pragma unroll 1
      for (int q = 0; q < D4; ++q) {
        i32x4 j4 = jn;
        if constexpr (!AHEAD) j4 = __builtin_nontemporal_load(gp + (int64_t)q * nr);
        else if (q + 1 < D4) jn = __builtin_nontemporal_load(gp + (int64_t)(q + 1) * nr);
        T v[4];
        ld_vals(q, v);
        const int64_t jj[4] = {j4.x, j4.y, j4.z, j4.w};
        C x[4][NC];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < NC; ++c) x[e][c] = ld<T>(cur + 2 * ((int64_t)c * N + jj[e]));
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            ar[c] = fma(v[e], x[e][c].x, ar[c]);
            ai[c] = fma(v[e], x[e][c].y, ai[c]);
          }
      }
    }
  };
  if (nc == CT) {
    accumulate(std::integral_constant<int, CT>{});
  } else if (CT > 1 && nc == CT - 1) {
    accumulate(std::integral_constant<int, (CT > 1 ? CT - 1 : 1)>{});
  } else {
    // other counts (not produced by ellw_columns_per_group): a branch per
    // column
    const CSP_GLOBAL int32_t* gp = (const CSP_GLOBAL int32_t*)(I.ellw_col) + qofs;
    for (int q = 0; q < D4; ++q) {
      T v[4];
      ld_vals(q, v);
      for (int e = 0; e < 4; ++e) {
        const int64_t j = gp[(int64_t)q * (4 * nr) + e];
        for (int c = 0; c < nc; ++c) {
          const C x = ld<T>(cur + 2 * ((int64_t)c * N + j));
          ar[c] = fma(v[e], x.x, ar[c]);
          ai[c] = fma(v[e], x.y, ai[c]);
        }
      }
    }
  }

  // ---- phi_{n+1} = 2 H~ phi_n - phi_{n-1} of row `row`, epilogues
  const T scale = sp.first ? T(0.5) : T(1);
  const T alpha = scale * static_cast<T>(I.alpha);
  const T beta0 = scale * static_cast<T>(I.beta0);
  const bool dots = MOM && (sp.dot_psi0 || sp.dot_self);
  // record sums of the waves, in the window's place
  double* red = reinterpret_cast<double*>(smem);
  if (dots) __syncthreads();
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    double rec[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (c < nc && valid) {
      const int64_t e = 2 * ((int64_t)c * N + row);
      const C cv = ld<T>(cur + e);
      const C pv = prev ? ld<T>(prev + e) : C{T(0), T(0)};
      C o;
      o.x = alpha * ar[c] + (beta0 * cv.x - pv.x);
      o.y = alpha * ai[c] + (beta0 * cv.y - pv.y);
      if (outv) st<T>(outv + e, o, true);
      if (copyv) st<T>(copyv + e, cv, true);
      if constexpr (CARRY) {
        if (sp.carry_mode && I.carry) {
          const T c0r = static_cast<T>(sp.cc0[0]), c0i = static_cast<T>(sp.cc0[1]);
          const T c1r = static_cast<T>(sp.ccl[0][0]), c1i = static_cast<T>(sp.ccl[0][1]);
          CSP_GLOBAL T* cy = (CSP_GLOBAL T*)(I.carry) + cofs + e;
          C b;
          if (sp.carry_mode == 1) {
            b.x = c0r * cv.x - c0i * cv.y;
            b.y = c0r * cv.y + c0i * cv.x;
          } else {
            b = ld<T>(cy);
          }
          b.x += c1r * o.x - c1i * o.y;
          b.y += c1r * o.y + c1i * o.x;
          st<T>(cy, b, false);
        }
      }
      if constexpr (MOM) {
        if (sp.dot_psi0) {
          const C q = ld<T>((const CSP_GLOBAL T*)(I.psi0) + cofs + e);
          rec[0] = (double)q.x * o.x + (double)q.y * o.y;
          rec[1] = (double)q.x * o.y - (double)q.y * o.x;
          rec[2] = (double)q.x * cv.x + (double)q.y * cv.y;
          rec[3] = (double)q.x * cv.y - (double)q.y * cv.x;
        }
        if (sp.dot_self) {
          rec[4] = (double)o.x * o.x + (double)o.y * o.y;
          rec[6] = (double)o.x * cv.x + (double)o.y * cv.y;
          rec[7] = (double)o.x * cv.y - (double)o.y * cv.x;
        }
      }
    }
    if constexpr (MOM) {
      if (dots) {
        // [kind][re, im]: <psi0|out>, <psi0|cur>, <out|out>, <out|cur>,
        // summed over the wave by a fixed butterfly
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          double x = rec[q];
#pragma unroll
          for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m);
          if (lane == q) red[(wave * CT + c) * 8 + q] = x;
        }
      }
    }
  }
  if constexpr (MOM) {
    if (dots) {
      __syncthreads();
      if (t < 8 * CT) {
        const int c = t >> 3, q = t & 7;
        if (c < nc) {
          const int64_t item = I.item0 + (int64_t)(c0 + c) * I.n_segs + slice;
          sp.partial[((int64_t)sp.mom_slot * sp.total_items + item) * 8 + q] =
              nr == 256 ? ((red[t] + red[8 * CT + t]) + red[16 * CT + t]) + red[24 * CT + t]
                        : red[t] + red[8 * CT + t];
        }
      }
    }
  }
}

}  // namespace ellw

// Columns per workgroup (tile width CT): the group's columns in tiles split
// evenly (25 in four: 7 + 6 + 6 + 6), so every tile holds CT or CT - 1
// columns, at most 8 and at most as many as fit the LDS budget with a window
// of `window` positions.  Every tile reads the matrix once per step (at
// little cost while it stays in the 256 MB of last-level cache); narrow tiles
// take fewer registers and less LDS.  The rule, with `waves` = waves per CU of
// one tile of all slices; figures are calls of 24 time steps of the moment
// form at the stated rows, D and columns (MI355X, ms):
//
// complex64, slices of 128 rows: a launch lasts as many rounds as its waves
// need, so the fewest tiles whose workgroups are all resident at once
// (registers, LDS) and that give a CU seven waves, except up to three columns
// in one tile (160000 rows, D = 61, 7 columns: 2.86 in one tile, 3.14 as
// 3 + 2 + 2 in two rounds; 90000, D = 121, 8 columns: 3.05 as 4 + 4, 3.57 as
// 3 + 3 + 2); tiles of 4 and 6 in twice as many of half the width while those
// still fit one round of 20 waves (160000, D = 121, 4 columns: 2.94 as 2 + 2,
// 3.22).  Where no width fits one round: up to 3 columns (a matrix up to
// 128 MB), 4 (up to 256 MB) or 8 (from HBM) a tile.  With less than five
// waves a CU for a tile, the latency of a workgroup counts: up to 3 columns
// and, if there are as many, three tiles (40000, D = 121, 3 columns: 1.47 as
// 1 + 1 + 1, 1.90; 10 columns: 2.23 as 3 + 3 + 2 + 2, 2.83 as 5 + 5; 73984, 9
// columns: 2.62 as 3 + 3 + 3, 3.15 as 5 + 4); with less than seven, up to 3
// columns where those tiles give no more than four waves per SIMD (84100, 9
// columns: 3.06, 3.51).
//
// In a form that keeps a ring of orders (`ring`: states, quasi-eigenstates,
// conductivity) the orders stream through the cache, so a further tile costs
// more: nine waves instead of seven, and from nine waves a tile on as few tiles
// of up to 7 columns as possible (24 steps: 160000, D = 121, 10 columns 10.5 as
// 5 + 5, 14.1 as 3 + 3 + 2 + 2; 122500, D = 61, 5 columns 3.30 as 3 + 2, 3.68).
//
// complex64, slices of 256 rows (matrices of 160 MB and more): as few tiles
// of up to 7 columns as possible (336400, D = 121: 7 columns 7.50, as 4 + 3
// 8.04; 8 columns 7.93 as 4 + 4, 8.19 in one), but of 6 only from HBM (409600:
// 7.67, as 3 + 3 8.25; 266256, in the cache: 6.11 and 5.39).
//
// complex128: the tiles of up to 6 columns, or 7 in slices of 256 rows, whose
// costs, fitted to 11 matrices of 2..12 columns (a matrix beyond the last-level
// cache, or a ring, adds half a unit a tile), sum to the least and that give a CU five
// waves, or 3.5 up to three columns (90000, D = 121,
// 5 columns: 3.45, as 3 + 2 4.28; 10 columns: 5.96 as 5 + 5, 6.91 as
// 3 + 3 + 2 + 2; 230400, 8 columns: 9.65 as 4 + 4, 12.35 in one; 336400, 9
// columns: 14.8 as 5 + 4, 16.6 as 3 + 3 + 3).  A tile of 6 at a window of 832
// takes 78 KB of LDS: 262144 rows 9.3, as 3 + 3 in 39 KB 9.9.
int ellw_columns_per_group(bool fp64, bool ring, int Rg, int64_t window, int nr, int64_t slices,
                           int64_t entries) {
  if (Rg <= 1) return 1;
  const int64_t value = std::max<int64_t>(window, 1) * (fp64 ? 16 : 8);   // LDS of a column
  const int fit =
      static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(8, kEllwLdsBytes / value)));
  const int64_t mb = (entries * (fp64 ? 10 : 6)) >> 20;
  const double waves = static_cast<double>(slices) * (nr / 64) / 256.0;
  auto width = [&](int tiles) { return (Rg + tiles - 1) / tiles; };
  auto at_most = [&](int cols) { return width((Rg + cols - 1) / cols); };
  if (fp64) {
    constexpr double kCost[7] = {0.6, 0.8, 1.0, 1.3, 1.7, 2.05, 3.0};
    const int most = std::min(nr == 256 ? 7 : 6, fit);
    double best = 1e300;
    int ct = 1;
    for (int k = 1; k <= Rg; ++k) {
      const int w = width(k);
      if (w > most || (k < Rg && waves * k < (w > 3 ? 5.0 : 3.5))) continue;
      const double c = k * (kCost[w - 1] + (ring || mb > 256 ? 0.5 : 0.0));
      if (c < best) {
        best = c;
        ct = w;
      }
    }
    return ct;
  }
  if (nr == 256) {
    const int w = at_most(std::min(7, fit));
    return w == 6 && mb <= 256 ? at_most(5) : w;
  }
  const int narrow = (Rg + std::min(3, fit) - 1) / std::min(3, fit);   // tiles of up to 3
  if (waves < 5.0) return width(std::max(narrow, std::min(Rg, 3)));
  if (!ring && waves < 7.0 && waves * narrow <= 16.0) return width(narrow);
  if (ring && waves >= 9.0) return at_most(std::min(7, fit));
  auto one_round = [&](int tiles) {
    constexpr int kWavesPerSimd[8] = {8, 8, 8, 4, 4, 4, 3, 3};   // from the registers of CT
    const int w = width(tiles);
    if (w > fit) return false;
    const int64_t lds = (w * value + 1279) / 1280 * 1280;
    const int64_t resident =
        std::min<int64_t>(160 * 1024 / lds * (nr / 64), 4 * kWavesPerSimd[w - 1]);
    return waves * tiles <= (double)resident;
  };
  for (int k = 1; k <= Rg; ++k) {
    const int w = width(k);
    if (w > 7 || (w > 3 && waves * k < (ring ? 9.0 : 7.0)) || !one_round(k)) continue;
    const bool halve = (w == 4 || w == 6) && mb <= 256 && waves * 2 * k <= 20.0 && one_round(2 * k);
    return halve ? width(2 * k) : w;
  }
  return at_most(std::min(mb > 256 ? 8 : mb > 128 ? 4 : 3, fit));
}

hipError_t launch_cheb_ellw(bool fp64, bool mom, bool carry, int ct, int nr, int64_t lds_cap,
                            const ChebInst* d_inst, int n_inst, int64_t wg_lo, int64_t wg_hi,
                            const ChebStep& st, hipStream_t s) {
  const int64_t n = wg_hi - wg_lo;
  if (n <= 0) return hipSuccess;
  if (st.nlev != 1 || (carry && !mom)) return hipErrorInvalidValue;
  if (ct < 1 || ct > (fp64 ? 7 : 8) || (nr != 128 && nr != 256)) return hipErrorInvalidValue;
  // LDS: the largest staged window of the run's instances times its
  // columns (lds_cap complex values)
  const size_t lds = std::max<size_t>((size_t)(lds_cap > 0 ? lds_cap : 1) * (fp64 ? 16 : 8),
                                      mom ? (size_t)(nr / 64) * ct * 64 : 0);
  if (lds > (size_t)kEllwLdsBytes) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(n)), block(nr);
#define CSP_ELLW(T, CT, M, CY) \
  hipLaunchKernelGGL((ellw::k_cheb_ellw<T, CT, M, CY>), grid, block, lds, s, d_inst, n_inst, wg_lo, wg_hi, st)
#define CSP_ELLW_CT(T, M, CY)      \
  do {                             \
    switch (ct) {                  \
      case 1: CSP_ELLW(T, 1, M, CY); break; \
      case 2: CSP_ELLW(T, 2, M, CY); break; \
      case 3: CSP_ELLW(T, 3, M, CY); break; \
      case 4: CSP_ELLW(T, 4, M, CY); break; \
      case 5: CSP_ELLW(T, 5, M, CY); break; \
      case 6: CSP_ELLW(T, 6, M, CY); break; \
      default: CSP_ELLW(T, 7, M, CY); break; \
    }                              \
  } while (0)
  if (fp64) {
    if (carry) CSP_ELLW_CT(double, true, true);
    else if (mom) CSP_ELLW_CT(double, true, false);
    else CSP_ELLW_CT(double, false, false);
  } else if (ct == 8) {
    if (carry) CSP_ELLW(float, 8, true, true);
    else if (mom) CSP_ELLW(float, 8, true, false);
    else CSP_ELLW(float, 8, false, false);
  } else {
    if (carry) CSP_ELLW_CT(float, true, true);
    else if (mom) CSP_ELLW_CT(float, true, false);
    else CSP_ELLW_CT(float, false, false);
  }
#undef CSP_ELLW_CT
#undef CSP_ELLW
  return hipGetLastError();
}

}  // namespace csp
