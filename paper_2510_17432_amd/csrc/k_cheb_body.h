// Chebyshev recursion (amxsy of Sec. II.B), several steps per pass over
// memory:  phi_{n+l} = 2 H~ phi_{n+l-1} - phi_{n+l-2},  l = 1..nlev (nlev <=
// KT), with H~ = (H - H0)/|H| the rescaled lattice Hamiltonian of Sec. II.A
// applied as a stencil (no matrix in memory).  The first step of a time
// block is phi_1 = H~ phi_0.
//
// Layout.  A column group is stored column-major: column c of the group is
// one lattice vector, cstride values from the previous one, rows of `opr`
// values in the orbital order of the lattice and `pitch` values apart, so
// the in-row stencil neighbours are at +-1 and the vertical ones one row up
// or down.  The propagation forms pad rows whose length is not a multiple
// of 16 values to one, so that rows start 128-byte aligned (unaligned rows
// measured about a tenth slower); vectors the caller passes in are unpadded
// (pitch = opr).
//
// Work decomposition.  One wave (64 lanes) owns a strip of a row segment of
// one column and is independent of every other wave: no LDS, no barriers.
// Lane l holds the V consecutive positions p0 + V l .. p0 + V l + V - 1 of
// the strip, so a lane loads and stores V values with wide accesses and the
// whole wave touches 64 V consecutive values.  In-row neighbours are in the
// lane's own registers except at its two ends, which come from the adjacent
// lane by a DPP wavefront shift.  On the honeycomb lattice the vertical
// partner of an orbital is the other orbital of its (even, odd) pair one row
// up or down, which is in the same lane (V is even, p0 is even).  A lattice
// of one row has no vertical neighbours: it runs in instantiations of its own
// (kLatRow) whose levels follow one another in registers without a row loop.
//
// The strip covers [os - MG, os - MG + 64 V); each level is valid one
// position further inside on each side than the one before, so after up to
// KT <= MG levels the owned positions [os, os + 64 V - 2 MG) are exact and
// neighbouring strips overlap by 2 MG positions that both compute (the
// redundant-margin form of temporal blocking).  MG is KT rounded up to a
// multiple of V, so every lane is either wholly owned or wholly margin.
// The wave marches down the rows y0 - nlev .. y1 + nlev - 1 of its segment
// keeping, for every level, the last three rows in registers; level l
// computes row r0 - l while level 0 loads row r0, so all levels advance
// together and only the owned rows [y0, y1) of every level are written.
// Per pass the memory traffic is one read of phi_n and phi_{n-1} (plus the
// 2 nlev-row segment margins) and one write per level kept, instead of two
// reads and one write per step.
//
// What bounds it.  On lattices whose vectors exceed the caches, HBM (rows in
// flight: 5.4-6.0 TB/s).  On small and ordinary lattices there are one to
// three waves per SIMD and a wave issues at most one instruction every four
// cycles, so the instructions of a row iteration set the pace: the row loop
// has no register moves (rows rotate by renaming), one 32-bit lane offset
// for all stores with a scalar base per level, incremental row pointers with
// one wrap, no tests in steady rows and one store region per iteration, and
// strips over the seam of a periodic row take the same form.  Against the
// form that moved rows, recomputed 64-bit addresses and ran seam strips
// position by position (MI355X, per launch of 8 steps): 64 x 64 sites 30.4
// -> 14.1 us (plain) and 38.5 -> 16 us (self products), graphene 1024^2 with
// 4 columns and self products 102 -> 74 us, 16 uneven lattices of 64..512
// sites a side 64 -> 30 us; bandwidth-bound launches (68 columns of graphene)
// 2078 -> 2010 us.
//
// Moment variants (moment-based form of Sec. II.A).  MOM = kMomBra: for every
// level and owned value the epilogue accumulates <psi0|phi_{n+l}>,
// <psi0|phi_n> (first level only), <phi_{n+l}|phi_{n+l}> and
// <phi_{n+l}|phi_{n+l-1}> (the products of Eq. cheby_prod), each kind when
// its flag is set; it can also accumulate the carried state
// s_{k+1} = sum_n c_n phi_n of a time block.  MOM = kMomSelf (one block with
// bra = ket, Sec. III DOS-Concurrent-M): only |phi_{n+l}|^2 and
// Re <phi_{n+l}|phi_{n+l-1}>, the two products that give every moment above
// the first two; psi0 is not read and holds no registers.  Products over the
// V values of a lane are summed in the working precision, then in FP64 over
// rows; each wave reduces with a fixed butterfly and writes one record per
// level, so the sums do not depend on the run.
#pragma once

#include <type_traits>

#include "csp_internal.h"

#define CSP_GLOBAL __attribute__((address_space(1)))

namespace csp {
namespace cheb {

// moment epilogue of the recursion kernel (template argument MOM)
constexpr int kMomNone = 0;   // state form: no inner products
constexpr int kMomBra = 1;    // products with psi0 and the self products, by flags
constexpr int kMomSelf = 2;   // self products only (bra = ket, one block)

template <typename T> struct cx {
  T x, y;
};

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(8)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4w __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

// ---- V consecutive complex values of one lane (T units: 2 per value)
template <int V>
__device__ __forceinline__ void ldv(const CSP_GLOBAL float* p, cx<float> (&d)[V]) {
  const CSP_GLOBAL f32x4u* q = reinterpret_cast<const CSP_GLOBAL f32x4u*>(p);
#pragma unroll
  for (int k = 0; k < V / 2; ++k) {
    const f32x4u t = q[k];
    d[2 * k] = {t.x, t.y};
    d[2 * k + 1] = {t.z, t.w};
  }
}
template <int V>
__device__ __forceinline__ void stv(CSP_GLOBAL float* p, const cx<float> (&d)[V]) {
  CSP_GLOBAL f32x4u* q = reinterpret_cast<CSP_GLOBAL f32x4u*>(p);
#pragma unroll
  for (int k = 0; k < V / 2; ++k) {
    f32x4u t;
    t.x = d[2 * k].x;
    t.y = d[2 * k].y;
    t.z = d[2 * k + 1].x;
    t.w = d[2 * k + 1].y;
    q[k] = t;
  }
}
// The orders of a state form are written once and read back only after many
// other vectors have streamed through the caches: non-temporal stores.  The
// moment forms write the two vectors that the next launch reads: cached.
template <int V>
__device__ __forceinline__ void stv_nt(CSP_GLOBAL float* p, const cx<float> (&d)[V]) {
  CSP_GLOBAL f32x4u* q = reinterpret_cast<CSP_GLOBAL f32x4u*>(p);
#pragma unroll
  for (int k = 0; k < V / 2; ++k) {
    f32x4u t;
    t.x = d[2 * k].x;
    t.y = d[2 * k].y;
    t.z = d[2 * k + 1].x;
    t.w = d[2 * k + 1].y;
    __builtin_nontemporal_store(t, q + k);
  }
}
template <int V>
__device__ __forceinline__ void ldv(const CSP_GLOBAL double* p, cx<double> (&d)[V]) {
  const CSP_GLOBAL f64x2u* q = reinterpret_cast<const CSP_GLOBAL f64x2u*>(p);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const f64x2u t = q[v];
    d[v] = {t.x, t.y};
  }
}
template <int V>
__device__ __forceinline__ void stv(CSP_GLOBAL double* p, const cx<double> (&d)[V]) {
  CSP_GLOBAL f64x2u* q = reinterpret_cast<CSP_GLOBAL f64x2u*>(p);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    f64x2u t;
    t.x = d[v].x;
    t.y = d[v].y;
    q[v] = t;
  }
}
template <int V>
__device__ __forceinline__ void stv_nt(CSP_GLOBAL double* p, const cx<double> (&d)[V]) {
  CSP_GLOBAL f64x2u* q = reinterpret_cast<CSP_GLOBAL f64x2u*>(p);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    f64x2u t;
    t.x = d[v].x;
    t.y = d[v].y;
    __builtin_nontemporal_store(t, q + v);
  }
}
__device__ __forceinline__ cx<float> ld1(const CSP_GLOBAL float* p) {
  const f32x2u t = *reinterpret_cast<const CSP_GLOBAL f32x2u*>(p);
  return {t.x, t.y};
}
__device__ __forceinline__ void st1(CSP_GLOBAL float* p, cx<float> v) {
  f32x2u t;
  t.x = v.x;
  t.y = v.y;
  *reinterpret_cast<CSP_GLOBAL f32x2u*>(p) = t;
}
__device__ __forceinline__ cx<double> ld1(const CSP_GLOBAL double* p) {
  const f64x2u t = *reinterpret_cast<const CSP_GLOBAL f64x2u*>(p);
  return {t.x, t.y};
}
__device__ __forceinline__ void st1(CSP_GLOBAL double* p, cx<double> v) {
  f64x2u t;
  t.x = v.x;
  t.y = v.y;
  *reinterpret_cast<CSP_GLOBAL f64x2u*>(p) = t;
}
// V consecutive on-site energies
template <int V>
__device__ __forceinline__ void ldr(const CSP_GLOBAL float* p, float (&d)[V]) {
  if constexpr (V == 4) {
    const f32x4w t = *reinterpret_cast<const CSP_GLOBAL f32x4w*>(p);
    d[0] = t.x;
    d[1] = t.y;
    d[2] = t.z;
    d[3] = t.w;
  } else {
#pragma unroll
    for (int k = 0; k < V / 2; ++k) {
      const f32x2u t = reinterpret_cast<const CSP_GLOBAL f32x2u*>(p)[k];
      d[2 * k] = t.x;
      d[2 * k + 1] = t.y;
    }
  }
}
template <int V>
__device__ __forceinline__ void ldr(const CSP_GLOBAL double* p, double (&d)[V]) {
#pragma unroll
  for (int k = 0; k < V / 2; ++k) {
    const f64x2u t = reinterpret_cast<const CSP_GLOBAL f64x2u*>(p)[k];
    d[2 * k] = t.x;
    d[2 * k + 1] = t.y;
  }
}

// ---- wavefront shifts by one lane (DPP): lane l receives lane l - 1 (shr)
// or lane l + 1 (shl); the lane without a source receives 0.
__device__ __forceinline__ int dpp_shr1_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x138, 0xF, 0xF, true);
}
__device__ __forceinline__ int dpp_shl1_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x130, 0xF, 0xF, true);
}
__device__ __forceinline__ float shr1(float x) {
  return __builtin_bit_cast(float, dpp_shr1_i(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ float shl1(float x) {
  return __builtin_bit_cast(float, dpp_shl1_i(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ double shr1(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)dpp_shr1_i((int)(unsigned)b);
  const unsigned hi = (unsigned)dpp_shr1_i((int)(unsigned)(b >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double shl1(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)dpp_shl1_i((int)(unsigned)b);
  const unsigned hi = (unsigned)dpp_shl1_i((int)(unsigned)(b >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

template <int V, int KT> struct Shape {
  static constexpr int MG = ((KT + V - 1) / V) * V;   // margin positions per side
  static constexpr int OW = 64 * V - 2 * MG;          // owned positions per strip
};

// ---- value of lane l ^ M (M = 1, 2, 4, 8: DPP inside rows of 16 lanes)
template <int M> __device__ __forceinline__ int xor_i(int x) {
  if constexpr (M == 8) return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, true);
  if constexpr (M == 4) {   // reversed inside 8, then inside 4
    x = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true);
    return __builtin_amdgcn_update_dpp(0, x, 0x1B, 0xF, 0xF, true);
  }
  if constexpr (M == 2) return __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true);
  return __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true);
}
// (a, b) -> {a of the lanes with bit M clear, b of those with it set} plus
// the value of lane l ^ M: one step of a sum over the wave that keeps half
// of the quantities in each half of the lanes
template <int M> __device__ __forceinline__ float pair_sum(float a, float b, bool up) {
  if constexpr (M >= 16) {
    const unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
    if constexpr (M == 32) {
      const auto r = __builtin_amdgcn_permlane32_swap(ua, ub, false, false);
      return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
    } else {
      const auto r = __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
      return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
    }
  } else {
    const float keep = up ? b : a, send = up ? a : b;
    return keep + __builtin_bit_cast(float, xor_i<M>(__builtin_bit_cast(int, send)));
  }
}
template <int M> __device__ __forceinline__ double pair_sum(double a, double b, bool up) {
  const unsigned long long la = __builtin_bit_cast(unsigned long long, a);
  const unsigned long long lb = __builtin_bit_cast(unsigned long long, b);
  if constexpr (M >= 16) {
    unsigned x0, x1, y0, y1;
    if constexpr (M == 32) {
      const auto r = __builtin_amdgcn_permlane32_swap((unsigned)la, (unsigned)lb, false, false);
      const auto q = __builtin_amdgcn_permlane32_swap((unsigned)(la >> 32), (unsigned)(lb >> 32),
                                                      false, false);
      x0 = r[0]; y0 = r[1]; x1 = q[0]; y1 = q[1];
    } else {
      const auto r = __builtin_amdgcn_permlane16_swap((unsigned)la, (unsigned)lb, false, false);
      const auto q = __builtin_amdgcn_permlane16_swap((unsigned)(la >> 32), (unsigned)(lb >> 32),
                                                      false, false);
      x0 = r[0]; y0 = r[1]; x1 = q[0]; y1 = q[1];
    }
    return __builtin_bit_cast(double, ((unsigned long long)x1 << 32) | x0) +
           __builtin_bit_cast(double, ((unsigned long long)y1 << 32) | y0);
  } else {
    const double keep = up ? b : a;
    const unsigned long long s = up ? la : lb;
    const unsigned lo = (unsigned)xor_i<M>((int)(unsigned)s);
    const unsigned hi = (unsigned)xor_i<M>((int)(unsigned)(s >> 32));
    return keep + __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
  }
}
// Sum of every x[k] over the wave, pairs of lanes 32, 16, 8, 4, 2, 1 apart
// added in that order (each quantity is added in the same order whatever
// its index); quantity k ends in lane sum_lane<N>(k).  A plain butterfly
// takes 6 N cross-lane moves; here each step halves the quantities a lane
// holds (N = 16: 17 moves).
template <int N, int M, typename T>
__device__ __forceinline__ T wave_sums(T (&x)[N], int lane) {
  constexpr int H = (N + 1) / 2;
  T y[H];
#pragma unroll
  for (int k = 0; k < H; ++k) y[k] = pair_sum<M>(x[k], k + H < N ? x[k + H] : x[k], (lane & M) != 0);
  if constexpr (M > 1) return wave_sums<H, M / 2>(y, lane);
  else return y[0];
}
template <int N, int M = 32> __device__ __forceinline__ int sum_lane(int k) {
  constexpr int H = (N + 1) / 2;
  const int bit = k >= H ? M : 0;
  if constexpr (M > 1) return bit + sum_lane<H, M / 2>(k >= H ? k - H : k);
  else return bit;
}

// Marks a register row as holding nothing: the slots of a level that has
// not started, or of a row that is not fetched, need not be kept (carrying
// them through the skipped iterations cost a third slot per level, 24-30
// VGPRs at 8 levels).
template <typename T, int V> __device__ __forceinline__ void any_row(cx<T> (&d)[V]) {
#pragma unroll
  for (int v = 0; v < V; ++v) {
    d[v].x = __builtin_nondeterministic_value(d[v].x);
    d[v].y = __builtin_nondeterministic_value(d[v].y);
  }
}

// insts: the instances of this launch (consecutive items item_lo..item_hi-1).
// DIAG: the Hamiltonian has a diagonal (on-site energies, or H0 != 0).
template <typename T, int V, int KT, int LAT, bool DIAG, int MOM, bool CARRY>
__global__ __launch_bounds__(256) void k_cheb(const ChebInst* __restrict__ insts, int n_inst,
                                              int64_t item_lo, int64_t item_hi, ChebStep st) {
  static_assert(V % 2 == 0, "lanes hold whole (even, odd) orbital pairs");
  static_assert(!CARRY || MOM != kMomSelf, "one block with bra = ket carries no state");
  constexpr bool HONEY = LAT == kLatHoney;
  // sequential form: the recursion with the carried state and, in a time
  // step's last launch, <psi0|carried state>, without moments
  constexpr bool SEQ = CARRY && MOM == kMomNone;
  // forms that keep the two newest levels of a launch only
  constexpr bool KEEP2 = CARRY || MOM != kMomNone;
  using C = cx<T>;
  using gT = CSP_GLOBAL T;
  using gB = CSP_GLOBAL char;
  constexpr int MG = Shape<V, KT>::MG;
  constexpr int OW = Shape<V, KT>::OW;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int64_t item = item_lo + xcd_remap(blockIdx.x, gridDim.x) * 4 + wave;
  if (item >= item_hi) return;                     // a whole wave; no barriers below
  // the last instance whose first item is not past this one: 64 at a time
  int ii = 0;
  if (n_inst > 1) {
    ii = -1;
    for (int k = 0; k < n_inst; k += 64)
      ii += __popcll(__ballot(k + lane < n_inst && item >= insts[k + lane].item0));
  }
  const ChebInst& I = insts[ii];

  // ---- geometry of this work item (wave-uniform)
  const int n_strips = static_cast<int>(I.n_strips);
  const int64_t per_col = I.n_strips * I.n_segs;
  const int64_t local = item - I.item0;
  int64_t col;
  int rem;                                          // n_strips x n_segs <= N < 2^31
  if (local < ((int64_t)1 << 31)) {
    const unsigned c32 = static_cast<unsigned>(local) / static_cast<unsigned>(per_col);
    col = c32;
    rem = static_cast<int>(static_cast<unsigned>(local) - c32 * static_cast<unsigned>(per_col));
  } else {
    col = local / per_col;
    rem = static_cast<int>(local - col * per_col);
  }
  const int seg = static_cast<int>(static_cast<unsigned>(rem) / static_cast<unsigned>(n_strips));
  const int strip = rem - seg * n_strips;
  // positions, rows and offsets inside one lattice vector fit in 32 bits
  // (the host checks N < 2^31)
  const int opr = static_cast<int>(I.opr), Ly = static_cast<int>(I.Ly);
  const int os = strip * OW;                         // first owned position
  const int p0 = os - MG;                            // first position of the strip
  const int y0 = seg * st.seg_rows;
  const int y1 = (y0 + st.seg_rows < Ly) ? y0 + st.seg_rows : Ly;
  const int H = y1 - y0;                             // owned rows
  const int nlev = st.nlev;
  const bool px = I.px != 0, py = I.py != 0;
  const int64_t coff = 2 * col * I.cstride;          // column offset in T units
  const int64_t pitch = I.pitch;
  const int64_t pitchB = pitch * (int64_t)sizeof(C);
  // iterations: the segment's rows and nlev margin rows on each side, in
  // whole triples (the extra iterations compute rows past the segment, which
  // are neither stored nor summed, from loads of rows that are inside the
  // lattice or absent and read as zero)
  const int n_iter = (H + 2 * nlev + 2) / 3 * 3;
  const int rbase = y0 - nlev;                       // level-0 row of iteration 0

  // ---- per-lane positions.  Whole lanes: every lane's V positions are
  // sites that follow each other in memory, after wrapping too, and are
  // owned together; every row is inside the lattice after wrapping; and the
  // segment spans less than 2^32 bytes.  True of strips inside a row, and of
  // those over the seam of a periodic row of a multiple of V values, away
  // from open edges: wide loads and stores at one 32-bit lane offset.
  const int lq = V * lane;
  const bool inside = p0 >= 0 && p0 + 64 * V <= opr;
  const bool whole = (inside || (px && opr % V == 0)) &&
                     (py || (rbase >= (CARRY ? nlev : 1) && rbase + n_iter <= Ly)) &&
                     pitchB * (n_iter + 2) < ((int64_t)1 << 32);
  const bool lane_in = lq >= MG && lq < MG + OW;

  gB* base = (gB*)(I.base);
  const int64_t slotB = I.slot_stride * (int64_t)sizeof(C);
  const int64_t coffB = coff * (int64_t)sizeof(T);
  const gB* curv =
      (st.slot_cur < 0 ? (const gB*)(I.src) : base + st.slot_cur * slotB) + coffB;
  const gB* prevv = st.first ? nullptr : base + st.slot_prev * slotB + coffB;
  gB* copyv = st.copy_slot >= 0 ? base + st.copy_slot * slotB + coffB : nullptr;
  const gT* eps = (const gT*)(I.eps);
  const gB* psi0 = (const gB*)(I.psi0) + coffB;
  gB* carry = CARRY && I.carry ? (gB*)(I.carry) + coffB : nullptr;

  // output slot of each level (nullptr: not stored); the moment forms store
  // the two newest levels of a launch only
  gB* outv[KT];
#pragma unroll
  for (int l = 0; l < KT; ++l)
    outv[l] = st.slot_out[l] >= 0 ? base + st.slot_out[l] * slotB + coffB : nullptr;

  // ---- register rows: rr[l][.] = the last three rows of level l.  The
  // three slots rotate with the row index: before an iteration of phase
  // P = i mod 3, slot P holds the oldest row, P + 1 the middle and P + 2 the
  // newest; the iteration overwrites slot P with the new row, and the row
  // loop is unrolled by three so every slot index is a constant (rotation by
  // renaming, no register moves).
  C rr[KT][3][V];
#pragma unroll
  for (int l = 0; l < KT; ++l)
#pragma unroll
    for (int k = 0; k < 3; ++k) any_row(rr[l][k]);
  T br[DIAG ? KT + 1 : 1][V];                        // diagonal of 2 H~ in rows r0 - k
#pragma unroll
  for (int k = 0; k < (DIAG ? KT + 1 : 1); ++k)
#pragma unroll
    for (int v = 0; v < V; ++v) br[k][v] = T(0);

  // Moment sums.  kMomBra: quantity q = 5 (l - 1) + j for level l: j = 0, 1
  // <psi0|out>, 2 |out|^2, 3, 4 <out|cur>; q = 5 KT + 0, 1: <psi0|cur> of
  // the first level.  kMomSelf: q = 2 (l - 1) + j: j = 0 |out|^2, 1
  // Re <out|cur>.  sq holds this lane's working-precision sums of the last
  // rows; every kFlush rows each is summed over the wave and added in FP64
  // into accq of lane sum_lane(q).
  constexpr int kFlush = 16;
  constexpr int NQ = MOM == kMomBra ? 5 * KT + 2 : (MOM == kMomSelf ? 2 * KT : 1);
  T sq[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) sq[k] = T(0);
  double accq = 0.0;
  // psi0 rows r0 - k (moment epilogue)
  C pq[MOM == kMomBra ? KT + 1 : 1][V];
#pragma unroll
  for (int k = 0; k < (MOM == kMomBra ? KT + 1 : 1); ++k)
#pragma unroll
    for (int v = 0; v < V; ++v) pq[k][v] = {T(0), T(0)};
  const bool dots = MOM == kMomSelf || (MOM == kMomBra && (st.dot_psi0 || st.dot_self));
  const bool want_psi0 = MOM == kMomBra && st.dot_psi0;
  const bool dot_carry = SEQ && st.dot_psi0;
  T sd[2] = {T(0), T(0)};                            // <psi0|carried state> of this lane
  // carried state: partial sums of rows r0 - 1 - j (j < KT) in registers;
  // a row is read (carry_mode 2), completed and written once per launch
  const bool carry_on = CARRY && carry && st.carry_mode != 0;
  const bool carry_in = CARRY && carry && st.carry_mode == 2;
  C cpr[CARRY ? KT : 1][V];
#pragma unroll
  for (int k = 0; k < (CARRY ? KT : 1); ++k)
#pragma unroll
    for (int v = 0; v < V; ++v) cpr[k][v] = {T(0), T(0)};

  // phi_{n+l} = alpha (sum of neighbours) + (diagonal phi_{n+l-1} - phi_{n+l-2});
  // the first step of a block takes half of both coefficients (exact)
  const T alpha = static_cast<T>(I.alpha);
  const T beta0 = static_cast<T>(I.beta0);
  const T oscale = static_cast<T>(I.onsite_scale);
  const T half1 = st.first ? T(0.5) : T(1);
  const T alpha1 = half1 * alpha;

  // Rows loaded ahead of their use: with one wave per SIMD (small lattices)
  // an iteration takes less time than a load from HBM, so the plain and
  // self-product forms keep three rows in flight, one per phase; the forms
  // that also read psi0 or the carried state, one.
  constexpr int PF = MOM == kMomBra || CARRY || (MOM == kMomSelf && sizeof(T) == 8) ? 1 : 3;

  auto run = [&](auto whole_tag) {
    constexpr bool WHOLE = decltype(whole_tag)::value;
    // general form: positions one by one
    int wpos[V];          // position inside the row (wrapped), valid when present
    bool pres[V];         // position is a site of the lattice
    bool own[V];          // position owned by this strip
    unsigned lb = 0;      // WHOLE: byte offset of the lane's values in a row
    bool lane_own = lane_in;
    if constexpr (WHOLE) {
      int w = p0 + lq;
      lane_own = lane_in && w < opr;
      if (!inside) {
        w %= opr;
        if (w < 0) w += opr;
      }
      lb = static_cast<unsigned>(w) * static_cast<unsigned>(sizeof(C));
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int p = p0 + lq + v;
        if (px) {
          int w = p % opr;
          if (w < 0) w += opr;
          wpos[v] = w;
          pres[v] = true;
        } else {
          pres[v] = p >= 0 && p < opr;
          wpos[v] = pres[v] ? p : 0;
        }
        own[v] = lane_in && p >= 0 && p < opr;
      }
    }
    auto load_row = [&](const gB* rowp, bool rp, C (&d)[V]) {
      if constexpr (WHOLE) {
        ldv<V>((const gT*)(rowp + lb), d);
      } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
          d[v] = rp && pres[v] ? ld1((const gT*)rowp + 2 * (int64_t)wpos[v]) : C{T(0), T(0)};
      }
    };
    auto store_row = [&](gB* rowp, const C (&o)[V]) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (own[v]) st1((gT*)rowp + 2 * (int64_t)wpos[v], o[v]);
    };
    // WHOLE: rows are written at base[level] + i pitchB + lane offset
    // (32 bits), base[l] = the level's row of iteration 0
    gB* outb[KT];
    gB* copyb = copyv + (int64_t)rbase * pitchB;
    gB* carryb = carry + (int64_t)(rbase - nlev) * pitchB;
#pragma unroll
    for (int l = 1; l <= KT; ++l) outb[l - 1] = outv[l - 1] + (int64_t)(rbase - l) * pitchB;
    unsigned so = lb;                                // lb + i pitchB

    C nc[PF][V], np[PF][V], nq[MOM == kMomBra ? PF : 1][V], nk[CARRY ? PF : 1][V];
    C nd[SEQ ? PF : 1][V], cd[V];                    // psi0 rows of the completed carried rows
    T ne[DIAG ? PF : 1][V];
    C pv[V], car[V];
#pragma unroll
    for (int k = 0; k < PF; ++k)
#pragma unroll
      for (int v = 0; v < V; ++v) np[k][v] = {T(0), T(0)};
    // next row to load: index (wrapped in a periodic lattice) and byte
    // offset; the row before it (phi_{n-1} lags one row, the carried state
    // nlev rows)
    int lrow = rbase;
    if (py) {
      lrow %= Ly;
      if (lrow < 0) lrow += Ly;
    }
    int64_t lo = lrow * pitchB;
    int prow = lrow - 1;
    if (py && prow < 0) prow += Ly;
    int64_t po = prow * pitchB;
    int krow = lrow - nlev;
    if (CARRY && py) {
      krow %= Ly;
      if (krow < 0) krow += Ly;
    }
    int64_t ko = krow * pitchB;
    auto owned_row = [&](int k) { return static_cast<unsigned>(k) < static_cast<unsigned>(H); };
    auto row_in = [&](int r) { return static_cast<unsigned>(r) < static_cast<unsigned>(Ly); };
    auto fetch = [&](auto slot_tag) {
      constexpr int B = decltype(slot_tag)::value;
      const bool rp = WHOLE || row_in(lrow);
      load_row(curv + lo, rp, nc[B]);
      if (prevv) load_row(prevv + po, WHOLE || row_in(prow), np[B]);
      if constexpr (DIAG) {
        if (!eps) {
#pragma unroll
          for (int v = 0; v < V; ++v) ne[B][v] = T(0);
        } else {
          const gT* rowp = eps + (int64_t)lrow * opr;
          if constexpr (WHOLE) {
            ldr<V>((const gT*)((const gB*)rowp + lb / 2), ne[B]);
          } else {
#pragma unroll
            for (int v = 0; v < V; ++v) ne[B][v] = rp && pres[v] ? rowp[wpos[v]] : T(0);
          }
        }
      }
      if constexpr (MOM == kMomBra)
        if (want_psi0) load_row(psi0 + lo, rp, nq[B]);
      if constexpr (CARRY) {
        if (carry_in) load_row(carry + ko, WHOLE || row_in(krow), nk[B]);
        if constexpr (SEQ)
          if (dot_carry) load_row(psi0 + ko, WHOLE || row_in(krow), nd[B]);
        ++krow;
        ko += pitchB;
        if (py && krow == Ly) {
          krow = 0;
          ko = 0;
        }
      }
      prow = lrow;
      po = lo;
      ++lrow;
      lo += pitchB;
      if (py && lrow == Ly) {
        lrow = 0;
        lo = 0;
      }
    };
    fetch(std::integral_constant<int, 0>{});
    if constexpr (PF == 3) {
      fetch(std::integral_constant<int, 1>{});
      fetch(std::integral_constant<int, 2>{});
    }

    int flush_in = kFlush;                           // rows left before the next flush
    // one iteration: level 0 takes row r0 = rbase + i, level l computes row
    // r0 - l; the phase selects the register slots.  STEADY iterations are
    // those in which all KT levels run and compute rows of the segment
    // (i in [2 KT, H + KT + 1) with nlev = KT): no level or row tests.
    // Launches that copy phi_n have none.
    auto iter = [&](auto phase_tag, auto steady_tag, int i) {
      constexpr int P = decltype(phase_tag)::value;
      constexpr bool STEADY = decltype(steady_tag)::value;
      // slots after this iteration's new rows: oldest, middle, newest
      constexpr int SLO = (P + 1) % 3, SMI = (P + 2) % 3, SHI = P;
      constexpr int B = PF == 3 ? P : 0;
      const int r0 = rbase + i;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        rr[0][SHI][v] = nc[B][v];
        pv[v] = np[B][v];
      }
      if constexpr (DIAG) {
#pragma unroll
        for (int k = KT; k >= 1; --k)
#pragma unroll
          for (int v = 0; v < V; ++v) br[k][v] = br[k - 1][v];
#pragma unroll
        for (int v = 0; v < V; ++v) br[0][v] = beta0 + oscale * ne[B][v];
      }
      if constexpr (MOM == kMomBra) {
#pragma unroll
        for (int k = KT; k >= 1; --k)
#pragma unroll
          for (int v = 0; v < V; ++v) pq[k][v] = pq[k - 1][v];
#pragma unroll
        for (int v = 0; v < V; ++v) pq[0][v] = nq[B][v];
      }
      if constexpr (CARRY) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          car[v] = nk[B][v];
          if constexpr (SEQ) cd[v] = nd[B][v];
        }
#pragma unroll
        for (int k = KT - 1; k >= 1; --k)
#pragma unroll
          for (int v = 0; v < V; ++v) cpr[k][v] = cpr[k - 1][v];
#pragma unroll
        for (int v = 0; v < V; ++v) cpr[0][v] = {T(0), T(0)};
      }
      // (a steady iteration of four or more levels always has PF rows to go)
      if ((STEADY && KT > PF) || i + PF < n_iter) {
        fetch(std::integral_constant<int, B>{});
      } else {
        any_row(nc[B]);
        if (prevv) any_row(np[B]);
      }
      // phi_n itself for the contraction (order 0 of a block; no steady form)
      if (!STEADY && copyv && owned_row(i - nlev)) {
        if constexpr (WHOLE) {
          if (lane_own) stv_nt<V>((gT*)(copyb + so), rr[0][SHI]);
        } else {
          store_row(copyv + (int64_t)r0 * pitchB, rr[0][SHI]);
        }
      }
      C olast[V];                                    // level KT (the others are in rr)
      // levels that have their three input rows
      const int lmax = i / 2 < nlev ? i / 2 : nlev;

#pragma unroll
      for (int l = 1; l <= KT; ++l) {
        if constexpr (!STEADY) {
          if (l > lmax) {                            // not started: any contents
            if (l < KT) any_row(rr[l < KT ? l : 0][SHI]);
            else any_row(olast);
            continue;
          }
        }
        const int r = r0 - l;
        // a row outside an open lattice is zero: its neighbours count for
        // nothing and its own rows of the two levels before are zero
        T as = l == 1 ? alpha1 : alpha;
        if constexpr (!WHOLE)
          if (!py && !row_in(r)) as = T(0);
        // level l-1 rows r - 1, r, r + 1 and level l-2 row r (phi_{n+l-2})
        const C(&up)[V] = rr[l - 1][SLO];
        const C(&c)[V] = rr[l - 1][SMI];
        const C(&dn)[V] = rr[l - 1][SHI];
        C o[V];
        const T lx = shr1(c[V - 1].x), ly = shr1(c[V - 1].y);
        const T rx = shl1(c[0].x), ry = shl1(c[0].y);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          T nx = (v > 0 ? c[v - 1].x : lx) + (v < V - 1 ? c[v + 1].x : rx);
          T ny = (v > 0 ? c[v - 1].y : ly) + (v < V - 1 ? c[v + 1].y : ry);
          if constexpr (HONEY) {
            // even orbital: partner one row up (pos + 1); odd: one row down (pos - 1)
            if (v % 2 == 0) {
              nx += up[v + 1].x;
              ny += up[v + 1].y;
            } else {
              nx += dn[v - 1].x;
              ny += dn[v - 1].y;
            }
          } else {
            // (a chain's rows -1 and 1 are absent: zero)
            nx += up[v].x + dn[v].x;
            ny += up[v].y + dn[v].y;
          }
          const C p = l == 1 ? pv[v] : rr[l - 2 >= 0 ? l - 2 : 0][SLO][v];
          if constexpr (DIAG) {
            const T beta = l == 1 ? half1 * br[1][v] : br[l][v];
            o[v].x = as * nx + (beta * c[v].x - p.x);
            o[v].y = as * ny + (beta * c[v].y - p.y);
          } else {
            o[v].x = as * nx - p.x;
            o[v].y = as * ny - p.y;
          }
        }
        if constexpr (!WHOLE) {
#pragma unroll
          for (int v = 0; v < V; ++v)
            if (!pres[v]) o[v] = {T(0), T(0)};
        }
        if (l < KT) {
#pragma unroll
          for (int v = 0; v < V; ++v) rr[l][SHI][v] = o[v];
        }
        if constexpr (WHOLE) {
          if (l == KT) {
#pragma unroll
            for (int v = 0; v < V; ++v) olast[v] = o[v];
          }
        }
        if (STEADY || owned_row(i - nlev - l)) {
          if constexpr (!WHOLE)
            if (!KEEP2 || (l >= nlev - 1 && outv[l - 1]))
              store_row(outv[l - 1] + (int64_t)r * pitchB, o);
          if constexpr (MOM == kMomSelf) {
            const int q0 = 2 * (l - 1);
#pragma unroll
            for (int v = 0; v < V; ++v) {
              const bool w = WHOLE ? true : own[v];
              const C oo = w ? o[v] : C{T(0), T(0)};
              // one accumulating FMA per product
              sq[q0] += oo.x * oo.x;
              sq[q0] += oo.y * oo.y;
              sq[q0 + 1] += oo.x * c[v].x;
              sq[q0 + 1] += oo.y * c[v].y;
            }
          }
          if constexpr (MOM == kMomBra) {
            if (dots) {
              // values outside the owned positions take no part in the sums
              // (whole lanes: masked when the sums are flushed)
              C oo[V], cc[V];
#pragma unroll
              for (int v = 0; v < V; ++v) {
                const bool w = WHOLE ? true : own[v];
                oo[v] = w ? o[v] : C{T(0), T(0)};
                cc[v] = w ? c[v] : C{T(0), T(0)};
              }
              const C(&q)[V] = pq[l];
              const int q0 = 5 * (l - 1);
#pragma unroll
              for (int v = 0; v < V; ++v) {
                if (want_psi0) {
                  sq[q0] += q[v].x * oo[v].x;
                  sq[q0] += q[v].y * oo[v].y;
                  sq[q0 + 1] += q[v].x * oo[v].y;
                  sq[q0 + 1] -= q[v].y * oo[v].x;
                  if (l == 1) {
                    sq[5 * KT] += q[v].x * cc[v].x;
                    sq[5 * KT] += q[v].y * cc[v].y;
                    sq[5 * KT + 1] += q[v].x * cc[v].y;
                    sq[5 * KT + 1] -= q[v].y * cc[v].x;
                  }
                }
                if (st.dot_self) {
                  sq[q0 + 2] += oo[v].x * oo[v].x;
                  sq[q0 + 2] += oo[v].y * oo[v].y;
                  sq[q0 + 3] += oo[v].x * c[v].x;
                  sq[q0 + 3] += oo[v].y * c[v].y;
                  sq[q0 + 4] += oo[v].x * c[v].y;
                  sq[q0 + 4] -= oo[v].y * c[v].x;
                }
              }
            }
          }
          if constexpr (CARRY) {
            // level l adds c_{n+l} phi_{n+l} (and the first launch of a
            // block c_n phi_n) to the partial carried row r = r0 - l
            if (carry_on) {
              const T clr = static_cast<T>(st.ccl[l - 1][0]), cli = static_cast<T>(st.ccl[l - 1][1]);
              const T c0r = static_cast<T>(st.cc0[0]), c0i = static_cast<T>(st.cc0[1]);
#pragma unroll
              for (int v = 0; v < V; ++v) {
                C& b = cpr[l - 1][v];
                b.x += clr * o[v].x - cli * o[v].y;
                b.y += clr * o[v].y + cli * o[v].x;
                if (l == 1 && st.carry_mode == 1) {
                  b.x += c0r * c[v].x - c0i * c[v].y;
                  b.y += c0r * c[v].y + c0i * c[v].x;
                }
              }
              if (l == nlev) {                       // row r is complete
                C b[V];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                  b[v] = cpr[l - 1][v];
                  if (st.carry_mode == 2) {
                    b[v].x += car[v].x;
                    b[v].y += car[v].y;
                  }
                }
                if constexpr (SEQ) {
                  if (dot_carry) {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                      const bool w = WHOLE ? true : own[v];
                      const C q = w ? cd[v] : C{T(0), T(0)};
                      sd[0] += q.x * b[v].x;
                      sd[0] += q.y * b[v].y;
                      sd[1] += q.x * b[v].y;
                      sd[1] -= q.y * b[v].x;
                    }
                  }
                }
                if constexpr (WHOLE) {
                  if (lane_own) stv<V>((gT*)(carryb + so), b);
                } else {
                  store_row(carry + (int64_t)r * pitchB, b);
                }
              }
            }
          }
        }
      }
      // Whole lanes are stored after all levels, so that one test of the
      // lane covers them and the level loop is straight-line code
      if constexpr (WHOLE) {
        if (lane_own) {
#pragma unroll
          for (int l = 1; l <= KT; ++l) {
            if constexpr (STEADY) {
              if (KEEP2 && l < KT - 1) continue;
            } else {
              if (l > lmax) break;
              if (!owned_row(i - nlev - l) || (KEEP2 && l < nlev - 1)) continue;
            }
            if constexpr (SEQ)
              if (!outv[l - 1]) continue;            // a time step's last launch keeps none
            const C(&row)[V] = l < KT ? rr[l < KT ? l : 0][SHI] : olast;
            if constexpr (!KEEP2) stv_nt<V>((gT*)(outb[l - 1] + so), row);
            else stv<V>((gT*)(outb[l - 1] + so), row);
          }
        }
        so += static_cast<unsigned>(pitchB);
      }
      if constexpr (MOM != kMomNone) {
        if (dots && (--flush_in == 0 || i + 1 == n_iter)) {
          flush_in = kFlush;
          T x[NQ];
#pragma unroll
          for (int k = 0; k < NQ; ++k) {
            x[k] = (WHOLE && !lane_own) ? T(0) : sq[k];
            sq[k] = T(0);
          }
          accq += static_cast<double>(wave_sums<NQ, 32>(x, lane));
        }
      }
    };
    // iterations [i0, i1), multiples of three
    auto iter_range = [&](auto steady_tag, int i0, int i1) {
#pragma unroll 1
      for (int i = i0; i < i1; i += 3) {
        iter(std::integral_constant<int, 0>{}, steady_tag, i);
        iter(std::integral_constant<int, 1>{}, steady_tag, i + 1);
        iter(std::integral_constant<int, 2>{}, steady_tag, i + 2);
      }
    };
    if constexpr (WHOLE) {
      // steady iterations [ia, ib), rounded inwards to multiples of three
      int ia = n_iter, ib = n_iter;
      if (nlev == KT && !copyv) {
        ia = (2 * KT + 2) / 3 * 3;
        ib = (H + KT + 1) / 3 * 3;
        if (ib < ia) ia = ib = n_iter;
      }
      iter_range(std::false_type{}, 0, ia);
      iter_range(std::true_type{}, ia, ib);
      iter_range(std::false_type{}, ib, n_iter);
      if (!lane_own) sd[0] = sd[1] = T(0);
    } else {
      iter_range(std::false_type{}, 0, n_iter);
    }
  };
  // One open row (a chain): a level needs only the row of the level before
  // and no margin rows; a launch is one read of phi_n and phi_{n-1} and the
  // stores.  The row loop takes 2 nlev + 1 iterations for it, and positions
  // one by one (4e6 sites x 4 columns, complex128, MI355X: one block of 32
  // steps by self products 19.7 -> 2.7 ms, 32 sequential steps 188 -> 25 ms,
  // two blocks of states 66 -> 40 ms, 16.9 of them in the recursion: 4 TB/s).
  auto run_chain = [&]() {
    const bool wide = inside || (px && opr % V == 0);
    int wpos[V];
    bool pres[V], own[V];
    bool lane_own = lane_in;
    {
      int w = p0 + lq;
      lane_own = lane_in && w < opr;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int p = p0 + lq + v;
        int u = p;
        if (px) {
          u %= opr;
          if (u < 0) u += opr;
          pres[v] = true;
        } else {
          pres[v] = p >= 0 && p < opr;
          if (!pres[v]) u = 0;
        }
        wpos[v] = u;
        own[v] = lane_in && p >= 0 && p < opr;
      }
    }
    auto load = [&](const gB* rowp, C (&d)[V]) {
      if (wide) {
        ldv<V>((const gT*)rowp + 2 * (int64_t)wpos[0], d);
      } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
          d[v] = pres[v] ? ld1((const gT*)rowp + 2 * (int64_t)wpos[v]) : C{T(0), T(0)};
      }
    };
    auto store = [&](gB* rowp, const C (&o)[V], bool nt) {
      if (wide) {
        if (!lane_own) return;
        if (nt) stv_nt<V>((gT*)rowp + 2 * (int64_t)wpos[0], o);
        else stv<V>((gT*)rowp + 2 * (int64_t)wpos[0], o);
      } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (own[v]) st1((gT*)rowp + 2 * (int64_t)wpos[v], o[v]);
      }
    };
    C a[V], c[V], q[V], b[V];                        // phi_{n+l-2}, phi_{n+l-1}, psi0, carry
    T beta[DIAG ? V : 1];
    load(curv, c);
#pragma unroll
    for (int v = 0; v < V; ++v) a[v] = q[v] = b[v] = {T(0), T(0)};
    if (prevv) load(prevv, a);
    if (want_psi0 || dot_carry) load(psi0, q);
    if (carry_in) load(carry, b);
    if constexpr (DIAG) {
#pragma unroll
      for (int v = 0; v < V; ++v) beta[v] = beta0 + oscale * (eps && pres[v] ? eps[wpos[v]] : T(0));
    }
    if (copyv) store(copyv, c, true);
    C part[V];                                       // sum_l c_{n+l} phi_{n+l}
#pragma unroll
    for (int v = 0; v < V; ++v) part[v] = {T(0), T(0)};
#pragma unroll
    for (int l = 1; l <= KT; ++l) {
      if (l > nlev) break;
      const T as = l == 1 ? alpha1 : alpha;
      C o[V];
      const T lx = shr1(c[V - 1].x), ly = shr1(c[V - 1].y);
      const T rx = shl1(c[0].x), ry = shl1(c[0].y);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const T nx = (v > 0 ? c[v - 1].x : lx) + (v < V - 1 ? c[v + 1].x : rx);
        const T ny = (v > 0 ? c[v - 1].y : ly) + (v < V - 1 ? c[v + 1].y : ry);
        if constexpr (DIAG) {
          const T be = l == 1 ? half1 * beta[v] : beta[v];
          o[v].x = as * nx + (be * c[v].x - a[v].x);
          o[v].y = as * ny + (be * c[v].y - a[v].y);
        } else {
          o[v].x = as * nx - a[v].x;
          o[v].y = as * ny - a[v].y;
        }
        if (!pres[v]) o[v] = {T(0), T(0)};
      }
      if ((!KEEP2 || l >= nlev - 1) && outv[l - 1]) store(outv[l - 1], o, !KEEP2);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const C oo = own[v] ? o[v] : C{T(0), T(0)};
        const C cc = own[v] ? c[v] : C{T(0), T(0)};
        if constexpr (MOM == kMomSelf) {
          const int q0 = 2 * (l - 1);
          sq[q0] += oo.x * oo.x;
          sq[q0] += oo.y * oo.y;
          sq[q0 + 1] += oo.x * cc.x;
          sq[q0 + 1] += oo.y * cc.y;
        }
        if constexpr (MOM == kMomBra) {
          const int q0 = 5 * (l - 1);
          if (want_psi0) {
            sq[q0] += q[v].x * oo.x;
            sq[q0] += q[v].y * oo.y;
            sq[q0 + 1] += q[v].x * oo.y;
            sq[q0 + 1] -= q[v].y * oo.x;
            if (l == 1) {
              sq[5 * KT] += q[v].x * cc.x;
              sq[5 * KT] += q[v].y * cc.y;
              sq[5 * KT + 1] += q[v].x * cc.y;
              sq[5 * KT + 1] -= q[v].y * cc.x;
            }
          }
          if (st.dot_self) {
            sq[q0 + 2] += oo.x * oo.x;
            sq[q0 + 2] += oo.y * oo.y;
            sq[q0 + 3] += oo.x * cc.x;
            sq[q0 + 3] += oo.y * cc.y;
            sq[q0 + 4] += oo.x * cc.y;
            sq[q0 + 4] -= oo.y * cc.x;
          }
        }
        if constexpr (CARRY) {
          const T clr = static_cast<T>(st.ccl[l - 1][0]), cli = static_cast<T>(st.ccl[l - 1][1]);
          part[v].x += clr * o[v].x - cli * o[v].y;
          part[v].y += clr * o[v].y + cli * o[v].x;
          if (l == 1 && st.carry_mode == 1) {
            const T c0r = static_cast<T>(st.cc0[0]), c0i = static_cast<T>(st.cc0[1]);
            part[v].x += c0r * c[v].x - c0i * c[v].y;
            part[v].y += c0r * c[v].y + c0i * c[v].x;
          }
        }
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        a[v] = c[v];
        c[v] = o[v];
      }
    }
    if constexpr (CARRY) {
      if (carry_on) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          b[v].x = part[v].x + b[v].x;
          b[v].y = part[v].y + b[v].y;
          if (SEQ && dot_carry) {
            const C w = own[v] ? q[v] : C{T(0), T(0)};
            sd[0] += w.x * b[v].x;
            sd[0] += w.y * b[v].y;
            sd[1] += w.x * b[v].y;
            sd[1] -= w.y * b[v].x;
          }
        }
        store(carry, b, false);
      }
    }
    if constexpr (MOM != kMomNone) {
      if (dots) accq += static_cast<double>(wave_sums<NQ, 32>(sq, lane));
    }
  };
  if constexpr (LAT == kLatRow) {
    run_chain();
  } else {
    if (whole) run(std::true_type{});
    else run(std::false_type{});
  }

  if constexpr (SEQ) {
    if (dot_carry) {                                 // one record per item
      T x[2] = {sd[0], sd[1]};
      const double v = static_cast<double>(wave_sums<2, 32>(x, lane));
      if (lane == sum_lane<2>(0) || lane == sum_lane<2>(1))
        st.partial[((int64_t)st.mom_slot * st.total_items + item) * 2 +
                   (lane == sum_lane<2>(0) ? 0 : 1)] = v;
    }
  }

  if constexpr (MOM != kMomNone) {
    if (dots) {
      // one record of 8 doubles per level, [kind][re, im] with kinds
      // <psi0|out>, <psi0|cur> (first level only), <out|out>, <out|cur>
      // (kMomSelf: the real parts of the last two, zeros elsewhere);
      // lane m writes element m % 8 of level m / 8
      const int m = lane;
      const int l = m >> 3, slot = m & 7;
      int q = -1;
      if constexpr (MOM == kMomSelf) {
        if (slot == 4) q = 2 * l;
        else if (slot == 6) q = 2 * l + 1;
      } else {
        if (slot == 0 || slot == 1) q = 5 * l + slot;
        else if (slot == 4) q = 5 * l + 2;
        else if (slot == 6 || slot == 7) q = 5 * l + slot - 3;
        else if ((slot == 2 || slot == 3) && l == 0) q = 5 * KT + slot - 2;
      }
      const double val = __shfl(accq, q < 0 || q >= NQ ? 0 : sum_lane<NQ>(q));
      if (l < nlev && l < KT) {
        double* out = st.partial + (((int64_t)st.mom_slot * KT + l) * st.total_items + item) * 8;
        out[slot] = q < 0 ? 0.0 : val;
      }
    }
  }
}

}  // namespace cheb
}  // namespace csp

// Launch helper for one instantiation file: (V, KT) pairs are listed by the
// including file.
#define CSP_CHEB_LAUNCH_LAT(T, V, KT, LAT, MOM, CARRY)                                         \
  do {                                                                                         \
    if (diag) hipLaunchKernelGGL((cheb::k_cheb<T, V, KT, LAT, true, MOM, CARRY>), grid, block, \
                                 0, s, d_inst, n_inst, item_lo, item_hi, st);                  \
    else hipLaunchKernelGGL((cheb::k_cheb<T, V, KT, LAT, false, MOM, CARRY>), grid, block, 0,  \
                            s, d_inst, n_inst, item_lo, item_hi, st);                          \
  } while (0)
#define CSP_CHEB_LAUNCH(T, V, KT, MOM, CARRY)                                                  \
  do {                                                                                         \
    if (lat == kLatHoney) CSP_CHEB_LAUNCH_LAT(T, V, KT, kLatHoney, MOM, CARRY);                \
    else if (lat == kLatRow) CSP_CHEB_LAUNCH_LAT(T, V, KT, kLatRow, MOM, CARRY);               \
    else CSP_CHEB_LAUNCH_LAT(T, V, KT, kLatSquare, MOM, CARRY);                                \
  } while (0)
