// Chebyshev recursion launches: the kernel itself (k_cheb_body.h) is
// instantiated per precision and epilogue in k_cheb_f32*.hip and
// k_cheb_f64*.hip; this file picks the instantiation for each run of
// instances with the same lattice class, and sums the moment records.
#include "csp_internal.h"

namespace csp {

#define CSP_CHEB_LAUNCHER(name)                                                                 \
  hipError_t name(int vec, int kt, int lat, bool diag, const ChebInst* d_inst, int n_inst,   \
                  int64_t item_lo, int64_t item_hi, const ChebStep& st, hipStream_t s);
CSP_CHEB_LAUNCHER(launch_cheb_f32)
CSP_CHEB_LAUNCHER(launch_cheb_f32m)
CSP_CHEB_LAUNCHER(launch_cheb_f64)
CSP_CHEB_LAUNCHER(launch_cheb_f64m)
CSP_CHEB_LAUNCHER(launch_cheb_f32mc)
CSP_CHEB_LAUNCHER(launch_cheb_f64mc)
CSP_CHEB_LAUNCHER(launch_cheb_f32s)
CSP_CHEB_LAUNCHER(launch_cheb_f64s)
CSP_CHEB_LAUNCHER(launch_cheb_f64q)
#undef CSP_CHEB_LAUNCHER

bool cheb_shape_supported(bool fp64, int vec, int kt, bool mom) {
  // (complex128 moments at 8 steps: the self products of one block only)
  if (fp64) return vec == 2 && (kt == 1 || kt == 2 || kt == 4 || kt == 8);
  if (vec != 2 && vec != 4) return false;
  return kt == 1 || kt == 2 || kt == 4 || (kt == 8 && (!mom || vec == 2));
}

bool cheb_carry_supported(bool fp64, int vec, int kt) {
  return vec == 2 && (kt == 1 || kt == 2 || kt == 4 || (kt == 8 && !fp64));
}

int cheb_margin(int vec, int kt) { return (kt + vec - 1) / vec * vec; }

hipError_t launch_cheb(bool fp64, int vec, int kt, bool mom, bool carry, const ChebInst* d_inst,
                       const std::vector<ChebRun>& runs, const ChebStep& st, hipStream_t s) {
  if (st.nlev < 1 || st.nlev > kt) return hipErrorInvalidValue;
  // the carried state without moments: the sequential form's kernel
  const bool seq = carry && !mom;
  if (seq ? !fp64 || vec != 2 || kt != kSeqSteps : !cheb_shape_supported(fp64, vec, kt, mom))
    return hipErrorInvalidValue;
  if (carry && mom && !cheb_carry_supported(fp64, vec, kt)) return hipErrorInvalidValue;
  // only the self products (one block, bra = ket): the kernel without psi0
  const bool self = mom && !carry && !st.dot_psi0 && st.dot_self;
  if (st.ow != 64 * vec - 2 * cheb_margin(vec, kt)) return hipErrorInvalidValue;
  for (const ChebRun& r : runs) {
    const ChebInst* di = d_inst + r.inst0;
    const int64_t lo = r.item0, hi = r.item0 + r.n_items;
    hipError_t e;
    if (seq)
      e = r.sparse ? hipErrorInvalidValue
                   : launch_cheb_f64q(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s);
    else if (r.sparse && r.win)
      e = launch_cheb_ellw(fp64, mom, carry, r.ct, r.win, r.win_cap, di, r.n_inst, r.wave0,
                           r.wave0 + r.n_waves, st, s);
    else if (r.sparse)
      e = launch_cheb_ell(fp64, mom, carry, r.ct, di, r.n_inst, r.wave0, r.wave0 + r.n_waves, st,
                          s);
    else if (fp64)
      e = carry  ? launch_cheb_f64mc(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s)
          : self ? launch_cheb_f64s(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s)
          : mom  ? launch_cheb_f64m(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s)
                 : launch_cheb_f64(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s);
    else
      e = carry  ? launch_cheb_f32mc(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s)
          : self ? launch_cheb_f32s(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s)
          : mom  ? launch_cheb_f32m(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s)
                 : launch_cheb_f32(vec, kt, r.lat, r.diag, di, r.n_inst, lo, hi, st, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ------------------------------------------------------------------ sequential form
// <psi0|psi(t_{j0+1+slot})> of every column from the records of its work
// items ([slot][item] complex): thread t adds every 256th record, the 256
// partial sums in a fixed tree.
__global__ __launch_bounds__(256) void k_seq_corr(const SeqInst* __restrict__ si,
                                                  const double* __restrict__ partial,
                                                  int64_t total_items, int64_t j0) {
  __shared__ double2 red[256];
  const SeqInst& I = si[blockIdx.z];
  const int c = blockIdx.y, slot = blockIdx.x, t = threadIdx.x;
  if (c >= I.Rg) return;
  const double2* p = reinterpret_cast<const double2*>(partial) + (int64_t)slot * total_items +
                     I.item0 + c * I.items_per_col;
  double sx = 0.0, sy = 0.0;
  for (int64_t k = t; k < I.items_per_col; k += 256) {
    const double2 v = p[k];
    sx += v.x;
    sy += v.y;
  }
  red[t] = make_double2(sx, sy);
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) {
      red[t].x += red[t + w].x;
      red[t].y += red[t + w].y;
    }
    __syncthreads();
  }
  if (t == 0)
    reinterpret_cast<double2*>(I.corr)[(j0 + 1 + slot) * I.ldc + I.col0 + c] = red[0];
}

hipError_t launch_seq_corr(const SeqInst* d_si, int n_inst, int rg_max, int n_slots,
                           const double* partial, int64_t total_items, int64_t j0, hipStream_t s) {
  if (n_slots <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_seq_corr, dim3(n_slots, rg_max, n_inst), dim3(256), 0, s, d_si, partial,
                     total_items, j0);
  return hipGetLastError();
}

// ------------------------------------------------------------------ moment sums
// One workgroup per (launch slot, level), column and instance: thread t sums
// value t % 8 ([kind][re, im]) of every 32nd of the column's records in four
// interleaved partial sums (whole 64-byte records of neighbouring items read
// together); the 32 lanes of a value are then added in order.  (One
// workgroup for all columns took 32 us at 2048 records x 5 columns.)
__global__ __launch_bounds__(256) void k_cheb_mom_finish(const MomInst* __restrict__ mi,
                                                         const double* __restrict__ partial,
                                                         int64_t total_items, int n0,
                                                         int max_row) {
  __shared__ double red[256];
  const int sl = blockIdx.x;                     // slot * kt + level
  const int row = n0 + sl;                       // order produced by that level
  const MomInst& M = mi[blockIdx.z];
  const int c = blockIdx.y;
  if (c >= M.Rg || row > max_row) return;
  const int t = threadIdx.x, vi = t & 7, lanei = t >> 3;
  const int64_t ipc = M.n_tiles / M.Rg;          // work items per column
  const double* base = partial + ((int64_t)sl * total_items + M.tile0 + c * ipc) * 8 + vi;
  double q[4] = {0, 0, 0, 0};
  int64_t k = lanei;
  for (; k + 3 * 32 < ipc; k += 4 * 32) {
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] += base[(k + u * 32) * 8];
  }
  for (int u = 0; k < ipc; k += 32, ++u) q[u] += base[k * 8];
  red[t] = (q[0] + q[1]) + (q[2] + q[3]);
  __syncthreads();
  if (t < 8) {
    double sum = 0.0;
    for (int l = 0; l < 32; ++l) sum += red[l * 8 + t];
    // dots row `row`, layout [kind][Rg][re, im]
    M.dots[(int64_t)row * 8 * M.Rg + ((t >> 1) * M.Rg + c) * 2 + (t & 1)] = sum;
  }
}

hipError_t launch_cheb_mom_finish(const MomInst* d_mi, int n_inst, int rg_max,
                                  const double* partial, int64_t total_items, int kt, int n_slots,
                                  int n0, int max_row, hipStream_t s) {
  if (n_slots <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_cheb_mom_finish, dim3(n_slots * kt, rg_max, n_inst), dim3(256), 0, s, d_mi,
                     partial, total_items, n0, max_row);
  return hipGetLastError();
}

}  // namespace csp
