// Instantiations of the Chebyshev recursion kernel: complex128, recursion with the carried state
// (sequential form).  Seven steps per launch: the 20 orders of a time step of pi take three
// launches and 16 vectors (four launches of five steps: 21).  326-378 registers, one wave per
// SIMD; graphene 1024^2 x 4 columns, one time step: 4 x 199 us with five steps, 3 x 171 us with
// seven; ten steps need 440-498 registers for two launches of more margin work.
#include "k_cheb_body.h"

namespace csp {

hipError_t launch_cheb_f64q(int vec, int kt, int lat, bool diag, const ChebInst* d_inst, int n_inst,
                            int64_t item_lo, int64_t item_hi, const ChebStep& st, hipStream_t s) {
  const int64_t n = item_hi - item_lo;
  if (n <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(ceil_div(n, 4))), block(256);
  if (vec != 2 || kt != kSeqSteps) return hipErrorInvalidValue;
  CSP_CHEB_LAUNCH(double, 2, kSeqSteps, cheb::kMomNone, true);
  return hipGetLastError();
}

}  // namespace csp
