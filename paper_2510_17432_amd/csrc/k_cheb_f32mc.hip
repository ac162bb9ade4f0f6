// Instantiations of the Chebyshev recursion kernel: complex64, moment epilogue and carried state.
#include "k_cheb_body.h"

namespace csp {

hipError_t launch_cheb_f32mc(int vec, int kt, int lat, bool diag, const ChebInst* d_inst, int n_inst,
                             int64_t item_lo, int64_t item_hi, const ChebStep& st, hipStream_t s) {
  const int64_t n = item_hi - item_lo;
  if (n <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(ceil_div(n, 4))), block(256);
  switch (vec * 100 + kt) {
    case 201: CSP_CHEB_LAUNCH(float, 2, 1, cheb::kMomBra, true); break;
    case 202: CSP_CHEB_LAUNCH(float, 2, 2, cheb::kMomBra, true); break;
    case 204: CSP_CHEB_LAUNCH(float, 2, 4, cheb::kMomBra, true); break;
    case 208: CSP_CHEB_LAUNCH(float, 2, 8, cheb::kMomBra, true); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace csp
