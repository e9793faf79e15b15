// The product-rule kernel with the low-order halves of bf16 pairs (see gemm_linear.h): five or six operand tiles a slab, so
// the wide tiles take 32-deep slabs and the 256-wide one does not fit.
#include "gemm_linear.h"

namespace hf {

template <bool TB>
static hipError_t launch_lo(int cfg, int nt, const LinP& p, int nb, int ks, hipStream_t st) {
  if (nt == 5) {
    switch (cfg) {
      case LIN_64x64: return launch_linear_one<64, 64, 32, 32, 16, 64, 4, 4, 2, false, TB, 5>(p, nb, ks, st);
      case LIN_64x128: return launch_linear_one<64, 128, 32, 32, 16, 64, 4, 2, 2, false, TB, 5>(p, nb, ks, st);
      case LIN_128x128: return launch_linear_one<128, 128, 64, 32, 16, 64, 2, 2, 2, false, TB, 5>(p, nb, ks, st);
      case LIN_128x192: return launch_linear_one<128, 192, 32, 96, 32, 32, 3, 3, 1, false, TB, 5>(p, nb, ks, st);
      default: return hipErrorNotSupported;
    }
  }
  switch (cfg) {
    case LIN_64x64: return launch_linear_one<64, 64, 32, 32, 16, 64, 3, 3, 2, false, TB, 6>(p, nb, ks, st);
    case LIN_64x128: return launch_linear_one<64, 128, 32, 32, 16, 64, 2, 2, 2, false, TB, 6>(p, nb, ks, st);
    default: return hipErrorNotSupported;
  }
}

hipError_t launch_linear_lo(int cfg, int nt, int transB, const LinP& p, int nb, int ks, hipStream_t st) {
  return transB ? launch_lo<true>(cfg, nt, p, nb, ks, st) : launch_lo<false>(cfg, nt, p, nb, ks, st);
}

}  // namespace hf
