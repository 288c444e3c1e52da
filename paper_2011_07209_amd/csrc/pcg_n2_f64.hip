// Instances of the preconditioned CG for stencil half-width n = 2, FP64.
#include "pcg_impl.h"

namespace exx {

hipError_t pcg_n2_f64(const SolveKArgs& a, int cols, int threads, int groups, size_t lds, hipStream_t s, int* occ) {
  return pcg_dispatch<2, false>(a, cols, threads, groups, lds, s, occ);
}

}  // namespace exx
