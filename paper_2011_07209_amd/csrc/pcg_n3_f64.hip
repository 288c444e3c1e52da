// Instances of the preconditioned CG for stencil half-width n = 3, FP64.
#include "pcg_impl.h"

namespace exx {

hipError_t pcg_n3_f64(const SolveKArgs& a, int cols, int threads, int groups, size_t lds, hipStream_t s, int* occ) {
  return pcg_dispatch<3, false>(a, cols, threads, groups, lds, s, occ);
}

}  // namespace exx
