// Instances of the preconditioned CG for stencil half-width n = 3, mixed precision.
#include "pcg_impl.h"

namespace exx {

hipError_t pcg_n3_mixed(const SolveKArgs& a, int cols, int threads, int groups, size_t lds, hipStream_t s, int* occ) {
  return pcg_dispatch<3, true>(a, cols, threads, groups, lds, s, occ);
}

}  // namespace exx
