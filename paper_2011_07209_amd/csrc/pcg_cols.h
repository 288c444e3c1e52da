// Parts of the preconditioned CG (pcg_impl.h) in code that the host can also run:
// a column of the sphere as a sweep step uses it, and the update of the solution.
#pragma once

#include "exx_internal.h"

namespace exx {

template <bool GEN>
struct PCol {
  int hi, lo;   // its planes: -hi .. hi (no column: hi < 0), in a general cell lo .. hi
  int col;      // slot within a plane
  int low;      // LDS plane position, less the NS rows that the stencil reaches up

  // A thread without a column.  In a general cell its planes lie beyond those
  // of any sphere (in 16 bits, as PCols keeps them), so that no plane is near
  // one: with the interval (1, -1) the planes |z| < d were, and an arm along a
  // body diagonal read LDS in front of the plane from its position 0.
  static constexpr int kNoHi = GEN ? -0x4000 : -1, kNoLo = GEN ? 0x3fff : 1;
  static __host__ __device__ constexpr PCol none() { return {kNoHi, kNoLo, 0, 0}; }

  // whether sweep plane z holds a point of it (in an orthorhombic cell one
  // comparison with a scalar)
  __host__ __device__ constexpr bool valid(int z) const {
    if constexpr (GEN)
      return z >= lo && z <= hi;
    else
      return (z < 0 ? -z : z) <= hi;
  }
  __host__ __device__ constexpr bool has() const { return GEN ? lo <= hi : hi >= 0; }
  // whether a plane from z - d to z + d holds one (general cells)
  __host__ __device__ constexpr bool near(int z, int d) const {
    static_assert(GEN, "only arms leaving the sweep plane look at neighbouring planes");
    return z + d >= lo && z - d <= hi;
  }
};

// y + the steps w_i v_i, in the precision X of the solution they are added to: a
// reliable update of the mixed solve folds its FP32 vectors into the FP64
// solution without rounding their sum to FP32 first.
template <typename X, typename T>
__host__ __device__ constexpr X pcg_add_steps(T y, const X (&w)[kPcgRing], const T (&v)[kPcgRing]) {
  X s = (X)y;
#pragma unroll
  for (int i = 0; i < kPcgRing; ++i) s += w[i] * (X)v[i];
  return s;
}

}  // namespace exx
