// Preconditioned CG of the pair Poisson problems: the CG of solve_impl.h with
// an additive multilevel preconditioner (Bramble, Pasciak and Xu 1990) on the
// nested grids of every second, fourth, eighth and sixteenth point,
//
//   z = sum_l w_l P_l P_l^T r,   w_l = 1 / (diagonal of the level-l operator),
//
// with P_l trilinear interpolation (zero off the sphere).  The preconditioner
// holds no operator beyond its diagonals, so it serves every stencil width and
// cell, and it is symmetric positive definite by construction.  On the
// spheres of the water sets it takes CG from 250 iterations to 34: a pair's
// cost is those iterations' sweeps over HBM, so that count is the time.
//
// An iteration is the coarse phase and one z-marching sweep, which takes the
// end of iteration k and the start of k + 1 together:
//   r_k+1 = r_k - alpha q_k,
//   p_k+1 = w_0 r_k+1 + P_1 e_k+1 + beta p_k   (e: the coarse correction on level 1),
//   q_k+1 = A p_k+1 n planes behind, with p.q, |q|^2 and |r|^2,
//   P^T q_k+1 on levels 1 and 2, streamed with the sweep.
// The coarse residuals follow P^T r_k+1 = P^T r_k - alpha P^T q_k, so the coarse
// phase needs no sweep of its own before it, and beta is known before the sweep
// from products of the one before (PDir); the stop test and alpha take the
// sweep's own |r|^2.
// x is left alone for four iterations: their directions stay in four buffers in
// turn, and one stream adds the four steps (PRing).  Per point and iteration
// that is seven and a half accesses, one stencil and one barrier a plane.
// Updating x in every second sweep costs the same accesses but two more values
// per column in flight, which the sweep's registers don't hold (FP64, 1024
// threads, 3 columns each: an iteration on all CUs 800 us against 500 us).  The same
// iteration as two sweeps (direction and product; update and restriction) makes
// seven and a half accesses too but two stencils.
//
// Restriction: a column's planes of q are combined in registers (weights 1/2 1
// 1/2), every second plane the combination is staged in LDS and the level-1
// columns take their 9 in-plane neighbours; level 2 is formed from level 1 the
// same way.  Interpolation mirrors it: one level-1 plane per two sweep steps is
// staged, a column takes its (up to four) in-plane neighbours once per level-1
// plane, and odd planes average two of them.  The coarse phase holds levels 2 to
// 4 (a few thousand points) as dense boxes in LDS.
#pragma once

#include <type_traits>

#include "pcg_cols.h"
#include "solve_impl.h"

namespace exx {

// The scalars of a class's nested grids that the sweeps use, in scalar
// registers (every lane's value is the same: the class of the workgroup's pair).
struct MgU {
  int Z1, rw, rh, ew, eh;
  int d2x, d2xy, e2z;   // level-2 box: row, plane, and half-width along the sweep
};
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ MgU mg_uniform(const MgDev& M) {
  MgU u;
  u.Z1 = uniform(M.Z1);
  u.rw = uniform(M.rw);
  u.rh = uniform(M.rh);
  u.ew = uniform(M.ew);
  u.eh = uniform(M.eh);
  u.d2x = uniform(M.D2[0]);
  u.d2xy = uniform(M.D2[0] * M.D2[1]);
  u.e2z = uniform(M.E2[2]);
  return u;
}

// The slot's working vectors as one buffer resource: a lane whose offset lies
// past its end (kOob) reads zero and writes nothing (the scalar offset added to
// it always lies within).  The sweeps mask their
// lanes so instead of branching around the access: behind a branch the number
// of accesses in flight is unknown and the compiler waits for all of them,
// stores of the plane before included (mixed, 2,957 columns, one pair per CU:
// a solve 9.3 ms against 7.7 ms with 1024 threads).
struct PBuf {
  __amdgpu_buffer_rsrc_t r;
};
__device__ __forceinline__ PBuf pbuf(void* base, int bytes) {
  return {__builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000)};
}
template <typename T>
__device__ __forceinline__ T bload(const PBuf& b, unsigned voff, unsigned soff) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b.r, voff, soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b.r, voff, soff, 0));
}
template <typename T>
__device__ __forceinline__ void bstore(const PBuf& b, unsigned voff, unsigned soff, T v) {
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b.r, voff, soff, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), b.r, voff, soff, 0);
}
constexpr unsigned kOob = 0x80000000u;

// The general stencil, read anew from the kernel's arguments (one struct, at
// the start of their segment): the 60 scalar registers that its FP64 constants
// take are not there for a whole sweep, and kept ones were moved to lanes of
// vector registers and back (321 moves per two steps of the FP64 sweep).
template <typename T>
__device__ __forceinline__ GenStencilT<T> gen_args(const SolveKArgs&) {
  typedef const __attribute__((address_space(4))) SolveKArgs KArgs;
  KArgs* k = (KArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(k));
  GenStencilT<T> g;
  auto copy = [&](const auto& from) __attribute__((always_inline)) {
    g.diag = from.diag;
    g.cz = from.cz;
    g.n_in = from.n_in;
    g.n_tl = from.n_tl;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      g.w[q] = from.w[q];
      g.czw[q] = from.czw[q];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      g.in_off[i] = from.in_off[i];
      g.in_coef[i] = from.in_coef[i];
      g.tl_off[i] = from.tl_off[i];
      g.tl_coef[i] = from.tl_coef[i];
#pragma unroll
      for (int q = 0; q < 4; ++q) g.tl_cw[i][q] = from.tl_cw[i][q];
    }
  };
  if constexpr (sizeof(T) == 4)
    copy(k->G32);
  else
    copy(k->G);
  return g;
}

// A sweep's vectors, as byte offsets into the slot's buffer.  none: kOob before
// the first direction, when p and q are to read zero, else 0.
struct PVec {
  PBuf all;
  unsigned none, r, q, p, pn, e1, g1, g2;
};

// A value the compiler may not carry across loop steps: what is computed from
// it (LDS addresses, a few integer instructions) is formed again where it is
// used.  Kept over a sweep, those addresses cost more registers than the
// sweep has, and the plane loops spilled to scratch memory (FP64, 2,957
// columns, 2,356 pairs: 218 ms against 166 ms, with PBase's scalar bases).
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Columns of the sphere owned by a thread, t, t + NT, ... of the class's real
// columns.  Only what the sweeps cannot recompute in a few instructions is
// kept: the sweeps' windows need the registers.  PK (FP64, whose windows take
// twice the registers): a column's plane slot, height and position in one
// register, taken apart in each step.
constexpr int kPkCol = 12, kPkLow = 13;   // bits; the rest: the height + 1
template <int CPT, bool GEN, bool PK>
struct PCols {
  int a[CPT];                          // PK: packed; else the plane slot
  int h[PK && !GEN ? 1 : CPT];         // hi, in a general cell hi & 0xffff | lo << 16
  int p[PK ? 1 : CPT];                 // low
  unsigned re[CPT];   // position in the restriction's plane | in the level-1 plane << 16 | parities << 30
  __device__ __forceinline__ void put(int c, int hi, int lo, int col, int low) {
    if constexpr (PK)
      a[c] = (int)((unsigned)col | (unsigned)low << kPkCol | (GEN ? 0u : (unsigned)(hi + 1) << (kPkCol + kPkLow)));
    else
      a[c] = col;
    if constexpr (GEN)
      h[c] = (hi & 0xffff) | (int)((unsigned)lo << 16);
    else if constexpr (!PK)
      h[c] = hi;
    if constexpr (!PK) p[c] = low;
  }
  __device__ __forceinline__ PCol<GEN> get(int c) const {
    PCol<GEN> k;
    const int v = PK ? fresh(a[c]) : a[c];
    k.col = PK ? v & ((1 << kPkCol) - 1) : v;
    k.low = PK ? (v >> kPkCol) & ((1 << kPkLow) - 1) : fresh(p[PK ? 0 : c]);
    if constexpr (GEN) {
      const int w = fresh(h[c]);
      k.hi = (int)(short)(w & 0xffff);
      k.lo = w >> 16;
    } else {
      k.hi = PK ? (int)((unsigned)v >> (kPkCol + kPkLow)) - 1 : h[PK ? 0 : c];
      k.lo = 0;
    }
    return k;
  }
  __device__ __forceinline__ bool valid(int c, int z) const { return get(c).valid(z); }
  __device__ __forceinline__ bool has(int c) const { return get(c).has(); }
};

// Byte offset of the column's point in a plane, or kOob.
template <typename T, bool GEN>
__device__ __forceinline__ unsigned pcg_off(const PCol<GEN>& k, bool in) {
  return in ? (unsigned)k.col * (unsigned)sizeof(T) : kOob;
}

// (No column: positions that stay zero, where the sweeps may write zeros.)
template <int NS, int CPT, int NT, bool GEN, bool PK>
__device__ __forceinline__ void pcg_cols(const ClassDev& C, int cx, int cy, PCols<CPT, GEN, PK>& cl) {
  const MgDev& M = C.mg;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int k = threadIdx.x + c * NT;
    constexpr PCol<GEN> none = PCol<GEN>::none();
    cl.put(c, none.hi, none.lo, none.col, none.low);
    cl.re[c] = 0;
    if (k < C.n_fin) {
      const int4 f = C.fin_cols[k];
      const int x = GEN ? (int)(short)(f.w & 0xffff) : f.z;
      const int y = GEN ? (f.w >> 16) : f.w;
      cl.put(c, GEN ? f.z : f.y, GEN ? f.y : 0, f.x, (x + cx) + kLdsWX * (y + cy - NS));
      const int r1 = (x + M.rcx) + M.rw * (y + M.rcy);
      const int e = ((x >> 1) + M.ex + 1) + M.ew * ((y >> 1) + M.ey + 1);
      cl.re[c] = (unsigned)r1 | (unsigned)e << 16 | (unsigned)(x & 1) << 30 | (unsigned)(y & 1) << 31;
    }
  }
}

#define EXX_PVALID(c, zz) cl.valid(c, zz)
#define EXX_PHAS(c) cl.has(c)
#define EXX_PIDX(c, base) ((base) + (unsigned)cl.get(c).col)
// LDS plane position (from the stencil's first row on: its offsets are all
// positive and go into the instructions), and the one in the restriction's plane
#define EXX_PPOS(c) (cl.get(c).low + NS * kLdsWX)
#define EXX_PR1(c) (fresh((int)cl.re[c]) & 0xffff)

// First slots of the N planes z, z + 1, ... of a sweep step, in scalar
// registers.  Each step takes one new one from LDS and shifts: read where they
// are used, a step's loads waited for one LDS read each, one after the other.
template <int N>
struct PBase {
  unsigned b[N];
  static __device__ __forceinline__ unsigned at(const int* pst, int Zmax, int z) {
    return (unsigned)uniform(pst[min(max(z + Zmax, 0), 2 * Zmax + 1)]);
  }
  __device__ __forceinline__ PBase(const int* pst, int Zmax, int z) {
#pragma unroll
    for (int k = 0; k < N; ++k) b[k] = at(pst, Zmax, z + k);
  }
  // to the planes of step z + 1
  __device__ __forceinline__ void next(const int* pst, int Zmax, int z) {
#pragma unroll
    for (int k = 0; k + 1 < N; ++k) b[k] = b[k + 1];
    b[N - 1] = at(pst, Zmax, z + N);
  }
};

// A thread's level-1 columns (CC of them) and its level-2 column, two 16-bit
// values to a register.
template <int CC>
struct PCoarse {
  int iv[CC];     // planes: lo | hi << 16
  int ps[CC];     // position of the column's centre in the staged plane of the sphere | in the staged level-1 plane << 16
  int iv2, ps2;   // level-2 column: planes; centre in the staged level-1 plane | place in a plane of the level-2 box << 16
};
__device__ __forceinline__ int pack16(int a, int b) { return (a & 0xffff) | (int)((unsigned)b << 16); }
// the halves, formed again at each use; lower signed
struct PHalves {
  int a, b;
  __device__ __forceinline__ explicit PHalves(int v) {
    const int w = fresh(v);
    a = (int)(short)(w & 0xffff);
    b = w >> 16;
  }
};

template <int CC, int NT>
__device__ __forceinline__ void pcg_coarse_cols(const ClassDev& C, PCoarse<CC>& k) {
  const MgDev& M = C.mg;
  const int t = threadIdx.x;
#pragma unroll
  for (int u = 0; u < CC; ++u) {
    k.iv[u] = pack16(1, 0);
    k.ps[u] = M.rw + 1;
    const int i = t + u * NT;
    if (i < M.n_c1) {
      const int4 f = M.c1cols[i];
      k.iv[u] = pack16(f.z, f.w);
      k.ps[u] = pack16((2 * f.x + M.rcx) + M.rw * (2 * f.y + M.rcy), (f.x + M.ex + 1) + M.ew * (f.y + M.ey + 1));
    }
  }
  k.iv2 = pack16(1, 0);
  k.ps2 = M.ew + 1;
  if (t < M.n_c2) {
    const int4 f = M.c2cols[t];
    k.iv2 = pack16(f.z, f.w);
    k.ps2 = pack16((2 * f.x + M.ex + 1) + M.ew * (2 * f.y + M.ey + 1),
                   (f.x + M.E2[0] + 1) + M.D2[0] * (f.y + M.E2[1] + 1));
  }
}

// The in-plane part of the restriction: weights 1/4 1/2 1/4, 1/2 1 1/2, 1/4 1/2 1/4
template <typename T>
__device__ __forceinline__ T restrict9(const T* b, int w) {
  const T corner = (b[-w - 1] + b[-w + 1]) + (b[w - 1] + b[w + 1]);
  const T edge = (b[-w] + b[w]) + (b[-1] + b[1]);
  return b[0] + (T)0.5 * edge + (T)0.25 * corner;
}

// The in-plane part of the interpolation at a fine column (x, y): the average
// of the level-1 values at (x >> 1, x + 1 >> 1) x (y >> 1, y + 1 >> 1).
template <typename T>
__device__ __forceinline__ T prolong4(const T* E, unsigned re, const MgU& M) {
  re = (unsigned)fresh((int)re);
  const T* b = E + ((re >> 16) & 0x3fff);
  const int dx = (re >> 30) & 1, dy = (re >> 31) ? M.ew : 0;
  return (T)0.25 * ((b[0] + b[dx]) + (b[dy] + b[dx + dy]));
}

// -(Laplacian) of the window form: axis stencil, or the in-plane arms of a
// general cell.
template <int NS, bool GEN, typename T>
__device__ __forceinline__ T pcg_apply(const StencilT<T>& S, const GenStencilT<T>& G, T ctr, const T* pl, int pos,
                                       const T* wz) {
  if constexpr (GEN)
    return -gen_inplane<NS, T>(G, ctr, pl, pos, wz);
  else
    return apply_point<NS, T>(S, ctr, pl, pos, wz);
}

// Shared buffers of the sweeps: the planes of the sphere (two in turn, or one
// where two do not fit: plane 0, and a second barrier a step), one for the
// restriction from the sphere (R1), one level-1 plane for the restriction from
// level 1 (R2) and one for the interpolation (E).
template <typename T>
struct PLds {
  T* pl0;
  int plane;   // distance of the second plane
  int old;     // distance of the direction before's planes (pcg_sweep_rq)
  T *R1, *R2, *E;
};

// The restriction streamed with a sweep: level-2 sums of the level-1 columns.
template <int CC, typename T>
struct PRestrict {
  T acc2[CC];
};

// Level-1 part of an even sweep step (after its barrier), level-2 part of an
// odd one.  z is the step's centre plane; the combination staged at the odd
// plane z - 1 completes level-1 plane (z - 2) / 2.  c1 and b2: byte offsets of
// the results in buffer B.
template <int CC, int NT, typename T>
__device__ __forceinline__ void pcg_restrict_even(const MgU& M, const PCoarse<CC>& k, const PLds<T>& L,
                                                  const int* cst, int z, PRestrict<CC, T>& R, const PBuf& B,
                                                  unsigned c1) {
  const int kz = (z - 2) >> 1;
  const bool fin = kz & 1;   // completes a level-2 plane
  const unsigned base = PBase<1>::at(cst, M.Z1, kz) * sizeof(T);
#pragma unroll
  for (int u = 0; u < CC; ++u) {
    const PHalves iv(k.iv[u]), ps(k.ps[u]);
    const bool in = kz >= iv.a && kz <= iv.b;
    T v = 0;
    if (in) v = restrict9<T>(L.R1 + ps.a, M.rw);
    bstore<T>(B, in ? (threadIdx.x + u * NT) * (unsigned)sizeof(T) : kOob, c1 + base, v);
    if (fin) {
      if (iv.a <= iv.b) L.R2[ps.b] = R.acc2[u] + (T)0.5 * v;
      R.acc2[u] = (T)0.5 * v;
    } else {
      R.acc2[u] += v;
    }
  }
}
template <int CC, typename T>
__device__ __forceinline__ void pcg_restrict_odd(const MgU& M, const PCoarse<CC>& k, const PLds<T>& L, int z,
                                                 const PBuf& B, unsigned b2) {
  const int kz = (z - 3) >> 1;   // level-1 plane of the previous step
  const int k2 = (kz - 1) >> 1;
  const PHalves iv(k.iv2), ps(k.ps2);
  const bool in = (kz & 1) && k2 >= iv.a && k2 <= iv.b;
  const unsigned plane = (unsigned)uniform(M.d2xy * min(max(k2 + M.e2z + 1, 0), 2 * M.e2z + 2));
  T v = 0;
  if (in) v = restrict9<T>(L.R2 + ps.a, M.ew);
  bstore<T>(B, in ? (unsigned)ps.b * (unsigned)sizeof(T) : kOob, b2 + plane * (unsigned)sizeof(T), v);
}
template <int CC, int NT, typename T>
__device__ __forceinline__ void pcg_restrict_step(const MgU& M, const PCoarse<CC>& k, const PLds<T>& L,
                                                  const int* cst, int z, PRestrict<CC, T>& R, const PBuf& B,
                                                  unsigned c1, unsigned b2) {
  if (z & 1)
    pcg_restrict_odd<CC, T>(M, k, L, z, B, b2);
  else
    pcg_restrict_even<CC, NT, T>(M, k, L, cst, z, R, B, c1);
}

// Last sweep step that the streamed restriction needs.
__device__ __forceinline__ int pcg_last_step(const MgU& M, int Zmax) {
  // level-1 plane Z1 (or Z1 + 1, when Z1 is even, to complete level 2) is
  // formed at step 2 kz + 2, its level-2 plane at the step after
  const int kz = (M.Z1 & 1) ? M.Z1 : M.Z1 + 1;
  return max(Zmax, 2 * kz + 3);
}

// The products a sweep returns, each this thread's part.
struct PSums {
  double rr, pq, qq;
};

// The sweep, window form (orthorhombic cells; general cells without arms
// leaving the sweep plane): plane zc enters, plane z = zc - NS is its windows'
// centre.  r, p and q of the next plane are loaded between the use of this
// plane's and the barrier, so one register set holds them.  Steps go in pairs
// (an even plane, an odd one), so that what a plane's parity decides is decided
// at compile time.  Before the first direction alpha, beta, p and q are zero.
template <int NS, int CPT, int NT, bool GEN, int CC, typename T, bool PK>
__device__ __forceinline__ PSums pcg_sweep_w(const StencilT<T>& S, const GenStencilT<T>& G, const MgU& M,
                                             const PCols<CPT, GEN, PK>& cl, const PCoarse<CC>& ck, const int* pst,
                                             const int* cst, int Zmax, const PVec& V, T w0, T alpha, T beta,
                                             const PLds<T>& L) {
  T win[CPT][2 * NS + 1];
  T lr[CPT], lp[CPT], lq[CPT], Bc[CPT], acc[CPT], ev[CC];
  // FP64 in a general cell: branches, as in the sweep with arms leaving the plane
  // (hexagonal, 11,220 pairs: 1,293 ms against 1,936 ms masked)
  constexpr bool BR = GEN && sizeof(T) == 8;
  PRestrict<CC, T> R;
  PSums s{0.0, 0.0, 0.0};
  // an even plane below the first one: its step stages the level-1 plane that
  // the next (odd) step interpolates
  const int z0 = -Zmax - 2 + (Zmax & 1);
  const int zl = pcg_last_step(M, Zmax) + NS;
  PBase<NS + 2> pb(pst, Zmax, z0 - NS);   // planes zc - NS .. zc + 1
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    lr[c] = lp[c] = lq[c] = Bc[c] = acc[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) win[c][k] = 0;
  }
  auto load_e = [&](int kz) {   // a level-1 plane of the correction
    const unsigned base = V.e1 + PBase<1>::at(cst, M.Z1, kz) * (unsigned)sizeof(T);
#pragma unroll
    for (int u = 0; u < CC; ++u) {
      const PHalves iv(ck.iv[u]);
      ev[u] = bload<T>(V.all, kz >= iv.a && kz <= iv.b ? (threadIdx.x + u * NT) * (unsigned)sizeof(T) : kOob, base);
    }
  };
  load_e((z0 + 2) >> 1);
  auto body = [&](auto odd, int zc) __attribute__((always_inline)) {
    constexpr bool ODD = decltype(odd)::value, ZODD = ODD != (bool)(NS & 1);
    const int z = zc - NS;
    // byte offsets of planes zc - NS .. of a vector: V.x + at(k)
    auto at = [&](int k) __attribute__((always_inline)) { return pb.b[k] * (unsigned)sizeof(T); };
    if constexpr (ODD) load_e((zc + 3) >> 1);
    T* pl = L.pl0 + ((z & 1) ? L.plane : 0);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      T pe = Bc[c];
      if constexpr (ODD) {
        const T Bn = prolong4<T>(L.E, cl.re[c], M);
        pe = (T)0.5 * (pe + Bn);
        Bc[c] = Bn;
      }
      const PCol<GEN> k = cl.get(c);
#pragma unroll
      for (int m = 0; m < 2 * NS; ++m) win[c][m] = win[c][m + 1];
      const bool in = k.valid(zc);
      const unsigned vo = pcg_off<T>(k, in);
      T v = 0;
      if (!BR || in) {
        const T rn = lr[c] - alpha * lq[c];
        v = (w0 * rn + pe) + beta * lp[c];
        v = in ? v : (T)0;
        bstore<T>(V.all, vo, V.r + at(NS), rn);
        bstore<T>(V.all, vo, V.pn + at(NS), v);
        s.rr += (double)rn * (double)rn;
      }
      win[c][2 * NS] = v;
      pl[k.low + NS * kLdsWX] = win[c][NS];
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const PCol<GEN> k = cl.get(c);
      const bool in = k.valid(zc + 1);
      const unsigned vo = pcg_off<T>(k, in);
      if constexpr (BR) lr[c] = lp[c] = lq[c] = 0;
      if (!BR || in) {
        lr[c] = bload<T>(V.all, vo, V.r + at(NS + 1));
        lp[c] = bload<T>(V.all, vo | V.none, V.p + at(NS + 1));
        lq[c] = bload<T>(V.all, vo | V.none, V.q + at(NS + 1));
      }
    }
    if constexpr (!ODD) {   // level-1 plane (zc + 2) / 2, interpolated in the next step
#pragma unroll
      for (int u = 0; u < CC; ++u) {
        const PHalves iv(ck.iv[u]);
        if (iv.a <= iv.b) L.E[PHalves(ck.ps[u]).b] = ev[u];
      }
    }
    __syncthreads();
    if constexpr (ZODD)
      pcg_restrict_odd<CC, T>(M, ck, L, z, V.all, V.g2);
    else
      pcg_restrict_even<CC, NT, T>(M, ck, L, cst, z, R, V.all, V.g1);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const PCol<GEN> k = cl.get(c);
      const bool in = k.valid(z);
      T qv = 0;
      if (in) qv = pcg_apply<NS, GEN, T>(S, G, win[c][NS], pl, k.low + NS * kLdsWX, win[c]);
      if (!BR || in) bstore<T>(V.all, pcg_off<T>(k, in), V.q + at(0), qv);
      s.pq += (double)win[c][NS] * (double)qv;
      s.qq += (double)qv * (double)qv;
      if constexpr (ZODD) {
        const T h = (T)0.5 * qv;
        L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += qv;
      }
    }
    pb.next(pst, Zmax, zc - NS);
    if (L.plane == 0) __syncthreads();   // one plane: its readers are done
  };
  for (int zc = z0; zc <= zl; zc += 2) {
    body(std::false_type(), zc);
    body(std::true_type(), zc + 1);
  }
  __syncthreads();
  return s;
}

// The window form without a stored q: q of the direction before is formed again
// from p, whose plane zc is staged with the new direction's plane z.  Five and a
// half accesses per point for a second stencil: the choice where the registers
// hold both windows (FP32 with 512 or 768 threads).
template <int NS, int CPT, int NT, bool GEN, int CC, typename T, bool PK>
__device__ __forceinline__ PSums pcg_sweep_rq(const StencilT<T>& S, const GenStencilT<T>& G, const MgU& M,
                                              const PCols<CPT, GEN, PK>& cl, const PCoarse<CC>& ck, const int* pst,
                                              const int* cst, int Zmax, const PVec& V, T w0, T alpha, T beta,
                                              const PLds<T>& L) {
  T wo[CPT][2 * NS + 1], wn[CPT][2 * NS + 1];   // windows of p around zc and of the new p around z
  T lr[CPT], lp[CPT], pe[CPT], Bc[CPT], acc[CPT], ev[CC];
  PRestrict<CC, T> R;
  PSums s{0.0, 0.0, 0.0};
  const int z0 = -Zmax - 2 + (Zmax & 1);
  const int zl = pcg_last_step(M, Zmax) + NS;
  PBase<2 * NS + 2> pb(pst, Zmax, z0 - NS);   // planes zc - NS .. zc + NS + 1
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
  auto off = [&](int c, int zz) __attribute__((always_inline)) {
    const PCol<GEN> k = cl.get(c);
    return pcg_off<T>(k, k.valid(zz));
  };
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    lr[c] = Bc[c] = acc[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) {
      wn[c][k] = 0;
      wo[c][k] = 0;
      if (k > NS) wo[c][k] = bload<T>(V.all, off(c, z0 - NS - 1 + k) | V.none, V.p + pb.b[k > 0 ? k - 1 : 0] * (unsigned)sizeof(T));
    }
    lp[c] = bload<T>(V.all, off(c, z0 + NS) | V.none, V.p + pb.b[2 * NS] * (unsigned)sizeof(T));
  }
  auto load_e = [&](int kz) {   // a level-1 plane of the correction
    const unsigned base = V.e1 + PBase<1>::at(cst, M.Z1, kz) * (unsigned)sizeof(T);
#pragma unroll
    for (int u = 0; u < CC; ++u) {
      const PHalves iv(ck.iv[u]);
      ev[u] = bload<T>(V.all, kz >= iv.a && kz <= iv.b ? (threadIdx.x + u * NT) * (unsigned)sizeof(T) : kOob, base);
    }
  };
  load_e((z0 + 2) >> 1);
  auto body = [&](auto odd, int zc) __attribute__((always_inline)) {
    constexpr bool ODD = decltype(odd)::value, ZODD = ODD != (bool)(NS & 1);
    const int z = zc - NS;
    // byte offsets of planes zc - NS .. of a vector: V.x + at(k)
    auto at = [&](int k) __attribute__((always_inline)) { return pb.b[k] * (unsigned)sizeof(T); };
    if constexpr (ODD) load_e((zc + 3) >> 1);
    T* pl = L.pl0 + ((zc & 1) ? L.plane : 0);
    T* po = pl + L.old;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
#pragma unroll
      for (int k = 0; k < 2 * NS; ++k) {
        wo[c][k] = wo[c][k + 1];
        wn[c][k] = wn[c][k + 1];
      }
      wo[c][2 * NS] = lp[c];
      const int pos = EXX_PPOS(c);
      po[pos] = wo[c][NS];
      pl[pos] = wn[c][NS];
      pe[c] = Bc[c];
      if constexpr (ODD) {
        const T Bn = prolong4<T>(L.E, cl.re[c], M);
        pe[c] = (T)0.5 * (pe[c] + Bn);
        Bc[c] = Bn;
      }
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) lp[c] = bload<T>(V.all, off(c, zc + NS + 1) | V.none, V.p + at(2 * NS + 1));
    if constexpr (!ODD) {   // level-1 plane (zc + 2) / 2, interpolated in the next step
#pragma unroll
      for (int u = 0; u < CC; ++u) {
        const PHalves iv(ck.iv[u]);
        if (iv.a <= iv.b) L.E[PHalves(ck.ps[u]).b] = ev[u];
      }
    }
    __syncthreads();
    if constexpr (ZODD)
      pcg_restrict_odd<CC, T>(M, ck, L, z, V.all, V.g2);
    else
      pcg_restrict_even<CC, NT, T>(M, ck, L, cst, z, R, V.all, V.g1);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const PCol<GEN> k = cl.get(c);
      const bool in = k.valid(zc);
      T qo = 0;
      if (in) qo = pcg_apply<NS, GEN, T>(S, G, wo[c][NS], po, k.low + NS * kLdsWX, wo[c]);
      const T rn = lr[c] - alpha * qo;
      T v = (w0 * rn + pe[c]) + beta * wo[c][NS];
      v = in ? v : (T)0;
      bstore<T>(V.all, pcg_off<T>(k, in), V.r + at(NS), rn);
      bstore<T>(V.all, pcg_off<T>(k, in), V.pn + at(NS), v);
      s.rr += (double)rn * (double)rn;
      wn[c][2 * NS] = v;
      lr[c] = bload<T>(V.all, pcg_off<T>(k, k.valid(zc + 1)), V.r + at(NS + 1));
      T qv = 0;
      if (k.valid(z)) qv = pcg_apply<NS, GEN, T>(S, G, wn[c][NS], pl, k.low + NS * kLdsWX, wn[c]);
      s.pq += (double)wn[c][NS] * (double)qv;
      s.qq += (double)qv * (double)qv;
      if constexpr (ZODD) {
        const T h = (T)0.5 * qv;
        L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += qv;
      }
    }
    pb.next(pst, Zmax, zc - NS);
    if (L.plane == 0) __syncthreads();   // one plane: its readers are done
  };
  for (int zc = z0; zc <= zl; zc += 2) {
    body(std::false_type(), zc);
    body(std::true_type(), zc + 1);
  }
  __syncthreads();
  return s;
}

// tl_scatter with the arms of a stencil read anew (constant indices only: the
// copy is then never in memory).
template <int NS, typename T>
__device__ __forceinline__ void pcg_scatter(const GenStencilT<T>& S, T v, bool point, const T* pl, int pos, T* acc) {
  if (point) {
    T s = S.diag * v;
    const T* bp = pl + pos;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (k >= S.n_in) break;
      const int off = S.in_off[k];
      T t = 0;
#pragma unroll
      for (int q = 1; q <= NS; ++q) t += S.w[q] * (bp[q * off] + bp[-q * off]);
      s += S.in_coef[k] * t;
    }
    acc[NS] += s;
  }
#pragma unroll
  for (int q = 1; q <= NS; ++q) {
    const T t = S.czw[q] * v;
    acc[NS - q] += t;
    acc[NS + q] += t;
  }
  gen_tilted<NS, NS, T>(S, pl, pos, acc);
}

// The same with arms leaving the sweep plane: a plane of the new p is staged
// as it enters and scattered into the partial sums of its columns' points; the
// point n planes behind completes (see cg_pass_a_tl).  p.q is summed as the
// planes enter, A being symmetric: p times its own plane's part and twice what
// the planes before have left in its sum, so no window of p is kept.
template <int NS, int CPT, int NT, int CC, typename T, bool GEN = true, bool PK = false>
__device__ __forceinline__ PSums pcg_sweep_tl(const SolveKArgs& a, const MgU& M,
                                              const PCols<CPT, GEN, PK>& cl, const PCoarse<CC>& ck, const int* pst,
                                              const int* cst, int Zmax, const PVec& V, T w0, T alpha, T beta,
                                              const PLds<T>& L) {
  T sum[CPT][2 * NS + 1], pv[CPT];   // partial sums of planes z .. zc + NS; p of plane zc
  T lr[CPT], lp[CPT], lq[CPT], Bc[CPT], acc[CPT], ev[CC];
  // FP64: the sums leave no registers for several columns' accesses in flight;
  // columns without a point are branched around
  constexpr bool BR = sizeof(T) == 8;
  PRestrict<CC, T> R;
  PSums s{0.0, 0.0, 0.0};
  const int z0 = -Zmax - 2 + (Zmax & 1);
  const int zl = pcg_last_step(M, Zmax) + NS;
  PBase<NS + 2> pb(pst, Zmax, z0 - NS);   // planes zc - NS .. zc + 1
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    lr[c] = lp[c] = lq[c] = Bc[c] = acc[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) sum[c][k] = 0;
  }
  auto load_e = [&](int kz) {   // a level-1 plane of the correction
    const unsigned base = V.e1 + PBase<1>::at(cst, M.Z1, kz) * (unsigned)sizeof(T);
#pragma unroll
    for (int u = 0; u < CC; ++u) {
      const PHalves iv(ck.iv[u]);
      ev[u] = bload<T>(V.all, kz >= iv.a && kz <= iv.b ? (threadIdx.x + u * NT) * (unsigned)sizeof(T) : kOob, base);
    }
  };
  load_e((z0 + 2) >> 1);
  auto body = [&](auto odd, int zc) __attribute__((always_inline)) {
    constexpr bool ODD = decltype(odd)::value, ZODD = ODD != (bool)(NS & 1);
    const int z = zc - NS;
    // byte offsets of planes zc - NS .. of a vector: V.x + at(k)
    auto at = [&](int k) __attribute__((always_inline)) { return pb.b[k] * (unsigned)sizeof(T); };
    if constexpr (ODD) load_e((zc + 3) >> 1);
    const GenStencilT<T> G = gen_args<T>(a);
    T* pl = L.pl0 + ((zc & 1) ? L.plane : 0);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      T pe = Bc[c];
      if constexpr (ODD) {
        const T Bn = prolong4<T>(L.E, cl.re[c], M);
        pe = (T)0.5 * (pe + Bn);
        Bc[c] = Bn;
      }
      const PCol<GEN> k = cl.get(c);
      const bool in = k.valid(zc);
      const unsigned vo = pcg_off<T>(k, in);
      T v = 0;
      if (!BR || in) {
        const T rn = lr[c] - alpha * lq[c];
        v = (w0 * rn + pe) + beta * lp[c];
        v = in ? v : (T)0;
        bstore<T>(V.all, vo, V.r + at(NS), rn);
        bstore<T>(V.all, vo, V.pn + at(NS), v);
        s.rr += (double)rn * (double)rn;
      }
      pv[c] = v;
      pl[k.low + NS * kLdsWX] = v;
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const PCol<GEN> k = cl.get(c);
      const bool in = k.valid(zc + 1);
      const unsigned vo = pcg_off<T>(k, in);
      if constexpr (BR) lr[c] = lp[c] = lq[c] = 0;
      if (!BR || in) {
        lr[c] = bload<T>(V.all, vo, V.r + at(NS + 1));
        lp[c] = bload<T>(V.all, vo | V.none, V.p + at(NS + 1));
        lq[c] = bload<T>(V.all, vo | V.none, V.q + at(NS + 1));
      }
    }
    if constexpr (!ODD) {   // level-1 plane (zc + 2) / 2, interpolated in the next step
#pragma unroll
      for (int u = 0; u < CC; ++u) {
        const PHalves iv(ck.iv[u]);
        if (iv.a <= iv.b) L.E[PHalves(ck.ps[u]).b] = ev[u];
      }
    }
    __syncthreads();
    if constexpr (ZODD)
      pcg_restrict_odd<CC, T>(M, ck, L, z, V.all, V.g2);
    else
      pcg_restrict_even<CC, NT, T>(M, ck, L, cst, z, R, V.all, V.g1);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const PCol<GEN> k = cl.get(c);
      const T below = sum[c][NS];
      if (k.near(zc, NS)) pcg_scatter<NS, T>(G, pv[c], k.valid(zc), pl, k.low + NS * kLdsWX, sum[c]);
      s.pq -= (double)pv[c] * ((double)below + (double)sum[c][NS]);
      const bool in = k.valid(z);
      const T qv = in ? -sum[c][0] : (T)0;
      if (!BR || in) {
        bstore<T>(V.all, pcg_off<T>(k, in), V.q + at(0), qv);
        s.qq += (double)qv * (double)qv;
      }
#pragma unroll
      for (int k = 0; k < 2 * NS; ++k) sum[c][k] = sum[c][k + 1];
      sum[c][2 * NS] = 0;
      if constexpr (ZODD) {
        const T h = (T)0.5 * qv;
        L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += qv;
      }
    }
    pb.next(pst, Zmax, zc - NS);
    if (L.plane == 0) __syncthreads();   // one plane: its readers are done
  };
  for (int zc = z0; zc <= zl; zc += 2) {
    body(std::false_type(), zc);
    body(std::true_type(), zc + 1);
  }
  __syncthreads();
  return s;
}

// The restriction of a residual that is not followed from the one before (the
// first one): the streamed part of the sweep alone.
template <int CPT, int NT, int CC, typename T, bool GEN, bool PK>
__device__ __forceinline__ void pcg_pass_r(const MgU& M, const PCols<CPT, GEN, PK>& cl, const PCoarse<CC>& ck, const int* pst,
                           const int* cst, int Zmax, const T* r, const PVec& V, unsigned c1, unsigned b2,
                           const PLds<T>& L) {
  T cr[CPT], acc[CPT];
  PRestrict<CC, T> R;
  PBase<2> pb(pst, Zmax, -Zmax);
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    acc[c] = 0;
    cr[c] = EXX_PVALID(c, -Zmax) ? gload(r, EXX_PIDX(c, pb.b[0])) : (T)0;
  }
  const int zl = pcg_last_step(M, Zmax);
  for (int z = -Zmax; z <= zl; ++z) {
    T nr[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) nr[c] = EXX_PVALID(c, z + 1) ? gload(r, EXX_PIDX(c, pb.b[1])) : (T)0;
    __syncthreads();
    pcg_restrict_step<CC, NT, T>(M, ck, L, cst, z, R, V.all, c1, b2);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      if (z & 1) {
        const T h = (T)0.5 * cr[c];
        if (EXX_PHAS(c)) L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += cr[c];
      }
      cr[c] = nr[c];
    }
    pb.next(pst, Zmax, z);
  }
  __syncthreads();
}

// The FP64 true residual b - A x, stored times rs as the working residual
// (FP32 in the mixed solve's reliable updates, see cg_true_residual), and the
// restriction of that.  pl0 and pl0 + plane are FP64 planes; L holds the
// working precision's buffers of the restriction.  Returns this thread's sum of
// the true residual^2.
template <int NS, int CPT, int NT, bool GEN, int CC, typename T, bool PK>
__device__ __forceinline__ double pcg_residual(const SolveKArgs& a, const MgU& M, const PCols<CPT, GEN, PK>& cl, const PCoarse<CC>& ck,
                               const int* pst, const int* cst, int Zmax, const double* __restrict__ x,
                               const double* __restrict__ b, T* __restrict__ r, double rs, double* pl0,
                               int plane, const PVec& V, unsigned c1, unsigned b2, const PLds<T>& L) {
  double win[CPT][2 * NS + 1];
  T acc[CPT];
  PRestrict<CC, T> R;
  double sum = 0.0;
  PBase<NS + 2> pb(pst, Zmax, -Zmax);   // planes z .. z + NS + 1
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    acc[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) {
      const int zz = -Zmax - NS + k;
      win[c][k] = zz >= -Zmax && EXX_PVALID(c, zz) ? gload(x, EXX_PIDX(c, pb.b[max(k - NS, 0)])) : 0.0;
    }
  }
  const int zl = pcg_last_step(M, Zmax);
  for (int z = -Zmax; z <= zl; ++z) {
    double nx[CPT], cb[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      nx[c] = EXX_PVALID(c, z + NS + 1) ? gload(x, EXX_PIDX(c, pb.b[NS + 1])) : 0.0;
      cb[c] = EXX_PVALID(c, z) ? gload(b, EXX_PIDX(c, pb.b[0])) : 0.0;
    }
    double* pl = pl0 + ((z & 1) ? plane : 0);
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (EXX_PHAS(c)) pl[EXX_PPOS(c)] = win[c][NS];
    __syncthreads();
    pcg_restrict_step<CC, NT, T>(M, ck, L, cst, z, R, V.all, c1, b2);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      T rn = 0;
      if (EXX_PVALID(c, z)) {
        const double rt = cb[c] - pcg_apply<NS, GEN, double>(a.S, a.G, win[c][NS], pl, EXX_PPOS(c), win[c]);
        rn = (T)(rt * rs);
        gstore(r, EXX_PIDX(c, pb.b[0]), rn);
        sum += rt * rt;
      }
      if (z & 1) {
        const T h = (T)0.5 * rn;
        if (EXX_PHAS(c)) L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += rn;
      }
#pragma unroll
      for (int k = 0; k < 2 * NS; ++k) win[c][k] = win[c][k + 1];
      win[c][2 * NS] = nx[c];
    }
    pb.next(pst, Zmax, z);
    if (plane == 0) __syncthreads();
  }
  __syncthreads();
  return sum;
}

template <int NS, int CPT, int NT, int CC, typename T, bool GEN = true, bool PK = false>
__device__ __forceinline__ double pcg_residual_tl(const SolveKArgs& a, const MgU& M, const PCols<CPT, GEN, PK>& cl, const PCoarse<CC>& ck,
                                  const int* pst, const int* cst, int Zmax, const double* __restrict__ x,
                                  const double* __restrict__ b, T* __restrict__ r, double rs, double* pl0,
                                  int plane, const PVec& V, unsigned c1, unsigned b2, const PLds<T>& L) {
  double acc[CPT][2 * NS + 1], cx[CPT];
  T ra[CPT];
  PRestrict<CC, T> R;
  double sum = 0.0;
  PBase<NS + 2> pb(pst, Zmax, -Zmax - NS);   // planes z - NS .. z + 1
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    ra[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) acc[c][k] = 0.0;
    cx[c] = EXX_PVALID(c, -Zmax) ? gload(x, EXX_PIDX(c, pb.b[NS])) : 0.0;
  }
  const int zl = pcg_last_step(M, Zmax) + NS;
  for (int z = -Zmax; z <= zl; ++z) {
    const int zo = z - NS;
    double nx[CPT], ob[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      nx[c] = EXX_PVALID(c, z + 1) ? gload(x, EXX_PIDX(c, pb.b[NS + 1])) : 0.0;
      ob[c] = EXX_PVALID(c, zo) ? gload(b, EXX_PIDX(c, pb.b[0])) : 0.0;
    }
    double* pl = pl0 + ((z & 1) ? plane : 0);
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (EXX_PHAS(c)) pl[EXX_PPOS(c)] = cx[c];
    __syncthreads();
    pcg_restrict_step<CC, NT, T>(M, ck, L, cst, zo, R, V.all, c1, b2);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      if (EXX_PHAS(c) && z <= Zmax + NS)
        tl_scatter<NS, double>(a.G, cx[c], EXX_PVALID(c, z), pl, EXX_PPOS(c), acc[c]);
      T rn = 0;
      if (EXX_PVALID(c, zo)) {
        const double rt = ob[c] + acc[c][0];   // b - A x, A x = -acc
        rn = (T)(rt * rs);
        gstore(r, EXX_PIDX(c, pb.b[0]), rn);
        sum += rt * rt;
      }
      if (zo & 1) {
        const T h = (T)0.5 * rn;
        if (EXX_PHAS(c)) L.R1[EXX_PR1(c)] = ra[c] + h;
        ra[c] = h;
      } else {
        ra[c] += rn;
      }
#pragma unroll
      for (int k = 0; k < 2 * NS; ++k) acc[c][k] = acc[c][k + 1];
      acc[c][2 * NS] = 0.0;
      cx[c] = nx[c];
    }
    pb.next(pst, Zmax, z - NS);
    if (plane == 0) __syncthreads();
  }
  __syncthreads();
  return sum;
}

// Trilinear interpolation of the box of the next coarser level (half-widths E,
// dims D, one zero cell on each side) at point (x, y, z) of this level.
template <typename T>
__device__ __forceinline__ T prolong8(const T* B, const int* E, const int* D, int x, int y, int z) {
  const T* b = B + ((x >> 1) + E[0] + 1) + D[0] * (((y >> 1) + E[1] + 1) + D[1] * ((z >> 1) + E[2] + 1));
  const int dx = x & 1, dy = (y & 1) ? D[0] : 0, dz = (z & 1) ? D[0] * D[1] : 0;
  return (T)0.125 * (((b[0] + b[dx]) + (b[dy] + b[dx + dy])) + ((b[dz] + b[dx + dz]) + (b[dy + dz] + b[dx + dy + dz])));
}
// Restriction of a box (half-widths E, dims D) at point (x, y, z) of the next coarser level.
template <typename T>
__device__ __forceinline__ T restrict27(const T* B, const int* E, const int* D, int x, int y, int z) {
  const int w2 = D[0] * D[1];
  const T* b = B + (2 * x + E[0] + 1) + D[0] * ((2 * y + E[1] + 1) + D[1] * (2 * z + E[2] + 1));
  return restrict9<T>(b, D[0]) + (T)0.5 * (restrict9<T>(b - w2, D[0]) + restrict9<T>(b + w2, D[0]));
}

// for (k = tid; k < n; k += NT) with a trip count that every lane shares: the
// loop's branch is scalar and no lane leaves it early.
#define EXX_PFOR(k, n) \
  for (int k##_0 = 0, k##_n = uniform((int)(n)); k##_0 < k##_n; k##_0 += NT) \
    if (const int k = k##_0 + (int)threadIdx.x; k < k##_n)

// The coarse phase: the residuals of levels 1 and 2, c1 and b2, take the step
// - alpha P^T q (g1, g2; not with fresh residuals), levels 2 to 4 follow as boxes
// in LDS, then the correction e1 over the level-1 points.  sums: this
// thread's parts of r_1.e_1, e_1.g_1 of the e_1 before, and e_1.g_1 (and zero:
// block_sum4 takes four).  The boxes lie in
// the sweeps' LDS and are cleared at the end (positions off the sphere must read
// zero there).
template <int NT, typename T>
__device__ __forceinline__ void pcg_coarse(const MgDev& M, const double* wl, T* lds, T* c1, const T* g1, T* e1, T* b2,
                                           const T* g2, bool step, T alpha, double (&sums)[4]) {
  const int n2 = uniform(M.D2[0] * M.D2[1] * M.D2[2]), n3 = uniform(M.D3[0] * M.D3[1] * M.D3[2]),
            n4 = uniform(M.D4[0] * M.D4[1] * M.D4[2]);
  T *B2 = lds, *B3 = lds + n2, *B4 = B3 + n3;
  constexpr int U = 4;   // loads in flight per thread (at clamped indices: only the stores are conditional)
  for (int k0 = 0; k0 < n2; k0 += U * NT) {
    T v[U], g[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = min(k0 + j * NT + (int)threadIdx.x, n2 - 1);
      v[j] = b2[k];
      g[j] = step ? g2[k] : (T)0;
    }
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (const int k = k0 + j * NT + (int)threadIdx.x; k < n2) {
        const T w = v[j] - alpha * g[j];
        B2[k] = w;
        if (step) b2[k] = w;
      }
  }
  EXX_PFOR(k, n3 + n4) B3[k] = 0;
  __syncthreads();
  EXX_PFOR(k, M.n_p3) {
    const short4 o = M.p3[k];
    B3[(o.x + M.E3[0] + 1) + M.D3[0] * ((o.y + M.E3[1] + 1) + M.D3[1] * (o.z + M.E3[2] + 1))] =
        restrict27<T>(B2, M.E2, M.D2, o.x, o.y, o.z);
  }
  __syncthreads();
  EXX_PFOR(k, M.n_p4) {
    const short4 o = M.p4[k];
    B4[(o.x + M.E4[0] + 1) + M.D4[0] * ((o.y + M.E4[1] + 1) + M.D4[1] * (o.z + M.E4[2] + 1))] =
        (T)wl[4] * restrict27<T>(B3, M.E3, M.D3, o.x, o.y, o.z);
  }
  __syncthreads();
  EXX_PFOR(k, M.n_p3) {
    const short4 o = M.p3[k];
    T* b = B3 + (o.x + M.E3[0] + 1) + M.D3[0] * ((o.y + M.E3[1] + 1) + M.D3[1] * (o.z + M.E3[2] + 1));
    *b = (T)wl[3] * *b + prolong8<T>(B4, M.E4, M.D4, o.x, o.y, o.z);
  }
  __syncthreads();
  EXX_PFOR(k, M.n_p2) {
    const short4 o = M.p2[k];
    T* b = B2 + (o.x + M.E2[0] + 1) + M.D2[0] * ((o.y + M.E2[1] + 1) + M.D2[1] * (o.z + M.E2[2] + 1));
    *b = (T)wl[2] * *b + prolong8<T>(B3, M.E3, M.D3, o.x, o.y, o.z);
  }
  __syncthreads();
  sums[0] = sums[1] = sums[2] = sums[3] = 0.0;
  const T w1 = (T)wl[1];
  const int np1 = uniform(M.n_p1);
  for (int k0 = 0; k0 < np1; k0 += U * NT) {
    short4 o[U];
    T rv[U], gv[U], ov[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = min(k0 + j * NT + (int)threadIdx.x, np1 - 1);
      o[j] = M.p1[k];
      rv[j] = c1[k];
      gv[j] = step ? g1[k] : (T)0;
      ov[j] = step ? e1[k] : (T)0;
    }
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (const int k = k0 + j * NT + (int)threadIdx.x; k < np1 && !o[j].w) {
        const T rn = rv[j] - alpha * gv[j];
        const T v = w1 * rn + prolong8<T>(B2, M.E2, M.D2, o[j].x, o[j].y, o[j].z);
        if (step) c1[k] = rn;
        e1[k] = v;
        sums[0] += (double)rn * (double)v;
        sums[1] += (double)ov[j] * (double)gv[j];
        sums[2] += (double)v * (double)gv[j];
      }
  }
  __syncthreads();
  EXX_PFOR(k, n2 + n3 + n4) lds[k] = 0;
  __syncthreads();
}

template <int NS, int CPT, int NT, bool GEN, bool TL, bool RQ, int CC, typename T, bool PK>
__device__ __forceinline__ PSums pcg_sweep(const SolveKArgs& a, const StencilT<T>& S, const GenStencilT<T>& G, const MgU& M,
                                           const PCols<CPT, GEN, PK>& cl, const PCoarse<CC>& ck, const int* pst,
                                           const int* cst, int Zmax, const PVec& V, T w0, T alpha, T beta,
                                           const PLds<T>& L) {
  w0 = uniform(w0);
  alpha = uniform(alpha);
  beta = uniform(beta);
  if constexpr (TL)
    return pcg_sweep_tl<NS, CPT, NT, CC, T>(a, M, cl, ck, pst, cst, Zmax, V, w0, alpha, beta, L);
  else if constexpr (RQ)
    return pcg_sweep_rq<NS, CPT, NT, GEN, CC, T>(S, G, M, cl, ck, pst, cst, Zmax, V, w0, alpha, beta, L);
  else
    return pcg_sweep_w<NS, CPT, NT, GEN, CC, T>(S, G, M, cl, ck, pst, cst, Zmax, V, w0, alpha, beta, L);
}

// The last directions and their steps, not yet added to x: buffers lo .. n - 1
// of kPcgRing; the next sweep writes buffer n (after a flush of a full ring, 0).
struct PRing {
  int lo = 0, n = 0;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  __device__ __forceinline__ void push(double alpha) {
    a0 = n == 0 ? alpha : a0;
    a1 = n == 1 ? alpha : a1;
    a2 = n == 2 ? alpha : a2;
    a3 = n == 3 ? alpha : a3;
    ++n;
  }
};
static_assert(kPcgRing == 4, "PRing holds four steps");

// x = (zero ? 0 : x) + scale * (y + sum of the ring's steps), y absent (null)
// or one more vector: a stream over the sphere's points.
template <int NT, typename X, typename T>
__device__ __forceinline__ void pcg_flush(X* x, bool zero, double scale, const T* y, PRing R, const T* p0,
                                          long long stride, int npe) {
  constexpr int U = 4;   // points in flight per thread
  const X w[kPcgRing] = {(X)uniform(R.a0), (X)uniform(R.a1), (X)uniform(R.a2), (X)uniform(R.a3)};
  for (int k0 = 0; k0 < npe; k0 += U * NT) {
    T yv[U], v[U][kPcgRing];
    X xv[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = min(k0 + j * NT + (int)threadIdx.x, npe - 1);   // clamped: only the stores are conditional
      xv[j] = zero ? (X)0 : x[k];
      yv[j] = y ? y[k] : (T)0;
#pragma unroll
      for (int i = 0; i < kPcgRing; ++i) v[j][i] = i >= R.lo && i < R.n ? p0[i * stride + k] : (T)0;
    }
    if constexpr (sizeof(X) != sizeof(T)) {
      // the conversions to X stay behind all the loads: moved up to each, they
      // wait for it (mixed, 4,789 pairs of 2,957 columns: an evaluation 268 ms against
      // 255 ms)
#pragma unroll
      for (int j = 0; j < U; ++j) {
        asm volatile("" : "+v"(yv[j]));
#pragma unroll
        for (int i = 0; i < kPcgRing; ++i) asm volatile("" : "+v"(v[j][i]));
      }
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const X s = pcg_add_steps<X, T>(yv[j], w, v[j]);
      if (const int k = k0 + j * NT + (int)threadIdx.x; k < npe) x[k] = xv[j] + (X)scale * s;
    }
  }
}

// The scalars that a direction needs before its sweep: beta makes the new
// direction z + beta p conjugate to p, and z.q = w_0 (r.q - alpha q.q) + e.g,
// where r.q of the step before follows from p.q (see the file comment).  Once
// the sweep has measured |r|^2, r.q is known without that; what is left of p.q'
// (rounding, which would double relative to r each iteration: FP64 solves
// slowed from 33 iterations to 54) is taken into account in the next r.q.
struct PDir {
  double beta = 0.0, cross = 0.0, eng = 0.0;
  // with eg = e.g of the direction's own correction, en the new correction's
  __device__ __forceinline__ void next(double w0, double alpha, double pq, double qq, double eg, double en) {
    const double rq = (pq - beta * cross - eg) / w0;
    eng = en;
    const double b = -(w0 * (rq - alpha * qq) + en) / pq;
    beta = b > 0.0 ? b : 0.0;   // rounding at convergence, or a NaN (which the sweep's products show)
  }
  // rr and rrn: |r|^2 before and after the step
  __device__ __forceinline__ void measured(double w0, double alpha, double pq, double qq, double rr, double rrn) {
    const double rq = (rr - rrn + alpha * alpha * qq) / (2.0 * alpha);
    cross = w0 * (rq - alpha * qq) + eng + beta * pq;
  }
};

// The slot of a solve in precision T, from base: r, q, the ring of p, the
// level-1 residual, its step and the correction, the level-2 residual box and
// its step.
template <typename T>
struct PSlot {
  T *r, *q, *p0, *c1, *g1, *e1, *b2, *g2;
  int bytes;
  __device__ __forceinline__ PSlot(T* base, const SolveKArgs& a) {
    r = base;
    q = r + a.sstride;
    p0 = q + a.sstride;
    c1 = p0 + kPcgRing * a.sstride;
    g1 = c1 + a.c1stride;
    e1 = g1 + a.c1stride;
    b2 = e1 + a.c1stride;
    g2 = b2 + a.b2stride;
    bytes = uniform((int)((char*)(g2 + a.b2stride) - (char*)base));
  }
  __device__ __forceinline__ unsigned off(const T* v) const { return (unsigned)uniform((int)((char*)v - (char*)r)); }
  // the vectors of a sweep from the direction in buffer `from` of the ring to `to`
  __device__ __forceinline__ PVec vec(const SolveKArgs& a, int from, int to, bool first) const {
    PVec V;
    V.all = pbuf(r, bytes);
    V.none = first ? kOob : 0u;
    V.r = 0;
    V.q = off(q);
    V.p = off(p0 + from * a.sstride);
    V.pn = off(p0 + to * a.sstride);
    V.e1 = off(e1);
    V.g1 = off(g1);
    V.g2 = off(g2);
    return V;
  }
};

// A right-hand side with ||b||^2 below kPcgTiny is solved times kPcgUnit: its
// products would otherwise be too small for numbers of full precision, and the
// solve end in NaNs (densities below about 1e-136).
constexpr double kPcgTiny = 0x1p-900, kPcgUnit = 0x1p+600;

// FP64 solve: one workgroup per pair, as k_solve.
template <int NS, int CPT, int NT, bool GEN, bool TL>
__global__ __launch_bounds__(NT) void k_pcg(SolveKArgs a) {
  extern __shared__ double lds[];
  __shared__ double red[4 * (NT / 64)];
  __shared__ int s_item;
  __shared__ double s_unit;   // (in LDS: the sweeps need the registers)
  constexpr int CC = NT >= 1024 ? 1 : 2;
  const int plane = kLdsWX * a.lds_wy;
  int* pst = reinterpret_cast<int*>(lds + a.pcg_lds);
  int* cst = pst + a.pcg_ints;
  const PSlot<double> W((double*)((char*)a.slot_ws + (long long)blockIdx.x * a.slot_bytes), a);

  long long lo, hi;
  solve_range(a, &lo, &hi);
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.queue, 1);
    __syncthreads();
    const long long row = lo + uniform(s_item);
    __syncthreads();
    if (row >= hi) break;
    const long long item = row - a.p0;
    const int pid = uniform(a.order[row]);
    const ClassDev& C = a.cls[uniform(a.pairs[pid].cls)];
    const MgU M = mg_uniform(C.mg);
    const int Zmax = uniform(C.Zmax);
    const int npe = uniform((int)C.n_pe);
    double* x = a.bx_ws + item * a.rstride;
    PLds<double> L;
    L.pl0 = lds;
    L.plane = a.pcg_planes == 2 ? plane : 0;
    L.old = 0;
    L.R1 = lds + a.pcg_planes * plane;
    L.R2 = L.R1 + M.rw * M.rh;
    L.E = L.R2 + M.ew * M.eh;

    EXX_PFOR(k, a.pcg_lds) lds[k] = 0.0;
    EXX_PFOR(k, 2 * Zmax + 2) pst[k] = C.plane_start[k];
    EXX_PFOR(k, 2 * M.Z1 + 2) cst[k] = C.mg.c1start[k];
    EXX_PFOR(k, M.d2xy * C.mg.D2[2]) W.b2[k] = W.g2[k] = 0.0;
    PCols<CPT, GEN, true> cl;
    pcg_cols<NS, CPT, NT, GEN>(C, a.lds_cx, a.lds_cy, cl);
    PCoarse<CC> ck;
    pcg_coarse_cols<CC, NT>(C, ck);
    const bool padded = uniform((int)C.n_real) != npe;
    double bb = 0.0;
    EXX_PFOR(k, npe) {
      const double v = x[k];
      bb += v * v;
      if (padded) {   // padding slots, which no sweep writes, hold zero
#pragma unroll
        for (int i = 0; i < kPcgRing; ++i) W.p0[i * a.sstride + k] = 0.0;
      }
    }
    if (threadIdx.x == 0) s_unit = 1.0;
    bb = uniform(block_sum(bb, red));
    // (told to be rare, or the branch takes registers from the sweeps: tilted arms,
    // 356 pairs, 50.9 ms against 54.3 ms)
    if (__builtin_expect(bb > 0.0 && bb < kPcgTiny, 0)) {
      double t = 0.0;
      EXX_PFOR(k, npe) {
        const double v = x[k] * kPcgUnit;
        x[k] = v;
        t += v * v;
      }
      bb = uniform(block_sum(t, red));
      if (threadIdx.x == 0) s_unit = kPcgUnit;
    }
    const double bnorm = sqrt(bb);
    int it = 0, code = kCgConverged;
    double rr = bb, rz = 0.0;
    bool x_zero = true;
    bool conv = bnorm == 0.0;   // b == 0: x = b = 0 already
    if (!conv && !(bnorm < INFINITY)) code = kCgNonFinite;   // b holds a NaN or an infinity
    // the first residual and its restriction: b with x = 0, or b - A x of the
    // previous solution
    if (!conv && code == kCgConverged) {
      if (warm_gather<double>(a, C, pid, W.p0)) {
        __syncthreads();
        if (__builtin_expect(uniform(s_unit) != 1.0, 0)) {
          EXX_PFOR(k, npe) W.p0[k] *= s_unit;
          __syncthreads();
        }
        double t;
        if constexpr (TL)
          t = pcg_residual_tl<NS, CPT, NT, CC, double>(a, M, cl, ck, pst, cst, Zmax, W.p0, x, W.r, 1.0, lds, L.plane,
                                                       W.vec(a, 0, 0, true), W.off(W.c1), W.off(W.b2), L);
        else
          t = pcg_residual<NS, CPT, NT, GEN, CC, double>(a, M, cl, ck, pst, cst, Zmax, W.p0, x, W.r, 1.0, lds, L.plane,
                                                         W.vec(a, 0, 0, true), W.off(W.c1), W.off(W.b2), L);
        rr = uniform(block_sum(t, red));
        EXX_PFOR(k, npe) x[k] = W.p0[k];
        x_zero = false;
        if (sqrt(rr) <= a.tol * bnorm) conv = true;
        if (!(rr < INFINITY)) code = kCgNonFinite;
        __syncthreads();
      } else {
        EXX_PFOR(k, npe) W.r[k] = x[k];
        __syncthreads();
        pcg_pass_r<CPT, NT, CC, double, GEN>(M, cl, ck, pst, cst, Zmax, W.r, W.vec(a, 0, 0, true), W.off(W.c1), W.off(W.b2), L);
      }
    }
    PRing ring;
    bool first = true;
    double alpha = 0.0, pq = 0.0, qq = 0.0;
    PDir dir;
    while (!conv && code == kCgConverged) {
      double t[4];
      pcg_coarse<NT, double>(C.mg, a.wl, lds, W.c1, W.g1, W.e1, W.b2, W.g2, !first, alpha, t);
      block_sum4(t, red);
      const double re = uniform(t[0]);
      if (first)
        dir = PDir();
      else
        dir.next(a.wl[0], alpha, pq, qq, uniform(t[1]), uniform(t[2]));
      if (ring.n == kPcgRing) {
        pcg_flush<NT, double, double>(x, x_zero, 1.0, nullptr, ring, W.p0, a.sstride, npe);
        __syncthreads();
        x_zero = false;
        ring.lo = ring.n = 0;
      }
      const PVec V = W.vec(a, (ring.n + kPcgRing - 1) % kPcgRing, ring.n, first);
      const PSums s = pcg_sweep<NS, CPT, NT, GEN, TL, false, CC, double>(a, a.S, a.G, M, cl, ck, pst, cst, Zmax, V,
                                                                         a.wl[0], alpha, dir.beta, L);
      double v[4] = {s.rr, s.pq, s.qq, 0.0};
      block_sum4(v, red);
      const double rrn = uniform(v[0]);
      if (!first) dir.measured(a.wl[0], alpha, pq, qq, rr, rrn);
      rr = rrn;
      rz = a.wl[0] * rr + re;
      pq = uniform(v[1]);
      qq = uniform(v[2]);
      if (!first) {
        ++it;
        if (sqrt(rr) <= a.tol * bnorm) conv = true;
      }
      first = false;
      if (conv) break;
      if (!(rr == rr)) {
        rr = NAN;
        code = kCgNonFinite;
      } else if (!(pq > 0.0) || !(pq < INFINITY) || !(rz > 0.0) || !(rz < INFINITY)) {
        // A and the preconditioner are positive definite: only non-finite
        // values get here
        code = kCgBreakdown;
      } else if (it >= a.max_iter) {
        break;
      }
      alpha = rz / pq;
      ring.push(alpha);
    }
    if (ring.n > 0) {
      pcg_flush<NT, double, double>(x, x_zero, 1.0, nullptr, ring, W.p0, a.sstride, npe);
      __syncthreads();
    } else if (x_zero && bnorm > 0.0 && code != kCgNonFinite) {
      EXX_PFOR(k, npe) x[k] = 0.0;
      __syncthreads();
    }
    if (!conv && code == kCgConverged) code = kCgCap;
    if (__builtin_expect(uniform(s_unit) != 1.0, 0)) {
      EXX_PFOR(k, npe) x[k] *= 1.0 / kPcgUnit;
      __syncthreads();
    }
    warm_store_solution(a, npe, pid, x);
    if (threadIdx.x == 0) {
      a.outIt[pid] = it;
      a.outRes[pid] = bnorm > 0.0 ? sqrt(rr) / bnorm : 0.0;
      a.outUpd[pid] = 0;
      a.outSav[pid] = it / 4;   // seven and a half accesses an iteration
      a.outExit[pid] = code;
    }
    __syncthreads();
  }
}

// Mixed-precision solve: FP32 recursion in units of ||b|| with FP64 dots and
// reliable updates, as k_solve_mixed, with the preconditioner's vectors in
// FP32.  A reliable update replaces the residual and its restrictions and keeps
// the direction.  Slot: x (FP64), the correction y, then the working vectors.
template <int NS, int CPT, int NT, bool GEN, bool TL>
__global__ __launch_bounds__(NT) void k_pcg_mixed(SolveKArgs a) {
  extern __shared__ double lds[];
  __shared__ double red[4 * (NT / 64)];
  __shared__ int s_item;
  constexpr int CC = NT >= 1024 ? 1 : 2;
  constexpr bool RQ = !TL && NT < 1024;
  const int plane = kLdsWX * a.lds_wy;
  float* fl = reinterpret_cast<float*>(lds);
  int* pst = reinterpret_cast<int*>(fl + a.pcg_lds);
  int* cst = pst + a.pcg_ints;
  double* x = (double*)((char*)a.slot_ws + (long long)blockIdx.x * a.slot_bytes);
  float* y = reinterpret_cast<float*>(x + a.sstride);
  const PSlot<float> W(y + a.sstride, a);
  const StencilT<float> S32 = stencil_cast<float>(a.S);

  long long lo, hi;
  solve_range(a, &lo, &hi);
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.queue, 1);
    __syncthreads();
    const long long row = lo + uniform(s_item);
    __syncthreads();
    if (row >= hi) break;
    const long long item = row - a.p0;
    const int pid = uniform(a.order[row]);
    const int cls = uniform(a.pairs[pid].cls);
    const ClassDev& C = a.cls[cls];
    const double delta = a.cls_delta[cls];
    const MgU M = mg_uniform(C.mg);
    const int Zmax = uniform(C.Zmax);
    const int npe = uniform((int)C.n_pe);
    double* bx = a.bx_ws + item * a.rstride;
    // (a reliable update's FP64 plane takes the place of two FP32 ones)
    PLds<float> L;
    L.pl0 = fl;
    L.plane = RQ && a.pcg_planes == 1 ? 0 : plane;
    L.old = a.pcg_planes == 1 ? plane : 2 * plane;
    L.R1 = fl + 2 * a.pcg_planes * plane;
    L.R2 = L.R1 + M.rw * M.rh;
    L.E = L.R2 + M.ew * M.eh;

    EXX_PFOR(k, 2 * Zmax + 2) pst[k] = C.plane_start[k];
    EXX_PFOR(k, 2 * M.Z1 + 2) cst[k] = C.mg.c1start[k];
    EXX_PFOR(k, M.d2xy * C.mg.D2[2]) W.b2[k] = W.g2[k] = 0.0f;
    PCols<CPT, GEN, false> cl;
    pcg_cols<NS, CPT, NT, GEN>(C, a.lds_cx, a.lds_cy, cl);
    PCoarse<CC> ck;
    pcg_coarse_cols<CC, NT>(C, ck);
    const bool padded = uniform((int)C.n_real) != npe;
    double bb = 0.0;
    EXX_PFOR(k, npe) {
      const double v = bx[k];
      bb += v * v;
      if (padded) {   // padding slots, which no sweep writes, hold zero
        y[k] = 0.0f;
#pragma unroll
        for (int i = 0; i < kPcgRing; ++i) W.p0[i * a.sstride + k] = 0.0f;
      }
    }
    bb = uniform(block_sum(bb, red));
    const double bnorm = sqrt(bb);
    const double inv_b = bnorm > 0.0 ? 1.0 / bnorm : 0.0;

    int it = 0, upd = 0, rst = 0, code = kCgConverged;
    double rr = 1.0, rr_true = bb, rmax = 1.0, rz = 0.0;
    bool first = true, x_zero = true, y_zero = true;
    bool conv = bnorm == 0.0;
    if (!conv && !(bnorm < INFINITY)) code = kCgNonFinite;   // b holds a NaN or an infinity
    // need: what the recursion lacks before its next sweep: 0 nothing, 1 the
    // residual of x = 0 (b / ||b||) and its restriction, 2 the FP64 true
    // residual of x and its restriction
    int need = 1;
    if (!conv && code == kCgConverged && warm_gather<double>(a, C, pid, x)) {
      __syncthreads();
      x_zero = false;
      need = 2;
    }
    PRing ring;
    double alpha = 0.0, pq = 0.0, qq = 0.0;
    PDir dir;
    while (!conv && code == kCgConverged) {
      bool step = !first;   // the coarse residuals follow the last ones
      if (need != 0) {
        EXX_PFOR(k, a.pcg_lds) fl[k] = 0.0f;   // the FP32 and FP64 plane views share LDS
        if (need == 1)
          EXX_PFOR(k, npe) W.r[k] = (float)(bx[k] * inv_b);
        __syncthreads();
        if (need == 1) {
          pcg_pass_r<CPT, NT, CC, float, GEN>(M, cl, ck, pst, cst, Zmax, W.r, W.vec(a, 0, 0, true), W.off(W.c1), W.off(W.b2), L);
          rr_true = bb;
        } else {
          double t;
          const int pl2 = a.pcg_planes == 2 ? plane : 0;
          if constexpr (TL)
            t = pcg_residual_tl<NS, CPT, NT, CC, float>(a, M, cl, ck, pst, cst, Zmax, x, bx, W.r, inv_b, lds, pl2,
                                                        W.vec(a, 0, 0, true), W.off(W.c1), W.off(W.b2), L);
          else
            t = pcg_residual<NS, CPT, NT, GEN, CC, float>(a, M, cl, ck, pst, cst, Zmax, x, bx, W.r, inv_b, lds, pl2,
                                                          W.vec(a, 0, 0, true), W.off(W.c1), W.off(W.b2), L);
          rr_true = uniform(block_sum(t, red));
        }
        EXX_PFOR(k, a.pcg_lds) fl[k] = 0.0f;
        __syncthreads();
        need = 0;
        y_zero = true;
        rr = rr_true * inv_b * inv_b;
        rmax = sqrt(rr);
        if (sqrt(rr_true) <= a.tol * bnorm) conv = true;
        if (!(rr < INFINITY)) code = kCgNonFinite;   // the FP64 solution itself is not finite
        if (conv || code != kCgConverged || it >= a.max_iter) break;
      }
      double t[4];
      pcg_coarse<NT, float>(C.mg, a.wl, fl, W.c1, W.g1, W.e1, W.b2, W.g2, step, (float)alpha, t);
      block_sum4(t, red);
      const double re = uniform(t[0]);
      if (first)
        dir = PDir();
      else
        dir.next(a.wl[0], alpha, pq, qq, uniform(t[1]), uniform(t[2]));
      if (ring.n == kPcgRing) {
        pcg_flush<NT, float, float>(y, y_zero, 1.0, nullptr, ring, W.p0, a.sstride, npe);
        __syncthreads();
        y_zero = false;
        ring.lo = ring.n = 0;
      }
      const PVec V = W.vec(a, (ring.n + kPcgRing - 1) % kPcgRing, ring.n, first);
      const PSums s = pcg_sweep<NS, CPT, NT, GEN, TL, RQ, CC, float>(a, S32, a.G32, M, cl, ck, pst, cst, Zmax, V,
                                                                     (float)a.wl[0], (float)alpha, (float)dir.beta, L);
      double v[4] = {s.rr, s.pq, s.qq, 0.0};
      block_sum4(v, red);
      const double rrn = uniform(v[0]);
      if (!first) dir.measured(a.wl[0], alpha, pq, qq, rr, rrn);
      rr = rrn;
      rz = a.wl[0] * rr + re;
      pq = uniform(v[1]);
      qq = uniform(v[2]);
      if (!first) ++it;
      int bad = kCgConverged;
      if (!(rr == rr) || !(rr < INFINITY))
        bad = kCgNonFinite;
      else if (!(pq > 0.0) || !(pq < INFINITY) || !(rz > 0.0) || !(rz < INFINITY))
        bad = kCgBreakdown;
      const double rnorm = sqrt(rr);
      if (bad != kCgConverged) {
        // restart from the last FP64 solution (steepest descent from its
        // residual); the FP32 correction is dropped
        if (rst >= kCgMaxRestarts) {
          code = bad;
          break;
        }
        ++rst;
        first = true;
        alpha = 0.0;
        ring.lo = ring.n = 0;
        need = x_zero ? 1 : 2;
        continue;
      }
      if (!first && (rnorm < delta * rmax || rnorm <= a.tol || it >= a.max_iter)) {
        // reliable update: the FP32 correction folded into the FP64 solution,
        // x = x + ||b|| y, with the deferred step
        pcg_flush<NT, double, float>(x, x_zero, bnorm, y_zero ? nullptr : y, ring, W.p0, a.sstride, npe);
        ring.lo = ring.n;
        x_zero = false;
        ++upd;
        need = 2;
      }
      first = false;
      alpha = rz / pq;
      ring.push(alpha);
    }
    if (!conv && code == kCgConverged) code = kCgCap;
    // the FP64 solution replaces the right-hand side
    __syncthreads();
    if (!x_zero) {
      EXX_PFOR(k, npe) bx[k] = x[k];
    } else if (bnorm > 0.0) {
      EXX_PFOR(k, npe) bx[k] = 0.0;
    }
    __syncthreads();
    warm_store_solution(a, npe, pid, bx);
    if (threadIdx.x == 0) {
      a.outIt[pid] = it;
      a.outRes[pid] = bnorm > 0.0 ? sqrt(rr_true) / bnorm : 0.0;
      a.outUpd[pid] = upd;
      a.outSav[pid] = RQ ? 5 * it / 4 : it / 4;   // five and a half, seven and a half accesses an iteration
      a.outExit[pid] = code | (rst << 8);
    }
    __syncthreads();
  }
}

template <int NS, int CPT, int NT, bool GEN, bool TL, bool MIXED>
hipError_t pcg_instance_g(const SolveKArgs& a, int groups, size_t lds, hipStream_t s, int* occ) {
  const void* fn;
  if constexpr (MIXED)
    fn = (const void*)k_pcg_mixed<NS, CPT, NT, GEN, TL>;
  else
    fn = (const void*)k_pcg<NS, CPT, NT, GEN, TL>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (occ) return hipOccupancyMaxActiveBlocksPerMultiprocessor(occ, fn, NT, lds);
  if constexpr (MIXED)
    k_pcg_mixed<NS, CPT, NT, GEN, TL><<<groups, NT, lds, s>>>(a);
  else
    k_pcg<NS, CPT, NT, GEN, TL><<<groups, NT, lds, s>>>(a);
  return hipGetLastError();
}

template <int NS, int CPT, int NT, bool MIXED>
hipError_t pcg_instance(const SolveKArgs& a, int groups, size_t lds, hipStream_t s, int* occ) {
  if (!a.gen) return pcg_instance_g<NS, CPT, NT, false, false, MIXED>(a, groups, lds, s, occ);
  if (a.G.n_tl > 0) return pcg_instance_g<NS, CPT, NT, true, true, MIXED>(a, groups, lds, s, occ);
  return pcg_instance_g<NS, CPT, NT, true, false, MIXED>(a, groups, lds, s, occ);
}

template <int NS, bool MIXED>
hipError_t pcg_dispatch(const SolveKArgs& a, int cols, int threads, int groups, size_t lds, hipStream_t s, int* occ) {
  switch (16 * threads + pcg_cpt(cols, threads)) {
    case 16 * 1024 + 1: return pcg_instance<NS, 1, 1024, MIXED>(a, groups, lds, s, occ);
    case 16 * 1024 + 2: return pcg_instance<NS, 2, 1024, MIXED>(a, groups, lds, s, occ);
    case 16 * 1024 + 3: return pcg_instance<NS, 3, 1024, MIXED>(a, groups, lds, s, occ);
    case 16 * 1024 + 4: return pcg_instance<NS, 4, 1024, MIXED>(a, groups, lds, s, occ);
    case 16 * 768 + 2: return pcg_instance<NS, 2, 768, MIXED>(a, groups, lds, s, occ);
    case 16 * 768 + 4: return pcg_instance<NS, 4, 768, MIXED>(a, groups, lds, s, occ);
    case 16 * 512 + 4: return pcg_instance<NS, 4, 512, MIXED>(a, groups, lds, s, occ);
    case 16 * 512 + 6: return pcg_instance<NS, 6, 512, MIXED>(a, groups, lds, s, occ);
    case 16 * 512 + 8: return pcg_instance<NS, 8, 512, MIXED>(a, groups, lds, s, occ);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace exx
