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

#include "solve_impl.h"

namespace exx {

// The scalars of a class's nested grids that the sweeps use, in scalar
// registers (every lane's value is the same: the class of the workgroup's pair).
struct MgU {
  int Z1, rw, rh, ew, eh;
  int cx, cy;           // LDS plane origin (the sphere's centre)
  int dx, dy;           // that of the restriction's plane is (cx - dx, cy - dy)
  int e0;               // level-1 plane position of the sphere's centre
  int d2x, d2xy, e2z;   // level-2 box: row, plane, and half-width along the sweep
};
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ MgU mg_uniform(const MgDev& M, int cx, int cy) {
  MgU u;
  u.Z1 = uniform(M.Z1);
  u.cx = cx;
  u.cy = cy;
  u.dx = cx - uniform(M.rcx);
  u.dy = cy - uniform(M.rcy);
  u.rw = uniform(M.rw);
  u.rh = uniform(M.rh);
  u.ew = uniform(M.ew);
  u.eh = uniform(M.eh);
  u.e0 = uniform(M.ex) + 1 + u.ew * (uniform(M.ey) + 1);
  u.d2x = uniform(M.D2[0]);
  u.d2xy = uniform(M.D2[0] * M.D2[1]);
  u.e2z = uniform(M.E2[2]);
  return u;
}

// Columns of the sphere owned by a thread, t, t + NT, ... of the class's real
// columns.  Only what the sweeps cannot recompute in an instruction or two is
// kept: the sweeps' windows need the registers.
template <int CPT, bool GEN>
struct PCols {
  int hi[CPT];              // the column's planes: -hi .. hi (hi -1: no column), or
  int lo_[GEN ? CPT : 1];   // lo .. hi in a general cell
  int col[CPT];             // slot within a plane
  int xy[CPT];              // LDS plane coordinates: x + cx | (y + cy) << 16
  // whether sweep plane z holds a point of column c (in an orthorhombic cell
  // one comparison with a scalar), and whether c is a column at all
  __device__ __forceinline__ bool valid(int c, int z) const {
    if constexpr (GEN)
      return z >= lo_[c] && z <= hi[c];
    else
      return abs(z) <= hi[c];
  }
  __device__ __forceinline__ bool has(int c) const {
    if constexpr (GEN)
      return lo_[c] <= hi[c];
    else
      return hi[c] >= 0;
  }
};

template <int CPT, int NT, bool GEN>
__device__ __forceinline__ void pcg_cols(const ClassDev& C, int cx, int cy, PCols<CPT, GEN>& cl) {
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int k = threadIdx.x + c * NT;
    cl.hi[c] = -1;
    if constexpr (GEN) cl.lo_[c] = 1;
    cl.col[c] = 0;
    cl.xy[c] = 0;
    if (k < C.n_fin) {
      const int4 f = C.fin_cols[k];
      const int x = GEN ? (int)(short)(f.w & 0xffff) : f.z;
      const int y = GEN ? (f.w >> 16) : f.w;
      cl.col[c] = f.x;
      if constexpr (GEN) cl.lo_[c] = f.y;
      cl.hi[c] = GEN ? f.z : f.y;
      cl.xy[c] = (x + cx) | ((y + cy) << 16);
    }
  }
}

// A value the compiler may not carry across loop steps: what is computed from
// it (LDS addresses, a few integer instructions) is formed again where it is
// used.  Kept over a sweep, those addresses cost more registers than the
// sweep has, and the plane loops spilled to scratch memory (FP64, 2,957
// columns, 2,356 pairs: 218 ms against 166 ms, with PBase's scalar bases).
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

#define EXX_PX(v) ((v) & 0xffff)
#define EXX_PY(v) ((v) >> 16)
#define EXX_PVALID(c, zz) cl.valid(c, zz)
#define EXX_PHAS(c) cl.has(c)
#define EXX_PIDX(c, base) ((base) + (unsigned)cl.col[c])
// LDS plane position, and the one in the restriction's plane
__device__ __forceinline__ int pcg_pos(int xy) {
  xy = fresh(xy);
  return EXX_PX(xy) + kLdsWX * EXX_PY(xy);
}
__device__ __forceinline__ int pcg_pos1(const MgU& M, int xy) {
  xy = fresh(xy);
  return (EXX_PX(xy) - M.dx) + M.rw * (EXX_PY(xy) - M.dy);
}
#define EXX_PPOS(c) pcg_pos(cl.xy[c])
#define EXX_PR1(c) pcg_pos1(M, cl.xy[c])

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

// A thread's level-1 columns (CC of them) and its level-2 column.
template <int CC>
struct PCoarse {
  int lo[CC], hi[CC];
  int r1[CC];       // position of the column's centre in the staged plane of the sphere
  int ep[CC];       // position in the staged level-1 plane
  int lo2, hi2, r2; // level-2 column: its interval and centre in the staged level-1 plane
  int b2;           // its position in a plane of the level-2 box
};

template <int CC, int NT>
__device__ __forceinline__ void pcg_coarse_cols(const ClassDev& C, PCoarse<CC>& k) {
  const MgDev& M = C.mg;
  const int t = threadIdx.x;
#pragma unroll
  for (int u = 0; u < CC; ++u) {
    k.lo[u] = 1;
    k.hi[u] = 0;
    k.r1[u] = M.rw + 1;
    k.ep[u] = 0;
    const int i = t + u * NT;
    if (i < M.n_c1) {
      const int4 f = M.c1cols[i];
      k.lo[u] = f.z;
      k.hi[u] = f.w;
      k.r1[u] = (2 * f.x + M.rcx) + M.rw * (2 * f.y + M.rcy);
      k.ep[u] = (f.x + M.ex + 1) + M.ew * (f.y + M.ey + 1);
    }
  }
  k.lo2 = 1;
  k.hi2 = 0;
  k.r2 = M.ew + 1;
  k.b2 = 0;
  if (t < M.n_c2) {
    const int4 f = M.c2cols[t];
    k.lo2 = f.z;
    k.hi2 = f.w;
    k.r2 = (2 * f.x + M.ex + 1) + M.ew * (2 * f.y + M.ey + 1);
    k.b2 = (f.x + M.E2[0] + 1) + M.D2[0] * (f.y + M.E2[1] + 1);
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
__device__ __forceinline__ T prolong4(const T* E, int xy, const MgU& M) {
  xy = fresh(xy);
  const int x = EXX_PX(xy) - M.cx, y = EXX_PY(xy) - M.cy;
  const T* b = E + ((x >> 1) + M.ew * (y >> 1) + M.e0);
  const int dx = x & 1, dy = (y & 1) ? M.ew : 0;
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

// The restriction streamed with a pass B.  `done` is called with the sweep
// plane z just finished (before its barrier's successor): column sums in acc.
template <int CC, typename T>
struct PRestrict {
  T acc2[CC];
};

// Level-1 and level-2 part of one sweep step (after its barrier).  z is the
// step's centre plane; the combination staged at the odd plane z - 1 completes
// level-1 plane (z - 2) / 2.
template <int CC, int NT, typename T>
__device__ __forceinline__ void pcg_restrict_step(const MgU& M, const PCoarse<CC>& k, const PLds<T>& L,
                                                  const int* cst, int z, PRestrict<CC, T>& R, T* c1, T* b2) {
  if (!(z & 1)) {
    const int kz = (z - 2) >> 1;
    if (kz >= -M.Z1 && kz <= M.Z1 + 1) {
      const bool fin = kz & 1;   // completes a level-2 plane
      const unsigned base = kz <= M.Z1 ? plane_base(cst, kz + M.Z1) : 0u;
#pragma unroll
      for (int u = 0; u < CC; ++u) {
        if (u > 0 && k.lo[u] > k.hi[u]) continue;
        T v = 0;
        if (kz >= k.lo[u] && kz <= k.hi[u]) {
          v = restrict9<T>(L.R1 + fresh(k.r1[u]), M.rw);
          gstore(c1, base + (unsigned)(threadIdx.x + u * NT), v);
        }
        if (fin) {
          if (k.lo[u] <= k.hi[u]) L.R2[fresh(k.ep[u])] = R.acc2[u] + (T)0.5 * v;
          R.acc2[u] = (T)0.5 * v;
        } else {
          R.acc2[u] += v;
        }
      }
    }
  } else {
    const int kz = (z - 3) >> 1;   // level-1 plane of the previous step
    if ((kz & 1) && kz >= -M.Z1 && kz <= M.Z1 + 1) {
      const int k2 = (kz - 1) >> 1;
      if (k2 >= k.lo2 && k2 <= k.hi2) b2[k.b2 + M.d2xy * (k2 + M.e2z + 1)] = restrict9<T>(L.R2 + fresh(k.r2), M.ew);
    }
  }
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
// plane's and the barrier, so one register set holds them.  pn receives the
// new p.  first: p = w_0 r + P e, nothing else read.
template <int NS, int CPT, int NT, bool GEN, int CC, typename T>
__device__ __forceinline__ PSums pcg_sweep_w(const StencilT<T>& S, const GenStencilT<T>& G, const MgU& M,
                                             const PCols<CPT, GEN>& cl, const PCoarse<CC>& ck, const int* pst,
                                             const int* cst, int Zmax, T* r, T* q, const T* p, T* pn,
                                             const T* __restrict__ e1, T w0, T alpha, T beta, bool first,
                                             T* g1, T* g2, const PLds<T>& L) {
  T win[CPT][2 * NS + 1];
  T lr[CPT], lp[CPT], lq[CPT], Bc[CPT], acc[CPT], ev[CC];
  PRestrict<CC, T> R;
  PSums s{0.0, 0.0, 0.0};
  // an even plane below the first one: its step stages the level-1 plane that
  // the next (odd) step interpolates
  const int z0 = -Zmax - 2 + (Zmax & 1);
  const int zl = pcg_last_step(M, Zmax) + NS;
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    lr[c] = lp[c] = lq[c] = Bc[c] = acc[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) win[c][k] = 0;
  }
  auto load_e = [&](int kz) {
    const unsigned base = PBase<1>::at(cst, M.Z1, kz) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < CC; ++u) {
      ev[u] = 0;
      if (kz >= ck.lo[u] && kz <= ck.hi[u]) ev[u] = gload(e1, base + u * NT);
    }
  };
  load_e((z0 + 2) >> 1);
  PBase<NS + 2> pb(pst, Zmax, z0 - NS);   // planes zc - NS .. zc + 1
  for (int zc = z0; zc <= zl; ++zc) {
    const int z = zc - NS;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      T pe = Bc[c];
      if (zc & 1) {
        const T Bn = EXX_PHAS(c) ? prolong4<T>(L.E, cl.xy[c], M) : (T)0;
        pe = (T)0.5 * (pe + Bn);
        Bc[c] = Bn;
      }
#pragma unroll
      for (int k = 0; k < 2 * NS; ++k) win[c][k] = win[c][k + 1];
      T v = 0;
      if (EXX_PVALID(c, zc)) {
        const unsigned idx = EXX_PIDX(c, pb.b[NS]);
        T rn = lr[c];
        if (!first) {
          rn -= alpha * lq[c];
          gstore(r, idx, rn);
        }
        v = w0 * rn + pe;
        if (!first) v += beta * lp[c];
        gstore(pn, idx, v);
        s.rr += (double)rn * (double)rn;
      }
      win[c][2 * NS] = v;
      lr[c] = lp[c] = lq[c] = 0;
      if (EXX_PVALID(c, zc + 1)) {
        const unsigned idx = EXX_PIDX(c, pb.b[NS + 1]);
        lr[c] = gload(r, idx);
        if (!first) {
          lp[c] = gload(p, idx);
          lq[c] = gload(q, idx);
        }
      }
    }
    T* pl = L.pl0 + ((z & 1) ? L.plane : 0);
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (EXX_PHAS(c)) pl[EXX_PPOS(c)] = win[c][NS];
    if (!(zc & 1)) {   // level-1 plane (zc + 2) / 2, interpolated in the next step
#pragma unroll
      for (int u = 0; u < CC; ++u)
        if (ck.lo[u] <= ck.hi[u]) L.E[fresh(ck.ep[u])] = ev[u];
    }
    __syncthreads();
    if (zc & 1) load_e((zc + 3) >> 1);
    if (z >= -Zmax) pcg_restrict_step<CC, NT, T>(M, ck, L, cst, z, R, g1, g2);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      T qv = 0;
      if (EXX_PVALID(c, z)) {
        qv = pcg_apply<NS, GEN, T>(S, G, win[c][NS], pl, EXX_PPOS(c), win[c]);
        gstore(q, EXX_PIDX(c, pb.b[0]), qv);
        s.pq += (double)win[c][NS] * (double)qv;
        s.qq += (double)qv * (double)qv;
      }
      if (z & 1) {
        const T h = (T)0.5 * qv;
        if (EXX_PHAS(c)) L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += qv;
      }
    }
    pb.next(pst, Zmax, zc - NS);
    if (L.plane == 0) __syncthreads();   // one plane: its readers are done
  }
  __syncthreads();
  return s;
}

// The window form without a stored q: q of the direction before is formed again
// from p, whose plane zc is staged with the new direction's plane z.  Five and a
// half accesses per point for a second stencil: the choice where the registers
// hold both windows (FP32 with 512 or 768 threads).
template <int NS, int CPT, int NT, bool GEN, int CC, typename T>
__device__ __forceinline__ PSums pcg_sweep_rq(const StencilT<T>& S, const GenStencilT<T>& G, const MgU& M,
                                              const PCols<CPT, GEN>& cl, const PCoarse<CC>& ck, const int* pst,
                                              const int* cst, int Zmax, T* r, const T* p, T* pn,
                                              const T* __restrict__ e1, T w0, T alpha, T beta, bool first, T* g1, T* g2,
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
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    lr[c] = Bc[c] = acc[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) {
      wn[c][k] = 0;
      const int zz = z0 - NS - 1 + k;
      wo[c][k] = 0;
      if (k > NS && !first && EXX_PVALID(c, zz)) wo[c][k] = gload(p, EXX_PIDX(c, pb.b[k > 0 ? k - 1 : 0]));
    }
    lp[c] = !first && EXX_PVALID(c, z0 + NS) ? gload(p, EXX_PIDX(c, pb.b[2 * NS])) : (T)0;
  }
  auto load_e = [&](int kz) {
    const unsigned base = PBase<1>::at(cst, M.Z1, kz) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < CC; ++u) {
      ev[u] = 0;
      if (kz >= ck.lo[u] && kz <= ck.hi[u]) ev[u] = gload(e1, base + u * NT);
    }
  };
  load_e((z0 + 2) >> 1);
  for (int zc = z0; zc <= zl; ++zc) {
    const int z = zc - NS;
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
      lp[c] = 0;
      if (!first && EXX_PVALID(c, zc + NS + 1)) lp[c] = gload(p, EXX_PIDX(c, pb.b[2 * NS + 1]));
      if (EXX_PHAS(c)) {
        const int pos = EXX_PPOS(c);
        po[pos] = wo[c][NS];
        pl[pos] = wn[c][NS];
      }
      pe[c] = Bc[c];
      if (zc & 1) {
        const T Bn = EXX_PHAS(c) ? prolong4<T>(L.E, cl.xy[c], M) : (T)0;
        pe[c] = (T)0.5 * (pe[c] + Bn);
        Bc[c] = Bn;
      }
    }
    if (!(zc & 1)) {   // level-1 plane (zc + 2) / 2, interpolated in the next step
#pragma unroll
      for (int u = 0; u < CC; ++u)
        if (ck.lo[u] <= ck.hi[u]) L.E[fresh(ck.ep[u])] = ev[u];
    }
    __syncthreads();
    if (zc & 1) load_e((zc + 3) >> 1);
    if (z >= -Zmax) pcg_restrict_step<CC, NT, T>(M, ck, L, cst, z, R, g1, g2);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      T v = 0;
      if (EXX_PVALID(c, zc)) {
        const unsigned idx = EXX_PIDX(c, pb.b[NS]);
        T rn = lr[c];
        if (!first) {
          rn -= alpha * pcg_apply<NS, GEN, T>(S, G, wo[c][NS], po, EXX_PPOS(c), wo[c]);
          gstore(r, idx, rn);
        }
        v = w0 * rn + pe[c];
        if (!first) v += beta * wo[c][NS];
        gstore(pn, idx, v);
        s.rr += (double)rn * (double)rn;
      }
      wn[c][2 * NS] = v;
      lr[c] = EXX_PVALID(c, zc + 1) ? gload(r, EXX_PIDX(c, pb.b[NS + 1])) : (T)0;
      T qv = 0;
      if (EXX_PVALID(c, z)) {
        qv = pcg_apply<NS, GEN, T>(S, G, wn[c][NS], pl, EXX_PPOS(c), wn[c]);
        s.pq += (double)wn[c][NS] * (double)qv;
        s.qq += (double)qv * (double)qv;
      }
      if (z & 1) {
        const T h = (T)0.5 * qv;
        if (EXX_PHAS(c)) L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += qv;
      }
    }
    pb.next(pst, Zmax, zc - NS);
    if (L.plane == 0) __syncthreads();   // one plane: its readers are done
  }
  __syncthreads();
  return s;
}

// The same with arms leaving the sweep plane: a plane of the new p is staged
// as it enters and scattered into the partial sums of its columns' points; the
// point n planes behind completes (see cg_pass_a_tl).
template <int NS, int CPT, int NT, int CC, typename T, bool GEN = true>
__device__ __forceinline__ PSums pcg_sweep_tl(const GenStencilT<T>& G, const MgU& M, const PCols<CPT, GEN>& cl,
                                              const PCoarse<CC>& ck, const int* pst, const int* cst, int Zmax,
                                              T* r, T* q, const T* p, T* pn, const T* __restrict__ e1, T w0, T alpha,
                                              T beta, bool first, T* g1, T* g2, const PLds<T>& L) {
  T pd[CPT][NS + 1], sum[CPT][2 * NS + 1];
  T lr[CPT], lp[CPT], lq[CPT], Bc[CPT], acc[CPT], ev[CC];
  PRestrict<CC, T> R;
  PSums s{0.0, 0.0, 0.0};
  const int z0 = -Zmax - 2 + (Zmax & 1);
  const int zl = pcg_last_step(M, Zmax) + NS;
#pragma unroll
  for (int u = 0; u < CC; ++u) R.acc2[u] = 0;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    lr[c] = lp[c] = lq[c] = Bc[c] = acc[c] = 0;
#pragma unroll
    for (int k = 0; k < 2 * NS + 1; ++k) sum[c][k] = 0;
#pragma unroll
    for (int k = 0; k < NS + 1; ++k) pd[c][k] = 0;
  }
  auto load_e = [&](int kz) {
    const unsigned base = PBase<1>::at(cst, M.Z1, kz) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < CC; ++u) {
      ev[u] = 0;
      if (kz >= ck.lo[u] && kz <= ck.hi[u]) ev[u] = gload(e1, base + u * NT);
    }
  };
  load_e((z0 + 2) >> 1);
  PBase<NS + 2> pb(pst, Zmax, z0 - NS);   // planes zc - NS .. zc + 1
  for (int zc = z0; zc <= zl; ++zc) {
    const int z = zc - NS;
    T* pl = L.pl0 + ((zc & 1) ? L.plane : 0);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      T pe = Bc[c];
      if (zc & 1) {
        const T Bn = EXX_PHAS(c) ? prolong4<T>(L.E, cl.xy[c], M) : (T)0;
        pe = (T)0.5 * (pe + Bn);
        Bc[c] = Bn;
      }
#pragma unroll
      for (int k = 0; k < NS; ++k) pd[c][k] = pd[c][k + 1];
      T v = 0;
      if (EXX_PVALID(c, zc)) {
        const unsigned idx = EXX_PIDX(c, pb.b[NS]);
        T rn = lr[c];
        if (!first) {
          rn -= alpha * lq[c];
          gstore(r, idx, rn);
        }
        v = w0 * rn + pe;
        if (!first) v += beta * lp[c];
        gstore(pn, idx, v);
        s.rr += (double)rn * (double)rn;
      }
      pd[c][NS] = v;
      if (EXX_PHAS(c)) pl[EXX_PPOS(c)] = v;
      lr[c] = lp[c] = lq[c] = 0;
      if (EXX_PVALID(c, zc + 1)) {
        const unsigned idx = EXX_PIDX(c, pb.b[NS + 1]);
        lr[c] = gload(r, idx);
        if (!first) {
          lp[c] = gload(p, idx);
          lq[c] = gload(q, idx);
        }
      }
    }
    if (!(zc & 1)) {   // level-1 plane (zc + 2) / 2, interpolated in the next step
#pragma unroll
      for (int u = 0; u < CC; ++u)
        if (ck.lo[u] <= ck.hi[u]) L.E[fresh(ck.ep[u])] = ev[u];
    }
    __syncthreads();
    if (zc & 1) load_e((zc + 3) >> 1);
    if (z >= -Zmax) pcg_restrict_step<CC, NT, T>(M, ck, L, cst, z, R, g1, g2);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      if (EXX_PHAS(c) && zc <= Zmax + NS)
        tl_scatter<NS, T>(G, pd[c][NS], EXX_PVALID(c, zc), pl, EXX_PPOS(c), sum[c]);
      T qv = 0;
      if (EXX_PVALID(c, z)) {
        qv = -sum[c][0];
        gstore(q, EXX_PIDX(c, pb.b[0]), qv);
        s.pq += (double)pd[c][0] * (double)qv;
        s.qq += (double)qv * (double)qv;
      }
#pragma unroll
      for (int k = 0; k < 2 * NS; ++k) sum[c][k] = sum[c][k + 1];
      sum[c][2 * NS] = 0;
      if (z & 1) {
        const T h = (T)0.5 * qv;
        if (EXX_PHAS(c)) L.R1[EXX_PR1(c)] = acc[c] + h;
        acc[c] = h;
      } else {
        acc[c] += qv;
      }
    }
    pb.next(pst, Zmax, zc - NS);
    if (L.plane == 0) __syncthreads();   // one plane: its readers are done
  }
  __syncthreads();
  return s;
}

// The restriction of a residual that is not followed from the one before (the
// first one): the streamed part of the sweep alone.
template <int CPT, int NT, int CC, typename T, bool GEN>
__device__ __forceinline__ void pcg_pass_r(const MgU& M, const PCols<CPT, GEN>& cl, const PCoarse<CC>& ck, const int* pst,
                           const int* cst, int Zmax, const T* r, T* c1, T* b2, const PLds<T>& L) {
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
    pcg_restrict_step<CC, NT, T>(M, ck, L, cst, z, R, c1, b2);
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
template <int NS, int CPT, int NT, bool GEN, int CC, typename T>
__device__ __forceinline__ double pcg_residual(const SolveKArgs& a, const MgU& M, const PCols<CPT, GEN>& cl, const PCoarse<CC>& ck,
                               const int* pst, const int* cst, int Zmax, const double* __restrict__ x,
                               const double* __restrict__ b, T* __restrict__ r, double rs, double* pl0,
                               int plane, T* c1, T* b2, const PLds<T>& L) {
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
    pcg_restrict_step<CC, NT, T>(M, ck, L, cst, z, R, c1, b2);
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

template <int NS, int CPT, int NT, int CC, typename T, bool GEN = true>
__device__ __forceinline__ double pcg_residual_tl(const SolveKArgs& a, const MgU& M, const PCols<CPT, GEN>& cl, const PCoarse<CC>& ck,
                                  const int* pst, const int* cst, int Zmax, const double* __restrict__ x,
                                  const double* __restrict__ b, T* __restrict__ r, double rs, double* pl0,
                                  int plane, T* c1, T* b2, const PLds<T>& L) {
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
    if (zo >= -Zmax) pcg_restrict_step<CC, NT, T>(M, ck, L, cst, zo, R, c1, b2);
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
// thread's parts of r_1.e_1, e_1.g_1 of the e_1 before, and e_1.g_1.  The boxes lie in
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

template <int NS, int CPT, int NT, bool GEN, bool TL, bool RQ, int CC, typename T>
__device__ __forceinline__ PSums pcg_sweep(const StencilT<T>& S, const GenStencilT<T>& G, const MgU& M,
                                           const PCols<CPT, GEN>& cl, const PCoarse<CC>& ck, const int* pst,
                                           const int* cst, int Zmax, T* r, T* q, const T* p, T* pn, const T* e1, T w0,
                                           T alpha, T beta, bool first, T* g1, T* g2, const PLds<T>& L) {
  w0 = uniform(w0);
  alpha = uniform(alpha);
  beta = uniform(beta);
  if constexpr (TL)
    return pcg_sweep_tl<NS, CPT, NT, CC, T>(G, M, cl, ck, pst, cst, Zmax, r, q, p, pn, e1, w0, alpha, beta, first, g1,
                                            g2, L);
  else if constexpr (RQ)
    return pcg_sweep_rq<NS, CPT, NT, GEN, CC, T>(S, G, M, cl, ck, pst, cst, Zmax, r, p, pn, e1, w0, alpha, beta, first,
                                                 g1, g2, L);
  else
    return pcg_sweep_w<NS, CPT, NT, GEN, CC, T>(S, G, M, cl, ck, pst, cst, Zmax, r, q, p, pn, e1, w0, alpha, beta,
                                                first, g1, g2, L);
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
  const T w[kPcgRing] = {(T)uniform(R.a0), (T)uniform(R.a1), (T)uniform(R.a2), (T)uniform(R.a3)};
  for (int k0 = 0; k0 < npe; k0 += U * NT) {
    T s[U], v[U][kPcgRing];
    X xv[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int k = min(k0 + j * NT + (int)threadIdx.x, npe - 1);   // clamped: only the stores are conditional
      xv[j] = zero ? (X)0 : x[k];
      s[j] = y ? y[k] : (T)0;
#pragma unroll
      for (int i = 0; i < kPcgRing; ++i) v[j][i] = i >= R.lo && i < R.n ? p0[i * stride + k] : (T)0;
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
#pragma unroll
      for (int i = 0; i < kPcgRing; ++i) s[j] += w[i] * v[j][i];
      if (const int k = k0 + j * NT + (int)threadIdx.x; k < npe) x[k] = xv[j] + (X)scale * (X)s[j];
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
  __device__ __forceinline__ PSlot(T* base, const SolveKArgs& a) {
    r = base;
    q = r + a.sstride;
    p0 = q + a.sstride;
    c1 = p0 + kPcgRing * a.sstride;
    g1 = c1 + a.c1stride;
    e1 = g1 + a.c1stride;
    b2 = e1 + a.c1stride;
    g2 = b2 + a.b2stride;
  }
};

// FP64 solve: one workgroup per pair, as k_solve.
template <int NS, int CPT, int NT, bool GEN, bool TL>
__global__ __launch_bounds__(NT) void k_pcg(SolveKArgs a) {
  extern __shared__ double lds[];
  __shared__ double red[4 * (NT / 64)];
  __shared__ int s_item;
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
    const MgU M = mg_uniform(C.mg, a.lds_cx, a.lds_cy);
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
    PCols<CPT, GEN> cl;
    pcg_cols<CPT, NT, GEN>(C, a.lds_cx, a.lds_cy, cl);
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
    bb = uniform(block_sum(bb, red));
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
        double t;
        if constexpr (TL)
          t = pcg_residual_tl<NS, CPT, NT, CC, double>(a, M, cl, ck, pst, cst, Zmax, W.p0, x, W.r, 1.0, lds, L.plane,
                                                       W.c1, W.b2, L);
        else
          t = pcg_residual<NS, CPT, NT, GEN, CC, double>(a, M, cl, ck, pst, cst, Zmax, W.p0, x, W.r, 1.0, lds, L.plane,
                                                         W.c1, W.b2, L);
        rr = uniform(block_sum(t, red));
        EXX_PFOR(k, npe) x[k] = W.p0[k];
        x_zero = false;
        if (sqrt(rr) <= a.tol * bnorm) conv = true;
        if (!(rr < INFINITY)) code = kCgNonFinite;
        __syncthreads();
      } else {
        EXX_PFOR(k, npe) W.r[k] = x[k];
        __syncthreads();
        pcg_pass_r<CPT, NT, CC, double, GEN>(M, cl, ck, pst, cst, Zmax, W.r, W.c1, W.b2, L);
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
      double* pn = W.p0 + ring.n * a.sstride;
      const double* p = W.p0 + (ring.n + kPcgRing - 1) % kPcgRing * a.sstride;
      const PSums s = pcg_sweep<NS, CPT, NT, GEN, TL, false, CC, double>(a.S, a.G, M, cl, ck, pst, cst, Zmax, W.r, W.q, p, pn,
                                                                  W.e1, a.wl[0], alpha, dir.beta, first, W.g1, W.g2, L);
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
    const ClassDev& C = a.cls[uniform(a.pairs[pid].cls)];
    const MgU M = mg_uniform(C.mg, a.lds_cx, a.lds_cy);
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
    PCols<CPT, GEN> cl;
    pcg_cols<CPT, NT, GEN>(C, a.lds_cx, a.lds_cy, cl);
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
          pcg_pass_r<CPT, NT, CC, float, GEN>(M, cl, ck, pst, cst, Zmax, W.r, W.c1, W.b2, L);
          rr_true = bb;
        } else {
          double t;
          const int pl2 = a.pcg_planes == 2 ? plane : 0;
          if constexpr (TL)
            t = pcg_residual_tl<NS, CPT, NT, CC, float>(a, M, cl, ck, pst, cst, Zmax, x, bx, W.r, inv_b, lds, pl2,
                                                        W.c1, W.b2, L);
          else
            t = pcg_residual<NS, CPT, NT, GEN, CC, float>(a, M, cl, ck, pst, cst, Zmax, x, bx, W.r, inv_b, lds, pl2,
                                                          W.c1, W.b2, L);
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
      float* pn = W.p0 + ring.n * a.sstride;
      const float* p = W.p0 + (ring.n + kPcgRing - 1) % kPcgRing * a.sstride;
      const PSums s = pcg_sweep<NS, CPT, NT, GEN, TL, RQ, CC, float>(S32, a.G32, M, cl, ck, pst, cst, Zmax, W.r, W.q, p, pn,
                                                                 W.e1, (float)a.wl[0], (float)alpha, (float)dir.beta,
                                                                 first, W.g1, W.g2, L);
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
      if (!first && (rnorm < a.delta * rmax || rnorm <= a.tol || it >= a.max_iter)) {
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

// Columns per thread: up to 4 with 1024 and 768 threads, up to 8 with 512.
template <int NS, bool MIXED>
hipError_t pcg_dispatch(const SolveKArgs& a, int cols, int threads, int groups, size_t lds, hipStream_t s, int* occ) {
  const int cpt = (cols + threads - 1) / threads;
  if (threads == 1024) {
    switch (cpt) {
      case 1: return pcg_instance<NS, 1, 1024, MIXED>(a, groups, lds, s, occ);
      case 2: return pcg_instance<NS, 2, 1024, MIXED>(a, groups, lds, s, occ);
      case 3: return pcg_instance<NS, 3, 1024, MIXED>(a, groups, lds, s, occ);
      case 4: return pcg_instance<NS, 4, 1024, MIXED>(a, groups, lds, s, occ);
      default: return hipErrorInvalidValue;
    }
  }
  if (threads == 768) {
    if (cpt <= 2) return pcg_instance<NS, 2, 768, MIXED>(a, groups, lds, s, occ);
    if (cpt <= 4) return pcg_instance<NS, 4, 768, MIXED>(a, groups, lds, s, occ);
    return hipErrorInvalidValue;
  }
  if (threads == 512) {
    if (cpt <= 4) return pcg_instance<NS, 4, 512, MIXED>(a, groups, lds, s, occ);
    if (cpt <= 6) return pcg_instance<NS, 6, 512, MIXED>(a, groups, lds, s, occ);
    if (cpt <= 8) return pcg_instance<NS, 8, 512, MIXED>(a, groups, lds, s, occ);
  }
  return hipErrorInvalidValue;
}

}  // namespace exx
