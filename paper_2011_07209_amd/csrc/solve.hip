// Launchers of the persistent CG solve (the instances live in solve_n*.hip).
#include <algorithm>
#include <cstring>

#include "solve_impl.h"

namespace exx {

hipError_t solve_dispatch_n1(const SolveKArgs& a, bool mixed, int max_cols, int threads, int depth, int groups,
                             size_t lds, hipStream_t s, int* occ);
hipError_t solve_dispatch_n2(const SolveKArgs& a, bool mixed, int max_cols, int threads, int depth, int groups,
                             size_t lds, hipStream_t s, int* occ);
hipError_t solve_dispatch_n3(const SolveKArgs& a, bool mixed, int max_cols, int threads, int depth, int groups,
                             size_t lds, hipStream_t s, int* occ);

// The preconditioned CG's instances (pcg_n*.hip).
#define EXX_PCG_DECL(name) \
  hipError_t name(const SolveKArgs& a, int cols, int threads, int groups, size_t lds, hipStream_t s, int* occ)
EXX_PCG_DECL(pcg_n1_f64);
EXX_PCG_DECL(pcg_n2_f64);
EXX_PCG_DECL(pcg_n3_f64);
EXX_PCG_DECL(pcg_n1_mixed);
EXX_PCG_DECL(pcg_n2_mixed);
EXX_PCG_DECL(pcg_n3_mixed);
#undef EXX_PCG_DECL

// Two plane buffers, then the plane offsets of the class, with room for the
// sweeps' look-ahead reads a few planes past the last one (their values are
// discarded).
size_t solve_lds_bytes(const Geo& g, int max_zmax) {
  return (size_t)2 * kLdsWX * g.lds_wy * sizeof(double) + (size_t)(2 * max_zmax + 2 + 8) * sizeof(int);
}

long long solve_slot_bytes(bool mixed, long long sstride) {
  const long long b = mixed ? 24 * sstride : 16 * sstride;
  return (b + 255) & ~255LL;
}

// Elements of the preconditioned CG's LDS buffers: one or two planes (mixed:
// FP64 ones, whose FP32 views the sweeps use), the restriction's plane of the
// sphere and two level-1 planes; or the coarse phase's three boxes where they
// are more.
static long long pcg_lds_elems(const Geo& g, const MgDev& M, bool mixed, int planes) {
  const long long sweep = (mixed ? 2LL : 1LL) * planes * kLdsWX * g.lds_wy + (long long)M.rw * M.rh +
                          2LL * M.ew * M.eh;
  auto box = [](const int* D) { return (long long)D[0] * D[1] * D[2]; };
  const long long e = std::max(sweep, box(M.D2) + box(M.D3) + box(M.D4));
  return (e + 1) / 2 * 2;
}

static int pcg_ints(int zmax) { return 2 * zmax + 2 + 8; }

static size_t pcg_lds_bytes(const Geo& g, const MgDev& M, int zmax, bool mixed, int planes) {
  return (size_t)pcg_lds_elems(g, M, mixed, planes) * (mixed ? 4 : 8) +
         (size_t)(pcg_ints(zmax) + 2 * M.Z1 + 2 + 8) * sizeof(int);
}

// Two planes where they fit the CU's 160 KB (1 KB for the kernels' static LDS),
// one (a second barrier a plane) where only that does, else 0.
static int pcg_planes(const Geo& g, const MgDev& M, int zmax, bool mixed) {
  for (int planes = 2; planes >= 1; --planes)
    if (pcg_lds_bytes(g, M, zmax, mixed, planes) + 1024 <= 160 * 1024) return planes;
  return 0;
}

MgDev pcg_join(const MgDev& a, const MgDev& b) {
  MgDev m = a;
  m.Z1 = std::max(a.Z1, b.Z1);
  m.rw = std::max(a.rw, b.rw);
  m.rh = std::max(a.rh, b.rh);
  m.ew = std::max(a.ew, b.ew);
  m.eh = std::max(a.eh, b.eh);
  for (int k = 0; k < 3; ++k) {
    m.D2[k] = std::max(a.D2[k], b.D2[k]);
    m.D3[k] = std::max(a.D3[k], b.D3[k]);
    m.D4[k] = std::max(a.D4[k], b.D4[k]);
  }
  return m;
}

bool pcg_joins(const Geo& g, const MgDev& joined, const MgDev& one, int zmax, bool mixed) {
  const int planes = pcg_planes(g, joined, zmax, mixed);
  return planes > 0 && planes == pcg_planes(g, one, zmax, mixed);
}

long long pcg_slot_bytes(bool mixed, long long sstride, long long c1stride, long long b2stride) {
  // r, q and the ring of p; the mixed solve's x (FP64) and y
  const long long b = (mixed ? 12 * sstride : 0) +
                      (mixed ? 4 : 8) * ((2 + kPcgRing) * sstride + 3 * c1stride + 2 * b2stride);
  return (b + 255) & ~255LL;
}

// (the columns of each level one or two to a thread, and what the kernels pack
// into 16, 14, 13, 12 and 6 bits: see PCols and PCoarse)
bool pcg_supported(const Geo& g, const ClassHost& C, bool mixed) {
  const MgDev& M = C.mg;
  return M.n_c1 > 0 && M.n_c1 <= 1024 && M.n_c2 <= 512 && C.n_cols <= 4096 && (int)C.fin_cols.size() <= 4096 &&
         (long long)kLdsWX * g.lds_wy <= 8192 && C.Zmax < 126 && (long long)M.rw * M.rh <= 32768 &&
         (long long)M.ew * M.eh <= 16384 && (long long)M.D2[0] * M.D2[1] <= 32768 &&
         pcg_planes(g, C.mg, C.Zmax, mixed) > 0;
}

static hipError_t solve_dispatch(const SolveArgs& in, int max_cols, int max_zmax, int groups, hipStream_t s,
                                 int* occ) {
  SolveKArgs a;
  a.cls = in.cls;
  a.pairs = in.pairs;
  a.order = in.order;
  a.p0 = in.p0;
  a.npair = in.npair;
  a.n_eff = in.n_eff;
  a.warm_store = in.warm_store;
  a.warm_cap = in.warm_cap;
  a.warm_state = in.warm_state;
  a.warm_map = in.warm_map;
  a.prev_pairs = in.prev_pairs;
  a.n = in.g.n;
  for (int ax = 0; ax < 3; ++ax) a.N[ax] = in.g.N[ax];
  a.cls_id = in.cls_id;
  a.cls_lo = in.cls_lo >= 0 ? in.cls_lo : in.cls_id;
  a.class_cnt = in.class_cnt;
  a.ncls = in.ncls;
  a.queue = in.queue;
  a.bx_ws = in.bx_ws;
  a.rstride = in.rstride;
  a.slot_ws = in.slot_ws;
  a.sstride = in.sstride;
  a.slot_bytes = solve_slot_bytes(in.mixed, in.sstride);
  a.outIt = in.outIt;
  a.outRes = in.outRes;
  a.outUpd = in.outUpd;
  a.outSav = in.outSav;
  a.outExit = in.outExit;
  a.tol = in.tol;
  a.max_iter = in.max_iter;
  a.delta = in.delta;
  for (int q = 0; q < 4; ++q) a.S.w[q] = in.g.w2[q];
  for (int al = 0; al < 3; ++al) a.S.c[al] = in.g.inv_d2[al];
  a.S.diag = in.g.w2[0] * (a.S.c[0] + a.S.c[1] + a.S.c[2]);
  a.S.cd = 0.0;
  a.S.sd = 0;
  if (in.g.gen && in.quads) {
    // a general cell in the quad layout: its arms in the CG frame are the x',
    // y' and z' axes and at most one diagonal of the sweep plane
    double c[3] = {0.0, 0.0, 0.0}, sum = 0.0;
    for (int m = 0; m < in.g.n_arms; ++m) {
      const int ux = in.g.arm_u[m][in.g.perm[0]], uy = in.g.arm_u[m][in.g.perm[1]], uz = in.g.arm_u[m][in.g.perm[2]];
      const double cf = in.g.arm_coef[m];
      sum += cf;
      if (uz != 0) {
        if (ux != 0 || uy != 0) return hipErrorInvalidValue;
        c[2] += cf;
      } else if (ux != 0 && uy != 0) {
        if (a.S.sd != 0 || (ux != 1 && ux != -1) || (uy != 1 && uy != -1)) return hipErrorInvalidValue;
        a.S.cd = cf;
        a.S.sd = ux * uy;   // oriented so that one step raises x' by one
      } else if (ux != 0) {
        c[0] += cf;
      } else {
        c[1] += cf;
      }
    }
    for (int al = 0; al < 3; ++al) a.S.c[al] = c[al];
    a.S.diag = in.g.w2[0] * sum;
  }
  // general cell: the NK arms in the CG frame (x', y', z') = o[perm]
  a.gen = in.g.gen;
  a.quads = in.quads ? 1 : 0;
  std::memset(&a.G, 0, sizeof(a.G));
  if (a.gen) {
    for (int q = 0; q < 4; ++q) a.G.w[q] = in.g.w2[q];
    double sum = 0.0;
    for (int m = 0; m < in.g.n_arms; ++m) {
      const int ux = in.g.arm_u[m][in.g.perm[0]], uy = in.g.arm_u[m][in.g.perm[1]], uz = in.g.arm_u[m][in.g.perm[2]];
      const double cf = in.g.arm_coef[m];
      sum += cf;
      if (ux == 0 && uy == 0) {
        a.G.cz += cf;
      } else if (uz == 0) {
        if (a.G.n_in == 3) return hipErrorInvalidValue;
        a.G.in_off[a.G.n_in] = ux + kLdsWX * uy;
        a.G.in_coef[a.G.n_in++] = cf;
      } else {
        if (a.G.n_tl == 3 || (uz != 1 && uz != -1)) return hipErrorInvalidValue;
        a.G.tl_off[a.G.n_tl] = uz * (ux + kLdsWX * uy);   // oriented so that a step raises z' by one
        a.G.tl_coef[a.G.n_tl++] = cf;
      }
    }
    a.G.diag = in.g.w2[0] * sum;
  }
  for (int q = 0; q < 4; ++q) {
    a.G.czw[q] = a.G.cz * a.G.w[q];
    for (int k = 0; k < 3; ++k) a.G.tl_cw[k][q] = a.G.tl_coef[k] * a.G.w[q];
  }
  for (int q = 0; q < 4; ++q) {
    a.G32.czw[q] = (float)a.G.czw[q];
    for (int k = 0; k < 3; ++k) a.G32.tl_cw[k][q] = (float)a.G.tl_cw[k][q];
  }
  for (int q = 0; q < 4; ++q) a.G32.w[q] = (float)a.G.w[q];
  a.G32.cz = (float)a.G.cz;
  a.G32.diag = (float)a.G.diag;
  a.G32.n_in = a.G.n_in;
  a.G32.n_tl = a.G.n_tl;
  for (int k = 0; k < 3; ++k) {
    a.G32.in_off[k] = a.G.in_off[k];
    a.G32.in_coef[k] = (float)a.G.in_coef[k];
    a.G32.tl_off[k] = a.G.tl_off[k];
    a.G32.tl_coef[k] = (float)a.G.tl_coef[k];
  }
  a.lds_cx = in.g.lds_cx;
  a.lds_cy = in.g.lds_cy;
  a.lds_wx = in.g.lds_wx;
  a.lds_wy = in.g.lds_wy;
  if (in.pcg_cols > 0) {
    a.slot_bytes = pcg_slot_bytes(in.mixed, in.sstride, in.c1stride, in.b2stride);
    a.c1stride = in.c1stride;
    for (int k = 0; k < kMaxClasses; ++k) a.cls_delta[k] = in.cls_delta[k] > 0.0 ? in.cls_delta[k] : in.delta;
    a.b2stride = in.b2stride;
    a.pcg_planes = pcg_planes(in.g, in.mg, max_zmax, in.mixed);
    if (a.pcg_planes == 0) return hipErrorInvalidValue;
    a.pcg_lds = (int)pcg_lds_elems(in.g, in.mg, in.mixed, a.pcg_planes);
    a.pcg_ints = pcg_ints(max_zmax);
    // 1 / diagonal of the operator on the sphere, and of the 3-point operator
    // of each coarser grid in the scaling of P^T (see pcg_impl.h): the level's
    // steps are 2^l, a cell holds 8^l points
    double sum = 0.0;
    if (a.gen) {
      for (int m = 0; m < in.g.n_arms; ++m) sum += in.g.arm_coef[m];
    } else {
      for (int al = 0; al < 3; ++al) sum += in.g.inv_d2[al];
    }
    a.wl[0] = 1.0 / (-in.g.w2[0] * sum);
    for (int l = 1; l < 5; ++l) a.wl[l] = 1.0 / ((double)(1 << l) * 2.0 * sum);
    const size_t plds = pcg_lds_bytes(in.g, in.mg, max_zmax, in.mixed, a.pcg_planes);
    auto* fn = in.mixed ? (in.g.n == 1 ? pcg_n1_mixed : in.g.n == 2 ? pcg_n2_mixed : pcg_n3_mixed)
                        : (in.g.n == 1 ? pcg_n1_f64 : in.g.n == 2 ? pcg_n2_f64 : pcg_n3_f64);
    return fn(a, in.pcg_cols, in.threads, groups, plds, s, occ);
  }
  const size_t lds = solve_lds_bytes(in.g, max_zmax);
  switch (in.g.n) {
    case 1: return solve_dispatch_n1(a, in.mixed, max_cols, in.threads, in.depth, groups, lds, s, occ);
    case 2: return solve_dispatch_n2(a, in.mixed, max_cols, in.threads, in.depth, groups, lds, s, occ);
    case 3: return solve_dispatch_n3(a, in.mixed, max_cols, in.threads, in.depth, groups, lds, s, occ);
    default: return hipErrorInvalidValue;
  }
}

bool solve_supported(int max_cols, int threads) {
  if (threads == 1024) return max_cols <= 4 * 1024;
  if (threads == 768) return max_cols <= 4 * 768;   // quad layout only
  if (threads == 512) return max_cols <= 8 * 512;
  return false;
}

int solve_groups_per_cu(const Geo& g, int max_cols, int max_zmax, bool mixed, bool quads, int threads, int depth) {
  if (!solve_supported(max_cols, threads)) return 0;
  SolveArgs a;
  a.g = g;
  a.mixed = mixed;
  a.quads = quads;
  a.threads = threads;
  a.depth = depth;
  int occ = 0;
  if (solve_dispatch(a, max_cols, max_zmax, 1, nullptr, &occ) != hipSuccess) return 0;
  return occ;
}

int pcg_groups_per_cu(const Geo& g, const ClassHost& C, bool mixed, int threads) {
  SolveArgs a;
  a.g = g;
  a.mixed = mixed;
  a.threads = threads;
  a.pcg_cols = (int)C.fin_cols.size();
  a.mg = C.mg;
  int occ = 0;
  if (solve_dispatch(a, C.n_cols, C.Zmax, 1, nullptr, &occ) != hipSuccess) return 0;
  return occ;
}

hipError_t launch_solve(const SolveArgs& a, int max_cols, int max_zmax, int groups, hipStream_t s) {
  if (a.npair <= 0) return hipSuccess;
  return solve_dispatch(a, max_cols, max_zmax, groups, s, nullptr);
}

}  // namespace exx
