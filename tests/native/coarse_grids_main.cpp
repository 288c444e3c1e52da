// The coarse grids of the preconditioned CG, built for several spheres and
// cells: nested, complete, with every index of the tables inside the boxes,
// planes and slots that the kernels address with them.
#include <array>
#include <cstdio>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "exx_internal.h"

using namespace exx;

static int failures = 0;
#define CHECK(c) \
  do {           \
    if (!(c) && ++failures < 20) std::printf("%s:%d: %s\n", name, __LINE__, #c); \
  } while (0)

static void check(const char* name, const ClassHost& C) {
  const MgDev& M = C.mg;
  std::set<std::array<int, 3>> fine;
  for (long long k = 0; k < C.n_pe; ++k) {
    const short4 o = C.me_off[(size_t)k];
    if (o.w) continue;
    const int t[3] = {o.x, o.y, o.z};
    fine.insert({t[C.perm[0]], t[C.perm[1]], t[C.perm[2]]});
  }
  const int np[4] = {M.n_p1, M.n_p2, M.n_p3, M.n_p4};
  const int* E[4] = {nullptr, M.E2, M.E3, M.E4};
  const int* D[4] = {nullptr, M.D2, M.D3, M.D4};
  std::set<std::array<int, 3>> lev[4];
  for (int l = 0; l < 4; ++l) {
    CHECK(np[l] == (int)C.mg_pts[l].size());
    for (const short4 o : C.mg_pts[l])
      if (!o.w) CHECK(lev[l].insert({o.x, o.y, o.z}).second);
    const int s = 2 << l;
    size_t want = 0;
    for (const auto& p : fine)
      if (p[0] % s == 0 && p[1] % s == 0 && p[2] % s == 0) {
        ++want;
        CHECK(lev[l].count({p[0] / s, p[1] / s, p[2] / s}));
      }
    CHECK(want == lev[l].size());
    if (l == 0) continue;
    // the stencils of the restriction to this level, and of the interpolation
    // from it to the level below, stay inside its box
    auto inside = [&](int x, int y, int z, const int* e, const int* d) {
      return x + e[0] + 1 >= 0 && x + e[0] + 1 < d[0] && y + e[1] + 1 >= 0 && y + e[1] + 1 < d[1] &&
             z + e[2] + 1 >= 0 && z + e[2] + 1 < d[2];
    };
    for (const auto& p : lev[l]) CHECK(inside(p[0], p[1], p[2], E[l], D[l]));
    for (const auto& p : lev[l - 1])
      for (int q = 0; q < 8; ++q)
        CHECK(inside((p[0] + (q & 1)) >> 1, (p[1] + (q >> 1 & 1)) >> 1, (p[2] + (q >> 2)) >> 1, E[l], D[l]));
    if (l >= 2)
      for (const auto& p : lev[l])
        for (int q = 0; q < 27; ++q)
          CHECK(inside(2 * p[0] + q % 3 - 1, 2 * p[1] + q / 3 % 3 - 1, 2 * p[2] + q / 9 - 1, E[l - 1], D[l - 1]));
  }
  // level-1 slots: column i's point of plane z lies at c1start[z] + i
  CHECK((int)C.c1start.size() == 2 * M.Z1 + 2 && C.c1start.back() == M.n_p1);
  size_t seen = 0;
  for (int i = 0; i < M.n_c1; ++i) {
    const int4 c = C.c1cols[i];
    for (int z = c.z; z <= c.w; ++z, ++seen) {
      CHECK(z >= -M.Z1 && z <= M.Z1);
      const int k = C.c1start[z + M.Z1] + i;
      CHECK(k < C.c1start[z + M.Z1 + 1]);
      const short4 o = C.mg_pts[0][(size_t)k];
      CHECK(o.x == c.x && o.y == c.y && o.z == z && !o.w);
    }
    // the staged planes: the restriction's 9 points, the column's own place
    const int rx = 2 * c.x + M.rcx, ry = 2 * c.y + M.rcy, qx = c.x + M.ex + 1, qy = c.y + M.ey + 1;
    CHECK(rx >= 1 && rx + 1 < M.rw && ry >= 1 && ry + 1 < M.rh);
    CHECK(qx >= 1 && qx + 1 < M.ew && qy >= 1 && qy + 1 < M.eh);
  }
  CHECK(seen == lev[0].size());
  seen = 0;
  for (int i = 0; i < M.n_c2; ++i) {
    const int4 c = C.c2cols[i];
    seen += c.w - c.z + 1;
    const int qx = 2 * c.x + M.ex + 1, qy = 2 * c.y + M.ey + 1;
    CHECK(qx >= 1 && qx + 1 < M.ew && qy >= 1 && qy + 1 < M.eh);
  }
  CHECK(seen == lev[1].size());
  // the sphere's own columns: their place in the restriction's plane and the
  // four level-1 neighbours of the interpolation
  for (const auto& p : fine) {
    CHECK(p[0] + M.rcx >= 0 && p[0] + M.rcx < M.rw && p[1] + M.rcy >= 0 && p[1] + M.rcy < M.rh);
    for (int q = 0; q < 4; ++q) {
      const int x = ((p[0] + (q & 1)) >> 1) + M.ex + 1, y = ((p[1] + (q >> 1)) >> 1) + M.ey + 1;
      CHECK(x >= 0 && x < M.ew && y >= 0 && y < M.eh);
    }
  }
  std::printf("%s: points %zu %zu %zu %zu %zu failures %d\n", name, fine.size(), lev[0].size(), lev[1].size(),
              lev[2].size(), lev[3].size(), failures);
}

int main() {
  const double radii[] = {0.3, 0.7, 1.5, 3.1, 4.4};
  for (double R : radii)
    for (int n = 1; n <= 3; ++n)
      for (int quads = 0; quads < 2; ++quads) {
        const std::string id = "R " + std::to_string(R) + " n " + std::to_string(n) + " quads " + std::to_string(quads);
        const double L[3] = {12.0, 13.0, 11.0};
        const int N[3] = {50, 48, 56};
        ClassHost C;
        std::string e = build_class(L, N, R, R + 0.8, n, quads, &C);
        if (e.empty())
          check(("ortho " + id).c_str(), C);
        else
          std::printf("ortho %s: %s\n", id.c_str(), e.c_str());
        const double cells[2][9] = {{12.0, 0, 0, -6.0, 10.392, 0, 0, 0, 12.0}, {12.0, 0, 0, -2.1, 12.3, 0, 1.0, 2.0, 11.2}};
        for (int c = 0; c < 2; ++c) {
          std::vector<NkArm> arms;
          e = build_nk_arms(cells[c], N, &arms);
          ClassHost G;
          if (e.empty()) e = build_class_general(cells[c], N, c == 0 ? 2 : 0, R, R + 0.8, n, arms, false, quads && c == 0, &G);
          if (e.empty())
            check((std::string(c ? "tilted " : "hex ") + id).c_str(), G);
          else
            std::printf("general %d %s: %s\n", c, id.c_str(), e.c_str());
        }
      }
  std::printf("failures %d\n", failures);
  return failures != 0;
}
