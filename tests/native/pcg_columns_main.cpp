// LDS reads of the arms that leave the sweep plane (the preconditioned CG's
// sweep of general cells), for every position that a thread may hold, one
// without a column included: where a plane counts as near a column, each arm's
// 2 n slots lie inside the staged plane, and a plane from which a point of the
// column takes a value always counts as near.
#include <cstdio>
#include <string>
#include <vector>

#include "pcg_cols.h"

using namespace exx;

static int failures = 0;
#define CHECK(c) \
  do {           \
    if (!(c) && ++failures < 20) std::printf("%s:%d: %s\n", name, __LINE__, #c); \
  } while (0)

static int check(const char* name, const ClassHost& C, const std::vector<NkArm>& arms, int n) {
  const int cx = C.Rc[0] + n, cy = C.Rc[1] + n, slots = kLdsWX * (2 * cy + 1);
  std::vector<int> off;   // one step of an arm, oriented so that it raises the plane by one
  for (const NkArm& A : arms) {
    const int ux = A.u[C.perm[0]], uy = A.u[C.perm[1]], uz = A.u[C.perm[2]];
    if (uz != 0 && (ux != 0 || uy != 0)) off.push_back(uz * (ux + kLdsWX * uy));
  }
  std::vector<PCol<true>> cols(1, PCol<true>::none());
  for (const int4& f : C.fin_cols) {
    const int x = (int)(short)(f.w & 0xffff), y = f.w >> 16;
    cols.push_back({f.z, f.y, f.x, (x + cx) + kLdsWX * (y + cy - n)});
  }
  CHECK(!cols[0].has());
  for (size_t i = 0; i < cols.size(); ++i) {
    const PCol<true>& k = cols[i];
    // as PCols keeps the planes: two 16-bit values
    const int w = (k.hi & 0xffff) | (int)((unsigned)k.lo << 16);
    CHECK((int)(short)(w & 0xffff) == k.hi && w >> 16 == k.lo);
    CHECK(i == 0 || k.has());
    for (int z = -C.Zmax - 3 * n - 4; z <= C.Zmax + 3 * n + 4; ++z) {
      CHECK(!k.valid(z) || k.has());
      for (int q = -n; q <= n; ++q) CHECK(!k.valid(z + q) || k.near(z, n));
      if (!k.near(z, n)) continue;
      const int pos = k.low + n * kLdsWX;
      CHECK(pos >= 0 && pos < slots);
      for (int o : off) CHECK(pos - n * o >= 0 && pos + n * o >= 0 && pos - n * o < slots && pos + n * o < slots);
    }
  }
  std::printf("%s: columns %zu arms leaving the plane %zu\n", name, cols.size() - 1, off.size());
  return (int)off.size();
}

int main() {
  // rhombohedral (angle 111 degrees), triclinic, monoclinic
  const double cells[3][9] = {
      {12.0, 0, 0, -4.300415, 11.202878, 0, -4.300415, -6.255543, 9.293262},
      {12.0, 0, 0, -2.1, 12.3, 0, 1.0, 2.0, 11.2},
      {12.0, 0, 0, 0, 11.0, 0, -3.0, 0, 11.5}};
  const int N[3] = {48, 48, 48};
  int body = 0, tilted = 0;
  for (int c = 0; c < 3; ++c) {
    std::vector<NkArm> arms;
    const std::string e = build_nk_arms(cells[c], N, &arms);
    if (!e.empty()) {
      std::printf("cell %d: %s\n", c, e.c_str());
      ++failures;
      continue;
    }
    for (const NkArm& A : arms) body += A.u[0] != 0 && A.u[1] != 0 && A.u[2] != 0;
    for (int sweep = 0; sweep < 3; ++sweep)
      for (int n = 1; n <= 3; ++n)
        for (double R : {0.7, 2.0, 4.0}) {
          const std::string id = "cell " + std::to_string(c) + " sweep " + std::to_string(sweep) + " n " +
                                 std::to_string(n) + " R " + std::to_string(R);
          ClassHost C;
          const std::string b = build_class_general(cells[c], N, sweep, R, R + 3.0, n, arms, false, false, &C);
          if (!b.empty()) {
            std::printf("%s: %s\n", id.c_str(), b.c_str());
            ++failures;
            continue;
          }
          tilted += check(id.c_str(), C, arms, n);
        }
  }
  if (body == 0 || tilted == 0) {
    std::printf("no arm along a body diagonal, or none that leaves the sweep plane\n");
    ++failures;
  }
  std::printf("failures %d\n", failures);
  return failures != 0;
}
