// The sum of a solution update of the preconditioned CG against extended
// precision: for an FP64 solution FP32 vectors are summed with FP64 steps and
// sums (four products and sums of terms of total size m leave at most 8 eps m).
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "pcg_cols.h"

using namespace exx;

static double value(double scale) { return scale * (2.0 * std::rand() / RAND_MAX - 1.0); }

template <typename X, typename T>
static int check(const char* name, double eps) {
  int failures = 0;
  std::srand(7);
  for (int k = 0; k < 20000; ++k) {
    const T y = (T)value(1.0);
    X w[kPcgRing];
    T v[kPcgRing];
    long double want = y, size = std::fabs((long double)y);
    for (int i = 0; i < kPcgRing; ++i) {
      w[i] = (X)value(0.05);
      v[i] = (T)value(3.0);
      want += (long double)w[i] * (long double)v[i];
      size += std::fabs((long double)w[i] * (long double)v[i]);
    }
    const long double err = std::fabs((long double)pcg_add_steps<X, T>(y, w, v) - want);
    if (!(err <= 8 * eps * size) && ++failures < 5)
      std::printf("%s: error %Lg of %Lg\n", name, err, size);
  }
  return failures;
}

int main() {
  const int failures = check<double, float>("FP64 x, FP32 steps", 1.2e-16) + check<double, double>("FP64", 1.2e-16) +
                       check<float, float>("FP32", 6e-8);
  std::printf("failures %d\n", failures);
  return failures != 0;
}
