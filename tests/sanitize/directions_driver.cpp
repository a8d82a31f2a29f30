// The refinement's search direction (csrc/directions.h) on the CPU: what is
// left of it for coefficients around -1 where the ring's oldest buffer is the
// new direction's.
#include <cmath>
#include <cstdio>

#include "../../paper_2512_12151_amd/csrc/directions.h"

using bfal::Directions;

// One entry of the direction, as the kernel forms it.
static double entry(double z, const Directions& d, const double* out) {
  double v = z;
  for (int j = 0; j < d.n; ++j) v = std::fma(d.a[j], d.p[j] == out ? v : *d.p[j], v);
  return v;
}

int main() {
  int failures = 0;
  const double p0 = 0.25, p1 = -0.5, p2 = 2.0, out = 7.0, z = 1.5;
  const double coef[] = {-1.0, std::nextafter(-1.0, 0.0), std::nextafter(-1.0, -2.0), -0.5, 0.0, 3.0};
  for (double a : coef) {
    Directions d;
    d.add(0.5, &p0, &out);
    d.add(-1.0, &p1, &out);   // (another buffer: -1 is a coefficient like any other)
    d.add(0.125, &p2, &out);
    const double before = entry(z, d, &out);
    if (before != 1.5 + 0.125 + 0.5 + 0.25 || d.n != 3) ++failures;
    d.add(a, &out, &out);
    const double v = entry(z, d, &out);
    const double want = a == -1.0 ? before : std::fma(a, before, before);
    std::printf("a = %.17g: %.17g\n", a, v);
    if (v == 0.0 || v != want) ++failures;
  }
  if (failures) {
    std::printf("%d failures\n", failures);
    return 1;
  }
  std::printf("all checks passed\n");
  return 0;
}
