// Host check of the energies that the float32 CG adds up for p.Ap: terms that cancel in float32,
// and random ones whose error is that of the exact products summed in float64.
#include <cmath>
#include <cstdio>
#include <random>

#include "energy.h"

using namespace sfem;

int main() {
  // neither 2^24 + 1 nor 4096.5^2 is a float32
  const float big = 4096.0f;
  const double a = add_energy(0.0, 1.0f, 1.0f, big, big, -big, big);
  const double b = add_energy(add_energy(0.0, 1.0f, 1.0f), 4096.5f, 4096.5f, -big, big, 0.0f, 0.0f);
  if (a != 1.0) std::printf("FAIL cancelled sum %.17g\n", a);
  if (b != 1.0 + 4096.25) std::printf("FAIL inexact product %.17g\n", b);
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<float> U(-1.0f, 1.0f);
  double got = 0.0, worst = 0.0;
  long double ref = 0.0L, scale = 0.0L;
  for (int i = 0; i < 4000; ++i) {
    float x[8];
    for (float &v : x) v = U(rng) * std::ldexp(1.0f, (i * 7) % 21 - 10);
    got = add_energy(add_energy(got, x[0], x[1]), x[2], x[3], x[4], x[5], x[6], x[7]);
    for (int k = 0; k < 8; k += 2) {
      ref += (long double)x[k] * x[k + 1];
      scale += std::fabs((long double)x[k] * x[k + 1]);
    }
    worst = std::fmax(worst, (double)(std::fabs((long double)got - ref) / scale));
  }
  // four float64 additions a point
  if (!(worst <= 4000 * 4 * 0x1p-53)) std::printf("FAIL error %g\n", worst);
  std::printf("worst %g\n", worst);
  return 0;
}
