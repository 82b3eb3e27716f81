/* The rounding of a slab's faces in a ray's walk, against 64-bit arithmetic: one
 * difference and one quotient, so within two roundings (2^-24 of its value each)
 * of the exact one; and in the order of the faces, which the walk takes for
 * granted.  Over grids and origins from inside the box to a million boxes away.
 * Exits 0 and prints "ok" on success. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include "walk.hpp"

static uint64_t rng_state = 0x9E3779B97F4A7C15ull;
static double uniform() {  // splitmix64, [0, 1)
  uint64_t z = (rng_state += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return ldexp(static_cast<double>((z ^ (z >> 31)) >> 11), -53);
}

int main() {
  const double u = ldexp(1.0, -24);
  for (int i = 0; i < 4000000; ++i) {
    const float w = static_cast<float>(exp2(uniform() * 20.0 - 10.0));
    const float pa = static_cast<float>((uniform() - 0.5) * 2048.0) * w;
    const float om = static_cast<float>((uniform() - 0.5) * exp2(uniform() * 32.0)) * w;
    const float dm = static_cast<float>((uniform() < 0.5 ? -1.0 : 1.0) * exp2(uniform() * 20.0 - 10.0) * (1.0 + uniform()));
    const float pb = pa + w;
    const float ta = gb::plane_t(pa, om, dm), tb = gb::plane_t(pb, om, dm);
    const double x = (static_cast<double>(pa) - om) / dm;
    if (fabs(ta - x) > 2.0 * u * fabs(x) * (1.0 + u) || (dm > 0 ? ta > tb : ta < tb)) {
      fprintf(stderr, "FAIL: %.9g (next %.9g) of p %.9g w %.9g om %.9g dm %.9g, exact %.17g (%.3f roundings)\n", ta, tb, pa, w, om,
              dm, x, fabs(ta - x) / (u * fabs(x)));
      return 1;
    }
  }
  puts("ok");
  return 0;
}
