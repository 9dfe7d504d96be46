// The coarse bound grid's bytes (bound_shares, coarse_byte of ctd_bound.h)
// against the float32 selection, evaluated as the transport evaluates it:
// random tables and majorants, energies anywhere in the grid including the
// nodes and the top, and for each a voxel of random density with the words
// around the byte's edge and random ones.  A rejected word must be fictitious:
// u1 * majorant at or above the selection sum.  Prints "ok <rejected>
// <fictitious>" or the first violation.  Arguments: seed trials.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "ctd_bound.h"

namespace {

struct Rng {
  uint64_t s;
  double u() {   // [0, 1)
    s = s * 6364136223846793005ull + 1442695040888963407ull;
    return (double)(s >> 11) * 0x1p-53;
  }
};

float lerp(float a, float b, float w) { return std::fma(w, b - a, a); }

// the transport's uniform of a 32-bit word: (2 (w >> 9) + 1) 2^-24
float unif(uint32_t w) { return (float)((double)(2u * (w >> 9) + 1u) * 0x1p-24); }

}  // namespace

int main(int argc, char **argv) {
  Rng g{argc > 1 ? std::strtoull(argv[1], nullptr, 10) : 1ull};
  const int trials = argc > 2 ? std::atoi(argv[2]) : 200;
  long rejected = 0, fictitious = 0;
  for (int t = 0; t < trials; ++t) {
    const int M = 1 + (int)(g.u() * 6), ne = 3 + (int)(g.u() * 300);
    const float e0 = (float)(1.0 + g.u() * 4.0), de = (float)(0.25 + g.u() * 2.0);
    const bool rayleigh = g.u() < 0.5;
    std::vector<float> tab((size_t)M * ne * 3), mu_max((size_t)ne);
    std::vector<double> top((size_t)M);
    for (int m = 0; m < M; ++m) {
      top[m] = std::pow(10.0, -3.0 + 3.3 * g.u());
      for (int k = 0; k < 3; ++k) {
        double v = std::pow(10.0, -3.0 + 4.0 * g.u());
        const bool zero = k > 0 && g.u() < 0.1;
        for (int j = 0; j < ne; ++j) {
          v *= std::exp((g.u() - 0.5) * 0.1);
          if (g.u() < 0.01) v *= 1.0 + 3.0 * g.u();
          tab[((size_t)m * ne + j) * 3 + k] = zero ? 0.0f : (float)v;
        }
      }
    }
    // the majorant of the largest densities, rounded up (as the library's)
    for (int j = 0; j < ne; ++j) {
      double best = 0.0;
      for (int m = 0; m < M; ++m) {
        const float *r = &tab[((size_t)m * ne + j) * 3];
        best = std::fmax(best, top[m] * ((double)r[0] + r[1] + (rayleigh ? r[2] : 0.0f)));
      }
      mu_max[j] = ctd::round_up_float(best * (1.0 + 0x1p-20));
    }
    std::vector<float> bnd((size_t)M * (ne - 1)), f((size_t)M);
    ctd::bound_sums(tab.data(), M, ne, rayleigh, bnd.data());
    ctd::bound_shares(bnd.data(), mu_max.data(), M, ne, f.data());
    const float inv_de = (float)(1.0 / (double)de);
    const double etop = (double)e0 + (double)(ne - 1) * (double)de;
    for (int q = 0; q < 400; ++q) {
      double Ed;
      const double r = g.u();
      if (r < 0.1) Ed = etop;
      else if (r < 0.4) Ed = (double)e0 + (int)(g.u() * (ne - 1)) * (double)de;
      else Ed = (double)e0 + g.u() * (etop - (double)e0);
      float E = (float)Ed;
      if ((double)E > etop) E = std::nextafter(E, 0.0f);
      const float fj = (E - e0) * inv_de;
      const int j = std::min(std::max((int)fj, 0), ne - 2);
      const float w = fj - (float)j, mumax = lerp(mu_max[j], mu_max[j + 1], w);
      const int m = (int)(g.u() * M);
      const float rho = (float)(top[m] * (q % 3 == 0 ? 1.0 : std::pow(g.u(), 2.0)));
      const unsigned char c = ctd::coarse_byte(rho * f[m]);
      const float *x0 = &tab[((size_t)m * ne + j) * 3], *x1 = x0 + 3;
      float sum = rho * lerp(x0[0], x1[0], w);
      sum = sum + rho * lerp(x0[1], x1[1], w);
      if (rayleigh) sum = sum + rho * lerp(x0[2], x1[2], w);
      for (int n = 0; n < 6; ++n) {
        uint32_t word = (uint32_t)(g.u() * 0x1p32);
        if (n < 3) word = (((uint32_t)c + 1u) << 24) + (n == 0 ? 0u : n == 1 ? ~0u : 511u);
        const bool fict = unif(word) * mumax >= sum;
        fictitious += fict;
        if (!ctd::coarse_rejects(word, c)) continue;
        ++rejected;
        if (!fict) {
          std::printf("violation: word %08x byte %d sum %.9g majorant %.9g\n", word, (int)c, sum,
                      mumax);
          return 0;
        }
      }
    }
  }
  std::printf("ok %ld %ld\n", rejected, fictitious);
  return 0;
}
