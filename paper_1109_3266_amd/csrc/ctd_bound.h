// Bound-test sums of the bound grid (host side, plain C++): for material m
// and energy cell j ([E_j, E_j+1]) a float at or above the interaction sum
// (photoelectric + Compton, + Rayleigh when on) that the Woodcock selection
// forms in float32 anywhere in the cell, so that a block's density level
// times it, rounded, bounds the selection at every density of the block.
//
// The sum over the processes of the largest value the column's linear
// interpolation takes in the cell, rounded up to float with a relative
// margin of 2^-20.  Inside the grid the interpolation weight w = f - j lies
// in [0, 1) exactly, and the float interpolation fma(w, x1 - x0, x0) stays
// within (1 + u)^2 of the larger node (u = 2^-24); the selection's products
// and sums of the non-negative rho-scaled terms add at most (1 + u)^3, and
// 2^-20 = 16u covers both and the final rounding.  In the top cell (E up to
// the last node) the rounding of f = (E - e0) / dE can put w past 1 by about
// 3u (ne - 1); there the column is extended to w = 1 + 4u ne.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>

namespace ctd {

inline float round_up_float(double x) {
  float f = (float)x;
  if ((double)f < x) f = std::nextafter(f, INFINITY);
  return f;
}

// mu_rho [M][ne][3] (pe, Compton, Rayleigh) cm^2/g; out [M][ne - 1].
inline void bound_sums(const float *mu_rho, int M, int ne, bool rayleigh, float *out) {
  const double w_top = 1.0 + 4.0 * 0x1p-24 * ne;
  for (int m = 0; m < M; ++m) {
    const float *r = mu_rho + (size_t)m * ne * 3;
    for (int j = 0; j + 1 < ne; ++j) {
      const float *x0 = r + (size_t)j * 3, *x1 = x0 + 3;
      const double w = j + 2 == ne ? w_top : 1.0;
      auto peak = [&](int k) {   // largest value of the column over the cell
        return std::max((double)x0[k], (double)x0[k] + w * ((double)x1[k] - (double)x0[k]));
      };
      double sum = peak(0) + peak(1);
      if (rayleigh) sum += peak(2);
      out[(size_t)m * (ne - 1) + j] = round_up_float(sum * (1.0 + 0x1p-20));
    }
  }
}

// Coarse bound grid: rejection without the energy.  The share of a voxel is its
// density times f[m], a float at or above material m's selection sum per unit
// density over the majorant anywhere on the energy grid (bnd from bound_sums,
// the majorant's nodes mu_max [ne]): the majorant interpolated in a cell is at
// least the smaller of its ends (the top cell's reaching w = 1 + 4u ne), and
// the margin of 2^-18 = 64u covers its float interpolation and the product
// u1 * majorant of the selection.  Infinite where the majorant may vanish.
inline void bound_shares(const float *bnd, const float *mu_max, int M, int ne, float *f) {
  const double w_top = 1.0 + 4.0 * 0x1p-24 * ne;
  for (int m = 0; m < M; ++m) {
    double top = 0.0;
    for (int j = 0; j + 1 < ne; ++j) {
      const double m0 = mu_max[j], m1 = mu_max[j + 1];
      const double end = j + 2 == ne ? m0 + w_top * (m1 - m0) : m1;
      const double low = std::min(m0, std::min(m1, end)), b = bnd[(size_t)m * (ne - 1) + j];
      top = std::max(top, b == 0.0 ? 0.0 : low > 0.0 ? b / low : INFINITY);
    }
    f[m] = round_up_float(top * (1.0 + 0x1p-18));
  }
}

// The byte c of a cell from its voxels' largest share: share * 256 rounded
// down, with a margin of 2^-20 for the float product rho * f.  A selection word
// w1 whose top byte is above c has a uniform u1 >= (c + 1) / 256 > share, so
// its collision is fictitious in every voxel of the cell; 255 rejects nothing.
constexpr unsigned char coarse_byte(float share) {
  const float x = share * (256.0f * (1.0f + 0x1p-20f));
  return x < 255.0f ? (unsigned char)x : (unsigned char)255;
}
constexpr bool coarse_rejects(unsigned int w1, unsigned char c) { return (w1 >> 24) > c; }

}  // namespace ctd
