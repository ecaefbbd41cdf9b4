// Host: the stencil and its pair counts per neighbour block, made once per process
// (safe from several threads at once: contexts of different threads share them).
#pragma once

#include <vector>

#include "fmm_common.h"

namespace fmm {

// Shell stencil 5 <= |d|^2 <= 36, dz slowest, then dy, then dx.
inline const std::vector<int>& stencil_host() {
  static const std::vector<int> s = [] {
    std::vector<int> v;
    for (int dz = -kRad; dz <= kRad; ++dz)
      for (int dy = -kRad; dy <= kRad; ++dy)
        for (int dx = -kRad; dx <= kRad; ++dx) {
          const int q = dx * dx + dy * dy + dz * dz;
          if (q >= 5 && q <= 36) {
            v.push_back(dx);
            v.push_back(dy);
            v.push_back(dz);
          }
        }
    return v;
  }();
  return s;
}

// pairs (target cell, offset) whose source lies in a block of `mask`
inline int64_t pairs_of_mask(uint32_t mask) {
  static const std::vector<int64_t> per_block = [] {
    std::vector<int64_t> v(27, 0);
    const std::vector<int>& st = stencil_host();
    for (int t = 0; t < kNTarget; ++t) {
      const int jx = t % 8 + 8, jy = (t / 8) % 8 + 8, jz = t / 64 + 8;
      for (size_t i = 0; i < st.size(); i += 3)
        v[(jx + st[i]) / 8 + 3 * ((jy + st[i + 1]) / 8) + 9 * ((jz + st[i + 2]) / 8)]++;
    }
    return v;
  }();
  int64_t n = 0;
  for (int b = 0; b < 27; ++b)
    if ((mask >> b) & 1u) n += per_block[b];
  return n;
}

}  // namespace fmm
