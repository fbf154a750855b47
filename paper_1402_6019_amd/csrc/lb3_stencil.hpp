// D3Q19 lattice and the force stencil of the 3-D kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace lb355 {

namespace d3 {

// D3Q19 in the canonical order of lb3.h; opposite links are adjacent (1-2, 3-4, ...).
__device__ constexpr int CX[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
__device__ constexpr int CY[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
__device__ constexpr int CZ[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};

constexpr int opp(int l) { return l == 0 ? 0 : (l & 1 ? l + 1 : l - 1); }
constexpr int cx(int l) { return l == 1 || l == 7 || l == 9 || l == 11 || l == 13 ? 1 : (l == 2 || l == 8 || l == 10 || l == 12 || l == 14 ? -1 : 0); }
constexpr int cy(int l) { return l == 3 || l == 7 || l == 10 || l == 15 || l == 17 ? 1 : (l == 4 || l == 8 || l == 9 || l == 16 || l == 18 ? -1 : 0); }
constexpr int cz(int l) { return l == 5 || l == 11 || l == 14 || l == 15 || l == 18 ? 1 : (l == 6 || l == 12 || l == 13 || l == 16 || l == 17 ? -1 : 0); }

__device__ inline int wrap(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

}  // namespace d3

// The 46 half-links of the 92-link cube stencil (one of each +-c pair), grouped by shell:
// c = (dx, dy, dz) with dz > 0, or dz == 0 and dy > 0, or dz == dy == 0 and dx > 0.
#define LB3_HALF_LINKS(X)                                                                        \
  /* shell 1 */ X(0, 1, 0, 0) X(0, 0, 1, 0) X(0, 0, 0, 1)                                       \
  /* shell 2 */ X(1, 1, 1, 0) X(1, -1, 1, 0) X(1, 1, 0, 1) X(1, -1, 0, 1) X(1, 0, 1, 1) X(1, 0, -1, 1) \
  /* shell 3 */ X(2, 1, 1, 1) X(2, -1, 1, 1) X(2, 1, -1, 1) X(2, -1, -1, 1)                      \
  /* shell 4 */ X(3, 2, 0, 0) X(3, 0, 2, 0) X(3, 0, 0, 2)                                        \
  /* shell 5 */ X(4, 2, 1, 0) X(4, -2, 1, 0) X(4, 1, 2, 0) X(4, -1, 2, 0) X(4, 2, 0, 1) X(4, -2, 0, 1) \
                X(4, 0, 2, 1) X(4, 0, -2, 1) X(4, 1, 0, 2) X(4, -1, 0, 2) X(4, 0, 1, 2) X(4, 0, -1, 2) \
  /* shell 6 */ X(5, 2, 1, 1) X(5, -2, 1, 1) X(5, 2, -1, 1) X(5, -2, -1, 1) X(5, 1, 2, 1) X(5, -1, 2, 1) \
                X(5, 1, -2, 1) X(5, -1, -2, 1) X(5, 1, 1, 2) X(5, -1, 1, 2) X(5, 1, -1, 2) X(5, -1, -1, 2) \
  /* shell 8 */ X(6, 2, 2, 0) X(6, -2, 2, 0) X(6, 2, 0, 2) X(6, -2, 0, 2) X(6, 0, 2, 2) X(6, 0, -2, 2)

}  // namespace lb355
