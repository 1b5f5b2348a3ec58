// Small pieces of the optimal unravelling that its batched kernel and the trajectory events share.
#pragma once
#include "common.h"

namespace mpsb {

using cd = c64d;

__device__ inline cd cz() { return cd{0.0, 0.0}; }
__device__ inline double cabs_(cd a) { return sqrt(norm2(a)); }

__device__ inline cd yy_flip(const cd (&v)[4], int i) {
  // (Y x Y) v*:  [ -v3*, v2*, v1*, -v0* ]
  switch (i) {
    case 0: return cd{-v[3].re, v[3].im};
    case 1: return cd{v[2].re, -v[2].im};
    case 2: return cd{v[1].re, -v[1].im};
    default: return cd{-v[0].re, v[0].im};
  }
}

struct UnravelOut {
  cd W[4][4];     // [i][j], i < r: K'_j = sum_i W[i][j] K_i
  double conc;
};

}  // namespace mpsb
