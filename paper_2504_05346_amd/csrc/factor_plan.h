// Order of a factorisation of nb blocks of columns.  Plain C++: the host tests compile it by itself.
#pragma once

namespace thanos {

constexpr int kOuter = 4;  // factor blocks to an outer block of the two-level updates
constexpr int kStepAll = 32, kStepLast = 24;

// The first block column that is left with one launch per step: 0 for up to kStepAll blocks, of more a multiple of kOuter
// with the last kStepLast (down to kStepLast - kOuter + 1) behind it.
constexpr int factor_first_step(int nb) {
  return nb <= kStepAll ? 0 : (nb - kStepLast + kOuter - 1) / kOuter * kOuter;
}

}  // namespace thanos
