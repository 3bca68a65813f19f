// Order of a factorisation of nb blocks of columns, and the forks onto its helper streams.  Plain C++: the host tests
// compile it by itself.
#pragma once

namespace thanos {

constexpr int kOuter = 4;  // factor blocks to an outer block of the two-level updates
constexpr int kStepAll = 32, kStepLast = 24;

// The first block column that is left with one launch per step: 0 for up to kStepAll blocks, of more a multiple of kOuter
// with the last kStepLast (down to kStepLast - kOuter + 1) behind it.
constexpr int factor_first_step(int nb) {
  return nb <= kStepAll ? 0 : (nb - kStepLast + kOuter - 1) / kOuter * kOuter;
}
// Outer blocks whose wide update has a rest on the helper stream
constexpr int factor_rests(int nb) { return factor_first_step(nb) / kOuter; }
// Batches of merges of the inverse beside the chain: one behind every outer block, if two block columns and more follow
constexpr int factor_tri_batches(int nb) { return nb < 2 ? 0 : (nb - 2) / kOuter; }

}  // namespace thanos
