// Order of a factorisation of nb blocks of columns, and the forks onto its helper streams.  Plain C++: the host tests
// compile it by itself.
#pragma once

namespace thanos {

constexpr int kOuter = 4;  // factor blocks to an outer block of the two-level updates

// Block rows that are factored with one launch per step (k_chol_step): up to kStepAll all of them, of more the last
// kStepLast.  A step updates every tile, (rows)^2 / 2 of them in 10 us a round of 512, beside 22.5 of its own; two-level
// updates move less.  Whole factorisations with the last 16, 24, 32, 40, 48, 64 blocks in such steps, us: 3000 columns 910,
// 768, 768, ..; 4096 1277, 1166, 1058, ..; 5120 1803, 1697, 1638, 1607, 1606, 1608; 6144 2355, 2284, 2250, 2245, 2340, 2338;
// 8192 3630, 3530, 3570, 3645, 3785, 4450; 11008 6625, 6560, 6500, 6510, 6580, 7290.  By themselves factorisations of 33
// to 48 blocks would want 40: up to 6 % of 5120 columns.  Next to the row losses, whose product leaves half of every compute
// unit, fewer are better: 5120 x 5120 4:8 with 16, 24, 32, 40 of 40 blocks 4581, 4520, 4581, 4700 us (4096: 2974, 2901, 2908
// of 32).  The same numbers for both, so that a factor has the same bits whatever runs beside it.  On both sides of kStepAll,
// without steps and with: 4096 columns 1696 and 1037, 4224 1848 and 1355, 4608 1930 and 1480, 5120 2100 and 1690.
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
