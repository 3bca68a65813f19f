// Workgroups of the unstructured selection.  Plain C++: the host tests compile it by itself.
#pragma once
#include <cstdint>

namespace thanos {

constexpr int kSelRows = 16;     // rows of a workgroup (one wavefront each)
constexpr int kSelMaxWgs = 256;  // at most one per compute unit: all resident at once

// The workgroups wait for each other at grid barriers, so that all of them have to be resident.  Calls that
// run at the same time compete for the units: `sharers` calls of one owner take no more of them together than
// the one with the most rows by itself, and two owners with several sweeps each are no closer to the
// limit than two with one.  (A workgroup alone waits for nobody.)
constexpr int select_workgroups(int64_t c, int units, int sharers) {
  const int64_t all = (c + kSelRows - 1) / kSelRows;
  const int64_t most = units < kSelMaxWgs ? units : kSelMaxWgs;
  const int64_t n = (all < most ? all : most) / sharers;
  return n < 1 ? 1 : (int)n;
}

}  // namespace thanos
