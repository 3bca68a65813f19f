// Division of the sweep's multiplier buffer.  Plain C++: the host tests compile it by itself.
#pragma once
#include <cstdint>

namespace thanos {

// Blocks whose selection only looks at their own columns (n:m, forced masks) are swept in
// super-blocks of kSuper blocks: inside a super-block the update of a block only reaches the
// end of the super-block, and everything right of it gets one update per super-block with a
// kSuper times longer reduction (the multipliers of all its blocks are kept, c x kSuper*B).
// The global residual mask needs current weights: there a super-block is one block.
constexpr int kSuper = 8;

constexpr int64_t lam_buffer_floats(int64_t c, int64_t B) { return c * B * kSuper * 2; }

// Offsets in floats of c x ldl matrices, ldl = B * super.  The multipliers of consecutive super-blocks
// sbi alternate between the first two; behind them lie, where a super-block is one block (room for
// 16), the operands of the complement products: every row of z is read by all column tiles of the
// product whose results are multipliers, so the two must never share memory.
// (rsc, one value per row, likewise: with super-blocks its two arrays are those of the selection, which
// does not run then.)
struct LamLayout {
  int64_t lam, z, wk, rsc;
};
constexpr LamLayout lam_layout(int64_t c, int64_t ldl, int64_t sbi) {
  return {(sbi & 1) * c * ldl, 2 * c * ldl, 3 * c * ldl, 4 * c * ldl};
}

}  // namespace thanos
