// Tile width, number of parts and workgroups of a 16-bit Hessian accumulation.  Plain C++: the host
// tests compile it by itself.
#pragma once
#include <algorithm>
#include <cstdint>

namespace thanos {

struct SyrkPlan {
  int tile;       // width
  int nt;         // tiles per side
  int ntiles;     // nt*(nt+1)/2
  int nkt;        // k-steps per tile
  int nsplit;     // parts a tile's k-steps are cut into; > 1: partial sums are added atomically
  int spread;     // which workgroup does what, see item_of
  unsigned grid;  // workgroups
};

// What a tile width costs, in us.
//   step   one k-step of a workgroup while the chip's power limit does not bind;
//   work   its multiplications relative to 256 x 256 x 32 tokens (the energy they take).  Beyond about 170 busy compute
//          units the chip clocks down in proportion (256-wide tiles of random data: 0.62 us a step on
//          136 units, 0.92 us on 256), so work, not the number of units, sets the time;
//   slots  workgroups the chip holds at once;
//   one, more   per work item: pipeline fill and write-out latency where all items run at once, and
//          where the next item waits behind the stores or atomics of the last one;
//   drift  share by which long items take longer: the workgroups of an XCD drift apart and share less
//          through its L2, in full from `far` steps on.
struct TileCost {
  int tile, kt, slots;
  double step, work, one, more, drift, far;
};

constexpr int64_t plan_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Whether k_syrk16_dma takes the rows: 16-byte aligned, and eight of them (what a wavefront loads from one
// descriptor, whose offsets have 32 bits) within 4 GB.
constexpr bool syrk_rows_aligned(uintptr_t X, int64_t ldx, int64_t b) {
  return X % 16 == 0 && ldx % 8 == 0 && b % 8 == 0 && ldx < (int64_t)1 << 28;
}

// What a wavefront reads of H (b x b) around the 32 x 32 tile at (i0, j0): from element `first` on, `bytes` bytes, which
// end where H ends, or none (zeros are read instead).  A tile whose one row is the last of H and whose columns are
// all past the last one starts behind H.
struct HWindow {
  int64_t first;
  uint32_t bytes;
};
constexpr HWindow h_window(int64_t b, int64_t i0, int64_t j0) {
  const int64_t left = i0 < b ? 4 * ((b - i0) * b - j0) : 0;
  return left > 0 ? HWindow{i0 * b + j0, (uint32_t)std::min<int64_t>(left, 0xffffffffll)} : HWindow{0, 0};
}

// Parts that fill whole rounds of the 32 compute units of an XCD with 256-wide tiles (12 k-steps per item
// for its fill and write-out).
inline int64_t round_parts(int64_t b, int64_t n_tok) {
  const int64_t nt = plan_div(b, 256), cnt = plan_div(nt * (nt + 1) / 2, 8), nkt = plan_div(n_tok, 32);
  auto cost = [&](int64_t S) { return (double)plan_div(cnt * S, 32) * ((double)nkt / (double)S + 12.0); };
  int64_t best = 1;
  for (int64_t S = 2; S <= std::min<int64_t>(64, nkt / 64); ++S)
    if (cost(S) < cost(best) * (best == 1 ? 0.97 : 1.0)) best = S;
  return best;
}

// Width of the tiles of k_syrk16_waves that fit the chip all at once, 0: more channels than that.
constexpr int64_t waves_tile(int64_t b) {
  const int64_t n32 = plan_div(b, 32), n64 = plan_div(b, 64);
  return n32 * (n32 + 1) / 2 <= 256 ? 32 : n64 * (n64 + 1) / 2 <= 256 ? 64 : 0;
}

// Tokens of one launch on rows of any alignment, in launches of equal length: no more than 4096 for any one
// sum (8192 in a 256-wide tile).  The rounding error of a sum grows with the root of its length (65536 x
// 4001 in one launch 1.4e-6 of the result, in eight 1e-7).  32-wide tiles have 16 sums each, 64-wide 8,
// 128-wide two.
constexpr int64_t syrk_launch_tokens(int64_t b, int64_t n_tok) {
  const int64_t w = waves_tile(b), most = w == 32 ? 65536 : w == 64 ? 32768 : 8192;
  const int64_t launches = plan_div(n_tok, most);
  return plan_div(plan_div(n_tok, launches), 128) * 128;
}

// The cheapest by this estimate: H is read and written once (4.5 TB/s), or, with parts, added to once
// per part with atomics (1.1 TB/s measured, which is why a narrower tile is preferred to a second
// part).  Start of a call 4 us.  Measured, 16-bit tokens x channels:
//                     256-wide whole tiles     chosen
//   2048 x 4096            73 us               192, 1 part     47 us
//   2048 x 2048            67 us               128, 1 part     26 us
//   32768 x 768            65 us (16 parts)    128, 11 parts   40 us
// aligned: 16-byte aligned rows (k_syrk16_dma), else k_syrk16.  Rows of any alignment are summed up
// in one part, in a fixed order, so that equal calls give equal bits and H is rounded once per
// launch: 2048 x 5121 128-wide 172 us, 256-wide 146, 2048 x 8191 394 and 414, 65536 x 8191 9.8 and 9.2 ms.
// Few channels, one part: k_syrk16_waves, while all of its tiles run at once.  2048 tokens:
//                     32-wide   64-wide   128-wide
//   256 channels         10        15        22 us      aligned
//   768                  21        16        22
//   1536                 62        34        24
//   237                  12        20        40         any alignment
//   700                  14        18        39
//   1365                 57        24        43
//   2047                123        64        46
inline SyrkPlan syrk_plan(int64_t b, int64_t n_tok, bool aligned) {
  static constexpr TileCost dma[] = {{256, 32, 256, 0.62, 1.0, 4, 12, 0.06, 8192},
                                     {192, 32, 256, 0.36, 0.58, 4, 12, 0.17, 512},
                                     {128, 64, 256, 0.43, 0.5, 4, 12, 0.06, 8192}};
  static constexpr TileCost any[] = {{256, 64, 256, 2.53, 2.0, 45, 45, 0.06, 8192},
                                     {128, 128, 256, 1.66, 1.0, 12, 12, 0.3, 512}};
  const TileCost* cand = aligned ? dma : any;
  const int ncand = aligned ? 3 : 2;
  const double hbytes = 4.0 * (double)b * (double)b / 2;
  // Parts: each rounds into H, in any order; the rounding error of a part grows with the root of the
  // length of its sums, which is half as long where two groups of wavefronts share the part (192, 128).  So
  // short calls have one part (20 calls of 2048 x 256 in 11 parts 2.1e-7 off float64, in one 0.7e-7),
  // and long ones as many as fill whole rounds, or down to half of them in two groups (65536 x 4096 in
  // 13 parts 1.2e-7, in 9 1.7e-7).
  const int64_t parts = aligned ? round_parts(b, n_tok) : 1;
  if (const int64_t w = waves_tile(b); w > 0 && parts == 1) {
    const int64_t nt = plan_div(b, w), ntiles = nt * (nt + 1) / 2;
    return {(int)w, (int)nt, (int)ntiles, (int)plan_div(n_tok, 32768 / w), 1, 1, 8u * (unsigned)plan_div(ntiles, 8)};
  }
  SyrkPlan p{};
  double best = 1e300;
  for (int q = 0; q < ncand; ++q) {
    const TileCost& k = cand[q];
    const int64_t nt = plan_div(b, k.tile), ntiles = nt * (nt + 1) / 2;
    const int64_t nkt = plan_div(n_tok, k.kt);
    for (int64_t S = k.tile == 256 ? parts : plan_div(parts, 2); S <= parts; ++S) {
      const bool spread = ntiles * S <= k.slots;
      // narrow tiles read the tokens more often: aligned ones only while everything is resident at once
      if (aligned && !spread && k.tile != 256) continue;
      const int64_t per_xcd = plan_div(ntiles, 8) * S, slots_xcd = k.slots / 8;
      const double steps = (double)plan_div(nkt, S);
      auto round_us = [&](double busy) {
        return steps * std::max(k.step, 0.62 * k.work * busy / 170.0) + (spread ? k.one : k.more);
      };
      const int64_t full = spread ? 0 : per_xcd / slots_xcd;
      const int64_t left = spread ? ntiles * S : 8 * (per_xcd - full * slots_xcd);
      const double rounds = (double)full + (left > 0 ? 1.0 : 0.0);
      double us = (double)full * round_us((double)k.slots) + (left > 0 ? round_us((double)left) : 0.0);
      if (aligned || !spread) us *= 1.0 + k.drift * std::min(1.0, steps / k.far);
      // the write-out of a round runs beside the multiplications of the next one
      const double out = S > 1 ? (double)S * hbytes / 1.1e6 : 2.0 * hbytes / 4.5e6;
      us = 4.0 + std::max(us + out / rounds * (rounds > 1.0 ? 0.5 : 1.0), out);
      if (us < best) {
        best = us;
        p = {k.tile,        (int)nt, (int)ntiles, (int)nkt, (int)S, spread ? 1 : 0,
             spread ? 8u * (unsigned)plan_div(ntiles * S, 8) : 8u * (unsigned)per_xcd};
      }
    }
  }
  return p;
}

}  // namespace thanos
