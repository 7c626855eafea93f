// Which variant of a pass a launch takes, as a function of the shape alone.  Plain host arithmetic (head_parts and grid_blocks are
// constexpr so that the device code that maps workgroup ids to tiles shares them), free of HIP, so that a test without a GPU can
// compile it and hold every rule against the times it was read from.
#pragma once
#include <algorithm>
#include <cmath>

namespace helix {

// Heads are dealt to the 8 XCDs as "virtual heads", P interleaved parts each (see map_block in helix_common.hpp): the smallest power
// of two that makes BH * P a multiple of 8.
constexpr int head_parts(int BH) { return (BH & 1) ? 8 : (BH & 2) ? 4 : (BH & 4) ? 2 : 1; }
// Number of workgroups to launch for BH slices of T tiles.  An eighth of them is the share of the fullest XCD, which has the
// tile more where T is not a multiple of P.
constexpr long long grid_blocks(int BH, int T) {
  const int P = head_parts(BH);
  return (long long)BH * P * ((T + P - 1) / P);
}

// The workgroups of a launch on the fullest XCD (32 compute units): how many, the 64-row (64-key) steps of the longest, and of all of them.
// `keys`: tiles of the dK/dV pass, which sweep the query rows from their first key on; else of query rows, which sweep the keys up
// to their last row.
struct Share { double blocks, longest, steps; };
inline Share share(int BH, int S, bool causal, int rows, bool keys) {
  const int P = head_parts(BH), T = (S + rows - 1) / rows;
  const double heads = (double)BH * P / 8, own = (T + P - 1) / P;   // virtual heads of an XCD and their tiles: the longest, then every P-th
  const double n = (S + 63) / 64, per_tile = rows / 64;
  double head = own * n;
  if (causal && keys) head -= per_tile * P * own * (own - 1) / 2;
  else if (causal) head = n + per_tile * ((own - 1) * T - P * own * (own - 1) / 2);
  return Share{own * heads, n, head * heads};
}
// Time of a pass whose workgroups go `slots` at a time per XCD, `per_step` for a step and `start` for a workgroup's first loads, its last
// tile and its results.  No mask: whole rounds of equal workgroups.  Causal: the longest workgroup, or the average of a slot if that
// is more (the longest go first).  The unit is a step of a 256-row workgroup.
inline double pass_time(const Share& w, bool causal, int slots, double per_step, double start) {
  const double rounds = std::ceil(w.blocks / slots);
  return per_step * (causal ? std::max(w.longest, w.steps / slots) : rounds * w.longest) + start * rounds;
}
inline double whole_rows_time(int BH, int S, bool causal) { return pass_time(share(BH, S, causal, 256, false), causal, 32, 1., 4.); }
inline double split_rows_time(int BH, int S, bool causal) { return pass_time(share(BH, S, causal, 128, false), causal, 32, 0.55, 4.5); }

// Whether a pass takes 128-row tiles with the keys split over two groups of waves instead of 256-row tiles.  A split workgroup needs little
// more than half of a whole one's time per key tile, a little more for its start and end, and there are twice as many: it pays where
// whole tiles leave compute units idle, or where they fill a round or an XCD badly.  Over 174 shapes (1 to 2048 heads, 65 to 32k tokens; forward
// at head dimension 128, dQ at both) the rule costs 0.2-0.3 % against the faster variant of each, 10 % at worst (252 x 761 causal).
// Whole -> split, us, forward / dQ (or the whole backward, b) at head dimension 128:
//   causal: 12 heads x 1500 39.0 -> 24.9 / 49 -> 31.5; 2 x 32k 708 -> 527 / 904 -> 693; 64 x 1024 32.4 -> 29.7; 500 x 200 59 -> 41 / b 182 -> 157;
//     128 x 512 21.9 -> 24.0; 256 x 256 19.4 -> 23.4 / b 77.7 -> 81.0; 16 x 8192 255 -> 282 / 339 -> 364; 256 x 2048 316 -> 367 / b 1353 -> 1394.
//   no mask: 32 x 1024 30.3 -> 22.3; 7 x 9000 446 -> 286 / b 1079 -> 875; 36 x 1700 94 -> 64; 12 x 8192 412 -> 399 / 533 -> 522;
//     275 x 987 341 -> 229 / b 824 -> 658;
//     32 x 1500 43.9 -> 53.8; 21 x 1216 38.5 -> 45.9; 120 x 3637 775 -> 848; 512 x 1024 301 -> 342; 36 x 16568 4585 -> 5196 / b 15128 -> 15659.
inline bool split_rows(int BH, int S, bool causal) {
  return split_rows_time(BH, S, causal) < whole_rows_time(BH, S, causal);
}

// The forward at head dimension 64 always splits: two split workgroups fit a compute unit (LDS and registers), where a whole one takes it
// alone, so the split is the faster one on full grids too.  Whole -> split, us: causal 267 heads x 209 75 -> 35, 962 x 40 48 -> 37, 512 x 1024
// 144 -> 116, 256 x 2048 204 -> 184, 64 x 8192 626 -> 609, 2 x 512 13.3 -> 10.0; no mask 2048 x 256 82 -> 68, 512 x 1024 175 -> 169, 16 x 32k
// 4614 -> 4547; at worst, where whole tiles just fill the chip, 128 x 300 11.4 -> 12.6, 32 x 2048 41.7 -> 42.6.  So at this head dimension O and
// LSE of a head depend on nothing but the head.
constexpr bool kForwardSplitsAlways(int D) { return D == 64; }
inline bool split_forward(int D, int BH, int S, bool causal) { return kForwardSplitsAlways(D) || split_rows(BH, S, causal); }

// Head dimension 64: whether two groups of waves share the query tiles of a key tile in the dK/dV pass, and that pass its launch with
// the dQ pass on split tiles (a launch of its own is what the stage calls make of it).  With one group a SIMD has one wave, which
// is bound by instruction issue, unless a second workgroup finds room beside it; two groups halve the sweep, and the common launch fills
// the compute units that a small grid or its last round leaves idle and saves a start.  Where the chip is full both only cost: the swap of
// partial sums, and one workgroup in the place of two.  The times of both ways, fitted to the whole backward at 282 shapes (2 to 2048
// heads, 20 to 32k tokens): the rule costs 0.4 % against the best of all variants, 6 % at worst.
// Separate passes (the faster way) -> one launch, us, key tiles in brackets:
//   causal: 2 heads x 512 [8] 33.7 -> 23.1; 12 x 1500 [144] 64 -> 44; 32 x 1024 [256] 51 -> 41; 32 x 1500 [384] 72.5 -> 70.5; 4 x 16k [512]
//     486 -> 484 (533 with one group); 60 x 900 [480] 69 -> 73; 128 x 512 [512] 51 -> 55; 256 x 256 [512] 43 -> 48; 256 x 2048 [4096] 730 -> 811.
//   no mask: 2 x 512 [8] 26.7 -> 16.2; 27 x 777 [189] 40.5 -> 39; 2 x 16k [256] 446 -> 443; 24 x 1500 [288] 80.5 -> 74; 40 x 1500 [480]
//     94 -> 102; 64 x 1024 [512] 72 -> 79; 24 x 3000 [576] 248 -> 214; 10 x 8192 [640] 626 -> 563; 11 x 8192 [704] 634 -> 649; 190 x 400 [760]
//     74 -> 81; 8 x 17920 [1120] 2244 -> 2128; 160 x 1024 [1280] 173 -> 187; 512 x 300 [1536] 102 -> 120; 80 x 6528 [4080] 2756 -> 2841.
inline bool two_query_groups(int BH, int S, bool causal) {
  const Share k = share(BH, S, causal, 128, true), q = share(BH, S, causal, 128, false);
  // one group: two workgroups beside one another on a compute unit, 1.6 a step; one alone takes 0.7 of that
  const double rest = std::fmod(k.blocks, 64.);
  double one = std::floor(k.blocks / 64) * (1.6 * k.longest + 6.) + (rest == 0. ? 0. : (rest <= 32. ? 0.7 : 1.) * 1.6 * k.longest + 6.);
  if (causal) one = 1.6 * std::max(0.7 * k.longest, k.steps / 64) + 6. * std::ceil(k.blocks / 64);
  const double separate = one + std::min(split_rows_time(BH, S, causal), whole_rows_time(BH, S, causal)) + 6.;   // a second launch
  // together: key tiles, 0.85 a step, then query tiles, 0.55; no mask: rounded up to a whole query tile
  const double query = 0.55 * q.longest + 4.5;
  const double work = 0.85 * k.steps + 8. * k.blocks + 0.55 * q.steps + 4.5 * q.blocks;
  const double together = causal ? std::max(0.85 * k.longest + 8., work / 32) : query * std::ceil(work / 32 / query);
  return together < separate;
}
inline bool split_dq(int D, int BH, int S, bool causal) {
  return (D == 64 && two_query_groups(BH, S, causal)) || split_rows(BH, S, causal);
}

}  // namespace helix
