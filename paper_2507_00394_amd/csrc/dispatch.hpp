// Which tile a workgroup takes, and which variant of a pass a launch takes, as functions of the shape alone.  Plain host arithmetic (what the device
// code shares is constexpr), free of HIP, so that a test without a GPU can compile it, count the tiles and hold every rule against the times it was
// read from.
#pragma once
#include <algorithm>
#include <cmath>

namespace helix {

// A launch's tiles are dealt to the 8 XCDs (workgroup id mod 8) in groups of P XCDs, P the smallest power of two that makes BH * P a multiple
// of 8: a group has BH * P / 8 heads of its own, so that no XCD idles whatever the number of heads - with 32 heads a group is an XCD, with the 4
// or 5 heads of one GPU's share of a tensor-parallel layer (Section 2.2) it is 2 or all 8 of them.
constexpr int head_parts_log2(int BH) { return (BH & 1) ? 3 : (BH & 2) ? 2 : (BH & 4) ? 1 : 0; }
constexpr int head_parts(int BH) { return 1 << head_parts_log2(BH); }
// Number of workgroups to launch for BH slices of T tiles: one for a tile, rounded up to the same number on every XCD.
constexpr long long grid_blocks(int BH, int T) { return ((long long)BH * T + 7) / 8 * 8; }

// The tile of workgroup n: slice `head`, the `rank`-th heaviest of its T tiles.
//
// A group's tiles form one running sequence, head after head, heaviest tiles first.  Its P XCDs take the sequence P tiles at a time, every
// other time backwards, so that none of them gets the heavier tile each time.  Only the last few workgroups of the grid are without a tile.
// (With a head's T tiles padded to a multiple of P the empty workgroups stand between the others and the tiles that they push into a compute unit's second round
// cost up to a third.  Padded, parts fixed / padded, parts rotating / one sequence, us, head dimension 128 unless said: forward 11 heads x 1399 no mask 34 /
// 18 / 17.9; 33 x 1984 no mask 104 / 108 / 89.5; 42 x 384 causal 12.9 / 14.5 / 9.8; 76 x 180 causal 8.5 / 10.0 / 7.4; 22 x 3840 x 64 no mask 105.5 / 110.8 / 105.6; 68 x
// 1080 x 64 no mask 36.1 / 37.9 / 34.8; backward 9 x 888 x 64 no mask 23.0 / 24.5 / 16.2.  Over 784 random shapes with BH no multiple of 8, time against
// rotating parts: forward 0.92, backward 0.90.)
//
// Causal tiles differ in length, so an XCD that takes its heads one after the other starts
// the longest tiles of the last one when hardly anything is left to fill the other compute units.
// The last heads therefore go side by side, all of their heaviest tiles first: as many as
// hold about four rounds of workgroups for the 32 compute units of an XCD, two at least.  More of
// them only cost L2 hits (4 instead of 2 at 32 heads x 32k tokens: dK/dV 4 % slower), fewer leave the
// imbalance.  One head after the other -> this rule, forward / dQ, us: 4 x 16 heads x 2k tokens 99 -> 77 /
// 132 -> 101; 5 x 32k 1472 -> 1249 / 1997 -> 1733; 24 x 4k 131 -> 108 / 174 -> 147; 32 x 32k 7552 -> 7441 /
// 10272 -> 10128.  Without a mask all tiles are equal and heads stay one after the other.
//
// Head dimension 128 with three or five tiles of a head to an XCD: only as many heads as hold about one and a half rounds.  Two or four tiles pair up,
// a long one of one head with a short one of another, and fill whole rounds; of an odd number one is left without a partner, so more heads
// side by side even nothing out and cost L2 hits.  One head after the other / four rounds / one and a half, forward, us: 272 heads x
// 570 59 / 73 / 55; 344 x 700 82 / 101 / 81; 360 x 520 72 / 74 / 65; 248 x 620 54 / 65 / 52; whole backward 272 x 570 225 / 247 / 208.  Over 43
// shapes with such heads the forward takes 0.93 of the time of four rounds, the backward 0.97.  At head dimension 64, where two workgroups
// share a compute unit, four rounds are the better choice there too (532 x 640 forward 69.6 / 65.4, backward 330 / 285).
struct TilePlace { int head, rank; bool valid; };
constexpr TilePlace tile_place(int n, int BH, int T, bool causal, int D) {
  const int l = head_parts_log2(BH), P = 1 << l;
  const int xcd = n & 7, s = n >> 3, part = xcd & (P - 1);
  const int m = (s << l) + ((s & 1) ? P - 1 - part : part);   // place in the group's sequence
  const int heads = (int)(((long long)BH << l) >> 3);         // of the group: xcd / P, and every 8 / P-th one after it
  int v = m / T, rank = m - v * T;
  if (causal) {
    const int per_xcd = (T + P - 1) >> l;                     // tiles of a head on an XCD
    const int blocks = D == 128 && (per_xcd == 3 || per_xcd == 5) ? 48 : 128;
    const int wanted = per_xcd >= 64 ? 2 : blocks / per_xcd;
    const int side = heads < wanted ? heads : wanted, m2 = m - (heads - side) * T;
    if (m2 >= 0) {
      rank = m2 / side;
      v = heads - side + m2 - rank * side;
    }
  }
  return TilePlace{(v << (3 - l)) + (xcd >> l), rank, m < heads * T};
}

// The workgroups of a launch on the fullest XCD (32 compute units): `heads` virtual heads with `own` tiles each, the longest of every
// head, the second longest of every head, ...  `keys`: tiles of the dK/dV pass, which sweep the query rows from their first key on;
// else of query rows, which sweep the keys up to their last row.  Lengths in steps of 64 rows or keys.
struct Share {
  bool causal, keys;
  int P, T, per_tile;          // parts of a head, tiles of a head, steps by which neighbouring tiles differ
  double heads, own, longest;
  // `even`: an average XCD's share in the place of the fullest one's (a fraction of a tile where T is no multiple of P).
  Share(int BH, int S, bool causal_, int rows, bool keys_, bool even = false)
      : causal(causal_), keys(keys_), P(head_parts(BH)), T((S + rows - 1) / rows), per_tile(rows / 64), heads((double)BH * P / 8),
        own(even ? (double)T / P : (T + P - 1) / P), longest((S + 63) / 64) {}
  double blocks() const { return own * heads; }
  double length(double i) const {   // of the i-th longest tile of a head
    if (!causal || i == 0.) return longest;
    return keys ? longest - per_tile * P * i : per_tile * (T - P * i);
  }
  double steps() const {
    if (!causal) return blocks() * longest;
    return heads * (keys ? own * longest - per_tile * P * own * (own - 1) / 2 : longest + per_tile * ((own - 1) * T - P * own * (own - 1) / 2));
  }
};
// Time of a pass whose workgroups go `slots` at a time, `per_step` for a step and `start` for a workgroup's first loads, its last tile and its
// results, the longest first: the average of a slot or, if that is more, what the longest ones take where k of them cannot help
// sharing a slot.  Without a mask all are equal, and that is whole rounds.  The unit is a step of a 256-row workgroup.
inline double pass_time(const Share& w, int slots, double per_step, double start) {
  const double rounds = std::ceil(w.blocks() / slots - 1e-9);
  double t = (per_step * w.steps() + start * w.blocks()) / slots;
  if (!w.causal) return std::max(t, rounds * (per_step * w.longest + start));
  for (int k = 0; k < 3 && k < rounds; k++) t = std::max(t, (k + 1) * (per_step * w.length(std::floor(k * slots / w.heads)) + start));
  return t;
}
inline double whole_rows_time(int BH, int S, bool causal) { return pass_time(Share(BH, S, causal, 256, false), 32, 1., 3.5); }
inline double split_rows_time(int BH, int S, bool causal) { return pass_time(Share(BH, S, causal, 128, false), 32, 0.58, 4.5); }

// Whether a pass takes 128-row tiles with the keys split over two groups of waves instead of 256-row tiles.  A split workgroup needs little
// more than half of a whole one's time per key tile, a little more for its start and end, and there are twice as many: it pays where
// whole tiles leave compute units idle, or where they fill a round or an XCD badly.  Over 467 shapes (1 to 2048 heads, 65 to 32k tokens; forward
// at head dimension 128, dQ at both) the rule costs 0.4 and 0.2 % against the faster variant of each, more than 10 % at four forward ones:
// 416 x 304 without a mask 64 for 52 us; causal 472 x 381 67 for 60, 252 x 761 95 for 86, 66 x 2521 166 for 151.
// Whole -> split, us, forward / dQ (or the whole backward, b) at head dimension 128:
//   causal: 12 heads x 1500 39.0 -> 24.9 / 49 -> 31.5; 2 x 32k 708 -> 527 / 904 -> 693; 64 x 1024 32.4 -> 29.7; 500 x 200 59 -> 41 / b 182 -> 157;
//     78 x 589 39.9 -> 32.7; 66 x 768 53 -> 41;
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
// partial sums, and one workgroup in the place of two.  The times of both ways, fitted to the whole backward at 465 shapes (1 to 2048
// heads, 20 to 32k tokens): the rule costs 0.3 % against the best of all variants, 10 % at worst.
// Separate passes (the faster way) -> one launch, us, key tiles in brackets:
//   causal: 2 heads x 512 [8] 33.7 -> 23.1; 12 x 1500 [144] 64 -> 44; 32 x 1024 [256] 51 -> 41; 32 x 1500 [384] 72.5 -> 70.5; 4 x 16k [512]
//     486 -> 484 (533 with one group); 60 x 900 [480] 69 -> 73; 128 x 512 [512] 51 -> 55; 256 x 256 [512] 43 -> 48; 256 x 2048 [4096] 730 -> 811.
//   no mask: 2 x 512 [8] 26.7 -> 16.2; 27 x 777 [189] 40.5 -> 39; 2 x 16k [256] 446 -> 443; 24 x 1500 [288] 80.5 -> 74; 40 x 1500 [480]
//     94 -> 102; 64 x 1024 [512] 72 -> 79; 24 x 3000 [576] 248 -> 214; 10 x 8192 [640] 626 -> 563; 11 x 8192 [704] 634 -> 649; 190 x 400 [760]
//     74 -> 81; 8 x 17920 [1120] 2244 -> 2128; 160 x 1024 [1280] 173 -> 187; 512 x 300 [1536] 102 -> 120; 80 x 6528 [4080] 2756 -> 2841.
inline bool two_query_groups(int BH, int S, bool causal) {
  const Share k(BH, S, causal, 128, true), q(BH, S, causal, 128, false);
  // one group: two workgroups beside one another on a compute unit, 1.6 a step; one alone takes 0.7 of that
  const double beside = 1.6 * k.longest + 7., alone = 0.7 * 1.6 * k.longest + 7., rest = std::fmod(k.blocks(), 64.);
  const double one = causal ? std::max((1.6 * k.steps() + 7. * k.blocks()) / 64, alone)
                            : std::floor(k.blocks() / 64) * beside + (rest == 0. ? 0. : rest <= 32. ? alone : beside);
  const double separate = one + std::min(split_rows_time(BH, S, causal), whole_rows_time(BH, S, causal)) + 7.;   // a second launch
  // together: key tiles, 0.8 a step, then query tiles, 0.55; no mask: rounded up to a whole query tile
  const double query = 0.55 * q.longest + 5.2;
  const double work = (0.8 * k.steps() + 10. * k.blocks() + 0.55 * q.steps() + 5.2 * q.blocks()) / 32;
  const double together = causal ? std::max(work, pass_time(k, 32, 0.8, 10.)) : query * std::ceil(work / query);
  return together < separate;
}
inline bool split_dq(int D, int BH, int S, bool causal) {
  return (D == 64 && two_query_groups(BH, S, causal)) || split_rows(BH, S, causal);
}


// Rows of a query tile: 256 with a wave for every 32 rows, or 128 or 64 with the keys split over two groups of waves, or 64 over four.
enum class Rows { k256, k128, k64, k64Quad };
inline int tiles(int S, Rows r) { const int n = r == Rows::k256 ? 256 : r == Rows::k128 ? 128 : 64; return (S + n - 1) / n; }

// Narrow workgroups: 64 rows (or keys) and four waves, one per SIMD, in the place of 128 and eight.  A wave that has its SIMD to itself takes a step
// in about 0.85 of the time that two side by side take theirs in, so that where narrow workgroups find compute units of their own every one of them
// ends earlier; beyond that they only cost.  The arithmetic of a row is that of the 128-row workgroups, bit for bit.
//
// Delta of the first rows: by the time on an average XCD, as above but with the tiles spread evenly, as the order of map_block does by now.  Over 145
// and 149 shapes (head dimension 128 and 64) the choice is 0.4 and 0.1 % off the fastest.  128 -> 64 rows, us: head dimension 128 12 heads x 1500
// 22.2 -> 17.9, 16 x 2048 29.7 -> 27.8, 64 x 2048 84 -> 116; head dimension 64 16 x 16384 23.3 -> 18.9.
// Narrow tiles that just fit the compute units at once do not where T is no multiple of P: workgroups without a tile are dealt out between
// the others, some compute units get two in their place, and without a mask that is a second round (11 heads x 1399 34 us for the 18 of one).
inline double rows_time(int BH, int S, bool causal, int rows, int slots, double per_step, double start) {
  const Share even(BH, S, causal, rows, false, true), fullest(BH, S, causal, rows, false);
  return pass_time(!causal && rows == 64 && slots == 32 && even.blocks() <= slots && fullest.blocks() > slots ? fullest : even, slots, per_step, start);
}
inline bool narrow_delta(int D, int BH, int S, bool causal) {
  const double wide = std::min(rows_time(BH, S, causal, 128, 32, 0.58, 4.5), rows_time(BH, S, causal, 256, 32, 1., 3.5));
  return (D == 64 ? rows_time(BH, S, causal, 64, 48, 0.42, 2.) : rows_time(BH, S, causal, 64, 32, 0.52, 3.2)) < wide;
}
// The forward at head dimension 64 shares a compute unit between two wide or more narrow workgroups, at a rate that grows with every one but less than
// in step, hence slots that are more than the compute units and no whole number of them.  Fitted to 441 shapes (1 to 200 heads, 65 to 6600 tokens, up to 4000 tiles of 64 rows), a
// wrong narrow choice counted three times: 1.4 (no mask) and 0.5 % (causal) off the faster one.  Narrow is at worst 1.11 times the wide one's time where it is taken (148 heads x 143 without a mask 8.8 / 9.8 us, causal 54 x 563 11.2 / 11.6), and
// where it is not, 0.72 (6 x 5164 79.8 / 57.7).  128 -> 64 rows, us, taken: 2 x 512 9.3 -> 7.6, 12 x 1500 18.7 -> 15.2; not: 120 x 1181 without a
// mask 64.5 -> 73.9, 60 x 896 15.8 -> 18.1, 16 x 16384 612 -> 693.
inline bool narrow_forward_64(int BH, int S, bool causal) {
  return causal ? rows_time(BH, S, true, 64, 64, 0.52, 3.8) < rows_time(BH, S, true, 128, 88, 0.58, 4.5)
                : rows_time(BH, S, false, 64, 48, 0.39, 2.1) < rows_time(BH, S, false, 128, 88, 0.58, 4.9);
}

// dK/dV and dQ: in their common launch, where 64-key and 64-row workgroups take their turns on the compute units.  Without a mask all take equally long, and
// the launch has to fit (half of the chip for either); causal ones differ in length and fill each other's gaps.  Over 420 shapes 0.3 %
// (head dimension 128, causal), 1.2 (no mask), 0.8 and 1.6 % (head dimension 64) off the better choice; at worst 10 x 819 x 64 without a mask 23.4 for 19.3 us.  128 -> 64, whole backward, us, 64-row
// tiles in brackets: causal 2 heads x 512 x 64 [16] 19.6 -> 17.1, 2 x 512 x 128 28 -> 22.8, 4 x 2048 [128] 75 -> 60, 2 x 8192 [256] 205 -> 167,
// 12 x 1500 [288] 62 -> 65, 16 x 2048 [512] 97 -> 109; no mask 4 x 2048 [128] 49 -> 38, 5 x 4187 [330] 187 -> 186, 27 x 777 x 64 [351] 37 -> 48.
inline bool narrow_gradients(int BH, int S, bool causal) {
  const long long tiles_64 = (long long)BH * ((S + 63) / 64);
  return tiles_64 <= (causal ? 288 : 128);
}

// The forward at head dimension 128 has both, narrow workgroups with two key groups, which start and end sooner, and eight waves in four, which have half the
// steps.  Over 519 shapes the choice among all four is 1.1 % (causal) and 1.9 % (no mask) off the fastest; at worst short sequences of many heads, 155 x 203
// 31 for 24 us, and full grids that miss a round by little, 101 x 851 without a mask 81 for 59.  256 / 128 / 64 / 64 in four groups, us: causal
// 4 heads x 1124 25.5 / 19.9 / 17.3 / 14.9, 12 x 1500 39 / 25.2 / 21.4 / 19.4, 2 x 8192 - / 107 / 91 / 70, 3 x 300 - / - / 8.25 / 8.6, 52 x 543 18.0 / 19.4 / 19.4 / 21.1.
inline Rows forward_rows(int D, int BH, int S, bool causal) {
  if (kForwardSplitsAlways(D)) return narrow_forward_64(BH, S, causal) ? Rows::k64 : Rows::k128;
  const double wide = std::min(rows_time(BH, S, causal, 256, 32, 1., 3.5), rows_time(BH, S, causal, 128, 32, 0.58, 4.5));
  const double narrow = rows_time(BH, S, causal, 64, 32, 0.52, 3.2), quad = rows_time(BH, S, causal, 64, 32, 0.38, 4.5);
  if (std::min(narrow, quad) < wide) return quad < narrow ? Rows::k64Quad : Rows::k64;
  return split_forward(D, BH, S, causal) ? Rows::k128 : Rows::k256;
}
inline Rows delta_rows(int D, int BH, int S, bool causal) {
  return narrow_delta(D, BH, S, causal) ? Rows::k64 : split_rows(BH, S, causal) ? Rows::k128 : Rows::k256;
}
inline Rows dq_rows(int D, int BH, int S, bool causal) {
  return narrow_gradients(BH, S, causal) ? Rows::k64 : split_dq(D, BH, S, causal) ? Rows::k128 : Rows::k256;
}
inline int key_tile(int BH, int S, bool causal) { return narrow_gradients(BH, S, causal) ? 64 : 128; }

}  // namespace helix
