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

// ---------------------------------------------------------------- which variant a pass takes
//
// Every variant has a time model of a few figures, fitted to its own times over 4700 random shapes (1 to 160, now and then 1000, heads, 48 to 131072
// tokens), and a launch takes the variant with the least.  With tile_place every XCD gets the same tiles, so an XCD's share is known.

// The workgroups of a pass on one XCD: `heads` heads (a fraction where XCDs share them) of T tiles each, the longest of every head, the second longest
// of every head, ...  `keys`: tiles of the dK/dV pass, which sweep the query rows from their first key on; else of query rows, which sweep the keys up
// to their last row.  Lengths in steps of 64 rows or keys.
struct XcdShare {
  bool causal, keys;
  int T, per_tile;             // tiles of a head, steps by which neighbouring tiles differ
  long long count;             // workgroups
  double heads, longest, mb;   // mb: what the pass reads and writes, MB: two tensors once, two by every XCD that a head's tiles are spread over
  XcdShare(int D, int BH, int S, bool causal_, int rows, bool keys_)
      : causal(causal_), keys(keys_), T((S + rows - 1) / rows), per_tile(rows / 64), count(grid_blocks(BH, T) / 8), heads(BH / 8.), longest((S + 63) / 64),
        mb((double)BH * S * D * 2 * (2 + 2 * std::min(head_parts(BH), T)) * 1e-6) {}
  double tiles() const { return heads * T; }
  double steps() const {
    if (!causal) return tiles() * longest;
    const double less = (double)per_tile * T * (T - 1) / 2;
    return heads * (keys ? T * longest - less : longest + less);
  }
  double length(double i) const {   // of the i-th longest tile of a head
    i = std::min(std::floor(i), T - 1.);
    return !causal || i == 0. ? longest : keys ? longest - per_tile * i : per_tile * (T - i);
  }
};
// us of a workgroup: per step with the chip full and with a compute unit (almost) to itself, and for its start and end; `tail`: the share of an average tile
// that causal tiles of unequal lengths leave idle at the end; us for a MB of XcdShare::mb.
struct Cost { double step, alone, fixed, tail, mb; };

// A pass whose workgroups have a compute unit each (32 on an XCD).  Without a mask all take equally long: whole rounds, the last one quicker the emptier it
// is.  Causal ones go longest first: the average of a compute unit or, if that is more, what the longest take where k of them have to share one.
inline double pass_time(const XcdShare& w, const Cost& c) {
  const double mb = c.mb * w.mb;
  if (!w.causal) {
    const double rounds = (double)((w.count - 1) / 32), rest = w.count - 32 * rounds;
    return rounds * (c.step * w.longest + c.fixed) + (c.alone + (c.step - c.alone) * rest / 32) * w.longest + c.fixed + mb;
  }
  const double step = c.alone + (c.step - c.alone) * std::min(1., w.count / 32.), work = step * w.steps() + c.fixed * w.tiles();
  double t = work / 32 + c.tail * work / w.tiles();
  for (int k = 0; k < 3 && 32 * k < w.count; k++) t = std::max(t, (k + 1) * (step * w.length(32 * k / w.heads) + c.fixed));
  return t + mb;
}
// A pass whose workgroups share a compute unit in pairs: up to 32 of them on an XCD have one alone.
inline double paired_time(const XcdShare& w, const Cost& c) {
  const double mb = c.mb * w.mb;
  if (!w.causal) {
    const double rounds = (double)((w.count - 1) / 64), rest = w.count - 64 * rounds;
    return rounds * (c.step * w.longest + c.fixed) + (rest <= 32 ? c.alone : c.step) * w.longest + c.fixed + mb;
  }
  const double pairs = std::min(1., std::max(0., (w.count - 32) / 32.)), step = c.alone + (c.step - c.alone) * pairs;
  const double work = step * w.steps() + c.fixed * w.tiles();
  double t = work / (32 + 32 * pairs) + c.tail * work / w.tiles();
  for (int k = 0; k < 3 && 64 * k < w.count; k++) t = std::max(t, (k + 1) * ((k == 0 ? c.alone : step) * w.length(64 * k / w.heads) + c.fixed));
  return t + mb;
}

// Rows of a query tile: 256 with a wave for every 32 rows, or 128 or 64 with the keys split over two groups of waves, or 64 over four.
enum class Rows { k256, k128, k64, k64Quad };
inline int tiles(int S, Rows r) { const int n = r == Rows::k256 ? 256 : r == Rows::k128 ? 128 : 64; return (S + n - 1) / n; }

// The forward.  A 128-row workgroup needs a little more than half of a 256-row one's time for a step and more for its start and end, and there are twice as
// many: it pays where 256-row ones leave compute units idle or fill a round badly.  Narrow workgroups of 64 rows and four waves, one to a SIMD, start and end
// sooner still; with the keys over four groups (eight waves, a merge of four) they have half the steps.  The arithmetic of a row is the same with 128 and
// with 64 rows, bit for bit; 256 rows and four groups have reference maxima of their own.
// Head dimension 128, 256 / 128 / 64 / 64 in four groups, us:
//   causal: 3 x 300 - / - / 8.25 / 8.6; 12 x 1500 36 / 24.9 / 21.4 / 18.7; 42 x 384 10.8 / 10.8 / 9.4 / 9.4; 38 x 949 26.4 / 22.1 / 27.4 / 27.8; 34 x 960 25.7 / 20.3 /
//     21.7 / 21.3; 155 x 203 11.6 / 14.8 / 17.5 / 19.5; 128 x 512 19.8 / 23.4 / 30.5 / 31.4; 2 x 32k 733 / 538 / 797 / 618; 16 x 16k 960 / 1063 / 1483 / 1244.
//   no mask: 7 x 1104 28.7 / 20.1 / 17.4 / 15.4; 12 x 1500 36.8 / 25.6 / 41 / 35; 11 x 2246 54 / 38.8 / 58 / 49; 101 x 851 60 / 61 / 87 / 80; 33 x 1984 110 / 103 / 99.7 / 91.2;
//     36 x 4096 329 / 326 / 441 / 362; 512 x 1024 284 / 358 / 501 / 487.
// Head dimension 64 never takes 256 rows: two 128-row workgroups share a compute unit (80 KB of LDS each, as the 64-row ones), where a 256-row one takes it
// alone.  128 / 64 rows, us: causal 2 x 512 8.8 / 7.2; 54 x 563 10.3 / 9.1; 60 x 896 15.1 / 16.4; 16 x 16k 600 / 690; no mask 6 x 5164 55.7 / 58.6; 10 x 819 12.0 / 9.9;
// 27 x 777 13.1 / 14.2; 148 x 143 8.4 / 6.5; 120 x 1181 60.9 / 67.1.
// Over all shapes the choice is 0.15 (head dimension 128, causal) and less than 0.1 % (no mask; 64) off the fastest variant.
inline Rows forward_rows(int D, int BH, int S, bool causal) {
  static constexpr Cost at128[2][4] = {{{1.6, 1.46, 3.97, 0, .0213}, {.932, .7, 5.63, 0, .0246}, {.706, .653, 4.2, 0, .0216}, {.549, .464, 5.49, 0, .0228}},
                                       {{1.52, 1.4, 4.49, .29, 0}, {.917, .629, 5.74, .15, .0115}, {.734, .592, 4.38, .183, .0257}, {.571, .372, 5.83, .219, .0158}}};
  static constexpr Cost at64[2][2] = {{{1.05, .565, 3.97, 0, .0249}, {.647, .418, 3.65, 0, .0401}}, {{1.09, .65, 4.09, .181, .0204}, {.652, .464, 3.68, .0707, .0238}}};
  const XcdShare wide(D, BH, S, causal, 128, false), narrow(D, BH, S, causal, 64, false);
  if (D == 64) return paired_time(narrow, at64[causal][1]) < paired_time(wide, at64[causal][0]) ? Rows::k64 : Rows::k128;
  const Cost* const c = at128[causal];
  const double t[4] = {pass_time(XcdShare(D, BH, S, causal, 256, false), c[0]), pass_time(wide, c[1]), pass_time(narrow, c[2]), pass_time(narrow, c[3])};
  return (Rows)(std::min_element(t, t + 4) - t);
}

// Delta of the first rows, likewise (S: the rows it is wanted for).  Its causal times serve full attention too, for which the backward does not ask for it.  The same bits
// with every one.  256 / 128 / 64 rows, us, head dimension 128: 2 x 512 14.5 / 9.8 / 8.1; 16 x 2048 45 / 28.4 / 26.8; 38 x 949 26 / 18.8 / 22.7; 64 x 2048 69 / 76 / 107;
// 128 x 512 19.9 / 19.5 / 24.8.  Head dimension 64, where two 64-row workgroups share a compute unit and 128 rows are not built (the fastest at 28 of 803 shapes, by 8 % at
// most): 2 x 512 10.6 / 8.0 / 6.1; 16 x 2048 32 / 21.8 / 16.6; 60 x 896 15.9 / 14.9 / 14.2; 256 x 256 8.0 / 9.8 / 8.7; 64 x 2048 43 / 51 / 47.
// 0.2 % off the fastest, at worst 1.25 times its time (99 x 404 x 64 12.3 for 9.8).
inline Rows delta_rows(int D, int BH, int S, bool causal) {
  static constexpr Cost at128[3] = {{1.46, 1.21, 3.53, .216, .0155}, {.827, .666, 3.94, .118, .027}, {.6, .598, 3.03, .201, .0372}};
  static constexpr Cost at64[2] = {{1.01, .799, 3.42, .177, .0084}, {.526, .444, 2.61, .19, .0218}};
  const XcdShare wide(D, BH, S, causal, 256, false), narrow(D, BH, S, causal, 64, false);
  if (D == 64) return paired_time(narrow, at64[1]) < pass_time(wide, at64[0]) ? Rows::k64 : Rows::k256;
  const double t[3] = {pass_time(wide, at128[0]), pass_time(XcdShare(D, BH, S, causal, 128, false), at128[1]), pass_time(narrow, at128[2])};
  return (Rows)(std::min_element(t, t + 3) - t);
}

// ---- the gradients

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


// Narrow workgroups: 64 rows (or keys) and four waves, one per SIMD, in the place of 128 and eight.  A wave that has its SIMD to itself takes a step
// in about 0.85 of the time that two side by side take theirs in, so that where narrow workgroups find compute units of their own every one of them
// ends earlier; beyond that they only cost.  The arithmetic of a row is that of the 128-row workgroups, bit for bit.
//
// dK/dV and dQ: in their common launch, where 64-key and 64-row workgroups take their turns on the compute units.  Without a mask all take equally long, and
// the launch has to fit (half of the chip for either); causal ones differ in length and fill each other's gaps.  Over 420 shapes 0.3 %
// (head dimension 128, causal), 1.2 (no mask), 0.8 and 1.6 % (head dimension 64) off the better choice; at worst 10 x 819 x 64 without a mask 23.4 for 19.3 us.  128 -> 64, whole backward, us, 64-row
// tiles in brackets: causal 2 heads x 512 x 64 [16] 19.6 -> 17.1, 2 x 512 x 128 28 -> 22.8, 4 x 2048 [128] 75 -> 60, 2 x 8192 [256] 205 -> 167,
// 12 x 1500 [288] 62 -> 65, 16 x 2048 [512] 97 -> 109; no mask 4 x 2048 [128] 49 -> 38, 5 x 4187 [330] 187 -> 186, 27 x 777 x 64 [351] 37 -> 48.
inline bool narrow_gradients(int BH, int S, bool causal) {
  const long long tiles_64 = (long long)BH * ((S + 63) / 64);
  return tiles_64 <= (causal ? 288 : 128);
}

inline Rows dq_rows(int D, int BH, int S, bool causal) {
  return narrow_gradients(BH, S, causal) ? Rows::k64 : split_dq(D, BH, S, causal) ? Rows::k128 : Rows::k256;
}
inline int key_tile(int BH, int S, bool causal) { return narrow_gradients(BH, S, causal) ? 64 : 128; }

}  // namespace helix
