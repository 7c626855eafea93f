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
// The dK/dV and the dQ pass in one launch: key tiles first, then query tiles, a compute unit each.  `sparse`: a step's time with the chip nearly empty
// over that with it full.
struct CommonCost { double key_step, key_fixed, query_step, query_fixed, tail, sparse, mb; };
inline double common_time(const XcdShare& k, const XcdShare& q, const CommonCost& c) {
  const double f = c.sparse + (1 - c.sparse) * std::min(1., (k.tiles() + q.tiles()) / 32), ks = c.key_step * f, qs = c.query_step * f;
  const double key = ks * k.longest + c.key_fixed, query = qs * q.longest + c.query_fixed, mb = c.mb * (k.mb + q.mb);
  if (!k.causal) {
    // Tile by tile: `late` compute units end their last key tile a key tile after the other ones, and every one takes query tiles as soon as it is free.
    // The end is that of the n-th query tile of one kind of compute unit or the other.
    const double rounds = (double)(k.count / 32), late = k.count - 32 * rounds, early = rounds * key, then = early + key;
    const auto done = [&](double t) { return late * std::max(0., std::floor((t - then) / query + 1e-9)) + (32 - late) * std::floor((t - early) / query + 1e-9); };
    double n = std::max(1., std::ceil((q.count + late * key / query) / 32) - 2), t = 1e30;
    while (done(early + n * query) < q.count) n++;
    t = early + n * query;
    if (late > 0) {
      n = std::max(0., std::ceil((q.count - (32 - late) * std::floor(key / query)) / 32) - 1);
      while (done(then + n * query) < q.count) n++;
      t = std::max(std::min(t, then + n * query), then);
    }
    return t + mb;
  }
  double t = (ks * k.steps() + c.key_fixed * k.tiles() + qs * q.steps() + c.query_fixed * q.tiles()) / 32 + c.tail * (qs * q.steps() / q.tiles() + c.query_fixed);
  for (int i = 0; i < 2 && 32 * i < k.count; i++) t = std::max(t, (i + 1) * (ks * k.length(32 * i / k.heads) + c.key_fixed));
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

// dK/dV and dQ: in a launch each, with 256 or 128 query rows to a dQ workgroup and 128 keys to a dK/dV one; in one launch likewise; or in one launch on narrow workgroups of 64 of
// either, which end sooner where the chip has room for all of them.  Head dimension 64: a launch each goes with one group of waves to a key tile, two workgroups of
// which share a compute unit; in one launch two groups share the query tiles of a key tile and end in half the time, which pays where the chip is not full.
// Both passes need the row statistics and nothing of each other, and a workgroup of either fills a compute unit in the common launch (LDS at head
// dimension 128, registers at 64), so one launch with the key tiles first fills the compute units that a small grid or its
// last, uneven round leaves idle, and pays for one start instead of two.  The work of a workgroup is that of the separate passes, bit for bit.
// A launch each 256 / 128 - together 256 / 128 / narrow, whole backward, us, head dimension 128:
//   causal: 2 x 512 44 / 39 - 28 / 26 / 20.5; 12 x 1500 98 / 82 - 66 / 57.3 / 58.8; 4 x 2048 123 / 102 - 81 / 69 / 54; 42 x 384 37 / 36 - 25.8 / 25.9 / 26.9; 16 x 2048 135 / 116 - 107 / 95 /
//     103; 128 x 512 75 / 77 - 74 / 75 / 91; 64 x 2048 309 / 318 - 304 / 313 / 368; 16 x 16k 3171 / 3272 - 3171 / 3270 / 3861; 5 x 32k 4109 / 4161 - 4100 / 4202 / -;
//     80 x 8000 3956 / 4075 - 3946 / 4062 / -; 256 x 2048 1350 / 1365 - 1320 / 1359 / -; 32 x 32k 24619 / 25399 - 24663 / 25438 / -.
//   no mask: 7 x 1104 69 / 57 - 42 / 36 / 28.7; 11 x 1399 81 / 67 - 52 / 49 / 53; 17 x 1438 93 / 81 - 95 / 80 / 99; 5 x 4187 211 / 169 - 150 / 188 / 184; 36 x 4096 1006 / 993 - 929 / 947 / 1089;
//     512 x 1024 946 / 1010 - 942 / 1015 / -; 12 x 8192 1231 / 1216 - 1246 / 1213 / 1409.
// Head dimension 64, a launch each 256 / 128 - together 128 / narrow:
//   causal: 2 x 512 31 / 27 - 17 / 15; 131 x 146 23 / 24 - 21 / 22; 54 x 563 39 / 36 - 29.5 / 36; 256 x 256 32 / 34 - 37 / 48; 4 x 16k 614 / 534 - 483 / 582; 16 x 16k 1718 / 1780 - 1834 / 2211.
//   no mask: 9 x 888 39 / 34 - 19.7 / 17.0; 10 x 819 37 / 31 - 18.9 / 22.9; 27 x 777 40 / 35 - 32 / 37; 22 x 3840 324 / 310 - 314 / 366; 120 x 1181 185 / 184 - 190 / 234.
// The choice is 0.3 (head dimension 128, causal) and 0.1 to 0.2 % (no mask; 64) off the fastest, at worst 1.19 times its time (81 x 135 causal 21.4 for 17.9).  At
// head dimension 128 a launch each is left to causal grids of more than 1024 key tiles, where one launch costs L2 hits in the change from one pass to the other: it takes
// 0.98 (up to 1500 key tiles) to 1.00 (beyond 5000) of the time on average, and up to 1.03 of it at single shapes.
enum class Gradients { kSeparate256, kSeparate128, kTogether256, kTogether128, kNarrow };
inline Gradients gradient_tiles(int D, int BH, int S, bool causal) {
  static constexpr CommonCost at128[2][3] = {{{1.65, 4.07, 2.01, 5.01, 0, .844, .0297}, {1.54, 4.97, 1.3, 4.48, 0, .861, .026}, {1.01, 4.26, .765, 4., 0, .955, .0428}},
                                             {{1.47, 6.08, 1.73, 3.01, .948, 1.02, .0166}, {1.4, 5.42, 1.43, 6.35, .0866, 1.15, .0269}, {1., 4.91, .789, 4.49, .34, .898, .0136}}};
  static constexpr CommonCost at64[2][2] = {{{.847, 4.19, .752, 2.93, 0, 1.04, .0263}, {.561, 3.62, .474, 2.73, 0, 1.12, .0355}},
                                            {{.882, 5.21, .776, 3.99, .242, 1.07, .0048}, {.608, 4.57, .422, 2.74, .597, 1.08, .0112}}};
  static constexpr Cost one_group[2] = {{1.4, .839, 4.32, 0, .0329}, {1.64, .863, 5.58, .392, .0099}}, query_256[2] = {{1.42, 1.38, 2.97, 0, .0329}, {1.24, 1.06, 4.01, 0, .0099}},
                        query_128[2] = {{.855, .699, 3.29, 0, .0329}, {.786, .824, 3.19, .503, .0099}};
  const XcdShare k128(D, BH, S, causal, 128, true), k64(D, BH, S, causal, 64, true), q256(D, BH, S, causal, 256, false), q128(D, BH, S, causal, 128, false),
      q64(D, BH, S, causal, 64, false);
  double t[5] = {1e30, 1e30, 1e30, 1e30, 1e30};
  if (D == 128) {
    if (causal && (long long)BH * k128.T > 1024) return Gradients::kSeparate256;
    t[2] = common_time(k128, q256, at128[causal][0]);
    t[3] = common_time(k128, q128, at128[causal][1]);
    t[4] = common_time(k64, q64, at128[causal][2]);
  } else {
    const double keys = paired_time(k128, one_group[causal]);
    t[0] = keys + pass_time(q256, query_256[causal]);
    t[1] = keys + pass_time(q128, query_128[causal]);
    t[3] = common_time(k128, q128, at64[causal][0]);
    t[4] = common_time(k64, q64, at64[causal][1]);
  }
  return (Gradients)(std::min_element(t, t + 5) - t);
}
inline Rows dq_rows(Gradients g) { return g == Gradients::kNarrow ? Rows::k64 : g == Gradients::kSeparate256 || g == Gradients::kTogether256 ? Rows::k256 : Rows::k128; }
inline int key_tile(Gradients g) { return g == Gradients::kNarrow ? 64 : 128; }
inline bool one_launch(Gradients g) { return g >= Gradients::kTogether256; }

// ---------------------------------------------------------------- the linear layer's tiles
//
// Square tiles of C.  As above every variant has a time model fitted to its own times, here over 3300 shapes (32 to 131072 tokens, K to 5120, N to 3072).
enum class TileKind { k256, k128, k64 };
inline int tile_edge(TileKind k) { return k == TileKind::k256 ? 256 : k == TileKind::k128 ? 128 : 64; }
inline int tile_slots(TileKind k) { return k == TileKind::k256 ? 256 : 512; }   // workgroups that the chip holds: one or two on a compute unit
// Workgroups of a product with `I` x `J` results: its tiles, rounded up to the same number on every XCD.
inline double tile_blocks(int I, int J, TileKind k) {
  const int e = tile_edge(k);
  return 8 * std::ceil(((I + e - 1) / e) * (double)((J + e - 1) / e) / 8);
}
// How far a round of n workgroups is on its way from the pace of one alone (0) to that of a full chip (1); where two share a compute unit, the step comes
// with the first pair.
inline double pace(TileKind k, double n) {
  const double x = n / tile_slots(k);
  return k == TileKind::k256 ? x : x <= 0.5 ? 0. : std::min(1., x);
}

// The forward.  us per 1000 contraction indices with the chip full and alone, for the start and end of a round and of the last one, per MB read (the weights by every
// XCD), per MB written, and for every one of those beyond `cached`, which the last cache no longer holds.
// 256 / 128 / 64, us: 64 x 2048 x 768 38.9 / 13.7 / 7.2; 2080 x 2048 x 768 40.6 / 17.4 / 13.3; 2080 x 4096 x 1536 75.0 / 36.3 / 58.7; 8192 x 2048 x 768
// 46.1 / 31.9 / 39.8; 16384 x 4096 x 1536 188 / 208 / 484; 131072 x 4096 x 1536 1310 / 1798 / 3863; 47776 x 256 x 1024 45.2 / 38.6 / 60.0; 123680 x 256
// x 2176 250 / 285 / 397.
// 0.1 % off the fastest tile, at worst 1.15 times its time (736 x 4864 x 2560 52.0 for 45.2).
inline TileKind linear_tile(int M, int K, int N) {
  struct Cost { double full, alone, round, last, mb_read, mb_written, mb_more, cached; };
  static constexpr Cost cost[3] = {{22.6, 15.3, 5.83, 6.72, .0176, .119, .0092, 314}, {16.7, 6.3, 0, 2.54, .0279, .0979, .415, 170},
                                   {6.73, 2.56, .742, 2.21, .0025, .0295, .619, 165}};
  const double k = K * 1e-3, read = ((double)M * K + 8. * K * N) * 2e-6, written = (double)M * N * 2e-6;
  double t[3];
  for (int i = 0; i < 3; i++) {
    const Cost& c = cost[i];
    const double n = tile_blocks(M, N, (TileKind)i), slots = tile_slots((TileKind)i), rounds = std::ceil(n / slots) - 1;
    t[i] = rounds * (c.full * k + c.round) + (c.alone + (c.full - c.alone) * pace((TileKind)i, n - rounds * slots)) * k + c.last + c.mb_read * read +
           c.mb_written * written + c.mb_more * std::max(0., written - c.cached);
  }
  return (TileKind)(std::min_element(t, t + 3) - t);
}

// The weight gradient has few output tiles and a long contraction (over all M tokens), so the
// contraction is cut into parts until the grid fills the chip about twice; the parts' fp32
// results go to the workspace and are summed in a fixed order (no atomics).
inline int linear_bwd_weight_parts(int M, int K, int N) {
  const long long tiles = (long long)((K + 255) / 256) * ((N + 255) / 256);
  long long parts = (512 + tiles - 1) / tiles;
  const long long most = M / 2048 > 0 ? M / 2048 : 1;      // at least 2048 tokens per part
  if (parts > most) parts = most;
  if (parts > 32) parts = 32;
  return (int)parts;
}

// The tiles of the two gradients, chosen as a pair: tiles that take a compute unit alike share a launch, the large one and a small one take one each (the input gradient on
// the small one; the other way round is not built, 5 % faster than any of these at most).  In a
// launch: the time in which the chip gets through all workgroups, that of the longest with a compute unit of its own, or somewhat more than the larger of the two
// where they are close (`sharp`), and no less than the input gradient's workgroup takes behind full rounds of others.
// Input / weight tile 256,256 - 256,128 - 128,256 - 128,128 - 128,64 - 64,256 - 64,128 - 64,64, us: 2080 x 2048 x 768 49.1 - 43.6 - 58.4 - 24.2 - 24.6 -
// 58.4 - 23.0 - 26.1; 131072 x 4096 x 1536 2825 - 3686 - 3903 - 4460 - 6929 - 5061 - 5669 - 8151; 352 x 4608 x 2560 63.0 - 79.2 - 49.0 - 51.1 - 48.9 -
// 43.4 - 44.4 - 45.7; 14880 x 128 x 2688 63.5 - 78.0 - 77.3 - 50.1 - 54.6 - 68.8 - 44.0 - 50.5; 92352 x 896 x 896 378 - 425 - 411 - 439 - 525 - 481 -
// 512 - 599; 82720 x 1792 x 256 268 - 288 - 269 - 293 - 329 - 325 - 351 - 383; 47776 x 256 x 1024 95.4 - 89.3 - 94.4 - 81.1 - 107 - 101 - 88.7 - 113;
// 1536 x 1280 x 2048 49.3 - 62.3 - 53.8 - 25.9 - 32.4 - 50.0 - 29.6 - 33.5.
// One launch for each product on its own fastest tile takes 32.5 us at 2080 x 2048 x 768 and 3015 at 131072 x 4096 x 1536.
// 0.6 % off the fastest pair, more than 5 % off at 5 % of the shapes, at worst 1.2 times its time (1472 x 256 x 3072 16.4 for 13.6).  Against a launch each on their own fastest
// tiles 9 of the 3300 shapes are more than 5 % slower (1888 x 1024 x 2816 38.4 -> 43.7 the most), and the mean is 0.76 of the time.
struct TilePair { TileKind input, weight; };
inline TilePair linear_gradient_tiles(int M, int K, int N, int parts) {
  // per 1000 contraction indices with the chip full and alone, start and end, of the input and of the weight gradient; of the launches; per MB read; per MB written beyond
  // `cached`
  struct Cost { int input, weight; double i_full, i_alone, i_fixed, w_full, w_alone, w_fixed, launch, mb_read, mb_written, sharp, cached; };
  static constexpr Cost cost[7] = {{0, 0, 24.7, 18.5, .0659, 21.8, 17.4, 1.53, 8.83, .0325, .19, 5.74, .0248},
                                   {1, 0, 20.3, 5.24, .0039, 24.6, 17.6, 2.55, 9.07, .0199, .165, 12., 221.},
                                   {1, 1, 16., 7.91, 1.07, 18.8, 6.47, 3.36, .284, .0615, .0091, 1.03, 137.},
                                   {1, 2, 5.29, 5.4, 1.99, 12.6, 2.6, 1.1, 1.35, .0892, 0, 1., 96.},
                                   {2, 0, 7.62, 3.37, .245, 24.8, 15.8, 0, 10.5, 0, .243, 1.08, 109.},
                                   {2, 1, 5.76, 2.56, .0135, 28.2, 7.52, 1.56, 1.75, 0, .0927, 4.13, .0065},
                                   {2, 2, .988, 3.08, 1.22, 13.3, 3.58, 2.07, .645, .0717, 0, 3.12, 4970.}};
  const double n = N * 1e-3, r = (double)M / parts * 1e-3;
  const double read = ((double)M * K + 2. * M * N + (double)K * N) * 2e-6, written = (2. * M * K + 4. * K * N * parts) * 1e-6;
  const Cost* best = cost;
  double least = 0;
  for (const Cost& c : cost) {
    const TileKind ki = (TileKind)c.input, kw = (TileKind)c.weight;
    const double blocks_i = tile_blocks(M, K, ki), blocks_w = tile_blocks(K, N, kw) * parts, slots = tile_slots(ki);
    const double full_i = c.i_full * n + c.i_fixed, full_w = c.w_full * r + c.w_fixed, alone_i = c.i_alone * n + c.i_fixed, alone_w = c.w_alone * r + c.w_fixed;
    double t;
    if (slots == tile_slots(kw)) {
      const double work = (blocks_i * full_i + blocks_w * full_w) / slots, chain = std::max(alone_i, alone_w), big = std::max(work, chain);
      t = big * std::pow(1 + std::pow(std::min(work, chain) / big, 1 + c.sharp), 1 / (1 + c.sharp));
      t = std::max(t, (std::ceil((blocks_i + blocks_w) / slots) - 1) * std::min(alone_i, alone_w) + alone_i);
    } else {
      const auto launch = [](TileKind k, double blocks, double full, double alone) {
        const double rounds = std::ceil(blocks / tile_slots(k)) - 1;
        return rounds * full + alone + (full - alone) * pace(k, blocks - rounds * tile_slots(k));
      };
      t = launch(ki, blocks_i, full_i, alone_i) + launch(kw, blocks_w, full_w, alone_w);
    }
    t += c.launch + c.mb_read * read + c.mb_written * std::max(0., written - c.cached);
    if (&c == cost || t < least) { least = t; best = &c; }
  }
  return TilePair{(TileKind)best->input, (TileKind)best->weight};
}

}  // namespace helix
