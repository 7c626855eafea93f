// Which variant of a pass a launch takes, as a function of the shape alone.  Plain host arithmetic (head_parts and grid_blocks are
// constexpr so that the device code that maps workgroup ids to tiles shares them), free of HIP, so that a test without a GPU can
// compile it and hold every rule against the times it was read from.
#pragma once
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

// Whether the forward and dQ passes take 128-row tiles with the keys split over two groups of waves instead
// of 256-row tiles.  A split workgroup needs 0.55-0.65 of the time of a whole one for the same keys, and there
// are twice as many: it pays where whole tiles leave compute units idle.  One workgroup per compute unit (256) is
// a round.
//   causal: tiles differ in length, so with up to one round the longest one sets the time.  Measured at head
//     dimension 128, whole -> split, forward / dQ, us: 12 heads x 1500 (72 tiles) 39.7 -> 25.9 / 49 -> 31.5;
//     2 x 32k (256) 710 -> 531 / 904 -> 693; 64 x 1024 (256) 33.5 -> 30.5 / 42 -> 39.5; just beyond,
//     40 x 2048 (320) 58 -> 61 / 75 -> 79; 16 x 8192 (512) 255 -> 282 / 339 -> 364.
//   no mask: all tiles are equal, so whole rounds are compared.  32 x 1024 (128) 31.8 -> 23.4 / 39 -> 30; 12 x 8192
//     (384: 2 rounds or 3) 412 -> 399 / 533 -> 522; 32 x 1500 (192: 1 or 2) 45.6 -> 54.5 / 58 -> 68.
// Head dimension 64 behaves alike (the sweep covered 1 to 64 heads, 200 to 32k tokens, both dimensions).
inline bool split_rows(int BH, int S, bool causal) {
  const long long whole = (long long)BH * ((S + 255) / 256), split = (long long)BH * ((S + 127) / 128);
  if (causal) return whole <= 256;
  return ((split + 255) / 256) * 5 < ((whole + 255) / 256) * 9;
}

// Head dimension 64: whether two groups of waves share the query tiles of a key tile in the dK/dV pass, and that pass its launch with
// the dQ pass on split tiles (a launch of its own is what the stage calls make of it).  With one group a SIMD has one wave, which
// is bound by instruction issue, unless a second workgroup finds room beside it; two groups halve the sweep, and the common launch fills
// the compute units that a small grid or its last round leaves idle.  Where the chip is full both only cost: the swap of partial sums,
// and one workgroup in the place of two.  The backward in separate passes (the faster way) -> in one launch, us; key tiles in brackets:
//   causal: 2 heads x 512 [8] 33.7 -> 23.1; 12 x 1500 [144] 64 -> 44; 32 x 1024 [256] 51 -> 41; 32 x 1500 [384] 72.5 -> 70.5; 4 x 16k [512]
//     486 -> 484 (533 with one group); 2 x 32k [512] 937 -> 931 (1033).  Short sweeps of more than 256 key tiles: 60 x 900 [480] 69 -> 73;
//     128 x 512 [512] 51 -> 55; 256 x 256 [512] 43 -> 48.  Beyond 512: one -> two groups, dK/dV alone, 40 x 2048 [640] 53 -> 64.
//   no mask, up to 256: 2 x 512 [8] 26.7 -> 16.2; 27 x 777 [189] 40.5 -> 39; 2 x 16k [256] 446 -> 443.  Up to 512 the separate passes do
//     with one round: 40 x 1500 [480] 94 -> 102; 64 x 1024 [512] 72 -> 79.  Just beyond they start a second one: 24 x 3000 [576] 248 -> 214;
//     10 x 8192 [640] 626 -> 563.  From there on 11 x 8192 [704] 634 -> 649; 12 x 8192 [768] 670 -> 671; 160 x 1024 [1280] 173 -> 187;
//     512 x 300 [1536] 102 -> 120; 80 x 6528 [4080] 2756 -> 2841.
// (Key tiles as launched: a head whose tiles the XCDs cannot share evenly counts for its fullest XCD.)
inline bool two_query_groups(int BH, int S, bool causal) {
  const long long tiles = grid_blocks(BH, (S + 127) / 128);
  if (tiles <= 256) return true;
  return causal ? tiles <= 512 && S >= 1024 : tiles > 512 && tiles <= 640;
}
inline bool split_dq(int D, int BH, int S, bool causal) {
  return (D == 64 && two_query_groups(BH, S, causal)) || split_rows(BH, S, causal);
}

}  // namespace helix
