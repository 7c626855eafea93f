"""Which tile a workgroup takes (csrc/dispatch.hpp), compiled for the host: every tile exactly once, hardly a workgroup without one, and an equal share
for each XCD."""
import pathlib
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2507_00394_amd" / "csrc"
PROGRAM = """
#include "dispatch.hpp"
#include <cstdio>
#include <vector>
int main() {
  int BH, T, causal, D;
  while (scanf("%d %d %d %d", &BH, &T, &causal, &D) == 4) {
    const long long blocks = helix::grid_blocks(BH, T);
    std::vector<int> seen((size_t)BH * T);
    int stray = 0, repeated = 0, early = 0, least = 1 << 30, most = 0;
    long long xcd_tiles[8] = {}, xcd_ranks[8] = {};
    for (int n = 0; n < blocks; n++) {
      const helix::TilePlace p = helix::tile_place(n, BH, T, causal, D);
      if (!p.valid) { early += n < blocks - 64; continue; }
      if (p.head < 0 || p.head >= BH || p.rank < 0 || p.rank >= T) { stray++; continue; }
      repeated += seen[(size_t)p.head * T + p.rank]++ > 0;
      xcd_tiles[n & 7]++;
      xcd_ranks[n & 7] += p.rank;
    }
    int missing = 0;
    for (int x : seen) missing += x == 0;
    long long lo = xcd_ranks[0], hi = xcd_ranks[0];
    for (int x = 0; x < 8; x++) {
      if (xcd_tiles[x] < least) least = (int)xcd_tiles[x];
      if (xcd_tiles[x] > most) most = (int)xcd_tiles[x];
      lo = xcd_ranks[x] < lo ? xcd_ranks[x] : lo;
      hi = xcd_ranks[x] > hi ? xcd_ranks[x] : hi;
    }
    printf("%lld %d %d %d %d %d %lld\\n", blocks, stray, repeated, missing, early, most - least, hi - lo);
  }
}
"""


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    d = tmp_path_factory.mktemp("places")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", str(CSRC), str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def ask(shapes):
        text = "".join(f"{bh} {t} {int(c)} {D}\n" for bh, t, c, D in shapes)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]

    return ask


@pytest.mark.parametrize("D,causal", [(64, True), (128, True), (128, False)])   # without a mask the head dimension does not enter
def test_every_tile_once_and_no_gaps(places, D, causal):
    shapes = [(bh, t, causal, D) for bh in (*range(1, 42), 66, 80, 101, 136, 272, 1000) for t in (*range(1, 26), 33, 40, 64, 65, 130, 513, 1024)
              if bh * t <= 40000]
    for (bh, t, *_), (blocks, stray, repeated, missing, early, uneven, _) in zip(shapes, places(shapes)):
        assert (stray, repeated, missing) == (0, 0, 0), (bh, t)
        assert blocks < bh * t + 8, (bh, t)
        assert early == 0, (bh, t)      # a workgroup without a tile is among the last eight of its XCD
        assert uneven <= 1, (bh, t)


def test_heavy_tiles_are_spread(places):
    """No XCD of a group gets the heavier tile of every row: the sums of the ranks differ by little more than a head's ranks."""
    shapes = [(bh, t, True, 128) for bh in (1, 3, 5, 12, 20, 34, 35, 66) for t in (8, 16, 24, 32, 64, 100, 256)]
    for (bh, t, *_), (*_, spread) in zip(shapes, places(shapes)):
        assert spread <= 2 * t, (bh, t, spread)


def test_far_ends_of_the_shape_limits(places):
    """A quarter of a billion workgroups: the first and the last ones' tiles (computed one by one elsewhere) stay in range."""
    program = """
#include "dispatch.hpp"
#include <cstdio>
int main() {
  const int BH[] = {1, 3, 8, 1023, 3355443, 26843545}, S[] = {1 << 24, 1 << 24, 1 << 24, 200000, 1, 1};
  for (int i = 0; i < 6; i++)
    for (int rows = 64; rows <= 256; rows *= 2) {
      const int T = (S[i] + rows - 1) / rows;
      const long long blocks = helix::grid_blocks(BH[i], T);
      if (blocks > 0x7fffffffLL) return 1;
      for (int c = 0; c < 2; c++)
        for (int k = 0; k < 2000; k++)
          for (int side = 0; side < 2; side++) {
            const long long n = side ? blocks - 1 - k : k;
            if (n < 0 || n >= blocks) continue;
            const helix::TilePlace p = helix::tile_place((int)n, BH[i], T, c, 128);
            if (p.valid && (p.head < 0 || p.head >= BH[i] || p.rank < 0 || p.rank >= T)) return 2;
          }
    }
  return 0;
}
"""
    import tempfile

    with tempfile.TemporaryDirectory() as d:
        (pathlib.Path(d) / "far.cpp").write_text(program)
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", str(CSRC), f"{d}/far.cpp",
                        "-o", f"{d}/far"], check=True)
        assert subprocess.run([f"{d}/far"]).returncode == 0
