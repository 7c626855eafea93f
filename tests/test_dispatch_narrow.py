"""The rules that give small grids narrow workgroups (csrc/dispatch.hpp), compiled for the host, against times measured on an MI355X."""
import pathlib
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2507_00394_amd" / "csrc"
PROGRAM = """
#include "dispatch.hpp"
#include <cstdio>
int main() {
  int D, BH, S, causal;
  while (scanf("%d %d %d %d", &D, &BH, &S, &causal) == 4)
    printf("%d %d\\n", helix::narrow_gradients(BH, S, causal), (int)helix::dq_rows(D, BH, S, causal));
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch_narrow")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", str(CSRC), str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def ask(shapes):
        text = "".join(f"{D} {bh} {s} {int(c)}\n" for D, bh, s, c in shapes)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]

    return ask


# head dimension, causal, heads, tokens; us of the forward on 256-, 128- and 64-row tiles (not used), of the causal delta of the
# first rows likewise (not used), and of the backward on wide and narrow gradient workgroups
MEASURED = """
64 N 31 190 | - 6.4 5.5 | - - - | 11.5 12.6
64 N 13 494 | - 9.2 7.5 | - - - | 15.0 14.0
64 N 53 118 | - 8.0 5.6 | - - - | 18.2 13.0
64 N 2 3963 | - 41.1 31.8 | - - - | 52.6 40.3
64 N 4 2235 | - 25.6 19.9 | - - - | 34.9 44.0
64 N 127 107 | - 10.1 8.1 | - - - | 25.7 24.4
64 N 131 303 | - 17.4 20.3 | - - - | 49.2 62.1
64 N 45 1677 | - 65.6 66.1 | - - - | 164.2 207.7
64 C 5 115 | - 5.9 5.0 | 5.4 4.9 4.1 | 12.4 11.4
64 C 2 331 | - 8.0 6.6 | 7.5 7.3 5.9 | 18.0 16.1
64 C 6 160 | - 6.1 5.3 | 6.1 5.3 4.4 | 13.8 12.2
64 C 23 50 | - 5.3 4.5 | 4.6 4.3 3.6 | 10.9 10.5
64 C 12 100 | - 5.9 5.0 | 5.4 4.9 4.1 | 12.6 11.5
64 C 4 877 | - 13.0 10.5 | 14.9 11.8 8.9 | 28.2 24.6
64 C 4 907 | - 12.9 10.5 | 16.8 11.9 9.4 | 29.2 25.4
64 C 11 389 | - 8.4 7.0 | 9.7 7.9 6.4 | 19.7 17.9
64 C 5 1243 | - 16.4 12.9 | 21.6 15.5 11.4 | 36.3 31.3
64 C 8 844 | - 12.7 10.2 | 14.9 11.9 9.1 | 28.8 25.0
64 C 3 2406 | - 26.7 21.2 | 32.0 21.9 16.1 | 60.4 50.7
64 C 2 6079 | - 60.5 47.2 | 32.1 21.8 15.9 | 105.0 82.7
64 C 2 8443 | - 81.5 65.1 | 32.0 21.9 15.9 | 135.3 115.6
64 C 134 123 | - 11.5 8.9 | 13.6 12.1 7.0 | 44.5 36.1
64 C 12 1767 | - 22.4 18.0 | 29.2 20.0 15.2 | 48.2 53.9
64 C 131 146 | - 11.8 9.7 | 16.1 13.7 8.0 | 46.7 40.2
64 C 1 27781 | - 257.9 202.3 | 31.7 21.2 15.5 | 398.4 444.5
64 C 25 1441 | - 21.8 19.0 | 25.8 21.3 16.4 | 67.3 75.3
64 C 88 673 | - 17.5 17.7 | 15.4 17.9 13.8 | 55.1 68.3
64 C 147 409 | - 21.1 21.9 | 28.6 23.6 19.0 | 79.9 86.6
128 N 13 62 | 5.9 6.3 5.4 | - - - | 10.1 9.3
128 N 3 329 | 13.3 10.5 8.7 | - - - | 17.5 14.4
128 N 7 243 | 10.8 8.9 7.4 | - - - | 15.4 13.3
128 N 2 1238 | 31.4 21.4 18.1 | - - - | 34.9 25.8
128 N 6 769 | 22.6 16.4 13.7 | - - - | 27.7 21.3
128 N 8 676 | 19.9 14.6 12.3 | - - - | 24.3 19.2
128 N 7 1104 | 29.6 21.0 17.9 | - - - | 35.9 41.1
128 N 2 8218 | 177.3 109.9 169.8 | - - - | 296.2 326.2
128 N 2 13140 | 280.8 189.7 278.9 | - - - | 568.6 678.4
128 N 6 5481 | 121.8 160.2 182.4 | - - - | 308.2 379.6
128 N 8 6220 | 163.4 183.7 273.0 | - - - | 524.3 602.3
128 N 11 7867 | 384.0 366.1 510.2 | - - - | 1090.8 1213.5
128 C 1 576 | 15.2 12.3 10.5 | 14.4 10.6 8.8 | 28.4 23.8
128 C 1 841 | 20.2 16.2 13.2 | 19.3 14.2 11.4 | 38.8 32.2
128 C 1 1434 | 34.1 22.8 19.4 | 33.0 20.6 16.6 | 56.1 45.6
128 C 5 286 | 10.4 9.5 8.2 | 9.6 7.9 6.7 | 20.7 18.1
128 C 10 142 | 8.8 7.8 6.8 | 7.5 6.4 5.5 | 16.0 14.4
128 C 1 2335 | 50.7 33.4 28.6 | 44.8 27.4 22.5 | 84.9 67.0
128 C 7 573 | 15.6 12.8 11.0 | 15.0 11.0 9.1 | 30.4 25.8
128 C 1 4760 | 100.3 62.8 53.8 | 44.9 27.3 22.6 | 130.8 97.9
128 C 1 5915 | 123.9 77.7 67.0 | 44.7 27.4 22.4 | 154.5 111.5
128 C 53 66 | 8.3 8.5 6.9 | 7.3 6.7 5.6 | 25.0 19.9
128 C 4 1952 | 45.2 29.5 25.2 | 43.5 26.7 21.6 | 70.4 57.0
128 C 5 3981 | 87.3 55.6 47.6 | 45.5 28.6 23.8 | 132.4 130.2
128 C 23 909 | 25.6 20.4 21.9 | 23.8 18.1 19.3 | 56.2 61.3
128 C 16 1364 | 32.0 23.8 19.9 | 30.1 20.8 16.9 | 60.6 65.4
128 C 39 577 | 17.9 22.4 22.9 | 16.7 18.8 20.0 | 55.8 58.8
128 C 1 37001 | 758.0 480.1 502.5 | 44.5 27.1 22.4 | 1122.9 1268.2
128 C 13 2913 | 69.0 48.9 61.1 | 47.7 31.0 31.0 | 147.0 175.0
128 C 3 13706 | 286.9 189.5 220.9 | 44.8 27.7 22.9 | 514.3 562.5
128 C 30 1599 | 41.9 37.5 45.0 | 39.4 34.2 39.3 | 128.9 143.2
128 C 8 11372 | 282.2 279.2 364.6 | 45.0 28.2 23.1 | 813.7 944.0"""


def _rows():
    for line in MEASURED.split("\n"):
        if line.strip():
            head, *groups = line.split("|")
            D, c, bh, s = head.split()
            yield int(D), c == "C", int(bh), int(s), [[float(x) if x != "-" else 1e9 for x in g.split()] for g in groups]


def test_choices_against_measured_times(rules):
    table = list(_rows())
    regret = {"gradients": []}
    for (D, c, bh, s, (_, _, g)), (rg, _) in zip(table, rules([r[:1] + r[2:4] + r[1:2] for r in table])):
        regret["gradients"].append(g[rg] / min(g))
    for name, r in regret.items():
        assert max(r) <= 1.3 and sum(r) / len(r) <= 1.02, (name, max(r), sum(r) / len(r))


def test_narrow_gradients_go_together(rules):
    """Narrow key tiles share their launch with narrow query tiles only, and never beyond the grids they were measured at."""
    for (D, bh, s, c), (narrow, dq) in zip(SHAPES, rules(SHAPES)):
        assert (dq == 2) == bool(narrow)
        assert not narrow or bh * ((s + 63) // 64) <= 288


SHAPES = [(D, bh, s, c) for D in (64, 128) for bh in (1, 2, 5, 8, 27, 64, 100, 289, 5000, 3355443) for s in (1, 64, 65, 500, 1024, 5000, 1 << 24)
          for c in (True, False) if bh * s < 1 << 26]
