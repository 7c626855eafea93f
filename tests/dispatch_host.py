"""The rules of csrc/dispatch.hpp, compiled for the host (a test without a GPU asks them which variant a launch takes)."""
import functools
import pathlib
import subprocess
import tempfile

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2507_00394_amd" / "csrc"


@functools.lru_cache(maxsize=None)
def _program(names, expressions):
    d = pathlib.Path(tempfile.mkdtemp(prefix="dispatch_host"))
    formats = " ".join(["%d"] * len(expressions))
    values = ", ".join(f"(int)({e})" for e in expressions)
    scan = ", ".join(f"&{n}" for n in names)
    (d / "main.cpp").write_text(f"""
#include "dispatch.hpp"
#include <cstdio>
using namespace helix;
int main() {{
  int {", ".join(names)};
  while (scanf("{" ".join(["%d"] * len(names))}", {scan}) == {len(names)}) printf("{formats}\\n", {values});
}}
""")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", str(CSRC), str(d / "main.cpp"), "-o", str(d / "main")], check=True)
    return d / "main"


def ask(shapes, *expressions, names=("D", "BH", "S", "causal")):
    """The C++ expressions (of the variables `names`) for every shape, a tuple of ints each."""
    shapes = list(shapes)
    text = "".join(" ".join(str(int(x)) for x in s) + "\n" for s in shapes)
    out = subprocess.run([str(_program(tuple(names), tuple(expressions)))], input=text, capture_output=True, text=True, check=True).stdout
    rows = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    assert len(rows) == len(shapes)
    return rows


def read_table(text):
    """(numbers of the shape, times) of `shape... | times...` entries, or `heads tokens times...`, separated by semicolons or lines."""
    for entry in text.replace("\n", ";").split(";"):
        if entry.strip():
            head, _, times = entry.partition("|") if "|" in entry else (" ".join(entry.split()[:2]), "", " ".join(entry.split()[2:]))
            yield tuple(int(x) for x in head.split()), [float(x) for x in times.split()]


def check(chosen, table, mean, worst):
    """The chosen variants (an index into the times of each shape) against the fastest of each."""
    regret = {shape: us[v] / min(us) for v, (shape, us) in zip(chosen, table)}
    assert len(set(chosen)) > 1
    assert max(regret.values()) <= worst, {s: r for s, r in regret.items() if r > worst}
    assert sum(regret.values()) / len(regret) <= mean, sum(regret.values()) / len(regret)
