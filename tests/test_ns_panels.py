"""The graded panels of the near-singular integrals (csrc/ns_panels.h, built for the
host with and without fused multiply-adds, as a device compiler may choose for
either function): for every closest point and width the panels are 0 .. n - 1, each
begins where another ends, and together they are [0, 1].  Widths whose triples meet
an end of the segment exactly are where the count and the bounds, rounded in other
ways, disagreed about the number of panels on a side: the last one was then left
out (a third of the segment for a node above its middle at a third of its length)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#define BS_HD static inline
#include "ns_panels.h"
#include <cstdio>
int main() {
    double ub, dl;
    while (std::scanf("%la %la", &ub, &dl) == 2) {
        COUNT
        std::printf("%d", p.n);
        for (int k = 0; k < p.n; k++) {
            double lo, hi;
            BOUNDS
            std::printf(" %a %a", lo, hi);
        }
        std::printf("\n");
    }
}
'''


def cases():
    rng = np.random.default_rng(7)
    out = []
    for ub in (0.0, 0.125, 0.25, 1 / 3, 0.375, 0.5, 0.625, 2 / 3, 0.75, 1.0):
        for side in (ub, 1.0 - ub):
            w = side
            for _ in range(24):      # triples that land on the end of a side, to rounding
                w /= 3.0
                for d in (w, np.nextafter(w, 0), np.nextafter(w, 1)):
                    out.append((ub, max(d, 1e-13)))
    out += [(u, d) for u, d in zip(rng.uniform(0, 1, 3000), 10.0 ** rng.uniform(-13, 1, 3000))]
    out += [(0.5, float("inf")), (0.5, float("nan")), (float("nan"), 0.1)]
    return out


def run(tmp_path, flags, split):
    """split: the count contracted, the bounds not, or the reverse (separate
    functions that no contraction spans)."""
    src = tmp_path / "p.cpp"
    src.write_text(PROGRAM.replace("COUNT", "bs::NsPanels p = bs::ns_panels(ub, dl);")
                   .replace("BOUNDS", "bs::ns_panel_bounds(ub, dl, p, k, &lo, &hi);"))
    header = open(os.path.join(ROOT, "paper_2406_07366_amd", "csrc", "ns_panels.h")).read()
    if split == "count fused":
        header = header.replace("e = ub - 3.0 * w", "e = fma(-3.0, w, ub)") \
                       .replace("e = ub + 3.0 * w", "e = fma(3.0, w, ub)")
    elif split == "bounds fused":
        header = header.replace("fmax(ub - 3.0 * w, 0.0)", "fmax(fma(-3.0, w, ub), 0.0)") \
                       .replace("fmin(ub + 3.0 * w, 1.0)", "fmin(fma(3.0, w, ub), 1.0)")
    (tmp_path / "ns_panels.h").write_text(header)
    exe = tmp_path / "p"
    subprocess.run(["g++", "-O2", "-std=c++17"] + flags + ["-I", str(tmp_path), str(src), "-o", str(exe)],
                   check=True)
    inp = "\n".join(f"{float(u).hex()} {float(d).hex()}" for u, d in cases())
    out = subprocess.run([str(exe)], input=inp, capture_output=True, text=True, check=True).stdout
    return out.splitlines()


@pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")
@pytest.mark.parametrize("split", ["as written", "count fused", "bounds fused"])
def test_panels_cover_the_segment(tmp_path, split):
    lines = run(tmp_path, ["-ffp-contract=off"], split)
    assert len(lines) == len(cases())
    most = 0
    for (ub, dl), line in zip(cases(), lines):
        f = line.split()
        n = int(f[0])
        if not dl == dl or not ub == ub:
            assert n == 0
            continue
        v = sorted((float.fromhex(a), float.fromhex(b)) for a, b in zip(f[1::2], f[2::2]))
        assert len(v) == n and n >= 1
        most = max(most, n)
        assert v[0][0] == 0.0 and v[-1][1] == 1.0, (ub, dl, v)
        for (_, b), (c, _) in zip(v[:-1], v[1:]):
            assert b == c, (ub, dl, v)
        assert all(b >= a for a, b in v)
    assert 50 < most < 64
