"""A quoted hardware counter is tied to the kernel's source: the file itself and
every header beside it that it includes, directly or through another (the bodies of
several kernels are in headers)."""
import os

from paper_2406_07366_amd import profsum

CSRC = os.path.join(os.path.dirname(os.path.abspath(profsum.__file__)), "csrc")


def test_headers_are_among_the_sources():
    names = [os.path.basename(p) for p in profsum.sources_of(os.path.join(CSRC, "pairs.hip"))]
    assert names[0] == "pairs.hip" and len(names) == len(set(names))
    assert {"pairs64.h", "erfcx_fit.h", "bs_device.h", "direct.h"} <= set(names)
    names = [os.path.basename(p) for p in profsum.sources_of(os.path.join(CSRC, "fft.hip"))]
    assert "fft_kernels.h" in names


def test_a_changed_header_makes_a_figure_stale(tmp_path):
    (tmp_path / "k.hip").write_text('#include <stdio.h>\n#include "a.h"\n')
    (tmp_path / "a.h").write_text('#pragma once\n#include "b.h"\n#include "a.h"\n')
    (tmp_path / "b.h").write_text("int x;\n")
    src, summary = str(tmp_path / "k.hip"), tmp_path / "s.txt"
    summary.write_text(f"traffic_bytes_per_launch: 1.5e+09\nsource: k.hip\n"
                       f"source_sha1: {profsum.sha1_of(src)}\n")
    assert profsum.read_traffic(str(summary), src) == 1.5e9
    for name in ("b.h", "a.h", "k.hip"):
        text = (tmp_path / name).read_text()
        (tmp_path / name).write_text(text + "// changed\n")
        assert profsum.read_traffic(str(summary), src) is None
        (tmp_path / name).write_text(text)
    assert profsum.read_traffic(str(summary), src) == 1.5e9
