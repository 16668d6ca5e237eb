"""Sub-tile and block shapes of every tile that the options accept, evaluated at compile time, where a
read of a value that has not been set is an error (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [(w, h, p) for w in range(11) for h in range(11) for p in range(3) if max(6 + p, 6) <= w + h <= min(10, 8 + p)]


def _best(w, h, parts):
    """(log2 w, log2 h, log2 columns) of the squarest split, the wider of two equals."""
    return min(((w - nx, h - parts + nx, nx) for nx in range(parts + 1) if w >= nx and h >= parts - nx),
               key=lambda s: (abs(s[0] - s[1]), -s[0]))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_shapes_are_the_squarest_and_set_before_they_are_read(tmp_path):
    lines = ['#include "subtiles.h"', "constexpr bool is(gs::Part p, int w, int h, int nx) {",
             "  return p.log2_w == w && p.log2_h == h && p.log2_nx == nx;", "}"]
    for w, h, p in SHAPES:
        sub = _best(w, h, w + h - 6 - p)
        assert sub[0] + sub[1] == 6 + p
        lines.append("static_assert(is(gs::split(%d, %d, %d), %d, %d, %d), \"\");" % (w, h, w + h - 6 - p, *sub))
        lines.append("static_assert(is(gs::split(%d, %d, %d), %d, %d, %d), \"\");" % (*sub[:2], p, *_best(*sub[:2], p)))
    src = tmp_path / "shapes.cpp"
    src.write_text("\n".join(lines) + "\n")
    res = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I", os.path.join(ROOT, "paper_2501_14534_amd", "csrc"),
                          str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
