"""Where reads of a row go (csrc/rows.h), checked on the CPU over every row of
graphs that do not hold each edge in both directions: vertices without
neighbours of their own, first, last and between others, are met as
neighbours. Every read must lie inside the arrays."""

from __future__ import annotations

import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_11188_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "rows.h"
int main() {  // "off deg" lines, then for each the reads of positions 0..299
  long long off; int deg;
  while (std::scanf("%lld %d", &off, &deg) == 2)
    for (int p = 0; p < 300; ++p)
      std::printf("%lld\n", (long long)(scan::row_start(off, deg) + scan::row_position(p, deg)));
}
"""


@pytest.fixture(scope="module")
def reads(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    exe = str(d / "rows")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-x", "c++", "-", "-o", exe],
                       input=PROGRAM, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(off):
        deg = np.diff(off)
        text = "".join(f"{o} {d}\n" for o, d in zip(off[:-1], deg))
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return np.array(out.split(), np.int64).reshape(len(deg), 300)

    return run


@pytest.mark.parametrize("deg", [[0, 3, 0, 2, 0], [0, 0, 1], [1, 0, 0], [5], [0, 65, 0, 129, 1, 0, 256, 0]])
def test_reads_stay_inside(reads, deg):
    off = np.concatenate([[0], np.cumsum(deg)])
    got = reads(off)
    assert got.min() >= 0 and got.max() < off[-1]
    for v, d in enumerate(deg):
        if d:  # the row's own positions, then its last one again
            assert np.array_equal(got[v], off[v] + np.minimum(np.arange(300), d - 1))
