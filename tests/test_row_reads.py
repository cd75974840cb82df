"""Where reads of a row go, and the numbers of ids without the isolated vertices
(csrc/rows.h), checked on the CPU over graphs that do not hold each edge in
both directions: vertices without neighbours of their own, first, last and
between others, are met as neighbours. Every read must lie inside the arrays,
every number inside the id windows."""

from __future__ import annotations

import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_11188_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "rows.h"
int main() {  // "off deg" lines, then for each the reads of positions 0..298 and of the last one
  long long off; int deg;
  while (std::scanf("%lld %d", &off, &deg) == 2)
    for (int p = 0; p < 300; ++p)
      std::printf("%lld\n", (long long)(scan::row_start(off, deg) + scan::row_position(p < 299 ? p : 0x7fffffff, deg)));
}
"""


def compiled(tmp_path_factory, program):
    exe = str(tmp_path_factory.mktemp("rows") / "rows")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-Wno-unused-function", "-I", CSRC, "-x", "c++", "-",
                        "-o", exe], input=program, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.fixture(scope="module")
def reads(tmp_path_factory):
    exe = compiled(tmp_path_factory, PROGRAM)

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
    missing = reads(np.concatenate([off[:1], off[:1] - 1]))  # a length of -1: the row's first slot
    assert np.all(missing == off[0])
    for v, d in enumerate(deg):
        if d:  # the row's own positions, then its last one again
            assert np.array_equal(got[v], off[v] + np.minimum(np.arange(300), d - 1))


NUMBERS = r"""
#include <cstdio>
#include "rows.h"
int main() {  // "used before" lines
  long long before; int used;
  while (std::scanf("%d %lld", &used, &before) == 2) std::printf("%d\n", scan::used_number(before, used));
}
"""


# the used vertices fill whole windows of 1024 ids, and one more or less
@pytest.mark.parametrize("used", [1, 1023, 1024, 1025, 2048])
def test_numbers_stay_inside_the_windows(tmp_path_factory, used):
    exe = compiled(tmp_path_factory, NUMBERS)
    deg = np.zeros(3 * used + 5, np.int64)
    place = np.sort(np.random.default_rng(used).permutation(len(deg) - 2)[:used])  # the last ids have no rows
    deg[place] = 1
    before = np.concatenate([[0], np.cumsum(deg > 0)])[:-1]
    out = subprocess.run([exe], input="".join(f"{used} {b}\n" for b in before), capture_output=True, text=True,
                         check=True).stdout
    got = np.array(out.split(), np.int64)
    windows = -(-used // 1024)
    assert got.min() >= 0 and got.max() < used and got.max() >> 10 < windows
    assert np.array_equal(got[place], np.arange(used))
    assert np.all(np.diff(got) >= 0)
