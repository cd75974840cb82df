"""The parameter sweep's many-clusterings kernels at the edges of their
batches and row units, against the oracle (exact integers, so bit for bit)."""

from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle
import paper_2012_11188_amd as scan
from gpu_util import gpu_build

pytestmark = pytest.mark.gpu


def wheel(rim, pendants):
    """A hub joined to `rim` ring vertices and to `pendants` leaves; ids are
    spread so that the hub lies between them."""
    hub = rim // 2
    ring = [i if i < hub else i + 1 for i in range(rim)]
    edges = [(hub, v) for v in ring] + [(ring[i], ring[(i + 1) % rim]) for i in range(rim)]
    edges += [(hub, rim + 1 + i) for i in range(pendants)]
    return graphgen.from_edges(rim + 1 + pendants, edges)


# clusterings are scored 32 at a time, rows in units of 128 slots
@pytest.mark.parametrize("batch", [31, 32, 33, 70])
@pytest.mark.parametrize("name", ["wheel", "sbm"])
def test_sweep_batches(batch, name):
    g = wheel(1300, 9) if name == "wheel" else graphgen.sbm(1003, 7, 0.08, 0.004, 9)
    gix = gpu_build(g)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    mus = np.array([2 + i % 6 for i in range(101)], np.int32)
    epss = np.array([0.02 + 0.009 * i for i in range(101)])
    q = scan.scan_sweep_modularity(gix, mus, epss, batch=batch)
    for i in range(101):
        want = oracle.modularity(g, oracle.query(oix, int(mus[i]), float(epss[i]))[0])[0]
        assert q[i].tobytes() == np.float64(want).tobytes(), (int(mus[i]), float(epss[i]))
