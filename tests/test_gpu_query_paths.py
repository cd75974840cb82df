"""Query kernels at the edges of their row classes (a lane group, a wavefront
and a workgroup each take a part of a row), over more queries than a slot has
mark values, over more than one set of launch descriptors, and on a capturing
stream, against the oracle."""

from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle
import paper_2012_11188_amd as scan
from gpu_util import assert_queries_equal, gpu_build

pytestmark = pytest.mark.gpu


def wheel(rim, pendants):
    """A hub joined to `rim` ring vertices and to `pendants` leaves; ids are
    spread so that the hub lies between them."""
    hub = rim // 2
    ring = [i if i < hub else i + 1 for i in range(rim)]
    edges = [(hub, v) for v in ring] + [(ring[i], ring[(i + 1) % rim]) for i in range(rim)]
    edges += [(hub, rim + 1 + i) for i in range(pendants)]
    return graphgen.from_edges(rim + 1 + pendants, edges)


# hub degrees around 64 (lane group), 64 + 8 * 256 (wavefront) and one, two workgroup steps of 4096 past it
@pytest.mark.parametrize("degree", [63, 64, 65, 320, 321, 2111, 2112, 2113, 6208, 6209, 10400])
def test_row_classes(degree):
    g = wheel(degree - 7, 7)
    gix = gpu_build(g)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    assert int(g.degrees().max()) == degree
    low = float(np.min(oix.sim))
    assert_queries_equal(gix, oix, [(mu, eps) for mu in (2, 3, 4, 5, degree + 1) for eps in (low, 0.5, 0.76)])


def test_more_queries_than_marks():
    g = graphgen.sbm(300, 6, 0.3, 0.02, 11)
    gix = gpu_build(g)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    pairs = [(2 + i % 7, 0.1 + 0.05 * (i % 9)) for i in range(300)]  # a slot has 127 mark values
    assert_queries_equal(gix, oix, pairs)


@pytest.mark.parametrize("count", [31, 32, 33, 70])
def test_batches_over_descriptor_sets(count):
    g = graphgen.rmat(10, 12, seed=3)
    gix = gpu_build(g)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    mus = [2 + i % 5 for i in range(count)]
    epss = [0.05 + 0.03 * (i % 13) for i in range(count)]
    for _ in range(2):
        got = scan.scan_query_batch(gix, mus, epss).cpu().numpy()
        for i in range(count):
            assert np.array_equal(got[i], oracle.query(oix, mus[i], epss[i])[0]), i


def test_pooled_query_refuses_capture():
    import torch

    gix = gpu_build(graphgen.sbm(300, 6, 0.3, 0.02, 11))
    memb, core = scan.scan_query_ex(gix, 3, 0.2)
    torch.cuda.synchronize()
    graph, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=s):
        memb.fill_(7)
        with pytest.raises(scan.ScanError):
            scan.scan_query_ex(gix, 3, 0.2, memb, core, stream=s)


# the one-workgroup kernel takes up to 2048 vertices and 64 * 2048 slots
@pytest.mark.parametrize("n,p", [(1, 0.0), (2, 1.0), (65, 0.9), (2047, 0.01), (2048, 0.01), (2049, 0.01),
                                 (2048, 0.0312), (2048, 0.04)])
def test_small_index_edges(n, p):
    g = graphgen.sbm(n, 1, p, 0.0, 5)
    gix = gpu_build(g)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    vals = np.unique(oix.sim) if g.nnz else np.array([0.5])
    assert_queries_equal(gix, oix, [(mu, float(e)) for mu in (2, 3, 17, 40) for e in vals[:: max(1, len(vals) // 6)]])


# A refused call leaves nothing behind: no workspace in the pool whose memory
# or cleared marks exist only inside the captured graph, and no event of a
# pooled workspace recorded there.
@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("n,call", [(300, "one"), (3000, "one"), (3000, "host"), (3000, "batch"), (3000, "sweep")])
def test_queries_after_refused_capture(n, call, warm):
    import torch

    g = graphgen.sbm(n, 6, 60.0 / n, 4.0 / n, 11)
    gix = gpu_build(g)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    memb = torch.zeros(n, dtype=torch.int32, device="cuda")
    core = torch.zeros(n, dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    if warm:
        scan.scan_query_ex(gix, 3, 0.2, memb, core, stream=s)
    torch.cuda.synchronize()
    graph, filled = torch.cuda.CUDAGraph(), torch.zeros(n, dtype=torch.int32, device="cuda")
    with torch.cuda.graph(graph, stream=s):
        filled.fill_(7)
        with pytest.raises(scan.ScanError, match="captured"):
            if call == "one":
                scan.scan_query_ex(gix, 3, 0.2, memb, core, stream=s)
            elif call == "host":
                scan.scan_query_ex(gix, 3, 0.2, stream=s, out_on_device=False)
            elif call == "batch":
                scan.scan_query_batch(gix, [3, 4, 5], [0.2, 0.3, 0.1], stream=s)
            else:
                scan.scan_sweep_modularity(gix, [3, 4], [0.2, 0.3], stream=s)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert int(filled.min()) == 7 and int(filled.max()) == 7
        filled.zero_()
        for mu, eps in ((2, 0.1), (3, 0.2), (5, 0.3)):
            for stream in (s, None):
                scan.scan_query_ex(gix, mu, eps, memb, core, stream=stream)
                torch.cuda.synchronize()
                want = oracle.query(oix, mu, eps)
                assert np.array_equal(memb.cpu().numpy(), want[0]) and np.array_equal(core.cpu().numpy(), want[1])
    gix.free()


# the one-workgroup kernel with rows past 256 entries: up to 32 * 2048 slots;
# hubs joined to all others, and cliques of 256 and 257
@pytest.mark.parametrize("n,hubs", [(2048, 1), (2048, 16), (2048, 17), (2048, 30), (256, 256), (257, 257), (257, 256)])
def test_small_index_long_rows(n, hubs):
    u, v = np.meshgrid(np.arange(hubs), np.arange(n), indexing="ij")
    g = graphgen.from_edges(n, np.stack([u.ravel(), v.ravel()], 1)[u.ravel() != v.ravel()].astype(np.int32))
    gix = gpu_build(g)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    vals = np.unique(oix.sim)
    assert_queries_equal(gix, oix, [(mu, float(e)) for mu in (2, 3, hubs, hubs + 1, n) if mu > 1
                                    for e in [0.0, *vals[:: max(1, len(vals) // 4)]]])
