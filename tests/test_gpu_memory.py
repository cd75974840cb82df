"""Refused device memory: what a call that is refused some leaves behind, and
what is answered without, against the oracle."""

from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle
import paper_2012_11188_amd as scan
from alloc_hooks import hooks
from gpu_util import assert_index_equal, device_csr, gpu_build

pytestmark = pytest.mark.gpu


# A batch that cannot have all of its workspaces keeps none of the new ones:
# their marks are still being cleared on its stream.
@pytest.mark.parametrize("warm,refused", [(0, 0), (0, 3), (2, 0), (2, 2)])
def test_batch_without_all_workspaces(warm, refused):
    import torch

    g = graphgen.sbm(3000, 6, 0.02, 0.001, 11)
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    mus, epss = [2, 3, 4, 5, 6, 3], [0.1, 0.2, 0.15, 0.1, 0.3, 0.05]
    want = np.stack([oracle.query(oix, m, e)[0] for m, e in zip(mus, epss)])
    with hooks() as h:
        gix = gpu_build(g)
        if warm:
            scan.scan_query_batch(gix, mus[:warm], epss[:warm])
        torch.cuda.synchronize()
        before = h.held
        out = torch.empty((len(mus), g.n), dtype=torch.int32, device="cuda")
        side = torch.cuda.Stream()
        with pytest.raises(scan.ScanError) as err:
            h.start(refuse=[refused])
            scan.scan_query_batch(gix, mus, epss, out, stream=side)
        assert err.value.status == scan.SCAN_ENOMEM
        assert h.held == before, "workspaces of the refused batch are still held"
        h.start()
        for stream in (None, side, None):
            got = scan.scan_query_batch(gix, mus, epss, out, stream=stream)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), want)
        gix.free()


def attempt(h, setup, run, refuse=(), budget=None):
    """run(setup()) with the hooks' limits on the run alone."""
    import torch

    given = setup()
    torch.cuda.synchronize()
    h.start(refuse, budget)
    try:
        got = run(given)
        torch.cuda.synchronize()
        return got
    finally:
        h.refuse, h.budget = frozenset(), None


def least_memory(h, setup, run, check):
    """The least peak of `run` over refusals of memory that it can do without
    (one call after the other is refused for good where the run still succeeds
    and holds less), and the number of those; every answer is checked."""
    check(attempt(h, setup, run))
    refused, least, calls, k = [], h.peak, h.calls, 0
    while k < calls:
        try:
            got = attempt(h, setup, run, refused + [k])
        except scan.ScanError as e:
            assert e.status == scan.SCAN_ENOMEM
        else:
            peak, made = h.peak, h.calls
            check(got)
            if peak < least:
                refused, least, calls = refused + [k], peak, made
        assert h.held == 0
        k += 1
    return least, len(refused)


# A build succeeds within the memory that it needs without the hub product and
# without ids numbered anew: what it needs is taken first. Dense rows of at
# most 4096 slots, whose sorts take no memory of their own, so that the peak is
# the intersection's; ids in one window, several, and ranges searched.
@pytest.mark.parametrize("n,tune", [(2400, None), (4000, {"wbits": 10}),
                                    (4000, {"wbits": 10, "flags": scan.SCAN_TUNE_SEARCH_WINDOWS})])
def test_builds_fit_without_optional_memory(n, tune):
    used = 2400
    rng = np.random.default_rng(n)
    place = np.sort(rng.permutation(n)[:used])
    u, v = np.nonzero(np.triu(rng.random((used, used)) < 0.6, 1))
    g = graphgen.from_edges(n, np.stack([place[u], place[v]], 1).astype(np.int32))
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    csr = device_csr(g)

    def run(_):
        return scan.scan_build_index(*csr, scan.COSINE, scan.SCAN_KEEP_SIMS | scan.SCAN_KEEP_COUNTS, tune=tune)

    def check(ix):
        assert_index_equal(ix, oix, g)
        ix.free()

    with hooks() as h:
        least, refused = least_memory(h, lambda: None, run, check)
        assert refused, "nothing that the build can do without"
        check(attempt(h, lambda: None, run, budget=least))


# A sweep succeeds within the memory that it needs for one clustering at a
# time: the queries' workspaces are taken before the tables that score many.
@pytest.mark.parametrize("batch", [5, 32])
def test_sweeps_fit_without_optional_memory(batch):
    g = graphgen.sbm(120000, 300, 0.02, 0.00001, 7)
    grid = [(mu, eps) for mu in (2, 3, 5, 9) for eps in (0.05, 0.1, 0.15, 0.2, 0.25, 0.3, 0.4, 0.5)]
    csr = device_csr(g)

    def run(ix):  # (an index without workspaces)
        try:
            return scan.scan_sweep_modularity(ix, [m for m, _ in grid], [e for _, e in grid], batch=batch)
        finally:
            ix.free()

    want = []

    def check(q):
        if not want:
            want.append(q)
            assert len(np.unique(q)) > 4
        assert np.array_equal(q, want[0])

    with hooks() as h:
        least, refused = least_memory(h, lambda: scan.scan_build_index(*csr), run, check)
        assert refused, "nothing that the sweep can do without"
        check(attempt(h, lambda: scan.scan_build_index(*csr), run, budget=least))


# Most of a large build's memory is what its sorts hold, 68 bytes per slot with
# the index (similarities by slot, by row and by segment, and the merges' two
# copies); beside them per vertex the offsets (8), degrees (4), ranks (16) and
# the lists of the row sort (60), and two chunks of 32 MiB. What the
# intersection alone needs (32 bytes per vertex) is not held then.
@pytest.mark.parametrize("weighted", [False, True])
def test_memory_of_a_large_build(weighted):
    import torch

    n = 1 << 20
    rng = np.random.default_rng(3)
    g = graphgen.from_edges(n, rng.integers(0, n, (2 * n, 2)).astype(np.int32))
    off, adj = device_csr(g)
    w = torch.rand(g.nnz, dtype=torch.float64, device="cuda")
    with hooks() as h:
        h.start()
        ix = scan.scan_build_index_weighted(off, adj, w) if weighted else scan.scan_build_index(off, adj)
        torch.cuda.synchronize()
        assert h.peak <= 68 * g.nnz + (8 + 4 + 16 + 60) * n + 2 * (32 << 20)
        ix.free()
