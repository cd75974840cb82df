"""Builds and sorts at the edges of their dispatch: the one-launch sort and the
per-class one, passes that find their own splits and passes that read them,
and the one-workgroup core-order preparation, against numpy and the oracle."""

from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle
import paper_2012_11188_amd as scan
from gpu_util import assert_index_equal, gpu_build

pytestmark = pytest.mark.gpu


# one launch for all classes up to 4 << 20 elements; own splits up to 1024 tiles of 4096
@pytest.mark.parametrize("big", [[], [4097], [9000, 4096 * 40, 4096 * 33 + 1], [4096 * 900], [4096 * 1023 + 5],
                                 [4096 * 1030, 8193, 50000]])
@pytest.mark.parametrize("fill", [0, 1 << 20])
def test_sort_paths(big, fill):
    rng = np.random.default_rng(len(big) + fill + sum(big))
    caps = [0, 1, 2, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096]
    lens = caps * 3 + big
    while fill > 0:
        part = rng.integers(0, 5000, 50).tolist()
        lens += part
        fill -= sum(part)
    lens = np.array(lens)[rng.permutation(len(lens))]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    keys = rng.integers(-50, 400, off[-1]) / 7.0  # many ties
    keys[keys == 0] = 0.5
    ids = np.concatenate([rng.permutation(n) for n in lens] or [np.zeros(0)]).astype(np.int32)
    ko, io = scan.scan_segmented_sort(off, keys, ids)
    seg = np.repeat(np.arange(len(lens)), lens)
    order = np.lexsort((ids, -keys, seg))
    assert np.array_equal(ko, keys[order]) and np.array_equal(io, ids[order])


def hub_and_ring(n, degree):
    """A ring of n vertices and one vertex joined to `degree` of them."""
    ring = [(i, (i + 1) % n) for i in range(n)]
    return graphgen.from_edges(n, ring + [(5, (7 + 2 * i) % n) for i in range(degree - 2)])


# one workgroup prepares the core order up to 32768 vertices and degree 4096
@pytest.mark.parametrize("n,degree", [(9001, 4095), (9001, 4096), (9001, 4097), (32767, 60), (32768, 4096),
                                      (32769, 60), (63, 5), (64, 5), (65, 5)])
def test_core_order_preparation(n, degree):
    g = hub_and_ring(n, degree)
    assert int(g.degrees().max()) == degree
    assert_index_equal(gpu_build(g), oracle.build_index(g, oracle.COSINE, threads=8), g)


# ids numbered without isolated vertices: several windows left, one left, and
# one or no id between used ones
@pytest.mark.parametrize("tune", [{"wbits": 10, "small_max": 8, "spc": 64}, {"wbits": 11, "small_max": 4},
                                  {"wbits": 10, "small_max": 8, "flags": scan.SCAN_TUNE_SEARCH_WINDOWS}])
@pytest.mark.parametrize("used,n", [(700, 5000), (1024, 2049), (1025, 4000), (3000, 3001), (3000, 9000)])
def test_isolated_vertices_left_out(used, n, tune):
    from gpu_util import device_csr

    base = graphgen.sbm(used, 5, 0.06, 0.02, 31)
    rng = np.random.default_rng(used + n)
    place = np.sort(rng.permutation(n)[:used])
    u = np.repeat(np.arange(used), base.degrees())
    g = graphgen.from_edges(n, np.stack([place[u], place[base.adj]], 1).astype(np.int32))
    for kind in (scan.COSINE, scan.JACCARD):
        ix = scan.scan_build_index(*device_csr(g), kind, scan.SCAN_KEEP_SIMS | scan.SCAN_KEEP_COUNTS, tune=tune)
        assert_index_equal(ix, oracle.build_index(g, kind, threads=8), g)


# a dense core (rows and columns of the hub product: tiles of 256, column
# blocks of 256) with a sparse rim whose ids lie between the core's; one id
# window, several, and ranges searched instead of tabled (no product)
@pytest.mark.parametrize("core,rim,tune", [(1535, 0, None), (1536, 100, None), (1537, 6000, None), (1700, 9000, None),
                                           (1537, 6000, {"wbits": 11}), (1700, 9000, {"wbits": 12, "spc": 96}),
                                           (1700, 3000, {"wbits": 10, "small_max": 900}),
                                           (1537, 6000, {"wbits": 11, "flags": scan.SCAN_TUNE_SEARCH_WINDOWS})])
def test_hub_product(core, rim, tune):
    from gpu_util import device_csr

    rng = np.random.default_rng(core + rim)
    n = core + rim
    place = rng.permutation(n)
    p = np.where(np.arange(core) < core // 3, 0.97, 0.6)  # two levels of degree
    u, v = np.nonzero(np.triu(rng.random((core, core)) < np.sqrt(p[:, None] * p[None, :]), 1))
    edges = [np.stack([place[u], place[v]], 1)]
    if rim:
        k = 6 * rim
        edges.append(np.stack([place[core + rng.integers(0, rim, k)], place[rng.integers(0, n, k)]], 1))
    g = graphgen.from_edges(n, np.concatenate(edges).astype(np.int32))
    for kind in (scan.COSINE, scan.JACCARD):
        ix = scan.scan_build_index(*device_csr(g), kind, scan.SCAN_KEEP_SIMS | scan.SCAN_KEEP_COUNTS, tune=tune)
        assert_index_equal(ix, oracle.build_index(g, kind, threads=8), g)


# lengths around a short range (128 ids), an item (512 with several windows,
# 1024 with one) and two of them, among large owners' lower neighbours; one
# window, a few, and more than a wavefront's lanes; a slot per chunk, few, a
# thread per slot
@pytest.mark.parametrize("tune", [{"small_max": 2100, "spc": 1024}, {"small_max": 2100, "spc": 1},
                                  {"small_max": 2100, "spc": 7, "wbits": 16}, {"small_max": 2100, "wbits": 10},
                                  {"small_max": 2100, "wbits": 12, "spc": 1024},
                                  {"small_max": 2100, "wbits": 13, "flags": scan.SCAN_TUNE_SEARCH_WINDOWS}])
@pytest.mark.parametrize("first", [True, False])
def test_range_lengths(tune, first):
    from gpu_util import device_csr

    n, owners = 70000, 3
    rng = np.random.default_rng(5)
    place = rng.permutation(n)
    if first:  # the owners have the ids 0 and n - 1 and one between as neighbours and ids
        place[[np.flatnonzero(place == 0)[0], 0]] = place[[0, np.flatnonzero(place == 0)[0]]]
        place[[np.flatnonzero(place == n - 1)[0], 1]] = place[[1, np.flatnonzero(place == n - 1)[0]]]
    edges = [np.stack([np.full(6000, o), rng.choice(np.arange(100, n), 6000, replace=False)], 1) for o in range(owners)]
    edges.append(np.array([(0, 1), (0, 2), (1, 2)]))
    pool = np.concatenate([e[:, 1] for e in edges[:owners]])
    at = owners
    for length in (2, 3, 15, 16, 17, 63, 64, 65, 127, 128, 129, 130, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2049):
        for seen in range(2):
            mates = rng.choice(pool if seen else np.arange(100, n), 4 * length + 40)
            mates = np.unique(mates[mates != at])[: length - owners] if length > owners else mates[:0]
            edges.append(np.stack([np.full(len(mates), at), mates], 1))
            edges.append(np.stack([np.full(owners, at), np.arange(owners)], 1)[:length])
            at += 1
    g = graphgen.from_edges(n, place[np.concatenate(edges)].astype(np.int32))
    ix = scan.scan_build_index(*device_csr(g), scan.COSINE, scan.SCAN_KEEP_SIMS | scan.SCAN_KEEP_COUNTS, tune=tune)
    assert_index_equal(ix, oracle.build_index(g, scan.COSINE, threads=8), g)


# rows around a step of the light kernel's groups (64 ids) and of the heavy
# one's (128), the largest of each, and ids that fill whole hash buckets (by
# the top bits of the low 24 of id * 10368889): more than one bucket holds
@pytest.mark.parametrize("tune", [None, {"small_max": 4096}, {"small_max": 1}, {"small_max": 700, "wbits": 10}])
@pytest.mark.parametrize("degree", [3, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257])
def test_small_owner_rows(degree, tune):
    from gpu_util import device_csr

    n = 1 << 17
    ids = np.arange(n, dtype=np.uint64)
    top = ((ids * 10368889) & 0xFFFFFF) >> 16
    same = np.flatnonzero((top == 7) | (top == 8))[:degree]  # close in the table
    rng = np.random.default_rng(degree)
    rest = rng.choice(np.setdiff1d(np.arange(n), same), degree + 40, replace=False)
    edges = [(a, b) for i, a in enumerate(same[:40]) for b in same[i + 1:]]  # a clique and its further members
    edges += [(a, b) for a, b in zip(same, rest)]
    edges += [(int(rest[0]), int(b)) for b in rest[1:degree]] + [(int(rest[1]), int(b)) for b in rest[5:degree]]
    g = graphgen.from_edges(n, np.array(edges, np.int64).astype(np.int32))
    ix = scan.scan_build_index(*device_csr(g), scan.COSINE, scan.SCAN_KEEP_SIMS | scan.SCAN_KEEP_COUNTS, tune=tune)
    assert_index_equal(ix, oracle.build_index(g, scan.COSINE, threads=8), g)


# The product over hub rows is formed where the cases above mean it to be: all
# vertices of a dense core are its rows and columns. It is not with searched
# ranges, several graphs or approximate similarities, nor where its memory is
# refused; the index is the same. (2037 ids: one window, or two of 1024.)
@pytest.mark.parametrize("how,tune", [("one", None), ("one", {"wbits": 10}), ("refused", None), ("refused", {"wbits": 10}),
                                      ("none", {"wbits": 10, "flags": scan.SCAN_TUNE_SEARCH_WINDOWS}),
                                      ("two", None), ("lsh", None)])
def test_hub_product_is_formed(how, tune):
    from alloc_hooks import hooks
    from gpu_util import device_csr

    core, rim = 1537, 500
    rng = np.random.default_rng(core)
    place = rng.permutation(core + rim)
    u, v = np.nonzero(np.triu(rng.random((core, core)) < 0.7, 1))
    edges = [np.stack([place[u], place[v]], 1),
             np.stack([place[core + np.arange(rim)], place[core + (np.arange(rim) + 1) % rim]], 1)]
    g = graphgen.from_edges(core + rim, np.concatenate(edges).astype(np.int32))
    csr = device_csr(g)
    flags = scan.SCAN_KEEP_SIMS | scan.SCAN_KEEP_COUNTS
    if how == "two":
        assert [scan.scan_index_hub_product(ix) for ix in scan.scan_build_index_batch([csr, csr])] == [(0, 0)] * 2
        return
    if how == "lsh":
        perm = graphgen.permutation(g.n, 3)
        import torch

        ix = scan.scan_build_index_lsh(*csr, scan.JACCARD, 64, perm=torch.from_numpy(perm).cuda())
        assert scan.scan_index_hub_product(ix) == (0, 0)
        return
    oix = oracle.build_index(g, oracle.COSINE, threads=8)
    want = (core, core) if how == "one" else (0, 0)
    if how != "refused":
        ix = scan.scan_build_index(*csr, scan.COSINE, flags, tune=tune)
        assert scan.scan_index_hub_product(ix) == want
        assert_index_equal(ix, oix, g)
        return
    without = 0
    with hooks() as h:
        h.start()
        scan.scan_build_index(*csr, scan.COSINE, flags, tune=tune).free()
        for k in range(h.calls):
            h.start(refuse=[k])
            try:
                ix = scan.scan_build_index(*csr, scan.COSINE, flags, tune=tune)
            except scan.ScanError as e:
                assert e.status == scan.SCAN_ENOMEM
                continue
            if scan.scan_index_hub_product(ix) == want:
                without += 1
                assert_index_equal(ix, oix, g)
            ix.free()
    assert without >= 1


# shapes left open: small owners up to 512 and chunks of 1024 slots where more
# than 2^20 vertices have neighbours, 256 and 768 else, whatever the ids span
@pytest.mark.parametrize("used,n,wide", [((1 << 20) + 1, (1 << 20) + 1, True), ((1 << 20) + 1, (1 << 21) + 77, True),
                                         (1 << 20, 1 << 20, False), (1 << 20, (1 << 21) + 77, False)])
def test_open_shapes(used, n, wide):
    from gpu_util import device_csr

    step = n / used
    place = (np.arange(used) * step).astype(np.int64)
    ring = np.stack([place, place[(np.arange(used) + 1) % used]], 1)
    hubs = [np.stack([np.full(d - 2, place[h]), place[3 * h + 7 + 5 * np.arange(d - 2)]], 1)
            for h, d in ((11, 257), (1000, 512), (50000, 513), (90000, 900))]
    g = graphgen.from_edges(n, np.concatenate([ring, *hubs]).astype(np.int32))
    assert int((g.degrees() > 0).sum()) == used
    deg = g.degrees()
    ix = scan.scan_build_index(*device_csr(g), scan.COSINE, scan.SCAN_KEEP_SIMS | scan.SCAN_KEEP_COUNTS | scan.SCAN_PROFILE)
    p = scan.scan_index_build_profile(ix)
    small, spc = (512, 1024) if wide else (256, 768)
    assert p["small_owners"] == int(((deg > 0) & (deg <= small)).sum())
    assert p["big_chunks"] == int((-(-deg[deg > small] // spc)).sum())
    assert_index_equal(ix, oracle.build_index(g, oracle.COSINE, threads=8), g)
