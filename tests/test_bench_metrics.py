"""Host-side metrics of bench.py: the adjusted Rand index of Section 7.2
(unclustered vertices as clusters of their own), pinned against a hand-worked
contingency table and scikit-learn's implementation."""

import numpy as np
import pytest

import bench


def test_ari_hand_worked():
    # C = {0,1,2} {3,4} ; G = {0,1} {2,3,4}; n = 5, C(5,2) = 10
    # n_ij: (C1,G1)=2, (C1,G2)=1, (C2,G2)=2 -> sum C(n_ij,2) = 1 + 0 + 1 = 2
    # rows 3, 2 -> 3 + 1 = 4; columns 2, 3 -> 1 + 3 = 4; expected 4*4/10 = 1.6
    # ARI = (2 - 1.6) / ((4 + 4)/2 - 1.6) = 0.4 / 2.4 = 1/6
    a = np.array([0, 0, 0, 3, 3])
    b = np.array([0, 0, 2, 2, 2])
    assert bench.adjusted_rand_index(a, b) == pytest.approx(1 / 6, abs=1e-15)
    assert bench.adjusted_rand_index(a, a) == 1.0
    # -1 entries are singletons: all unclustered on both sides is identical
    assert bench.adjusted_rand_index(np.full(4, -1), np.full(4, -1)) == 1.0


def test_ari_matches_sklearn():
    metrics = pytest.importorskip("sklearn.metrics")
    rng = np.random.default_rng(3)
    for n, k in [(50, 3), (400, 20), (2000, 200)]:
        a = rng.integers(-1, k, n)
        b = np.where(rng.random(n) < 0.7, a, rng.integers(-1, k, n))
        la, lb = bench._labels(a), bench._labels(b)
        assert bench.adjusted_rand_index(a, b) == pytest.approx(metrics.adjusted_rand_score(la, lb), abs=1e-12)


def test_source_hashes():
    """The marks that cut the kernels' source are in the sources."""
    import bench

    assert len(bench.kernel_source_hash()) == 64 and len(bench.library_source_hash()) == 64
    assert bench.counter_traffic({"small_max": 1, "spc": 1, "wbits": 1}, "none")[0] is None


def test_hub_split():
    """Edges between product rows and their answered ids, against the sets; the
    kernel's bytes leave the answered ids out."""
    import graphgen

    g = graphgen.rmat(9, 12, seed=4)
    deg = np.diff(g.off)
    ranked = np.sort(deg)[::-1]
    rows = int((deg >= ranked[60]).sum())
    cols = int((deg >= ranked[150]).sum())
    small_max = int(ranked[40])
    is_row, is_col = deg >= ranked[60], deg >= ranked[150]
    edges = answered = 0
    for u in np.flatnonzero(is_row):
        row = g.adj[g.off[u]:g.off[u + 1]]
        for h in row:
            if is_row[h] and deg[h] > small_max and (deg[u], u) < (deg[h], h):
                edges += 1
                answered += int(is_col[row].sum())
    hub = bench.hub_split(g, rows, cols, small_max)
    assert hub == {"edges": edges, "answered": answered} and edges > 100
    assert bench.hub_split(g, 0, 0, small_max) == {"edges": 0, "answered": 0}
    split, st = graphgen.owner_split(g, small_max), graphgen.degree_stats(g)
    whole = bench.byte_model(st, split, 4, deg, small_max)
    less = bench.byte_model(st, split, 4, deg, small_max, hub)
    assert whole["k_big_owner"] - less["k_big_owner"] == 4 * answered - 36 * edges
    assert {k: v for k, v in whole.items() if k != "k_big_owner"} == {k: v for k, v in less.items() if k != "k_big_owner"}
    phases = {"intersect_big_ms": 2.0, "plan_ms": 1.0}
    roof = bench.kernel_roofline(less, phases, {"small_max": small_max, "spc": 1, "wbits": 1}, "none")
    assert roof["achieved"] == pytest.approx(less["k_big_owner"] / 2e-3 / 1e9)
    assert roof["model_frac"] == pytest.approx(less["k_big_owner_model"] / 3e-3 / 1e9 / bench.HBM_PEAK_GBS)


@pytest.mark.parametrize("name,kernel", [("intersect.hip", True), ("hubs.hip", True), ("index.h", True),
                                         ("common.h", True), ("rows.h", True), ("query.hip", False)])
def test_kernel_hash_covers_its_sources(tmp_path, monkeypatch, name, kernel):
    """A change to any source that the large-owner kernel's traffic follows
    from makes counters taken before it stale; one elsewhere does not."""
    import shutil

    src = tmp_path / "csrc"
    shutil.copytree(bench.CSRC, src)
    monkeypatch.setattr(bench, "CSRC", str(src))
    before = bench.kernel_source_hash(), bench.library_source_hash()
    with open(src / name, "a") as f:
        f.write("// more\n")
    after = bench.kernel_source_hash(), bench.library_source_hash()
    assert (before[0] != after[0]) == kernel and before[1] != after[1]


def test_headline_is_one_short_line():
    """The printed line keeps the contract's fields and every summary, and does
    not grow with the number of queries, rates or trials."""
    import json

    row = {"offered_qps": 1234.5678901234567, "achieved_qps": 1234.5678901234567, "p50_ms": 0.12345678901234567,
           "p99_ms": 0.12345678901234567}

    def rec(k):
        return bench.record(1.5e9, 20, 5, 6.1, "f64", {"workload": "w", "tune": {"spc": 1}}, roofline={"frac": 0.5},
                            query={"queries": k, "batched": {"p50_ms": 0.5}, "per_query": [row] * k},
                            approx_quality=[{"graph": "g", "simhash_cosine": {"ari_mean": 0.9, "trials": [row] * k}}],
                            serving={"device": {"batched": {"max_slots": 4, "ladder": [row] * k},
                                                "batched_max_qps_within_budget": 5.0}})

    line, detail = bench.headline(rec(3))
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config"):
        assert line[key] == rec(3)[key]
    assert line["approx_quality"] == [{"graph": "g", "simhash_cosine": {"ari_mean": 0.9}}]
    assert line["serving"]["device"] == {"batched": {"max_slots": 4}, "batched_max_qps_within_budget": 5.0}
    assert {k: len(v) for k, v in detail.items()} == {"query.per_query": 3, "serving.device.batched.ladder": 3,
                                                      "approx_quality.0.simhash_cosine.trials": 3}
    assert len(json.dumps(bench.headline(rec(5000))[0])) < len(json.dumps(line)) + 10
    assert len(json.dumps(rec(200))) > 20000
