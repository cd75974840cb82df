"""Refused device memory: what a call that is refused some leaves behind, and
what is answered without, against the oracle."""

from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle
import paper_2012_11188_amd as scan
from alloc_hooks import hooks
from gpu_util import gpu_build

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
