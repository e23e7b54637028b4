"""Lists that the round kernels stage in LDS, long enough for a workgroup to go
over its share several times: full and half-full buffers between the passes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

FIELDS = ("n_i", "delta_i", "b_i", "r_i", "centers", "claimed", "conflicts")
SHARES = 512  # workgroups a list is cut for, 256 threads each


def _circulant(n, k):
    """Every vertex next to the k before and the k after it, on a ring."""
    step = np.concatenate([np.arange(-k, 0), np.arange(1, k + 1)])
    col = (np.arange(n, dtype=np.int64)[:, None] + step) % n
    col[:k].sort(axis=1)
    col[-k:].sort(axis=1)
    off = np.arange(n + 1, dtype=np.int64) * (2 * k)
    return graphgen.Graph(n=n, off=off, col=np.ascontiguousarray(col.ravel(), dtype=np.int32))


def _ring_and_hub():
    """A ring of degree 70 and a vertex next to 100 K others: its leaving ends the lazy search."""
    g, hub = _circulant(140_001, 35), 100_000
    rows = np.repeat(np.arange(g.n), np.diff(g.off))
    leaves = np.arange(g.n + 1, g.n + 1 + hub)
    return graphgen.from_edges(g.n + 1 + hub, np.concatenate(
        [np.stack([rows, g.col], 1)[rows < g.col], np.stack([np.full(hub, g.n), leaves], 1)]).astype(np.int32))


CASES = {
    # more active and claimed vertices than one pass of every workgroup; exact degrees
    "active": (lambda: graphgen.erdos_renyi(4 * SHARES * 256 + 77, 2.5, 1), 1000.0),
    "claimed": (lambda: graphgen.erdos_renyi(4 * SHARES * 256, 9.0, 2), 6.0),
    # rows recounted at the switch
    "switch": (_ring_and_hub, 0.5),
    # candidates of a Delta pass, four per thread and pass
    "candidates": (lambda: _circulant(4 * SHARES * 256 + 6000, 94), 8.0),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_several_passes(name):
    import torch
    import paper_1507_05086_amd as cc
    make, eps = CASES[name]
    g = make()
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = graphgen.permutation(g.n, 5)
    if name == "switch":
        order[np.flatnonzero(order == 140_001)[0]] = order[0]
        order[0] = 140_001
    for algo, run in ((oracle.C4, cc.cc_c4), (oracle.CW, cc.cc_clusterwild)):
        lab, st = run(gh, torch.from_numpy(order).cuda(), eps)
        ref = oracle.bsp(algo, g.off, g.col, order, eps)
        assert st.rounds == ref.rounds
        assert np.array_equal(lab.cpu().numpy(), ref.labels)
        for f in FIELDS:
            assert np.array_equal(st.trace[f], ref.trace[f]), f
