"""Rows that hold their own vertex, unvalidated: a center has nothing to claim
from itself, so C4's labels are those of the graph without the loops."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _with_loops(g, every):
    """A loop at each `every`-th vertex, in its place in the ascending row."""
    rows = np.repeat(np.arange(g.n), np.diff(g.off))
    loops = np.arange(0, g.n, every)
    r, c = np.concatenate([rows, loops]), np.concatenate([g.col, loops])
    k = np.lexsort((c, r))
    off = np.zeros(g.n + 1, np.int64)
    np.cumsum(np.bincount(r, minlength=g.n), out=off[1:])
    return off, c[k].astype(np.int32)


GRAPHS = {
    "one_workgroup": (lambda: graphgen.erdos_renyi(1500, 8.0, 1), 0.5),
    "one_xcd": (lambda: graphgen.erdos_renyi(20_000, 10.0, 2), 0.5),
    # rows that the workgroups share, roots and promoted alike; lazy and exact rounds
    "long_rows": (lambda: graphgen.erdos_renyi(6000, 2600.0, 3), 40.0),
    "power": (lambda: graphgen.chung_lu(40_009, 2.1, 40.0, 7), 0.5),
}


@pytest.mark.parametrize("every", [1, 7])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_c4_labels(name, every):
    import torch
    import paper_1507_05086_amd as cc
    make, eps = GRAPHS[name]
    g = make()
    off, col = _with_loops(g, every)
    gh = cc.cc_graph_from_csr(torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda())
    order = graphgen.permutation(g.n, 5)
    lab, _ = cc.cc_c4(gh, torch.from_numpy(order).cuda(), eps)
    assert np.array_equal(lab.cpu().numpy(), oracle.kwikcluster(g.off, g.col, order))


@pytest.mark.parametrize("every", [1, 7])
@pytest.mark.parametrize("n", [1500, 30_011])
def test_cost_counts_stored_entries(n, every):
    """m and m_in are half the stored entries, a loop's one among them."""
    import torch
    import paper_1507_05086_amd as cc
    g = graphgen.erdos_renyi(n, 9.0, n)
    off, col = _with_loops(g, every)
    gh = cc.cc_graph_from_csr(torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda())
    lab = np.random.default_rng(1).integers(0, n // 20, n).astype(np.int32)
    size = np.bincount(lab).astype(np.int64)
    same = int((np.repeat(lab, np.diff(off)) == lab[col]).sum())
    assert int(cc.cc_cost(gh, torch.from_numpy(lab).cuda())[0]) == int((size * (size - 1) // 2).sum()) + len(col) // 2 - same
