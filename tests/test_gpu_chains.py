"""Long dependences among the active vertices of C4: a path whose order follows
it, where each vertex waits for the one before.  The labels are the oracle's,
and a level of the dependence takes microseconds (the limits below are several
times what it takes, and a fraction of what it took with a barrier, or with a
round trip to memory, for every level)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _path(n):
    return graphgen.from_edges(n, np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32))


def _clique(n):
    return graphgen.from_edges(n, np.stack(np.triu_indices(n, 1), 1).astype(np.int32))


def _load(g):
    import torch
    import paper_1507_05086_amd as cc
    return cc, cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())


# conflict edges about the limits: 4096 in one workgroup of the team, 32768 in k_resolve
GRAPHS = {
    "pair": lambda: _path(2),
    "clique91": lambda: _clique(91),
    "clique92": lambda: _clique(92),
    "path4097": lambda: _path(4097),
    "path4098": lambda: _path(4098),
    "path32769": lambda: _path(32_769),
    "path32770": lambda: _path(32_770),
    "sparse": lambda: graphgen.erdos_renyi(3000, 2.5, 1),
    "sparse_wide": lambda: graphgen.erdos_renyi(24_000, 2.5, 2),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_all_active_at_once(name):
    import torch
    g = GRAPHS[name]()
    cc, gh = _load(g)
    up = np.arange(g.n, dtype=np.int32)
    for order in (up, up[::-1].copy(), graphgen.permutation(g.n, 3)):
        lab, st = cc.cc_c4(gh, torch.from_numpy(order).cuda(), 1000.0)
        ref = oracle.bsp(oracle.C4, g.off, g.col, order, 1000.0)
        assert st.rounds == ref.rounds == 1
        assert np.array_equal(lab.cpu().numpy(), ref.labels)
        assert st.blocked == ref.trace["conflicts"].sum()


@pytest.mark.parametrize("n,eps,most_ms", [(3000, 20.0, 4.0), (100_000, 0.5, 250.0)])
def test_time_of_a_level(n, eps, most_ms):
    import torch
    g = _path(n)
    cc, gh = _load(g)
    order = np.arange(n, dtype=np.int32)
    d_order = torch.from_numpy(order).cuda()
    times = []
    for _ in range(5):
        lab, st = cc.cc_c4(gh, d_order, eps)
        times.append(st.loop_ms)
    assert np.array_equal(lab.cpu().numpy(), oracle.kwikcluster(g.off, g.col, order))
    assert min(times) < most_ms, times
