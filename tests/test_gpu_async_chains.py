"""Asynchronous C4 where the vertices of one wave wait for each other: orders
that follow the graph, about the 64 positions a wave works on.  The limit on
the long path's time is several times what it takes, and a third of what it
took with a round trip to memory for every vertex of a chain."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _path(n, step=1):
    v = np.arange(n - step)
    return graphgen.from_edges(n, np.stack([v, v + step], 1).astype(np.int32))


def _clique(n):
    return graphgen.from_edges(n, np.stack(np.triu_indices(n, 1), 1).astype(np.int32))


def _band(n, width):
    return graphgen.from_edges(n, np.concatenate([np.stack([np.arange(n - d), np.arange(d, n)], 1) for d in
                                                  range(1, width + 1)]).astype(np.int32))


GRAPHS = {
    **{f"path{n}": (lambda n=n: _path(n)) for n in (2, 63, 64, 65, 129, 4100)},
    **{f"step{s}": (lambda s=s: _path(3000, s)) for s in (31, 32, 33, 63, 64, 65)},
    **{f"clique{n}": (lambda n=n: _clique(n)) for n in (33, 64, 65, 300)},
    # more undecided neighbours than a wave keeps as pairs, inside its chunk and before it
    "band20": lambda: _band(5000, 20),
    "band150": lambda: _band(5000, 150),
    "grid": lambda: graphgen.from_edges(10_000, [(i, i + 1) for i in range(9999) if i % 100 != 99] +
                                        [(i, i + 100) for i in range(9900)]),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("waves", [0, 1, 5])
def test_labels(name, waves):
    import torch
    import paper_1507_05086_amd as cc
    g = GRAPHS[name]()
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    up = np.arange(g.n, dtype=np.int32)
    for order in (up, up[::-1].copy(), graphgen.permutation(g.n, 3)):
        lab, _ = cc.cc_c4_async(gh, torch.from_numpy(order).cuda(), waves=waves)
        assert np.array_equal(lab.cpu().numpy(), oracle.kwikcluster(g.off, g.col, order))


def test_time_of_a_chain():
    import torch
    import paper_1507_05086_amd as cc
    g = _path(100_000)
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = torch.arange(g.n, dtype=torch.int32, device="cuda")
    times = []
    for _ in range(5):
        lab, st = cc.cc_c4_async(gh, order)
        times.append(st.loop_ms)
    assert np.array_equal(lab.cpu().numpy(), oracle.kwikcluster(g.off, g.col, order.cpu().numpy()))
    assert min(times) < 40.0, times
