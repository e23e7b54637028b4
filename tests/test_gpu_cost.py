"""cc_cost on the renumbered rows at the edges of its tiles (2048 entries)
and for clusterings that are not a run's own, against the oracle's count."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _graphs():
    yield "tile", graphgen.from_edges(1025, [(i, i + 1) for i in range(1024)])        # 2048 entries
    yield "tile_less", graphgen.from_edges(1024, [(i, i + 1) for i in range(1023)])   # 2046
    yield "tile_more", graphgen.from_edges(1026, [(i, i + 1) for i in range(1025)])   # 2050
    yield "row_ends_tile", graphgen.from_edges(4100, [(0, i) for i in range(1, 2049)] + [(i, i + 1) for i in range(2050, 4000)])
    yield "long_row", graphgen.from_edges(9001, [(0, i) for i in range(1, 9001)])
    yield "isolated", graphgen.from_edges(5000, [(7, 4999)])
    yield "edgeless", graphgen.from_edges(33, [])
    yield "power", graphgen.chung_lu(30_007, 2.1, 30.0, 3)


@pytest.mark.parametrize("name", [n for n, _ in _graphs()])
def test_cost_at_tile_edges(name):
    import torch
    import paper_1507_05086_amd as cc
    g = dict(_graphs())[name]
    off, col = torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col.copy() if g.nnz else np.zeros(1, np.int32)).cuda()[:g.nnz]
    gh = cc.cc_graph_from_csr(off, col)
    rng = np.random.default_rng(1)
    for labels in (np.zeros(g.n, np.int32), np.arange(g.n, dtype=np.int32),
                   rng.integers(0, g.n, g.n).astype(np.int32), rng.integers(0, min(3, g.n), g.n).astype(np.int32)):
        want = oracle.cost(g.off, g.col, labels)
        assert int(cc.cc_cost(gh, torch.from_numpy(labels).cuda())[0]) == want
        assert int(cc.cc_cost(gh, labels)[0]) == want
    bad = np.zeros(g.n, np.int32)
    for v in (-1, g.n):
        bad[g.n // 2] = v
        with pytest.raises(cc.CCError) as e:
            cc.cc_cost(gh, bad)
        assert e.value.code == cc.CC_ERR_INVALID_ARG
