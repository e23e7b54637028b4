"""The last tile of the cost's walk: a workgroup's threads behind its end have
nothing to look for among the tile's rows."""
import time

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

TILE = 2048  # entries


def _matching(n):
    return graphgen.from_edges(n, np.arange(n, dtype=np.int32).reshape(-1, 2))


def _least_time(n):
    import torch
    import paper_1507_05086_amd as cc
    g = _matching(n)
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    lab = np.random.default_rng(n).integers(0, n // 3, n).astype(np.int32)
    d_lab = torch.from_numpy(lab).cuda()
    best = 1.0
    for _ in range(30):
        t = time.perf_counter()
        c = cc.cc_cost(gh, d_lab)
        best = min(best, time.perf_counter() - t)
    assert int(c[0]) == oracle.cost(g.off, g.col, lab)
    return best


def test_a_ragged_tile_costs_no_more_than_a_full_one():
    """Rows of one entry: a walk from the first to the last of them, which the
    threads behind the end took, made the ragged one take twice as long."""
    full = _least_time(2 * TILE)
    for entries in (2 * TILE - 2, 2 * TILE - 600, TILE + 1400):
        assert _least_time(entries) < 1.5 * full, entries
