"""Rounds whose search for the next Delta needs a second or third pass, or
none finds it and the run switches to exact degrees, with more candidate rows
than k_team takes: each pass has a slot of the round kernels to itself."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

FIELDS = ("n_i", "delta_i", "b_i", "r_i", "centers", "claimed", "conflicts")
HUB, LEAVES = 100_000, 100_000


def _steps(hubs, degree):
    """One vertex of degree HUB, then `hubs` of the given degree, on other leaves."""
    rng = np.random.default_rng(degree)
    base = 1 + HUB
    edges = [np.stack([np.zeros(HUB, np.int64), 1 + np.arange(HUB)], 1)]
    for i in range(hubs):
        leaves = base + hubs + rng.choice(LEAVES, degree, replace=False)
        edges.append(np.stack([np.full(degree, base + i), leaves], 1))
    return graphgen.from_edges(base + hubs + LEAVES, np.concatenate(edges).astype(np.int32))


@pytest.mark.parametrize("algo", ["c4", "cw"])
@pytest.mark.parametrize("hubs,degree", [(60, 25_000), (60, 20_000), (60, 80_000), (4000, 400), (2, 1_500)])
def test_delta_passes(algo, hubs, degree):
    import torch
    import paper_1507_05086_amd as cc
    g = _steps(hubs, degree)
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda(), validate=True)
    order = graphgen.permutation(g.n, 3)
    order[np.flatnonzero(order == 0)[0]] = order[0]
    order[0] = 0  # the first round takes the largest row away
    run, ref_algo = (cc.cc_c4, oracle.C4) if algo == "c4" else (cc.cc_clusterwild, oracle.CW)
    ref = oracle.bsp(ref_algo, g.off, g.col, order, 0.5)
    for _ in range(2):
        lab, st = run(gh, torch.from_numpy(order).cuda(), 0.5)
        assert st.rounds == ref.rounds
        assert np.array_equal(lab.cpu().numpy(), ref.labels)
        for f in FIELDS:
            assert np.array_equal(st.trace[f], ref.trace[f]), f
    # a run that ends while the search would go on
    lab, st = run(gh, torch.from_numpy(order).cuda(), 0.5, max_rounds=1)
    assert st.rounds == 1 and st.trace["centers"][0] == ref.trace["centers"][0]
