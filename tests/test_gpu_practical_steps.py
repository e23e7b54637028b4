"""The practical schedule on one workgroup and on one XCD: rounds whose
positions take several selection steps, the last of them partly filled, and
consecutive rounds of rows that the workgroups share."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

FIELDS = ("n_i", "delta_i", "b_i", "r_i", "centers", "claimed", "conflicts")


def _matching(n):
    return graphgen.from_edges(n, np.arange(n, dtype=np.int32).reshape(-1, 2))


# one workgroup takes 2048 positions a step, 32 of them 65536
STEPS = {
    "one_workgroup_matching": (lambda: _matching(16_384), 0.9),
    "one_workgroup": (lambda: graphgen.erdos_renyi(11_000, 3.0, 1), 9.0),
    "one_workgroup_all": (lambda: graphgen.erdos_renyi(10_241, 3.0, 2), 1000.0),
    "one_workgroup_even": (lambda: graphgen.erdos_renyi(12_288, 2.0, 3), 5.0),
    "one_xcd": (lambda: graphgen.erdos_renyi(220_000, 0.6, 4), 4.0),
}


def _check(g, algo, eps, seeds, order_of=None):
    import torch
    import paper_1507_05086_amd as cc
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    kind, run = (oracle.C4, cc.cc_c4) if algo == "c4" else (oracle.CW, cc.cc_clusterwild)
    most = 0
    for seed in seeds:
        order = order_of(seed) if order_of else graphgen.permutation(g.n, 10 + seed)
        ref = oracle.bsp_binomial(kind, g.off, g.col, order, eps, seed, 0.1)
        cc.cc_set_eps_policy(cc.CC_EPS_BINOMIAL, (seed, 0.1))
        try:
            lab, st = run(gh, torch.from_numpy(order).cuda(), eps)
        finally:
            cc.cc_set_eps_policy(cc.CC_EPS_FIXED)
        assert st.rounds == ref.rounds
        assert np.array_equal(lab.cpu().numpy(), ref.labels)
        for f in FIELDS:
            assert np.array_equal(st.trace[f], ref.trace[f]), f
        most = max(most, int(ref.trace["b_i"].max()))
    return most


@pytest.mark.parametrize("algo", ["c4", "cw"])
@pytest.mark.parametrize("name", sorted(STEPS))
def test_several_steps(name, algo):
    make, eps = STEPS[name]
    most = _check(make(), algo, eps, range(4))
    assert most > (2 * 2048 if name.startswith("one_workgroup") else 65_536)


HUBS, LEAVES = 3000, 3000


def _shared_rows():
    """Hubs in cliques of four, each with over 2048 of the same leaves: a
    round's active hubs take few others with them."""
    rng = np.random.default_rng(5)
    e = [np.stack([np.full(2300, h), HUBS + rng.choice(LEAVES, 2300, replace=False)], 1) for h in range(HUBS)]
    e += [[(h + i, h + j) for h in range(0, HUBS, 4) for i in range(4) for j in range(i)]]
    return graphgen.from_edges(HUBS + LEAVES, np.concatenate(e).astype(np.int32))


@pytest.mark.parametrize("algo", ["c4", "cw"])
@pytest.mark.parametrize("eps", [0.9, 4.0])
def test_shared_rows_round_after_round(algo, eps):
    """Rows too long for a workgroup to keep are in a list that all of them
    read, filled again by the next round; cliques follow each other in pi, so
    most rounds have active neighbours."""
    _check(_shared_rows(), algo, eps, range(3), lambda seed: np.concatenate(
        [(4 * graphgen.permutation(HUBS // 4, seed)[:, None] + np.arange(4)).ravel(),
         HUBS + graphgen.permutation(LEAVES, seed)]).astype(np.int32))
