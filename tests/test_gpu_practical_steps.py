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


def _check(g, algo, eps, seeds):
    import torch
    import paper_1507_05086_amd as cc
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    kind, run = (oracle.C4, cc.cc_c4) if algo == "c4" else (oracle.CW, cc.cc_clusterwild)
    most = 0
    for seed in seeds:
        order = graphgen.permutation(g.n, 10 + seed)
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
