"""Rounds whose active vertices are hubs, so that they walk far more entries
than the graph's mean degree lets expect: the team lists them and leaves them to
the whole device before the election."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_common import TRACE_INT_FIELDS, torch_cuda

pytestmark = pytest.mark.gpu


def _hubs(hubs, leaves, degree, friends=0):
    """`hubs` vertices next to `degree` of the leaves each; the first `friends` of them a clique."""
    rng = np.random.default_rng(1)
    e = [np.stack([np.full(degree, h), hubs + rng.choice(leaves, degree, replace=False)], 1) for h in range(hubs)]
    if friends:
        e.append(np.stack(np.triu_indices(friends, 1), 1))
    return graphgen.from_edges(hubs + leaves, np.concatenate(e).astype(np.int32))


GRAPHS = {
    "hubs": lambda: _hubs(120, 60_000, 8000, 40),
    "star": lambda: _hubs(1, 700_000, 700_000),
    # short rows beside the long ones
    "mixed": lambda: graphgen.from_edges(160_100, np.concatenate(
        [np.stack([np.full(9000, h), 100 + 9 * np.arange(9000) + h % 9], 1) for h in range(100)] +
        [np.stack([np.arange(100, 160_000, 2), np.arange(101, 160_001, 2)], 1)]).astype(np.int32)),
}


@pytest.mark.parametrize("algo", ["c4", "cw"])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_against_oracle(name, algo):
    torch = torch_cuda()
    import paper_1507_05086_amd as cc
    g = GRAPHS[name]()
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda(), validate=True)
    kind, run = (oracle.C4, cc.cc_c4) if algo == "c4" else (oracle.CW, cc.cc_clusterwild)
    order = np.arange(g.n, dtype=np.int32)  # the hubs first
    for eps, seed in ((0.5, None), (30.0, None), (1000.0, None), (2.0, 3), (60.0, 4)):
        if seed is None:
            ref = oracle.bsp(kind, g.off, g.col, order, eps)
        else:
            ref = oracle.bsp_binomial(kind, g.off, g.col, order, eps, seed, 0.1)
            cc.cc_set_eps_policy(cc.CC_EPS_BINOMIAL, (seed, 0.1))
        try:
            lab, st = run(gh, torch.from_numpy(order).cuda(), eps)
        finally:
            cc.cc_set_eps_policy(cc.CC_EPS_FIXED)
        assert st.rounds == ref.rounds
        assert np.array_equal(lab.cpu().numpy(), ref.labels)
        for f in TRACE_INT_FIELDS:
            assert np.array_equal(st.trace[f], ref.trace[f]), (f, eps, seed)


def test_time_of_hub_rounds():
    """0.6 ms; 2.2 ms while the workgroups of one XCD walked twenty million entries."""
    torch = torch_cuda()
    import paper_1507_05086_amd as cc
    g = _hubs(2000, 400_000, 10_000)
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = torch.arange(g.n, dtype=torch.int32, device="cuda")
    assert min(cc.cc_clusterwild(gh, order, 50.0)[1].loop_ms for _ in range(8)) < 1.3
