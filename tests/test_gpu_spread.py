"""Rounds of a few active vertices that bring many entries with them: the team
shares the positions out one by one, so that no workgroup has all the claims."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_common import check_against_oracle, torch_cuda, upload

pytestmark = pytest.mark.gpu

GRAPHS = {
    "dense": (lambda: graphgen.erdos_renyi(5000, 300.0, 2), 0.5),
    "denser": (lambda: graphgen.erdos_renyi(2000, 700.0, 3), 2.0),
    "few_ahead": (lambda: graphgen.chung_lu(9000, 2.1, 90.0, 4), 0.9),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_against_oracle(name):
    torch_cuda()
    import paper_1507_05086_amd as cc
    cc.cc_set_eps_policy(cc.CC_EPS_FIXED)
    make, eps = GRAPHS[name]
    g = make()
    gh = upload(g)
    for seed in range(3):
        for algo in (oracle.C4, oracle.CW):
            check_against_oracle(algo, g, gh, graphgen.permutation(g.n, seed), eps)


def test_time_of_heavy_rounds():
    """0.85 ms; 1.7 ms while one workgroup peeled all that a round had claimed."""
    import paper_1507_05086_amd as cc
    torch = torch_cuda()
    g = graphgen.erdos_renyi(5000, 300.0, 2)
    gh = upload(g)
    order = torch.from_numpy(graphgen.permutation(g.n, 1)).cuda()
    assert min(cc.cc_clusterwild(gh, order, 0.5)[1].loop_ms for _ in range(8)) < 1.3
