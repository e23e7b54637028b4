"""Between 2^22 and 2^23 vertices a run has both the bucketed mapping of pi and
a team: rounds with Delta passes, the switch to exact degrees and what follows."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_common import check_against_oracle, torch_cuda, upload

pytestmark = pytest.mark.gpu


def test_delta_passes_on_mapped_orders():
    torch_cuda()
    import paper_1507_05086_amd as cc
    cc.cc_set_eps_policy(cc.CC_EPS_FIXED)
    g = graphgen.chung_lu(4_500_001, 2.1, 6.0, 7)
    gh = upload(g)
    order = graphgen.permutation(g.n, 5)
    for algo in (oracle.C4, oracle.CW):
        _, _, ref = check_against_oracle(algo, g, gh, order, 0.5)
        assert ref.trace["delta_i"][0] > 4096 and (np.diff(ref.trace["delta_i"]) < 0).sum() > 50
