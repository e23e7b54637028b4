"""What the round loop's host side keeps and counts, as the error of the
fault_round test hook tells it."""
import re

import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


def _inject(cc, run, k):
    """(round graphs kept, slots queued, slots counted) of a run that fails after round k."""
    with pytest.raises(cc.CCError) as e:
        run(fault_round=k)
    assert e.value.code == cc.CC_ERR_DEVICE
    return tuple(int(x) for x in re.search(r"kept: (\d+).*queued: (\d+).*counted: (\d+)", str(e.value)).groups())


@pytest.mark.parametrize("scale,entries", [(20, 16), (24, 1)])
def test_a_new_labels_buffer_builds_no_graphs(scale, entries):
    """Scale 20 has a team and rounds too wide for it, 24 round kernels alone."""
    import torch
    import paper_1507_05086_amd as cc
    g = graphgen.rmat(scale, entries, 0.57, 0.19, 0.19, seed=9)
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = torch.from_numpy(graphgen.permutation(g.n, 5)).cuda()
    kept, buffers = [], []
    for _ in range(4):
        buffers.append(torch.empty(g.n, dtype=torch.int32, device="cuda"))  # all alive: four addresses
        kept.append(_inject(cc, lambda **k: cc.cc_c4(gh, order, 0.5, labels=buffers[-1], **k), 40)[0])
    assert kept[0] > 0 and len(set(kept)) == 1, kept
