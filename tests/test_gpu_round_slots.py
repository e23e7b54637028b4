"""What the round loop's host side keeps and counts, as the error of the
fault_round test hook tells it."""
import re

import numpy as np
import pytest

import graphgen
import oracle

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


def _stale_bounds(hub=100_000, others=30_000, rows=60):
    """A vertex with `hub` leaves, and rows that share most of those leaves:
    once it has taken them, the rows' bounds are far above what remains."""
    rng = np.random.default_rng(3)
    base = 1 + hub
    e = [np.stack([np.zeros(hub, np.int64), 1 + np.arange(hub)], 1)]
    for i in range(rows):
        near, far = 1 + rng.choice(hub, 72_000, replace=False), base + rows + rng.choice(others, 8000, replace=False)
        e.append(np.stack([np.full(80_000, base + i), np.concatenate([near, far])], 1))
    return graphgen.from_edges(base + rows + others, np.concatenate(e).astype(np.int32))


@pytest.mark.parametrize("algo", ["c4", "cw"])
def test_every_slot_is_counted(algo):
    """The team leaves the first round to the device in its search for the next
    Delta, and the device needs more than one pass: a slot each, and each counted."""
    import torch
    import paper_1507_05086_amd as cc
    g = _stale_bounds()
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = graphgen.permutation(g.n, 3)
    order[np.flatnonzero(order == 0)[0]] = order[0]
    order[0] = 0  # the first round takes the hub's leaves away
    d_order = torch.from_numpy(order).cuda()
    fn, kind = (cc.cc_c4, oracle.C4) if algo == "c4" else (cc.cc_clusterwild, oracle.CW)
    ref = oracle.bsp(kind, g.off, g.col, order, 0.5)
    lab, st = fn(gh, d_order, 0.5)
    assert st.rounds == ref.rounds and np.array_equal(lab.cpu().numpy(), ref.labels)
    assert np.array_equal(st.trace["delta_i"], ref.trace["delta_i"])
    _, queued, counted = _inject(cc, lambda **k: fn(gh, d_order, 0.5, **k), min(6, ref.rounds))
    assert counted > 2 and queued - counted <= 2  # what is queued behind the failing slot is not run
