"""RunStats.trace holds what the library recorded and zeros elsewhere: a batch
records no rounds, and of a single graph's run the first 65536 are kept."""
import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


@pytest.fixture
def cc(monkeypatch):
    import paper_1507_05086_amd as cc
    plain = np.empty

    def used_memory(*a, **k):  # what np.empty returns once the heap has been used
        out = plain(*a, **k)
        if out.flags.c_contiguous:
            out.reshape(-1).view(np.uint8)[:] = 0xA5
        return out
    monkeypatch.setattr(np, "empty", used_memory)
    return cc


@pytest.mark.parametrize("capacity", [1 << 14, 3])
def test_batch_has_no_records(cc, capacity):
    import torch
    parts = [graphgen.erdos_renyi(n, 8.0, n) for n in (50, 400)]
    ptr = np.array([0, 50, 450], np.int64)
    off = np.concatenate([parts[0].off, parts[1].off[1:] + parts[0].nnz]).astype(np.int64)
    col = np.concatenate([g.col for g in parts]).astype(np.int32)
    gh = cc.cc_graph_from_csr(torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda(), vtx_ptr=ptr)
    order = torch.from_numpy(graphgen.batch_permutations(ptr, 1)).cuda()
    for run in (cc.cc_c4, cc.cc_clusterwild):
        _, st = run(gh, order, 0.5, trace_capacity=capacity)
        assert st.rounds == st.graph_rounds.max() > 3
        assert len(st.trace) == min(st.rounds, capacity)
        for f in st.trace.dtype.names:
            assert not st.trace[f].any(), f


def test_rounds_past_the_records_kept(cc):
    import torch
    n = 180_000  # one vertex a round: about 0.43 n rounds
    e = np.arange(n - 1, dtype=np.int32)
    g = graphgen.from_edges(n, np.stack([e, e + 1], 1))
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    _, st = cc.cc_c4(gh, torch.from_numpy(graphgen.permutation(n, 2)).cuda(), 1e-6, trace_capacity=1 << 17)
    kept = 1 << 16
    assert st.rounds > kept and len(st.trace) == st.rounds and st.truncated == 1
    assert (st.trace["n_i"][:kept] > 0).all() and (st.trace["b_i"][:kept] == 1).all()
    for f in st.trace.dtype.names:
        assert not st.trace[f][kept:].any(), f
