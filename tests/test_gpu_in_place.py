"""Labels written over the order they were computed from: a call may be given
one device buffer as both, on every path a run can take."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

PATHS = {
    "one_workgroup": lambda: graphgen.erdos_renyi(3001, 6.0, 1),
    "one_xcd": lambda: graphgen.erdos_renyi(20_011, 10.0, 2),
    "round_kernels": lambda: graphgen.erdos_renyi((1 << 23) + 5, 1.5, 3),
}


def _same_buffer(run, order, *args, **kw):
    import torch
    buf = torch.from_numpy(order).cuda()
    out, _ = run(buf, *args, labels=buf, **kw)
    assert out is buf
    return buf.cpu().numpy()


@pytest.mark.parametrize("path", sorted(PATHS))
def test_single_graph(path):
    import torch
    import paper_1507_05086_amd as cc
    g = PATHS[path]()
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = graphgen.permutation(g.n, 4)
    for algo, fn in ((oracle.C4, cc.cc_c4), (oracle.CW, cc.cc_clusterwild)):
        ref = oracle.bsp(algo, g.off, g.col, order, 0.5).labels
        assert np.array_equal(_same_buffer(lambda o, **k: fn(gh, o, 0.5, **k), order), ref)
    part = cc.cc_c4(gh, torch.from_numpy(order).cuda(), 0.5, max_rounds=2)[0].cpu().numpy()
    assert np.array_equal(_same_buffer(lambda o, **k: cc.cc_c4(gh, o, 0.5, max_rounds=2, **k), order), part)
    kwik = oracle.kwikcluster(g.off, g.col, order)
    assert np.array_equal(_same_buffer(lambda o, **k: cc.cc_c4_async(gh, o, **k), order), kwik)


def test_batch():
    import torch
    import paper_1507_05086_amd as cc
    parts = [graphgen.erdos_renyi(n, 8.0, n) for n in (40, 300, 1500, 5000)]
    ptr = np.concatenate([[0], np.cumsum([g.n for g in parts])]).astype(np.int64)
    base = np.concatenate([[0], np.cumsum([g.nnz for g in parts])])
    off = np.concatenate([[0]] + [g.off[1:] + b for g, b in zip(parts, base)]).astype(np.int64)
    col = np.concatenate([g.col for g in parts]).astype(np.int32)
    gh = cc.cc_graph_from_csr(torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda(), vtx_ptr=ptr)
    order = graphgen.batch_permutations(ptr, 4)
    lab = _same_buffer(lambda o, **k: cc.cc_c4(gh, o, 0.5, **k), order)
    for i, g in enumerate(parts):
        a, b = int(ptr[i]), int(ptr[i + 1])
        assert np.array_equal(lab[a:b], oracle.kwikcluster(g.off, g.col, order[a:b])), i
