"""Asynchronous C4 where a vertex's undecided neighbours outgrow the kept
list, rows are walked by a whole wave, or everything waits in a chain; and
labels delivered to a buffer that is not 16-byte aligned."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

CASES = {
    "clique": (lambda: graphgen.from_edges(700, [(i, j) for i in range(700) for j in range(i)]), True),
    "clique_random": (lambda: graphgen.from_edges(1100, [(i, j) for i in range(1100) for j in range(i)]), False),
    "pairs_512": (lambda: graphgen.from_edges(514, [(513, i) for i in range(513)]), True),
    "late_hubs": (lambda: graphgen.from_edges(20_000, [(19_999 - h, i) for h in range(4) for i in range(19_990)]), True),
    "chain": (lambda: graphgen.from_edges(50_000, [(i, i + 1) for i in range(49_999)]), True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_async_rows(name):
    import torch
    import paper_1507_05086_amd as cc
    make, identity = CASES[name]
    g = make()
    order = np.arange(g.n, dtype=np.int32) if identity else graphgen.permutation(g.n, 2)
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    want = oracle.kwikcluster(g.off, g.col, order)
    for _ in range(3):
        lab, _ = cc.cc_c4_async(gh, torch.from_numpy(order).cuda())
        assert np.array_equal(lab.cpu().numpy(), want)


@pytest.mark.parametrize("n", [1, 3, 4, 1027])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_labels_at_any_address(n, shift):
    import torch
    import paper_1507_05086_amd as cc
    g = graphgen.from_edges(n, [(i, i + 1) for i in range(0, n - 1, 2)])
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col.copy() if g.nnz else np.zeros(1, np.int32)).cuda()[:g.nnz])
    order = torch.from_numpy(graphgen.permutation(n, 1)).cuda()
    buf = torch.full((n + 8,), -7, dtype=torch.int32, device="cuda")
    want = oracle.kwikcluster(g.off, g.col, order.cpu().numpy())
    for run in (lambda o: cc.cc_c4(gh, order, 0.5, labels=o), lambda o: cc.cc_c4_async(gh, order, labels=o)):
        buf.fill_(-7)
        run(buf[shift:shift + n])
        got = buf.cpu().numpy()
        assert np.array_equal(got[shift:shift + n], want)
        assert (got[:shift] == -7).all() and (got[shift + n:] == -7).all()
