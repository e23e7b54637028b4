"""Rows of a batch member at the lengths where their walk changes: shorter
than a lane's four entries, whole steps and one entry more, a hub dealt to the
whole group, and the last row of the column array."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _graphs():
    clique = lambda n: graphgen.from_edges(n, [(i, j) for i in range(n) for j in range(i)])
    star = lambda n: graphgen.from_edges(n, [(0, i) for i in range(1, n)])
    hub = lambda n, m: graphgen.from_edges(n, [(0, i) for i in range(1, n)] + [(i, i + 1) for i in range(1, m)])
    sets = {
        "short": [graphgen.from_edges(2, [(0, 1)]), clique(3), clique(4), clique(5), clique(6), star(5)],
        "tiny_array": [graphgen.from_edges(2, [(0, 1)]), graphgen.from_edges(3, [])],  # fewer entries than a lane reads
        "steps": [clique(n) for n in (9, 17, 18, 33, 34, 65, 66, 129, 257, 258)],
        "hubs": [star(1024), star(1025), star(1026), hub(1537, 900), hub(5000, 4000), hub(2049, 2)],
        "dense": [clique(600), clique(1025), star(3000)],
        "end": [star(3000), clique(10), graphgen.from_edges(7, [(5, 6)])],
        "edgeless": [graphgen.from_edges(1, []), graphgen.from_edges(40, []), clique(7)],
    }
    return sets


@pytest.mark.parametrize("shape", [None, (1024, 0), (256, 5000), (1024, 64, 1100)])
@pytest.mark.parametrize("name", sorted(_graphs()))
def test_rows(name, shape):
    import torch
    import paper_1507_05086_amd as cc
    parts = _graphs()[name]
    ptr = np.concatenate([[0], np.cumsum([g.n for g in parts])]).astype(np.int64)
    base = np.concatenate([[0], np.cumsum([g.off[-1] for g in parts])])
    off = np.concatenate([[0]] + [g.off[1:] + b for g, b in zip(parts, base)]).astype(np.int64)
    col = np.concatenate([g.col for g in parts]).astype(np.int32)
    # borrowed, and exactly as long as the offsets say
    t_off, t_col = torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda()
    gh = cc.cc_graph_from_csr(t_off, t_col, vtx_ptr=ptr, validate=True, borrow=True)
    if shape:
        if shape[0] == 256 and max(g.n for g in parts) > 1100:
            shape = (256, 1100)  # four waves' slots fit
        cc.cc_batch_set_config(gh, *shape)
    order = graphgen.batch_permutations(ptr, 4)
    for algo, run in ((oracle.C4, cc.cc_c4), (oracle.CW, cc.cc_clusterwild)):
        for eps in (0.3, 8.0):
            lab, st = run(gh, torch.from_numpy(order).cuda(), eps)
            lab = lab.cpu().numpy()
            for i, g in enumerate(parts):
                a, b = int(ptr[i]), int(ptr[i + 1])
                ref = oracle.bsp(algo, g.off, g.col, order[a:b], eps)
                assert np.array_equal(lab[a:b], ref.labels), (i, algo, eps)
                assert st.graph_rounds[i] == ref.rounds
