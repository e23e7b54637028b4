"""Rounds run by one workgroup or by the workgroups of one XCD (cc_team.hip):
the sizes and shapes at which that path changes, against the oracle's loop,
labels and every trace field exactly."""
import threading

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

FIELDS = ("n_i", "delta_i", "b_i", "r_i", "centers", "claimed", "conflicts")


def _clique(n):
    return graphgen.from_edges(n, [(i, j) for i in range(n) for j in range(i)])


def _star_ring(n, hubs):
    e = [(h, v) for h in range(hubs) for v in range(hubs, n)]
    return graphgen.from_edges(n, e + [(v, v + 1) for v in range(hubs, n - 1)])


CASES = {
    # one workgroup: the largest run it takes, and one entry more
    "solo_edge": (lambda: graphgen.from_edges(16384, [(i, i + 1) for i in range(16383)]), 0.5),
    "past_solo": (lambda: graphgen.from_edges(16400, [(i, i + 1) for i in range(16399)]), 0.5),
    # more conflict edges than its LDS holds: the round kernels settle them
    "solo_conflicts": (lambda: _clique(200), 1000.0),
    "team_conflicts": (lambda: _clique(400), 1000.0),
    # the most conflict edges k_resolve keeps in registers, one row more, and a long chain of them
    "resolve_edge": (lambda: _clique(256), 1000.0),
    "resolve_past": (lambda: _clique(257), 1000.0),
    "chain_at_once": (lambda: graphgen.from_edges(30_000, [(i, i + 1) for i in range(29_999)]), 4.0),
    # rows longer than a workgroup keeps for itself, a chain of blocked vertices
    "long_rows": (lambda: _star_ring(30_000, 3), 2.0),
    "chain": (lambda: graphgen.from_edges(60_000, [(i, i + 1) for i in range(59_999)]), 0.05),
    # lazy Delta passes, the switch to exact degrees, and both after it
    "power": (lambda: graphgen.chung_lu(40_009, 2.1, 40.0, 7), 0.5),
    "power_wide": (lambda: graphgen.chung_lu(40_009, 2.1, 40.0, 7), 8.0),
    "rmat": (lambda: graphgen.rmat(17, 16, 0.57, 0.19, 0.19, seed=9), 0.5),
}


def _check(cc, gh, g, order, eps, algo):
    import torch
    lab, st = (cc.cc_c4 if algo == "c4" else cc.cc_clusterwild)(gh, torch.from_numpy(order).cuda(), eps)
    ref = oracle.bsp(oracle.C4 if algo == "c4" else oracle.CW, g.off, g.col, order, eps)
    assert st.rounds == ref.rounds
    assert np.array_equal(lab.cpu().numpy(), ref.labels)
    for f in FIELDS:
        assert np.array_equal(st.trace[f], ref.trace[f]), f


@pytest.mark.parametrize("algo", ["c4", "cw"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_team_against_oracle(name, algo):
    import torch
    import paper_1507_05086_amd as cc
    make, eps = CASES[name]
    g = make()
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = np.arange(g.n, dtype=np.int32) if name.startswith("chain") else graphgen.permutation(g.n, 5)
    for _ in range(2):  # the workspace of the first run serves the second
        _check(cc, gh, g, order, eps, algo)


@pytest.mark.parametrize("algo", ["c4", "cw"])
def test_more_active_rows_than_a_workgroup_keeps(algo):
    """A matching: the practical schedule's first round has 200 K active rows."""
    import torch
    import paper_1507_05086_amd as cc
    n = 400_000
    g = graphgen.from_edges(n, np.arange(n, dtype=np.int32).reshape(-1, 2))
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = graphgen.permutation(n, 6)
    cc.cc_set_eps_policy(cc.CC_EPS_BINOMIAL, (3, 0.1))
    try:
        lab, st = (cc.cc_c4 if algo == "c4" else cc.cc_clusterwild)(gh, torch.from_numpy(order).cuda(), 0.5)
    finally:
        cc.cc_set_eps_policy(cc.CC_EPS_FIXED)
    ref = oracle.bsp_binomial(oracle.C4 if algo == "c4" else oracle.CW, g.off, g.col, order, 0.5, 3, 0.1)
    assert st.rounds == ref.rounds
    assert np.array_equal(lab.cpu().numpy(), ref.labels)
    for f in FIELDS:
        assert np.array_equal(st.trace[f], ref.trace[f]), f


@pytest.mark.parametrize("n", [600, 40_000])
def test_partial_and_failing_runs(n):
    """A bounded run's labels, and errors that leave the labels alone."""
    import torch
    import paper_1507_05086_amd as cc
    g = graphgen.erdos_renyi(n, 12.0, 3)
    gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
    order = graphgen.permutation(n, 8)
    d_order = torch.from_numpy(order).cuda()
    full = oracle.bsp(oracle.C4, g.off, g.col, order, 0.5)
    lab, st = cc.cc_c4(gh, d_order, 0.5, max_rounds=3)
    lab = lab.cpu().numpy()
    assert st.rounds == 3
    done = lab >= 0
    assert np.array_equal(lab[done], full.labels[done])
    assert done.sum() == n - full.trace["n_i"][3]
    keep = torch.full((n,), 77, dtype=torch.int32, device="cuda")
    with pytest.raises(cc.CCError) as e:
        cc.cc_c4(gh, d_order, 0.5, labels=keep, fault_round=2)
    assert e.value.code == cc.CC_ERR_DEVICE
    for wrong in (order[0], n, -1):
        o = order.copy()
        o[n // 2] = wrong
        with pytest.raises(cc.CCError) as e:
            cc.cc_c4(gh, torch.from_numpy(o).cuda(), 0.5, labels=keep)
        assert e.value.code == cc.CC_ERR_NOT_PERMUTATION
    assert bool((keep == 77).all())
    host, _ = cc.cc_c4(gh, order, 0.5)  # host order and labels
    assert np.array_equal(host, full.labels)


def test_teams_of_several_threads_and_streams():
    import torch
    import paper_1507_05086_amd as cc
    graphs = [graphgen.chung_lu(30_011 + 1000 * i, 2.1, 30.0, 20 + i) for i in range(3)]
    refs, errors = [], []
    for i, g in enumerate(graphs):
        order = graphgen.permutation(g.n, 30 + i)
        refs.append((g, order, oracle.bsp(oracle.CW, g.off, g.col, order, 0.5).labels))

    def work(g, order, ref):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                gh = cc.cc_graph_from_csr(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.col).cuda())
                d = torch.from_numpy(order).cuda()
                for _ in range(10):  # the first builds the round graphs while others run
                    lab, _ = cc.cc_clusterwild(gh, d, 0.5)
                    assert np.array_equal(lab.cpu().numpy(), ref)
        except BaseException as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=r) for r in refs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
