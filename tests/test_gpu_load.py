"""cc_graph_from_csr's checks against their definition, entry by entry: the
validating pass searches one entry of each pair and counts both kinds, so every
way in which a pair can be broken must still give the code of a full search."""
import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


def _code(cc, off, col, ptr):
    """The smallest failing code over all entries; a column out of range outranks it."""
    codes = set()
    for a, b in zip(ptr[:-1], ptr[1:]):
        for v in range(a, b):
            row = col[off[v]:off[v + 1]]
            for i, u in enumerate(row):
                if not 0 <= u < b - a:
                    return cc.CC_ERR_OUT_OF_RANGE
                if u == v - a:
                    codes.add(cc.CC_ERR_SELF_LOOP)
                if i + 1 < len(row) and row[i + 1] <= u:
                    codes.add(cc.CC_ERR_DUPLICATE_EDGE)
                other = col[off[a + u]:off[a + u + 1]]
                lo, hi = 0, len(other)  # first entry not below, as a binary search finds it
                while lo < hi:
                    mid = (lo + hi) // 2
                    lo, hi = (mid + 1, hi) if other[mid] < v - a else (lo, mid)
                if not (lo < len(other) and other[lo] == v - a):
                    codes.add(cc.CC_ERR_NOT_SYMMETRIC)
    return min(codes, default=cc.CC_OK)


def _break(rows, how, rng):
    full = [v for v, r in enumerate(rows) if len(r)]
    v = full[rng.integers(len(full))]
    long = max(full, key=lambda x: len(rows[x]))
    if how == "drop":
        rows[v].pop(rng.integers(len(rows[v])))
    elif how == "drop_long":  # from the row whose entries are searched
        rows[long].pop(rng.integers(len(rows[long])))
    elif how == "drop_two":   # one entry of either kind: the counts stay equal
        u = rows[long].pop(0)
        for w in full:
            if w not in (u, long) and rows[w] and rows[w][0] == long:
                rows[w].pop(0)
                break
    elif how == "repeat":
        rows[v].insert(0, rows[v][0])
    elif how == "repeat_pair":  # an entry and its mirror twice
        u = rows[v][0]
        rows[v].insert(0, u)
        rows[u].insert(rows[u].index(v), v)
    elif how == "loop":
        rows[v] = sorted(rows[v] + [v])
    elif how == "swap":
        rows[long].reverse()
    elif how == "move":  # an entry points elsewhere
        u = next((x for x in range(len(rows)) if x not in rows[v] and x != v), rows[v][0])
        rows[v][0] = u
        rows[v].sort()
    elif how == "range":
        rows[v][-1] = len(rows)
    return rows


def _graphs():
    yield "er", graphgen.erdos_renyi(60, 200, 3)
    yield "power", graphgen.chung_lu(200, 2.1, 8.0, 2)
    yield "star", graphgen.from_edges(300, [(0, i) for i in range(1, 300)])
    yield "clique", graphgen.from_edges(40, [(i, j) for i in range(40) for j in range(i)])
    yield "pair", graphgen.from_edges(4, [(1, 2)])


@pytest.mark.parametrize("how", ["none", "drop", "drop_long", "drop_two", "repeat", "repeat_pair", "loop", "swap",
                                 "move", "range"])
def test_validate_codes(how):
    import torch
    import paper_1507_05086_amd as cc
    rng = np.random.default_rng(5)
    for name, g in _graphs():
        rows = [list(map(int, g.col[g.off[v]:g.off[v + 1]])) for v in range(g.n)]
        rows = _break(rows, how, rng)
        off = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        col = np.array([u for r in rows for u in r], np.int32)
        # alone, and as the middle graph of a batch of three
        gp = [0, g.n, 2 * g.n, 3 * g.n]
        boff = np.concatenate([g.off, g.off[-1] + off[1:], g.off[-1] + off[-1] + g.off[1:]]).astype(np.int64)
        bcol = np.concatenate([g.col, col, g.col]).astype(np.int32)
        for o, c, ptr, kw in ((off, col, [0, g.n], {}), (boff, bcol, gp, {"vtx_ptr": np.array(gp, np.int64)})):
            want = _code(cc, o, c, ptr)
            for dev in (False, True):
                args = (torch.from_numpy(o).cuda(), torch.from_numpy(c).cuda()) if dev else (o, c)
                if want == cc.CC_OK:
                    h = cc.cc_graph_from_csr(*args, validate=True, **kw)
                    order = np.concatenate([rng.permutation(b - a) for a, b in zip(ptr[:-1], ptr[1:])]).astype(np.int32)
                    cc.cc_c4(h, order, 0.5)
                    continue
                with pytest.raises(cc.CCError) as e:
                    cc.cc_graph_from_csr(*args, validate=True, **kw)
                assert e.value.code == want, (name, how, dev, len(ptr))


@pytest.mark.parametrize("n", [1, 256, 257, 70_001])
def test_offsets(n):
    """Refused before anything uses them, from either memory and in a batch."""
    import torch
    import paper_1507_05086_amd as cc
    for at in {0, 1, n // 2, n - 1, n}:
        off = np.zeros(n + 1, np.int64)
        off[at] += 1 if at < n else -1
        for kw in ({}, {"vtx_ptr": np.array([0, n // 2, n], np.int64)}):
            for dev in (False, True):
                o, c = (torch.from_numpy(off).cuda(), torch.zeros(1, dtype=torch.int32).cuda()) if dev else \
                    (off, np.zeros(1, np.int32))
                with pytest.raises(cc.CCError) as e:
                    cc.cc_graph_from_csr(o, c, **kw)
                assert e.value.code == cc.CC_ERR_INVALID_ARG
