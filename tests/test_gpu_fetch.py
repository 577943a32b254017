"""Fetched rows at the sizes where the transfer changes: tiles of 256 rows, the
small and the large transfer area, pieces of an area, segments, offsets."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SMALL, LARGE = 32768, 1 << 20  # 4-byte values per part of the two areas


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1807_07691_amd as G
    return G


@pytest.mark.parametrize("n", [1, 255, 256, 257, SMALL - 1, SMALL, SMALL + 1, 2 * SMALL + 3,
                               LARGE, LARGE + 1, 2 * LARGE + 259])
def test_fetch_edges(G, n):
    # vertex 0 has n objects; every tenth of them leads to two others
    x = np.arange(1, n + 1, dtype=np.int32)
    lead = x[x % 10 == 1]
    s = np.concatenate([np.zeros(n, np.int32), lead, lead])
    p = np.concatenate([np.zeros(n, np.int32), np.ones(2 * len(lead), np.int32)])
    o = np.concatenate([x, lead % 3, 3 + lead % 5]).astype(np.int32)
    st = G.gsmat_load_triples(s, p, o, n + 9, 2)
    G.gsmat_build_index(st)
    two = np.stack([np.repeat(lead, 2), np.stack([lead % 3, 3 + lead % 5], 1).ravel()], 1)
    for q, want, budget in (([[0, 0, -1]], x[:, None], 0),
                            ([[0, 0, -1], [-1, 1, -2]], two, 0),
                            ([[0, 0, -1], [-1, 1, -2]], two, max(800, 4 * len(two)))):
        pl = G.gsmat_plan(st, q, G.PLAN_ADAPTIVE)
        r = G.gsmat_join(st, pl, budget)
        print(f"[gpu] fetch n={n} cols={want.shape[1]} budget={budget}", flush=True)
        got = G.gsmat_fetch_bindings(r)
        order = np.lexsort(got.T[::-1])
        assert np.array_equal(got[order], want[np.lexsort(want.T[::-1])])
        m = len(got)
        for lo, cnt in ((0, 1), (m // 2, m), (m - 1, 5), (1, 256), (m // 3, m // 2), (m, 4)):
            page = G.gsmat_fetch_bindings(r, lo, cnt)
            assert np.array_equal(page, got[lo:lo + cnt]), (lo, cnt)
        r.close()
        pl.close()
    st.close()


@pytest.mark.parametrize("sizes", [[0], [1, 0, 7], [256] * 300, [SMALL // 2 + 1] * 5,
                                   [3, LARGE + 5, 0, 12, 2 * LARGE + 1, 255, 40_000]])
def test_fetch_many(G, sizes):
    # vertex i has sizes[i] objects along predicate 0 and two along predicate 1
    V = max(max(sizes), len(sizes)) + 2
    s = np.repeat(np.arange(len(sizes)), sizes)
    o = np.concatenate([np.arange(z) for z in sizes])
    k = np.arange(len(sizes))
    t = [np.concatenate([s, k, k]), np.concatenate([np.zeros(len(s)), np.ones(2 * len(k))]),
         np.concatenate([o, k % 2, 1 + k])]
    s, p, o = (np.asarray(x).astype(np.int32) for x in t)
    st = G.gsmat_load_triples(s, p, o, V, 2)
    G.gsmat_build_index(st)
    print(f"[gpu] fetch many {len(sizes)} results", flush=True)
    qs = [[[i, 0, -1]] for i in range(len(sizes))] + [[[0, 1, 0]], [[-1, 1, -2]]]
    plans, _ = G.gsmat_plan_batch(st, qs)
    res = [G.gsmat_join(st, pl) for pl in plans]
    got = G.gsmat_fetch_bindings_many(res)
    for i, z in enumerate(sizes):
        assert np.array_equal(got[i], np.arange(z, dtype=np.int32)[:, None]), i
    for a, r in zip(got, res):
        assert a.shape == (G.gsmat_result_info(r)["rows"], G.gsmat_result_info(r)["n_vars"])
        assert np.array_equal(a, G.gsmat_fetch_bindings(r))
        r.close()
    for pl in plans:
        pl.close()
    st.close()
