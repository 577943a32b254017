"""OPTIONAL and FILTER on parts at the size where one workgroup selects their
rows (4096 rows; up to 65536 matches), against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1807_07691_amd as G
    return G


@pytest.mark.parametrize("n,fan", [(1, 1), (64, 2), (4095, 1), (4096, 2), (4097, 2), (4096, 40),
                                   (300, 400)])
def test_small_parts(G, n, fan):
    from oracle import algebra
    r = np.random.default_rng(n + fan)
    V = n + fan + 8
    x = np.arange(1, n + 1)
    some = x[r.random(n) < 0.5]
    src = np.repeat(some, fan)
    t = [np.stack([np.zeros(n, int), np.zeros(n, int), x], 1),
         np.stack([src, np.full(len(src), 1), r.integers(0, V, len(src))], 1),
         np.stack([x, np.full(n, 2), r.permutation(x)], 1)]
    a = np.concatenate(t).astype(np.int32)
    s, p, o = (a[:, i].copy() for i in range(3))
    st = G.gsmat_load_triples(s, p, o, V, 3)
    G.gsmat_build_index(st)
    base = [[0, 0, -1, 0, 0]]
    opt = [[-1, 1, -2, 0, 1]]
    two = [[-1, 2, -3, 0, 2]]
    lo = int(x[n // 2])
    queries = [(base + opt, []), (base + opt + two, []), (base, [[G.F_LT, -1, lo, 0]]),
               (base, [[G.F_GE, -1, 0, 0]]), (base, [[G.F_LT, -1, 0, 0]]),
               (base + opt, [[G.F_NOT_BOUND, -2, 0, 0]]), (base + opt, [[G.F_BOUND, -2, 0, 0]]),
               (base + opt, [[G.F_NE, -1, -2, 0], [G.F_GT, -1, 1, 0]])]
    for pats, filt in queries:
        nv = -min(min(q[0], q[2]) for q in pats)
        want = algebra.join_ext(s, p, o, pats, filt, nv)
        for budget in (0, 64 << 10):
            res = G.gsmat_join_ext(st, pats, filt, nv, budget)
            got = G.gsmat_fetch_bindings(res)
            print(f"[gpu] ext small n={n} fan={fan} rows={len(got)} budget={budget}", flush=True)
            assert np.array_equal(got[np.lexsort(got.T[::-1])], want), (pats, filt)
            res.close()
    st.close()
