"""Single joins at the sizes where a step's launches change: offsets with or
without a scan of their own (2048 tiles of 2048 rows), splits by a wave or by a
thread (8192 tiles of the path), samples by a wave or by slices (256 rows)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

T = 2048


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1807_07691_amd as G
    return G


@pytest.mark.parametrize("n,fan", [(4097, 1), (2 * T, 3), (2 * T + 1, 3), (T * T - 1, 1),
                                   (T * T, 1), (T * T + 1, 1), (5 * T * T // 4, 3), (100_000, 170)])
def test_expand_sizes(G, n, fan):
    # n pairs (i, i % 97) along 0; vertex v has (v * 7) % (fan + 1) objects along 1
    V = max(n, 200)
    i = np.arange(n, dtype=np.int64)
    deg = (np.arange(97) * 7) % (fan + 1)
    s1 = np.repeat(np.arange(97), deg)
    o1 = np.concatenate([np.arange(d) for d in deg]).astype(np.int64) if deg.sum() else s1
    s = np.concatenate([i, s1]).astype(np.int32)
    p = np.concatenate([np.zeros(n), np.ones(len(s1))]).astype(np.int32)
    o = np.concatenate([i % 97, o1]).astype(np.int32)
    st = G.gsmat_load_triples(s, p, o, V, 2)
    G.gsmat_build_index(st)
    pl = G.gsmat_plan(st, [[-1, 0, -2], [-2, 1, -3]], G.PLAN_PAPER)
    nv, steps = G.gsmat_plan_info(pl)
    r = G.gsmat_join(st, pl)
    print(f"[gpu] expand n={n} fan={fan}", flush=True)
    m = int(deg[i % 97].sum())
    info = G.gsmat_result_info(r)
    assert info["rows"] == m
    got = G.gsmat_fetch_bindings(r)
    order = np.lexsort(got.T[::-1])
    want = np.repeat(i, deg[i % 97])
    assert np.array_equal(got[order, 0], want)
    assert np.array_equal(got[order, 1], want % 97)
    first = np.concatenate([[0], np.flatnonzero(np.diff(want)) + 1]) if m else np.zeros(0, int)
    run = np.arange(m) - np.repeat(first, np.diff(np.append(first, m)))
    assert np.array_equal(got[order, 2], run)
    r.close()
    pl.close()
    st.close()


@pytest.mark.parametrize("n", [255, 256, 257, 16383, 16385])
def test_samples(G, n):
    """600 queries (a batch that takes the rounds) whose bound table has n rows
    and several candidates: the batch takes the single join's steps."""
    r = np.random.default_rng(n)
    V = 20_000
    t = [np.stack([np.zeros(n, int), np.zeros(n, int), np.arange(1, n + 1)], 1)]
    for p, k in ((1, 30_000), (2, 25_000), (3, 28_000)):
        t.append(np.stack([r.integers(0, V, k), np.full(k, p), r.integers(0, V, k)], 1))
    a = np.concatenate(t).astype(np.int32)
    st = G.gsmat_load_triples(a[:, 0].copy(), a[:, 1].copy(), a[:, 2].copy(), V, 4)
    G.gsmat_build_index(st)
    q = [[0, 0, -1], [-1, 1, -2], [-1, 2, -3], [-4, 3, -1]]
    pl = G.gsmat_plan(st, q, G.PLAN_ADAPTIVE)
    one = G.gsmat_join(st, pl)
    want, wi = G.gsmat_fetch_bindings(one), G.gsmat_result_info(one)
    res, _ = G.gsmat_join_batch_bgp(st, [q] * 600, G.PLAN_ADAPTIVE)
    print(f"[gpu] samples n={n} rows={len(want)}", flush=True)
    for i in (0, 1, 299, 599):
        assert np.array_equal(G.gsmat_fetch_bindings(res[i]), want)
        assert G.gsmat_result_info(res[i])["step_rows_out"] == wi["step_rows_out"]
    for x in res:
        x.close()
    one.close()
    pl.close()
    st.close()


@pytest.mark.parametrize("fan", [1, 2, 3, 64])
@pytest.mark.parametrize("n", [700, 6000])
def test_filter_by_either_row(G, n, fan):
    """Triangles whose last expansion binds the subject of the closing pattern,
    below and above the run length (2) from which the pair is looked for in the
    object's row; with a budget the runs are cut.  Rows against numpy."""
    r = np.random.default_rng(n + fan)
    x = np.arange(n)
    y = n + x // 2  # two x for a y
    z = 2 * n + r.integers(0, n, (n, fan))  # subjects of y's pairs
    ys = n + np.arange(n)
    close = r.random((n, fan)) < 0.3
    cz, cx = z[x // 2][close], np.repeat(x, close.sum(1))  # (z, x) closes
    hub = 2 * n + np.arange(n)  # a long row: every z meets x = 0
    s = np.concatenate([x, z.ravel(), cz, hub])
    p = np.concatenate([np.zeros(n), np.ones(n * fan), np.full(len(cz) + n, 2)])
    o = np.concatenate([y, np.repeat(ys, fan), cx, np.zeros(n)])
    t = np.unique(np.stack([s, p, o], 1).astype(np.int32), axis=0)
    st = G.gsmat_load_triples(*(np.ascontiguousarray(t[:, i]) for i in range(3)), 3 * n, 3)
    G.gsmat_build_index(st)
    pairs = set(map(tuple, t[t[:, 1] == 2][:, [0, 2]].tolist()))
    zy = np.unique(t[t[:, 1] == 1][:, [2, 0]], axis=0)
    lo, hi = np.searchsorted(zy[:, 0], y), np.searchsorted(zy[:, 0], y, "right")
    want = sorted((int(a), int(b), int(c)) for a, b, l, h in zip(x, y, lo, hi)
                  for c in zy[l:h, 1] if (int(c), int(a)) in pairs)
    for mode in (G.PLAN_ADAPTIVE, G.PLAN_DEFAULT, G.PLAN_PAPER):
        for budget in (0, 20_000):
            pl = G.gsmat_plan(st, [(-1, 0, -2), (-3, 1, -2), (-3, 2, -1)], mode)
            res = G.gsmat_join(st, pl, budget)
            print(f"[gpu] filter rows n={n} fan={fan} mode={mode} budget={budget}", flush=True)
            assert sorted(map(tuple, G.gsmat_fetch_bindings(res).tolist())) == want
            res.close()
            pl.close()
    st.close()
