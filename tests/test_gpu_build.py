"""The index of graphs at the sizes where its kernels change: tiles of 2048 and
4096 keys, 8- and 9-bit digits, predicates with dense pointers, directories or
neither.  Exported matrices against numpy, lookups through one-pattern joins."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1807_07691_amd as G
    return G


def check(G, s, p, o, V, P, dense_div):
    st = G.gsmat_load_triples(s, p, o, V, P)
    G.gsmat_build_index(st, dense_div)
    d = np.unique(np.stack([p, s, o], 1).astype(np.int64), axis=0)
    assert G.gsmat_store_stats(st)["n_triples"] == len(d)
    for q in range(P):
        m = d[d[:, 0] == q]
        for orient, (row, mem) in enumerate(((1, 2), (2, 1))):
            e = m[np.lexsort((m[:, mem], m[:, row]))]
            keys, at = np.unique(e[:, row], return_index=True)
            got = G.gsmat_export_matrix(st, q, orient)
            assert np.array_equal(got[0], keys), (q, orient)
            assert np.array_equal(got[1], np.append(at, len(e))), (q, orient)
            assert np.array_equal(got[2], e[:, mem]), (q, orient)
    # every kind of row pointer answers the lookups of present and absent ids
    r = np.random.default_rng(len(d))
    ids = np.unique(np.concatenate([[0, V - 1], r.integers(0, V, 6)]))
    for q in range(min(P, 4)):
        m = d[d[:, 0] == q]
        for v in ids:
            for tp, want in (([int(v), q, -1], m[m[:, 1] == v, 2]), ([-1, q, int(v)], m[m[:, 2] == v, 1])):
                pl = G.gsmat_plan(st, [tp])
                res = G.gsmat_join(st, pl)
                assert np.array_equal(G.gsmat_fetch_bindings(res)[:, 0], np.sort(want)), tp
                res.close()
                pl.close()
    st.close()


@pytest.mark.parametrize("n", [0, 1, 2, 63, 2047, 2048, 2049, 4095, 4096, 4097, 8193, 40_000])
@pytest.mark.parametrize("V,P,dense_div", [(2, 1, 0), (300, 3, 0), (300, 3, 10 ** 6), (5000, 17, 8),
                                           (70_000, 130, 1000), (2 ** 26 + 3, 2, 0),
                                           (2 ** 31 - 1, 2, 1)])
def test_build_edges(G, n, V, P, dense_div):
    r = np.random.default_rng(n + V % 1000)
    # hubs, runs of equal keys and the largest ids
    s = np.minimum((r.random(n) ** 3 * V).astype(np.int64), V - 1)
    o = np.where(r.random(n) < 0.2, V - 1, r.integers(0, V, n))
    p = np.minimum((r.random(n) ** 2 * P).astype(np.int64), P - 1)
    if n > 4:
        s[n // 2:n // 2 + n // 4] = s[0]
        dup = r.integers(0, n, n // 5)
        s[:n // 5], p[:n // 5], o[:n // 5] = s[dup], p[dup], o[dup]
    print(f"[gpu] build n={n} V={V} P={P} dense_div={dense_div}", flush=True)
    check(G, s.astype(np.int32), p.astype(np.int32), o.astype(np.int32), V, P, dense_div)


def test_build_one_row_and_one_column(G):
    n = 6000
    x = np.arange(n, dtype=np.int32)
    z = np.zeros(n, np.int32)
    check(G, np.concatenate([z, x]), np.concatenate([z, z + 1]), np.concatenate([x, z]), n, 2, 0)


@pytest.mark.parametrize("n", [65_535, 65_536, 65_537, 1_050_001, 3_000_000])
@pytest.mark.parametrize("which", ["s", "p", "o"])
def test_bad_ids_on_the_device(G, n, which):
    """The id check of loads around the size from which it runs on the device
    (65536 triples): the first of several bad ids is named, at either end and
    between; then the same arrays with good ids load."""
    V, P = 50, 7
    r = np.random.default_rng(n)
    a = {"s": r.integers(0, V, n).astype(np.int32), "p": r.integers(0, P, n).astype(np.int32),
         "o": r.integers(0, V, n).astype(np.int32)}
    good = a[which].copy()
    kind = "predicate" if which == "p" else "vertex"
    for first in (0, 1023, n // 3, n - 1):
        for bad in (-1, np.iinfo(np.int32).min, P if which == "p" else V):
            a[which][:] = good
            for i in {first, (first + n) // 2, n - 1}:
                a[which][i] = bad
            with pytest.raises(G.GsmatError) as e:
                G.gsmat_load_triples(a["s"], a["p"], a["o"], V, P)
            assert e.value.status == G.GSMAT_EINVAL
            assert str(e.value).endswith(f"{kind} id out of range at triple {first}")
    a[which][:] = good
    st = G.gsmat_load_triples(a["s"], a["p"], a["o"], V, P)
    G.gsmat_build_index(st)
    d = np.unique(np.stack([a["s"], a["p"], a["o"]], 1), axis=0)
    assert G.gsmat_store_stats(st)["n_triples"] == len(d)
    st.close()


@pytest.mark.parametrize("V", [63, 64, 4095, 4096, 4097, 8191, 8192])
def test_dense_pointer_tiles(G, V):
    """Dense pointers at the edges of their tiles (4096 vertices, V + 1 of them):
    every row present, only the last, only the first of each 64."""
    x = np.arange(V, dtype=np.int32)
    parts = [x, x[-1:], x[::64]]
    s = np.concatenate(parts)
    p = np.concatenate([np.full(len(a), q, np.int32) for q, a in enumerate(parts)])
    check(G, s, p, s[::-1].copy(), V, 3, 10 ** 6)
