"""The load's id check, shared by the host threads, names the first bad triple
of large arrays.  Host only."""
import numpy as np
import pytest


@pytest.fixture(scope="module")
def G():
    import paper_1807_07691_amd as G
    return G


@pytest.mark.parametrize("n", [1, 4096, 4097, 1_000_003])
@pytest.mark.parametrize("which", ["s", "p", "o"])
def test_first_bad_triple(G, n, which):
    V, P = 50, 7
    r = np.random.default_rng(n)
    for first in {0, n // 3, n - 1}:
        a = {"s": r.integers(0, V, n).astype(np.int32), "p": r.integers(0, P, n).astype(np.int32),
             "o": r.integers(0, V, n).astype(np.int32)}
        for i in {first, (first + n) // 2, n - 1}:
            a[which][i] = -1 if i % 2 else (P if which == "p" else V)
        with pytest.raises(G.GsmatError) as e:
            G.gsmat_load_triples(a["s"], a["p"], a["o"], V, P)
        assert e.value.status == G.GSMAT_EINVAL
        kind = "predicate" if which == "p" else "vertex"
        assert str(e.value).endswith(f"{kind} id out of range at triple {first}")
