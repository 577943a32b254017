"""The step-by-step launches and the batched rounds by themselves: with the
one-launch runs of small tables off (gsmat_set_small_joins), the batch tests
reach every kernel of the rounds at every size, and both ways give the same
rows in the same order and the same step counters."""
import numpy as np
import pytest

import test_gpu_batch as B
from test_gpu_batch import (G, O, tiny, test_batch_random_graphs,  # noqa: F401
                            test_batch_shapes, test_batch_tuning_star_intersections,
                            test_batch_wide_tables)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def small_off(G):
    """Every store this module's tests build runs without the small launches."""
    build = G.gsmat_build_index

    def build_off(st, *a, **kw):
        build(st, *a, **kw)
        G.gsmat_set_small_joins(st, 0)

    mp = pytest.MonkeyPatch()
    mp.setattr(G, "gsmat_build_index", build_off)
    yield
    mp.undo()


def _rounds(G, st, queries, mode):
    """Tasks counted in the rounds of one batch."""
    plans, _ = G.gsmat_plan_batch(st, queries, mode, as_set=True)
    res, _ = G.gsmat_join_batch(st, plans, as_set=True)
    res.close()
    plans.close()
    return sum(r["tasks"] for r in G.gsmat_batch_round_stats(st))


def test_small_batches_take_the_rounds(G, tiny):
    spec, s, p, o, qs, st, want = tiny
    queries = [q.tps for q in qs]
    assert _rounds(G, st, queries, G.PLAN_ADAPTIVE) >= len(queries) / 2
    assert G.lib().gsmat_set_small_joins(None, 1) == G.GSMAT_EINVAL
    assert G.lib().gsmat_set_small_joins(st.h, 2) == G.GSMAT_EINVAL


@pytest.fixture(scope="module")
def alone(G, tiny):
    """The tiny workload's answers and counters one by one, per mode."""
    spec, s, p, o, qs, st, want = tiny
    got = {mode: [B._single(G, st, q.tps, mode) for q in qs] for mode in (0, 1, 2)}
    for (rows, _), w in zip(got[2], want):
        assert np.array_equal(B._sorted(rows), w)
    return got


@pytest.mark.parametrize("mode,sparse,regions,tuning", [
    (0, B.SPARSE[0], B.REGIONS[0], B.TUNING[0]), (1, B.SPARSE[0], B.REGIONS[1], B.TUNING[1]),
    (2, B.SPARSE[0], B.REGIONS[2], B.TUNING[2]), (0, B.SPARSE[2], B.REGIONS[3], B.TUNING[3]),
    (1, B.SPARSE[2], B.REGIONS[0], B.TUNING[4]), (2, B.SPARSE[2], B.REGIONS[1], B.TUNING[5]),
    (0, B.SPARSE[1], B.REGIONS[2], B.TUNING[6]), (1, B.SPARSE[2], B.REGIONS[3], B.TUNING[7]),
    (2, B.SPARSE[2], B.REGIONS[0], B.TUNING[8])])
def test_rounds_of_the_tiny_workload(G, tiny, alone, mode, sparse, regions, tuning):
    spec, s, p, o, qs, st, want = tiny
    print(f"[gpu] rounds mode={mode} {sparse} {regions} {tuning}", flush=True)
    G.gsmat_set_sparse_expand(st, *sparse)
    G.gsmat_set_batch_tuning(st, *tuning)
    queries = [q.tps for q in qs] * 2
    G.gsmat_set_batch_regions(st, *regions)
    plans, _ = G.gsmat_plan_batch(st, queries, mode)
    try:
        for engine in (1, 1, 0):  # the second batch starts from the first one's sizes
            got, stat = B._join_all(G, st, plans, engine=engine)
            assert stat == [0] * len(queries)
            for i, (a, b) in enumerate(zip(got, alone[mode] * 2)):
                assert np.array_equal(a[0], b[0]) and a[1] == b[1], (i, queries[i])
        fused, _ = G.gsmat_join_batch_bgp(st, queries, mode)
        for r, b in zip(fused, alone[mode] * 2):
            assert np.array_equal(G.gsmat_fetch_bindings(r), b[0])
            assert G.gsmat_result_info(r) == b[1]
            r.close()
    finally:
        for pl in plans:
            pl.close()
        G.gsmat_set_sparse_expand(st, 0.5, 4096)
        G.gsmat_set_batch_tuning(st, 8, G.ISECT_SEARCH)
        G.gsmat_set_batch_regions(st, 0, 0)


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_both_ways_agree(G, O, tiny, mode):
    """Singly, as a batch and served, small launches on and off."""
    import test_gpu_serve as S
    spec, s, p, o, qs, st, want = tiny
    wide = [B._chain(n, [0, 1], const_start=n) for n in (2, 5, 9)]
    queries = [q.tps for q in qs] + wide
    got = []
    try:
        for on in (0, 1):
            G.gsmat_set_small_joins(st, on)
            print(f"[gpu] both ways mode={mode} small={on}", flush=True)
            one = [B._single(G, st, q, mode) for q in queries]
            plans, _ = G.gsmat_plan_batch(st, queries, mode)
            many, _ = B._join_all(G, st, plans)
            served, _ = S._serve(G, st, queries, mode, [len(queries)])
            got.append((one, many, [served[i][:2] for i in range(len(queries))]))
            for pl in plans:
                pl.close()
    finally:
        G.gsmat_set_small_joins(st, 0)
    for off, on in zip(*got):
        for i, (a, b) in enumerate(zip(off, on)):
            assert np.array_equal(a[0], b[0]) and a[1] == b[1], (i, queries[i])


@pytest.mark.parametrize("mode", [1, 2])
def test_hub_bitmaps_at_any_size(G, O, tiny, mode):
    """Filters and intersections by bitmap over tables of few rows (the small
    launch searches the rows instead)."""
    spec, s, p, o, qs, st, want = tiny
    h = G.gsmat_load_triples(s, p, o, spec.V, spec.P)
    G.gsmat_set_hub_options(h, 2, 1 << 30)
    G.gsmat_build_index(h)
    queries = [[[-1, 0, int(o[0])], [-1, 1, -2], [-1, 2, int(o[5])]],
               [[int(s[3]), 0, -1], [-1, 1, -2], [int(s[3]), 2, -2]],
               [[-1, 0, -2], [-2, 1, -3], [-1, 2, -3]]] + [q.tps for q in qs]
    for q in queries:
        nv = int(-np.min(np.asarray(q)[:, [0, 2]]))
        print(f"[gpu] hub bitmaps mode={mode} {np.asarray(q).tolist()}", flush=True)
        assert np.array_equal(B._sorted(G.evaluate(h, q, mode)), O.join(s, p, o, q, nv))
    h.close()


def test_ext_both_ways(G, tiny):
    """OPTIONAL and FILTER over parts of few rows, selected by the launches
    that larger parts take."""
    from oracle import algebra
    spec, s, p, o, qs, st, want = tiny
    v = int(s[11])
    for pats, filt in [([[v, 0, -1, 0, 0], [-1, 1, -2, 0, 1]], [[G.F_NE, -1, -2, 0]]),
                       ([[-1, 3, -2, 0, 0], [-2, 0, -3, 0, 1], [-2, 1, -4, 0, 2]], []),
                       ([[-1, 5, -2, 0, 0]], [[G.F_LT, -1, int(np.median(s)), 0]])]:
        nv = -min(min(q[0], q[2]) for q in pats)
        rows = algebra.join_ext(s, p, o, pats, filt, nv)
        print(f"[gpu] ext without small parts rows={len(rows)}", flush=True)
        r = G.gsmat_join_ext(st, pats, filt, nv)
        assert np.array_equal(B._sorted(G.gsmat_fetch_bindings(r)), rows)
        r.close()


def test_autotuner_times_the_rounds(G):
    """Also of plans that a batch would finish in one small launch."""
    rng = np.random.default_rng(5)
    s, p, o = (rng.integers(0, hi, 3000).astype(np.int32) for hi in (400, 3, 400))
    st = B._store(G, s, p, o, 400, 3)
    G.gsmat_set_small_joins(st, 1)
    plans, _ = G.gsmat_plan_batch(st, [[[7, 0, -1], [-1, 1, -2]]] * 20, G.PLAN_ADAPTIVE,
                                  as_set=True)
    G.gsmat_autotune_batch(st, plans)
    assert sum(r["tasks"] for r in G.gsmat_batch_round_stats(st)) >= 20
    pl = G.gsmat_plan(st, [[7, 0, -1], [-1, 1, -2]], G.PLAN_ADAPTIVE)
    G.gsmat_prof_enable()
    G.gsmat_join(st, pl).close()
    n = sum(k["launches"] for k in G.gsmat_prof_read().values())
    G.gsmat_prof_enable(0)
    assert n <= 2, "the store's setting is as it was"
    pl.close()
    plans.close()
    st.close()


def test_round_stats_are_the_last_batchs(G, tiny):
    """A batch that took no rounds reports none, not an earlier batch's."""
    spec, s, p, o, qs, st, want = tiny
    assert _rounds(G, st, [q.tps for q in qs], G.PLAN_ADAPTIVE) > 0
    G.gsmat_set_small_joins(st, 1)
    try:
        assert _rounds(G, st, [[[int(s[0]), int(p[0]), -1]]] * 8, G.PLAN_ADAPTIVE) == 0
    finally:
        G.gsmat_set_small_joins(st, 0)
    assert _rounds(G, st, [q.tps for q in qs], G.PLAN_ADAPTIVE) > 0
    # a fused batch of which no query can be planned
    _, stat = G.gsmat_join_batch_bgp(st, [[[-1, -1, -2]]] * 600, raise_on_error=False)
    assert stat == [G.GSMAT_EUNSUPPORTED] * 600 and G.gsmat_batch_round_stats(st) == []
