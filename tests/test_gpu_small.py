"""Queries of few rows, which one launch takes from their first table to their
answer: at the edges of what the launch holds (rows entering a step, rows of a
step and of the answer), at the steps it leaves to the general path, and from
tables the general path has already produced.  Rows against the oracle and, in
order, against the batched join; step counters against the batched join."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS = 4096  # rows of a table inside the launch


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1807_07691_amd as G
    return G


def graph(n, fan, seed):
    """Vertex 0 has n objects along predicate 0; each of them `fan` objects
    along predicate 1 (every seventh none); predicate 2 closes a part of the
    pairs, predicate 3 leads on, 4 marks a part of the objects, 5 is random."""
    r = np.random.default_rng(seed)
    V = 2 * n + 40
    xs = np.arange(1, n + 1)
    t = [np.stack([np.zeros(n, np.int64), np.zeros(n, np.int64), xs], 1)]
    src = np.repeat(xs[xs % 7 != 0], fan)
    dst = r.integers(1, V, len(src))
    t.append(np.stack([src, np.full(len(src), 1), dst], 1))
    near = r.random(len(src)) < 0.5
    t.append(np.stack([src[near], np.full(near.sum(), 2), dst[near]], 1))
    t.append(np.stack([np.arange(1, V), np.full(V - 1, 3), r.integers(1, V, V - 1)], 1))
    some = xs[r.random(n) < 0.6]
    t.append(np.stack([some, np.full(len(some), 4), np.full(len(some), 5)], 1))
    t.append(np.stack([r.integers(0, V, 3000), np.full(3000, 5), r.integers(0, 9, 3000)], 1))
    a = np.concatenate(t).astype(np.int32)
    return a[:, 0].copy(), a[:, 1].copy(), a[:, 2].copy(), V, 6


QUERIES = [
    [[0, 0, -1]],
    [[0, 0, -1], [-1, 1, -2]],
    [[0, 0, -1], [-1, 1, -2], [-1, 2, -2]],
    [[0, 0, -1], [-1, 1, -2], [-2, 3, -3], [-1, 3, -4]],
    [[0, 0, -1], [-1, 4, 5], [-1, 3, -2]],
    [[-1, 4, 5], [-1, 1, -2], [-2, 5, 3]],
    [[-1, 4, 5], [0, 0, -1]],
    [[0, 0, 1], [1, 3, -1], [-1, 3, -2], [-2, 3, -3]],
    [[0, 0, -1], [-1, 3, -1]],
    [[0, 0, -1], [1, 3, -2]],
]


def rows_sorted(a):
    return a[np.lexsort(a.T[::-1])] if len(a) and a.shape[1] else a


@pytest.mark.parametrize("n,fan", [(1, 1), (63, 3), (ROWS - 1, 1), (ROWS, 1), (ROWS + 1, 1),
                                   (2048, 2), (2341, 2), (700, 7), (683, 24)])
def test_small_joins(G, n, fan):
    import oracle as O
    s, p, o, V, P = graph(n, fan, n + fan)
    st = G.gsmat_load_triples(s, p, o, V, P)
    G.gsmat_build_index(st)
    for mode in (G.PLAN_PAPER, G.PLAN_DEFAULT, G.PLAN_ADAPTIVE):
        for budget in (0, 40_000):
            plans, _ = G.gsmat_plan_batch(st, QUERIES, mode)
            # the batch's rounds, which never take the one-launch path
            G.gsmat_set_batch_engine(st, G.ENGINE_HOST)
            batch, _ = G.gsmat_join_batch(st, plans)
            for q, pl, b in zip(QUERIES, plans, batch):
                want = O.join(s, p, o, q, int(-np.min(np.array(q)[:, [0, 2]])))
                r = G.gsmat_join(st, pl, budget)
                got = G.gsmat_fetch_bindings(r)
                print(f"[gpu] small n={n} fan={fan} mode={mode} budget={budget} rows={len(got)}",
                      flush=True)
                assert np.array_equal(rows_sorted(got), want), (q, mode, budget)
                gi, bi = G.gsmat_result_info(r), G.gsmat_result_info(b)
                assert gi["step_rows_out"] == bi["step_rows_out"], (q, mode, budget)
                assert gi["step_rows_in"] == bi["step_rows_in"], (q, mode, budget)
                if budget == 0:
                    assert np.array_equal(got, G.gsmat_fetch_bindings(b)), (q, mode)
                r.close()
                b.close()
                pl.close()
    st.close()


@pytest.mark.parametrize("n,fan,count", [(63, 3, 10), (ROWS, 1, 10), (ROWS + 1, 2, 60), (700, 7, 512),
                                         (700, 7, 513), (2341, 2, 30)])
def test_small_batches(G, n, fan, count):
    """Batches around the size that first runs in one launch: rows, order and
    counters as in the host-driven rounds, also where most queries are left to
    the rounds, and through the server."""
    s, p, o, V, P = graph(n, fan, n + fan)
    st = G.gsmat_load_triples(s, p, o, V, P)
    G.gsmat_build_index(st)
    queries = [QUERIES[i % len(QUERIES)] for i in range(count)]
    for mode, budget in ((G.PLAN_ADAPTIVE, 0), (G.PLAN_ADAPTIVE, 40_000), (G.PLAN_DEFAULT, 0),
                         (G.PLAN_PAPER, 0)):
        plans, _ = G.gsmat_plan_batch(st, queries, mode)
        G.gsmat_set_batch_engine(st, G.ENGINE_HOST)
        want, _ = G.gsmat_join_batch(st, plans[:len(QUERIES)], budget)
        rows = [G.gsmat_fetch_bindings(r) for r in want]
        info = [G.gsmat_result_info(r) for r in want]
        G.gsmat_set_batch_engine(st, G.ENGINE_DEVICE)
        print(f"[gpu] small batch n={n} count={count} mode={mode} budget={budget}", flush=True)
        a, _ = G.gsmat_join_batch(st, plans, budget)
        b, _ = G.gsmat_join_batch_bgp(st, queries, mode, budget)
        sv = G.gsmat_server_new(st, 0, budget, -1, 4096)
        for i, pl in enumerate(plans):
            G.gsmat_server_submit(sv, pl, i)
        c = {}
        while len(c) < count:
            G.gsmat_server_step(sv)
            for tag, r, status in G.gsmat_server_poll(sv, count):
                assert status == 0
                c[tag] = r
        for i in range(count):
            w, wi = rows[i % len(QUERIES)], info[i % len(QUERIES)]
            for r in (a[i], b[i], c[i]):
                assert np.array_equal(G.gsmat_fetch_bindings(r), w), (i, mode)
                gi = G.gsmat_result_info(r)
                assert gi["step_rows_out"] == wi["step_rows_out"], (i, mode)
                assert gi["step_rows_in"] == wi["step_rows_in"], (i, mode)
                r.close()
        sv.close()
        for x in plans + want:
            x.close()
        # a row limit fails only the queries above it
        lim = sorted(len(w) for w in rows)[len(rows) // 2]
        res, stat = G.gsmat_join_batch_bgp(st, queries, mode, 0, lim, raise_on_error=False)
        for i in range(count):
            assert (stat[i] == G.GSMAT_ETOOBIG) == (len(rows[i % len(QUERIES)]) > lim), (i, mode)
            if res[i] is not None:
                res[i].close()
    st.close()


def launches(G, f):
    """Kernel launches of the library during f()."""
    G.gsmat_prof_enable()
    try:
        f()
        return sum(k["launches"] for k in G.gsmat_prof_read().values())
    finally:
        G.gsmat_prof_enable(0)


def test_no_launch_for_what_it_cannot_take(G):
    """A constant pattern the plan knows about, a product of two constants'
    rows, and a join whose answer is far above the allocation-free array cost
    the launches they cost without the small joins."""
    import torch
    s, p, o, V, P = graph(3000, 9, 3)
    n = 3_000_000  # predicate 6: pairs whose square is above the array
    big = np.stack([np.arange(n) % 1500, np.full(n, 6), np.arange(n) // 1500], 1).astype(np.int32)
    a = np.concatenate([np.stack([s, p, o], 1), big])
    st = G.gsmat_load_triples(a[:, 0].copy(), a[:, 1].copy(), a[:, 2].copy(), V, 7)
    G.gsmat_build_index(st)
    out = torch.empty(64, dtype=torch.int32, device="cuda")

    def join(q, mode):
        pl = G.gsmat_plan(st, q, mode)
        return lambda: G.gsmat_join(st, pl).close()

    def fails():
        pl = G.gsmat_plan(st, [[5, 6, -1], [-2, 6, -1], [-2, 6, -3]], G.PLAN_ADAPTIVE)
        n_rows = []

        def f():
            with pytest.raises(G.GsmatError) as e:
                n_rows.append(G.gsmat_join_noalloc(st, pl, out.data_ptr(), 16, 16))
            assert e.value.status == G.GSMAT_ENOMEM
        return f

    calls = [join([[0, 0, 1]], m) for m in (1, 2)]
    calls += [join([[0, 0, -1], [1, 3, -2]], m) for m in (0, 1, 2)]
    calls += [join([[0, 0, -1], [1, 3, -2], [-3, 4, 5]], m) for m in (1, 2)]
    calls.append(fails())
    for i, f in enumerate(calls):
        got = []
        for on in (0, 1):
            G.gsmat_set_small_joins(st, on)
            got.append(launches(G, f))
        print(f"[gpu] call {i}: launches without {got[0]}, with {got[1]}", flush=True)
        assert got[1] <= got[0] + (i == 7), i
    st.close()


class Counting:
    """A store's allocator: torch memory, with the bytes held."""

    def __init__(self, G):
        import torch
        self.held, self.bytes, self.peak = {}, 0, 0

        def alloc(size, stream):
            t = torch.empty(size, dtype=torch.uint8, device="cuda")
            self.held[t.data_ptr()] = t
            self.bytes += size
            self.peak = max(self.peak, self.bytes)
            return t.data_ptr()

        def free(p, size, stream):
            assert self.held.pop(p).numel() == size
            self.bytes -= size

        self.allocator = G.make_allocator(alloc, free)


def test_kept_answers_hold_little(G):
    """An answer of a small join holds at most four times its columns (which
    start on 256-byte boundaries), or 1 KiB."""
    s, p, o, V, P = graph(3000, 2, 5)
    # predicate 6: vertex i has the objects 1 to 2 ** i
    more = np.concatenate([np.stack([np.full(1 << i, i), np.full(1 << i, 6), 1 + np.arange(1 << i)], 1)
                           for i in range(13)]).astype(np.int32)
    a = np.concatenate([np.stack([s, p, o], 1), more])
    mem = Counting(G)
    st = G.gsmat_load_triples(*(a[:, i].copy() for i in range(3)), V, 7, allocator=mem.allocator)
    G.gsmat_build_index(st)
    for mode in (G.PLAN_DEFAULT, G.PLAN_ADAPTIVE):
        for i in range(13):
            pl = G.gsmat_plan(st, [[i, 6, -1], [-1, 3, -2], [-2, 3, -3]], mode)
            before = mem.bytes
            r = G.gsmat_join(st, pl)
            info = G.gsmat_result_info(r)
            n = info["rows"]
            assert n > 0
            held, own = mem.bytes - before, 4 * 3 * ((n + 63) // 64 * 64)
            print(f"[gpu] kept answer rows={n} holds {held}", flush=True)
            assert held <= max(1024, 4 * own), (n, held)
            r.close()
            assert mem.bytes == before
            pl.close()
    st.close()
    assert mem.bytes == 0


def test_batch_areas_stay_small(G):
    """What a batch's small launch takes follows each query's own patterns and
    stays within 256 MiB, and one kept answer holds the batch's answers and 2
    MiB at most, not every query's largest possible answer."""
    s, p, o, V, P = graph(700, 7, 5)
    mem = Counting(G)
    st = G.gsmat_load_triples(s, p, o, V, P, allocator=mem.allocator)
    G.gsmat_build_index(st)
    chain = [[1, 3, -1]] + [[-i, 3, -i - 1] for i in range(1, 25)]
    tiny = [[[i + 1, 1, -1], [-1, 3, -2]] for i in range(300)]
    for queries, most in [(tiny[:60], 24 << 20), (tiny + [chain], 128 << 20),
                          ([chain] * 300, 256 << 20)]:
        want = [G.evaluate(st, q) for q in queries]
        plans, _ = G.gsmat_plan_batch(st, queries, G.PLAN_ADAPTIVE)
        before = mem.peak = mem.bytes
        G.gsmat_set_batch_regions(st, 1 << 20, 1 << 20)
        res, _ = G.gsmat_join_batch(st, plans)
        print(f"[gpu] batch of {len(queries)}: peak {mem.peak - before}", flush=True)
        assert mem.peak - before <= most + (8 << 20)
        for r, w in zip(res, want):
            assert np.array_equal(G.gsmat_fetch_bindings(r), w)
        answers = sum(4 * w.shape[1] * ((len(w) + 63) // 64 * 64) for w in want)
        for r in res[1:]:
            r.close()
        if queries[0] != chain:  # those take the rounds
            assert mem.bytes - before <= answers + (2 << 20)
        res[0].close()
        assert mem.bytes == before
        for pl in plans:
            pl.close()
    st.close()
    assert mem.bytes == 0


def test_batch_routes(G):
    """Which batches take the small launch, the rounds, or neither: rounds only
    where too many queries cannot start in the launch, may outgrow it or have;
    the rows are those of the queries alone, in the same order."""
    s, p, o, V, P = graph(5000, 3, 8)
    st = G.gsmat_load_triples(s, p, o, V, P)
    G.gsmat_build_index(st)
    view = [[0, 0, -1]]
    two = [[1, 1, -1], [-1, 3, -2]]
    three = [[1, 1, -1], [-1, 3, -2], [-2, 3, -3]]
    wide = [[0, 0, -1], [-1, 3, -2]]                 # starts from 5000 rows
    grows = [[-1, 4, 5], [-1, 1, -2], [-2, 3, -3]]   # 3000 rows, then 7700
    for name, queries, rounds in [
            ("views", [view] * 7 + [[[-1, 4, 5]], [[3, 4, 5]], [[-1, 7, -2]]], False),
            ("two patterns", [two] * 300, False),
            ("two patterns, one wide", [two] * 30 + [wide], False),
            ("two patterns, many wide", [two] * 30 + [wide] * 9, True),
            ("three patterns", [three] * 64, False),
            ("more of three patterns", [three] * 65, True),
            ("two grow", [three] * 20 + [grows] * 2, False),
            ("many grow", [three] * 20 + [grows] * 20, True),
            ("one wide alone", [wide], False)]:
        plans, _ = G.gsmat_plan_batch(st, queries, G.PLAN_DEFAULT)
        res = []
        n = launches(G, lambda: res.extend(G.gsmat_join_batch(st, plans)[0]))
        took = sum(r["tasks"] for r in G.gsmat_batch_round_stats(st)) > 0
        print(f"[gpu] routes: {name}, {n} launches, rounds {took}", flush=True)
        assert took == rounds, name
        assert name != "views" or n == 0
        alone = {}
        for q, pl, r in zip(queries, plans, res):
            key = str(q)
            if key not in alone:
                one = G.gsmat_join(st, pl)
                alone[key] = G.gsmat_fetch_bindings(one), G.gsmat_result_info(one)
                one.close()
            assert np.array_equal(G.gsmat_fetch_bindings(r), alone[key][0]), name
            assert G.gsmat_result_info(r) == alone[key][1], name
            r.close()
            pl.close()
    sv = G.gsmat_server_new(st)
    plans, _ = G.gsmat_plan_batch(st, [view] * 6, G.PLAN_ADAPTIVE)
    for i, pl in enumerate(plans):
        G.gsmat_server_submit(sv, pl, i)
    assert launches(G, lambda: G.gsmat_server_step(sv)) == 0
    done = G.gsmat_server_poll(sv)
    assert len(done) == 6 and all(G.gsmat_result_info(r)["rows"] == 5000 for _, r, _ in done)
    for _, r, _ in done:
        r.close()
    sv.close()
    for pl in plans:
        pl.close()
    st.close()


def test_batch_outputs_within_the_budget(G):
    """Outputs that fit the budget each but not together: what is above it is
    left to the rounds, which take it a round at a time; the rows are the same."""
    s, p, o, V, P = graph(5000, 3, 8)
    st = G.gsmat_load_triples(s, p, o, V, P)
    G.gsmat_build_index(st)
    q = [[-1, 4, 5], [-1, 1, -2]]
    want = G.evaluate(st, q)
    one = 4 * 2 * ((len(want) + 63) // 64 * 64)
    assert len(want) > ROWS
    for n in (1, 3, 20):
        for budget, rounds in ((0, False), (n * one, False), (n * one - 1, n > 1),
                               (one, n > 1), (one // 3, False)):
            plans, _ = G.gsmat_plan_batch(st, [q] * n, G.PLAN_ADAPTIVE)
            res, _ = G.gsmat_join_batch(st, plans, budget)
            took = sum(r["tasks"] for r in G.gsmat_batch_round_stats(st)) > 0
            print(f"[gpu] {n} outputs of {one}, budget {budget}: rounds {took}", flush=True)
            assert took == rounds, (n, budget)
            for r in res:
                assert np.array_equal(G.gsmat_fetch_bindings(r), want)
                r.close()
            for pl in plans:
                pl.close()
    st.close()


@pytest.mark.parametrize("budget", [1 << 20, 8 << 20, 64 << 20])
def test_server_areas_within_its_budget(G, budget):
    """The small launch's areas count as memory the admitted queries hold."""
    s, p, o, V, P = graph(700, 7, 5)
    mem = Counting(G)
    st = G.gsmat_load_triples(s, p, o, V, P, allocator=mem.allocator)
    G.gsmat_build_index(st)
    queries = [[[i + 1, 1, -1], [-1, 3, -2], [-2, 3, -3]] for i in range(128)]
    want = [G.evaluate(st, q) for q in queries]
    plans, _ = G.gsmat_plan_batch(st, queries, G.PLAN_ADAPTIVE)
    before = mem.peak = mem.bytes
    sv = G.gsmat_server_new(st, budget)
    for i, pl in enumerate(plans):
        G.gsmat_server_submit(sv, pl, i)
    left = len(plans)
    while left:
        G.gsmat_server_step(sv)
        for tag, r, status in G.gsmat_server_poll(sv):
            assert status == 0 and np.array_equal(G.gsmat_fetch_bindings(r), want[tag])
            r.close()
            left -= 1
    print(f"[gpu] server budget {budget}: peak {mem.peak - before}", flush=True)
    assert mem.peak - before <= budget
    sv.close()
    for pl in plans:
        pl.close()
    st.close()
    assert mem.bytes == 0


def test_kept_selections_hold_little(G):
    """The rows an OPTIONAL or FILTER over a small part keeps hold at most four
    times their columns, or 1 KiB, and not the whole part."""
    s, p, o, V, P = graph(4000, 1, 5)
    mem = Counting(G)
    st = G.gsmat_load_triples(s, p, o, V, P, allocator=mem.allocator)
    G.gsmat_build_index(st)
    for keep in (1, 64, 65, 1000, 3999, 4000):
        before = mem.bytes
        r = G.gsmat_join_ext(st, [[0, 0, -1, 0, 0]], [[G.F_LE, -1, keep, 0]])
        n, held = G.gsmat_result_info(r)["rows"], mem.bytes - before
        print(f"[gpu] kept selection rows={n} holds {held}", flush=True)
        assert n == keep
        assert held <= max(1024, 4 * 4 * ((n + 63) // 64 * 64))
        assert np.array_equal(np.sort(G.gsmat_fetch_bindings(r)[:, 0]), np.arange(1, keep + 1))
        r.close()
        assert mem.bytes == before
    st.close()
    assert mem.bytes == 0
