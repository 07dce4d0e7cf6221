"""GPU parity at scale for the parts that small graphs do not reach.

* Predicate codes 1, 2, 4, 5 and 7 on the 10M-edge medium workload: full
  per-edge counts, pairs, certificate counts and |Sol| against the oracle
  (codes 0, 3 and 6 are covered in test_gpu_parity.py).
* Timestamps that need more than 32 bits.  The index keeps each list's first
  and last timestamp shifted right by tshift = bitlen(t_max) - 32 so that they
  fit 32 bits, and the time-range filter compares them with a slack.  Here the
  medium workload's timestamps become t * 4096 + 2^40 (tshift 9), and the tiny
  workload's a millisecond clock t * 1000 + 1.7e12 (tshift 9); windows are
  scaled ones and ones that are no multiple of 2^tshift.  Single queries (both
  filter modes), a plan, the smaller-side evaluation, the vertex queries and
  the exists-exists-exists query are compared with the oracle on the same
  timestamps.
"""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2507_17215_amd import folty, synth

pytestmark = pytest.mark.gpu
YEAR = synth.YEAR_S


def say(*a):
    print("[case]", *a, flush=True)


def assert_same(res, want, counts=True):
    if counts:
        got = res.counts()
        bad = np.nonzero(got != want["counts"])[0]
        assert bad.size == 0, f"{bad.size} count mismatches, first at {bad[:5]}: gpu {got[bad[:5]]} oracle {want['counts'][bad[:5]]}"
    assert res.n_certificates == want["n_certificates"]
    assert np.array_equal(res.pair_u, want["pair_u"])
    assert np.array_equal(res.pair_v, want["pair_v"])
    assert np.array_equal(res.n_cert, want["n_cert"])


@pytest.fixture(scope="module")
def medium():
    say("medium: generate")
    return synth.medium()


@pytest.mark.timeout(900)
def test_other_predicate_codes_full_counts_at_scale(medium):
    g = medium
    o = Oracle(g.n, g.src, g.dst, g.t)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build()
    for variant in (1, 2, 4, 5, 7):
        say("medium predicate", variant)
        cnt = o.counts(86400, variant)
        assert int((cnt > 0).sum() - (cnt == 0xFFFFFFFF).sum()) > 0, "the window leaves no non-zero count"
        for theta in ((1, 10), (1, 2)):
            assert_same(G.query(86400, theta, variant), o.query(86400, theta[0], theta[1], variant, counts=cnt))


def shifted(g, scale, offset):
    return synth.TemporalGraph(n=g.n, src=g.src, dst=g.dst, t=g.t * scale + offset, meta=dict(g.meta))


@pytest.mark.timeout(900)
def test_wide_timestamps_medium_workload(medium):
    g = shifted(medium, 4096, 1 << 40)
    assert int(g.t.max()).bit_length() - 32 >= 8
    o = Oracle(g.n, g.src, g.dst, g.t)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build()
    deltas = [3600 * 4096, 86400 * 4096, YEAR * 4096, 86400 * 4096 + 12345, 1_000_003]
    say("wide medium: oracle pool")
    pool = o.counts_pool(deltas, 0)
    for j, d in enumerate(deltas):
        say("wide medium", d)
        assert_same(G.query(d, (1, 4), 0), o.query(d, 1, 4, 0, counts=pool[:, j]))
    say("wide medium: predicate 3")
    d = 86400 * 4096 + 777
    assert_same(G.query(d, (1, 2), 3), o.query(d, 1, 2, 3))
    say("wide medium: plan")
    plan = folty.Plan([G], [(0, dict(delta=d_, theta=(1, 4))) for d_ in deltas])
    for r, j in zip(plan.run(), range(len(deltas))):
        assert np.array_equal(r.counts(), pool[:, j])
    plan.close()


@pytest.mark.timeout(600)
def test_wide_timestamps_tiny_workload_all_query_kinds():
    g = shifted(synth.tiny(seed=4), 1000, 1_700_000_000_000)
    assert int(g.t.max()).bit_length() - 32 >= 8
    o = Oracle(g.n, g.src, g.dst, g.t)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build()
    deltas = [0, 1, 511, 3_600_000, 3_600_001, 86_400_000 + 123, 10**9 + 7, folty.DELTA_INF]
    for d in deltas:
        for variant in (0, 3, 6):
            say("wide tiny", d, variant)
            want = o.query(d, 1, 4, variant)
            assert_same(G.query(d, (1, 4), variant), want)
            assert_same(G.query(d, (1, 4), variant, smaller_side=True), want)
        tr = G.triad_query(d, 0, edge_instances=True)
        assert np.array_equal(tr.triads()["triples"], o.triad_solutions(d, 0))
        assert np.array_equal(tr.edge_instances(), o.triad_instances(d, 0))
        vq = G.vertex_query(d, (1, 10), folty.INNER_EXISTS, (1, 2), 0)
        wv = o.vertex_query(d, 1, 10, 0, False)
        v, good = vq.vertices()
        assert np.array_equal(v, wv["vertices"]) and np.array_equal(good, wv["good"])
    say("wide tiny: plan")
    qs = [(0, dict(delta=d, theta=(1, 4), variant=v)) for d in deltas for v in (0, 3)]
    plan = folty.Plan([G], qs)
    for rep in range(2):
        for (gi, q), r in zip(qs, plan.run()):
            assert_same(r, o.query(q["delta"], 1, 4, q["variant"]))
    plan.close()
    # the one-pass filter (per-item triangle slots) on the same timestamps
    for d in (3_600_001, 10**9 + 7):
        r = G.query(d, (1, 4), 0, one_pass=True)
        assert r.stats["filter_passes"] == 1
        assert_same(r, o.query(d, 1, 4, 0))


def test_filter_output_larger_than_its_first_chunks():
    """A complete graph of 400 vertices has 10.6M triangles; with every edge at the
    same time all of them pass the filter, more than the 4.2M its chunks hold at
    first, so the pass is repeated with chunks that suffice.  A second query finds
    them large enough, and the same graph as a plan holds every triangle at once.
    All equal the closed form: 398 third vertices for a transitive edge order."""
    n = 400
    src, dst = (x.astype(np.int32) for x in np.triu_indices(n, 1))
    t = np.full(src.size, 1000, np.int64)
    G = folty.Graph(n, src, dst, t).build()
    # edges run from lower to higher id: (a, b, w) needs a -> w and b -> w, so w > b
    want = (n - 1 - dst).astype(np.uint32)
    for one in (False, True, False):
        say("complete graph", one)
        r = G.query(0, (1, 4), 0, one_pass=one)
        assert np.array_equal(r.counts(), want)
        assert r.stats["triangles"] == n * (n - 1) * (n - 2) // 6
    say("complete graph: fresh index, triples")
    G2 = folty.Graph(n, src, dst, t).build()
    assert G2.triad_query(0, 0, triples=False).triads()["n_instances"] == n * (n - 1) * (n - 2) // 6
    say("complete graph: plan")
    plan = folty.Plan([G, G2], [(0, dict(delta=0, theta=(1, 4))), (1, dict(delta=5, theta=(1, 2), variant=3))])
    r0, r1 = plan.run()
    assert np.array_equal(r0.counts(), want)
    assert np.array_equal(r1.counts(), src.astype(np.uint32))  # w -> a and w -> b: w < a


@pytest.mark.parametrize("d", [1, 4, 5, 63, 64, 65, 127, 128, 129, 255, 256, 257, 510, 511, 512, 513, 600])
def test_enumeration_at_row_length_edges(d):
    """Owner rows of up to d entries, probed from segments of every length below d:
    table sizes, the last staged row length and the first long one, items of one
    owner and of several (few probes each).  Random directions and times, all eight
    predicates (two for the larger cliques), against the oracle."""
    rng = np.random.default_rng(d)
    # a clique of d + 1 vertices (out-rows of d, d - 1, ..., 0) beside sparse ones
    k = d + 1
    i, j = np.triu_indices(k, 1)
    extra = rng.integers(0, k + 200, size=(400, 2))
    a = np.concatenate([i, extra[:, 0]])
    b = np.concatenate([j, extra[:, 1]])
    flip = rng.random(a.size) < 0.5
    src = np.where(flip, b, a).astype(np.int32)
    dst = np.where(flip, a, b).astype(np.int32)
    t = np.sort(rng.integers(0, 10_000, size=src.size)).astype(np.int64)
    n = k + 200
    o = Oracle(n, src, dst, t)
    for mode in (folty.RANK_DEGENERACY, folty.RANK_DEGREE)[:2 if d < 130 else 1]:
        G = folty.Graph(n, src, dst, t).build(rank_mode=mode)
        for v in range(8) if d < 130 else (0, 6):
            say("row edges", d, mode, v)
            for delta, one in ((300, False), (5_000, True)):
                r = G.query(delta, (1, 4), v, one_pass=one)
                assert np.array_equal(r.counts(), o.query(delta, 1, 4, v)["counts"])
    o.close()


@pytest.mark.parametrize("n,m,tmax,loops,shuffle", [
    (2, 5, 3, False, False), (7, 64, 1, True, True), (300, 4097, 0, True, False),
    (3000, 20_000, (1 << 62) - 1, True, True),       # pair and time bits do not fit one key, not in order
    (3000, 20_000, (1 << 62) - 1, True, False),      # nor their low bits with a table of steps
    (1 << 22, 30_000, (1 << 24) - 5, True, False),   # 46 + 24 bits: the low 18 in the key, 64 steps
    (1 << 22, 30_000, (1 << 30) - 9, False, False),  # 12 high bits: the most the steps take
    (1 << 22, 30_000, (1 << 31) - 9, False, False),  # 13: gathered
    (1 << 22, 30_000, (1 << 24) - 5, True, True),    # too long for one key, unsorted: sorted by time first
    (12_288, 39_000, 5_000, False, True), (12_289, 39_000, 5_000, False, True),  # the one-block core phase and past it
])
def test_grouping_keys_and_core_phase_sizes(n, m, tmax, loops, shuffle):
    """Every form of the grouping keys (timestamps beside the pair in one 64-bit
    key, their high bits from the input position, sorts by time and pair) and the
    core phase of small graphs at its size limit: counts and pairs against the
    oracle, core numbers and ranks against its peel."""
    rng = np.random.default_rng(n + m)
    hubs = rng.integers(0, n, size=40)
    src = np.where(rng.random(m) < 0.4, hubs[rng.integers(0, 40, m)], rng.integers(0, min(n, 2000), m)).astype(np.int32)
    dst = np.where(rng.random(m) < 0.4, hubs[rng.integers(0, 40, m)], rng.integers(0, min(n, 2000), m)).astype(np.int32)
    if not loops:
        keep = src != dst
        src, dst = src[keep], dst[keep]
    t = np.sort(rng.integers(0, tmax, size=src.size, endpoint=True)).astype(np.int64)
    if shuffle:
        p = rng.permutation(src.size)
        src, dst, t = src[p], dst[p], t[p]
    say("grouping", n, m, tmax, loops, shuffle)
    o = Oracle(n, src, dst, t)
    G = folty.Graph(n, src, dst, t).build()
    for d in (tmax // 50, tmax):
        for v in (0, 6):
            assert_same(G.query(d, (1, 4), v), o.query(d, 1, 4, v))
    assert np.array_equal(G.core_numbers(), o.core_numbers())
    assert np.array_equal(G.ranks(), o.degeneracy_rank())
    o.close()


@pytest.mark.parametrize("scale", [1, 1 << 30])
def test_list_lengths_at_search_steps(scale):
    """Triangles whose six lists take every pair of lengths around the steps of the
    searches (1 to 4 entries, 5, 16, 17, ...), the pieces of a run and the light limit,
    with many equal timestamps; in 32 bits, where lists of one or two entries come from
    the records, and beyond.  Direct and smaller-side counts, temporal triangles per
    edge and a plan (one query that a count of 0 meets, jobs that none does) against
    the oracle."""
    rng = np.random.default_rng(scale & 1023)
    lens = [0, 1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 20, 21, 63, 64, 65, 130]
    src, dst, v0 = [], [], 0
    for x in lens:
        for y in lens:
            ends = [(0, 1, x), (1, 0, y), (1, 2, int(rng.choice(lens))), (2, 1, x), (0, 2, y),
                    (2, 0, int(rng.choice(lens)))]
            for a, b, k in ends:
                src += [v0 + a] * k
                dst += [v0 + b] * k
            v0 += 3
    p = rng.permutation(len(src))
    src, dst = np.asarray(src, np.int32)[p], np.asarray(dst, np.int32)[p]
    t = np.sort(rng.integers(0, 400, size=src.size)).astype(np.int64) * scale
    o = Oracle(v0, src, dst, t)
    G = folty.Graph(v0, src, dst, t).build()
    for v in range(8):
        for delta in (0, 3 * scale, 60 * scale, 400 * scale):
            say("list lengths", scale, v, delta // scale)
            want = o.query(delta, 1, 1, v)
            assert_same(G.query(delta, (1, 1), v), want)
            assert_same(G.query(delta, (1, 1), v, smaller_side=True), want)
        got = G.triad_query(20 * scale, v, triples=False, edge_instances=True).edge_instances()
        assert np.array_equal(got, o.triad_instances(20 * scale, v))
    qs = [dict(delta=d * scale, theta=th, variant=v, exclude_other=x)
          for v, th, x in ((0, (1, 1), False), (3, (1, 2), True), (5, (0, 1), False), (6, (1, 2), False))
          for d in (2, 50)]
    plan = folty.Plan([G], [(0, q) for q in qs])
    for _ in range(3):
        for q, r in zip(qs, plan.run()):
            say("list lengths: plan", q)
            assert_same(r, o.query(q["delta"], *q["theta"], q["variant"], exclude_other=q["exclude_other"]))
    o.close()


@pytest.mark.parametrize("pairs", [1024, 1025, 262_144, 262_145, 1_572_864, 1_572_865])
def test_pair_sorts_at_their_size_limits(pairs):
    """As many solution pairs as each kind of sort takes at most and one more: with
    theta = 0 every directed pair is one, and they come sorted with their edges."""
    rng = np.random.default_rng(pairs)
    n = 40_000
    key = np.unique(rng.integers(0, n * n, size=pairs + pairs // 4 + 64))
    key = key[key // n != key % n]
    key = np.sort(rng.permutation(key)[:pairs])
    assert key.size == pairs
    p = rng.permutation(np.concatenate([key, key[: pairs // 3]]))
    say("pair sorts", pairs)
    r = folty.Graph(n, (p // n).astype(np.int32), (p % n).astype(np.int32), np.arange(p.size)).build().query(5, (0, 1), 0)
    assert np.array_equal(r.pair_u, key // n) and np.array_equal(r.pair_v, key % n)
    assert np.array_equal(r.n_cert, 1 + (np.arange(pairs) < pairs // 3))


# ---------------------------------------------------------------------------
# the filter's time ranges: 14 bits over the span that holds most timestamps
# ---------------------------------------------------------------------------
def squeezed(g, span, offset):
    t = g.t.astype(np.int64)
    return synth.TemporalGraph(n=g.n, src=g.src, dst=g.dst, t=t * span // (int(t.max()) + 1) + offset, meta=dict(g.meta))


@pytest.mark.parametrize("span, delta", [(86_400, 60), (1_000_000, 3600), (YEAR, 86_400)])
def test_filter_keeps_the_same_wherever_times_start(span, delta):
    """stats.tests counts the tests of the triangles that the filter kept: the same graph
    keeps the same ones from 0, from Unix seconds and from the last 32-bit second, and
    about as many (2 of 64 sampled timestamps may be strays) with stray edges at 0."""
    base = synth.tiny(seed=11)
    kept = []
    for offset in (0, 1_300_000_000, (1 << 32) - 1 - span):
        g = squeezed(base, span, offset)
        o = Oracle(g.n, g.src, g.dst, g.t)
        G = folty.Graph(g.n, g.src, g.dst, g.t).build()
        kept.append([G.query(delta, (1, 4), v).stats["tests"] for v in (0, 6)])
        for v in range(8):
            say("late times", span, offset, v)
            assert_same(G.query(delta, (1, 4), v), o.query(delta, 1, 4, v))
    say("kept", kept)
    assert kept[1] == kept[0] and kept[2] == kept[0]
    # edges between two vertices of their own, at time 0
    g = squeezed(base, span, 1_300_000_000)
    a = np.full(20, g.n, np.int32)
    strays = synth.TemporalGraph(n=g.n + 2, src=np.concatenate([a, g.src]), dst=np.concatenate([a + 1, g.dst]),
                                 t=np.concatenate([np.zeros(20, np.int64), g.t]))
    o = Oracle(strays.n, strays.src, strays.dst, strays.t)
    G = folty.Graph(strays.n, strays.src, strays.dst, strays.t).build()
    for v, k in zip((0, 6), kept[0]):
        say("strays", span, v)
        r = G.query(delta, (1, 4), v)
        assert_same(r, o.query(delta, 1, 4, v))
        assert abs(r.stats["tests"] - k) <= k // 8 + 64


@pytest.mark.parametrize("offset, span, low, high", [
    (0, 50, 0, 0), (5, 16_383, 0, 0), (5, 16_384, 0, 0), (1_000, 16_385, 1, 1),  # units of one, and the first of two
    (1 << 31, 90_000, 1, 0), (100, 90_000, 0, 1), (1 << 61, 1 << 40, 1, 0), ((1 << 32) - 40, 80, 0, 1)])
def test_range_codes_at_their_ends(offset, span, low, high):
    """Timestamps before the base and past the last unit count as its ends: parity on all
    predicates with a seventh of the edges moved to 0 and to the largest timestamp."""
    g = squeezed(synth.bruteforce_size(seed=21), span, offset)
    t = g.t.copy()
    if low:
        t[::14] = 0
    if high:
        t[7::14] = (1 << 62) - 1
    o = Oracle(g.n, g.src, g.dst, t)
    G = folty.Graph(g.n, g.src, g.dst, t).build()  # no longer in time order
    deltas = sorted({0, 1, span // 3, span, folty.DELTA_INF})
    for v in range(8):
        say("range ends", offset, span, low, high, v)
        for d in deltas:
            assert_same(G.query(d, (1, 4), v), o.query(d, 1, 4, v))
    plan = folty.Plan([G], [(0, dict(delta=d, theta=(1, 4), variant=v)) for d in deltas for v in (0, 5)])
    for r, (d, v) in zip(plan.run(), [(d, v) for d in deltas for v in (0, 5)]):
        assert_same(r, o.query(d, 1, 4, v))
    plan.close()


def cliques(count, size, span, seed):
    rng = np.random.default_rng(seed)
    a, b = np.triu_indices(size, 1)
    src = np.concatenate([a + c * size for c in range(count)]).astype(np.int32)
    dst = np.concatenate([b + c * size for c in range(count)]).astype(np.int32)
    return synth.TemporalGraph(n=count * size, src=src, dst=dst, t=np.sort(rng.integers(0, span, src.size)))


def test_filter_counts_first_when_memory_is_short():
    """An eighth of 1.02 billion triangles is 1.5 GB of chunks: with 1.2 GB of device
    memory free the filter counts what its window keeps and allocates that."""
    import torch
    g = cliques(12, 800, 10**7, 61)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build()
    assert G.stats()["triangles"] == 12 * (800 * 799 * 798 // 6)
    ws = folty.Workspace()
    folty.release_cached_memory()
    torch.cuda.synchronize()
    fill = []
    for _ in range(3):
        k = torch.cuda.mem_get_info()[0] - (1200 << 20)
        if k > 0:
            fill.append(torch.empty(k, dtype=torch.uint8, device="cuda:0"))
    say("short of memory:", torch.cuda.mem_get_info()[0])
    r = G.query(10_000, (1, 1000), 0, counts=False, workspace=ws)
    del fill
    torch.cuda.empty_cache()
    want = G.query(10_000, (1, 1000), 0, counts=False)
    assert r.pair_u.size > 0 and r.pairs() == want.pairs() and r.stats["tests"] == want.stats["tests"]
    ws.close()
    folty.release_cached_memory()


def test_triangles_known_are_not_counted_again():
    """After a query the triangle count is known: a one-pass query, a plan and a server
    request use it (nothing is added to the index), with the results of a graph on
    which they come first."""
    g = synth.tiny(seed=12)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build()
    fresh = folty.Graph(g.n, g.src, g.dst, g.t).build()
    G.query(10**6, (1, 4), 0)
    before = G.device_bytes()
    for d, v in ((10**6, 0), (3600, 3)):
        want = fresh.query(d, (1, 4), v, one_pass=True)
        got = G.query(d, (1, 4), v, one_pass=True)
        assert got.pairs() == want.pairs() and got.stats["triangles"] == want.stats["triangles"] > 0
    plan = folty.Plan([G], [(0, dict(delta=10**6, theta=(1, 4), variant=0))])
    assert plan.run()[0].pairs() == G.query(10**6, (1, 4), 0).pairs()
    plan.close()
    srv = folty.Server(workers=1)
    assert srv.wait(srv.submit(G, delta=10**6, theta=(1, 4))).pairs() == G.query(10**6, (1, 4), 0).pairs()
    srv.close()
    assert G.device_bytes() == before


def test_plan_results_state_the_filter_passes():
    """Known edges first, then triangles, as in a single query of a fresh graph; none
    without closing probes (a path).  Triangles alone when each graph's largest window
    spans its timestamps, with the results of single queries."""
    g = synth.tiny(seed=13)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build()
    ids = np.arange(9, dtype=np.int32)
    P = folty.Graph(10, ids, ids + 1, np.arange(9, dtype=np.int64)).build()
    plan = folty.Plan([G, P], [(0, dict(delta=10**6, theta=(1, 4))), (1, dict(delta=5, theta=(1, 4)))])
    for _ in range(2):
        assert [r.stats["filter_passes"] for r in plan.run()] == [2, 0]
    plan.close()
    assert G.query(3600, (1, 4), 0).stats["filter_passes"] == 2
    assert P.query(5, (1, 4), 0).stats["filter_passes"] == 0
    g2 = synth.bruteforce_size(seed=16)
    G2 = folty.Graph(g2.n, g2.src, g2.dst, g2.t).build(cache_triangles=True)
    for last, passes in ((folty.DELTA_INF, 1), (3600, 2)):
        qs = [(i, dict(delta=d, theta=(1, 4), variant=v)) for v in range(8)
              for i, d in ((0, folty.DELTA_INF), (0, 3600), (1, 600), (1, last))]
        plan = folty.Plan([G, G2], qs)
        for _ in range(2):
            for (i, q), r in zip(qs, plan.run()):
                say("plan passes", i, q)
                w = (G, G2)[i].query(**q)
                assert r.stats["filter_passes"] == passes
                assert np.array_equal(r.counts(), w.counts()) and r.pairs() == w.pairs()
        plan.close()


def test_a_failed_call_waits_for_its_stream():
    """Buffers of a failed call go back to pools that other streams take from: the call
    returns its error only when its stream is idle (40 products are queued on it here
    before a query whose first allocation fails), and the same query answers after."""
    import ctypes
    import torch
    g = synth.tiny(seed=14)
    stream = torch.cuda.Stream()
    G = folty.Graph(g.n, g.src, g.dst, g.t, stream=stream.cuda_stream)
    dev, refuse = torch.cuda.current_device(), []

    def alloc(nbytes, st, ctx):
        return None if refuse else torch.cuda.caching_allocator_alloc(int(nbytes), dev, int(st or 0))

    opts = folty.BuildOpts(0, 0, 0, folty.ALLOC_FN(alloc),
                           folty.FREE_FN(lambda p, nbytes, st, ctx: torch.cuda.caching_allocator_delete(p)), None)
    assert folty.load_library().folty_build_index(G._h, ctypes.byref(opts)) == folty.OK
    G.query(10**6, (1, 4), 0)
    a = torch.ones(8192, 8192, device="cuda:0", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(40):
            a @ a
    refuse.append(1)
    # N(a) & N(b): the per-edge triangle counts are made on first use, in the caller's memory
    with pytest.raises(folty.FoltyError) as ei:
        G.query(10**6, (1, 4), 0, folty.UNIVERSE_COMMON)
    idle = stream.query()
    say("failed query", ei.value.code, idle)
    assert ei.value.code == folty.ENOMEM and idle
    refuse.clear()
    o = Oracle(g.n, g.src, g.dst, g.t)
    assert_same(G.query(10**6, (1, 4), 0, folty.UNIVERSE_COMMON), o.query(10**6, 1, 4, 0, folty.UNIVERSE_COMMON))
    G.close()


def test_plan_takes_a_tuning_file_with_more_blocks_than_run(tmp_path):
    """A tuning file may name up to 2^20 blocks; the launch is held to what the heavy
    list's counter allows, results are the single queries' (a child process: the table
    lives as long as the process)."""
    import json
    import os
    import subprocess
    import sys
    path = tmp_path / "tune.json"
    path.write_text(json.dumps(dict(arch="gfx950", entries=[
        dict(tests_log2=a, edges_log2=b, tests_per_chunk=2, blocks=1 << 20, ms=1.0) for a in range(40) for b in range(32)])))
    code = r"""
import numpy as np
from paper_2507_17215_amd import folty
rng = np.random.default_rng(15)
n, m = 60, 60_000  # long lists: most triangles have more than 64 tests
src, dst, t = rng.integers(0, n, m), rng.integers(0, n, m), np.sort(rng.integers(0, 10**6, m))
G = folty.Graph(n, src.astype(np.int32), dst.astype(np.int32), t).build()
qs = [dict(delta=d, theta=(1, 4), variant=v) for d in (500, 20_000) for v in (0, 5)]
plan = folty.Plan([G], [(0, q) for q in qs])
for _ in range(2):
    for q, r in zip(qs, plan.run()):
        w = G.query(**q)
        assert np.array_equal(r.counts(), w.counts()) and r.pairs() == w.pairs()
assert plan.info()["temporal_blocks"] == 1 << 20 and plan.info()["tune_source"] == 2, plan.info()
print("ok")
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=110, cwd=root,
                         env=dict(os.environ, FOLTY_TUNE_CACHE=str(path)))
    say("tuning file:", out.stdout.strip(), out.stderr[-1500:])
    assert out.returncode == 0 and out.stdout.strip() == "ok"


@pytest.mark.parametrize("close, passes", [(1, 2), (2, 1)])
def test_switch_to_one_pass_at_one_triangle_in_twelve(close, passes):
    """24 separate triangles, `close` of them within the window: one in 12 kept switches
    later queries from half of that window on, one in 24 does not."""
    k = 24
    a = np.arange(k, dtype=np.int32) * 3
    gap = np.where(np.arange(k) < close, 10, 5000)
    src = np.concatenate([a, a, a + 1])
    dst = np.concatenate([a + 1, a + 2, a + 2])
    t = np.concatenate([np.zeros(k, np.int64), gap // 2, gap])
    o = Oracle(3 * k, src, dst, t)
    G = folty.Graph(3 * k, src, dst, t).build()
    got = []
    for delta in (100, 100, 50, 49):
        r = G.query(delta, (1, 2), 0)
        assert_same(r, o.query(delta, 1, 2, 0))
        got.append(r.stats["filter_passes"])
    assert got == [2, passes, passes, 2]


def test_row_table_with_ids_equal_in_their_low_bits():
    """The row table keeps the low 22 bits of ids: with more vertices than that, entries
    that agree in them are told apart by the row.  In the random orientation an
    id's rank does not depend on the edges: a complete graph on the ranks below 64
    and the ones 2^22 above them has such pairs in every row and among its probes."""
    n = (1 << 22) + 64
    e = np.zeros(1, np.int32)
    rank = folty.Graph(n, e, e + 1, e.astype(np.int64)).build(rank_mode=folty.RANK_RANDOM, rank_seed=9).ranks()
    ids = np.nonzero((rank < 64) | (rank >= 1 << 22))[0].astype(np.int32)
    assert ids.size == 128
    rng = np.random.default_rng(17)
    i, j = np.triu_indices(128, 1)
    keep = rng.random(i.size) < 0.7
    i, j = np.repeat(i[keep], 2), np.repeat(j[keep], 2)
    flip = rng.random(i.size) < 0.5
    src, dst = np.where(flip, ids[j], ids[i]), np.where(flip, ids[i], ids[j])
    t = rng.integers(0, 10_000, src.size)
    o = Oracle(n, src, dst, t)
    G = folty.Graph(n, src, dst, t).build(rank_mode=folty.RANK_RANDOM, rank_seed=9)
    assert np.array_equal(G.ranks(), rank)
    for delta, v, one in ((300, 0, False), (10_000, 5, False), (10_000, 0, True)):
        say("equal low bits", delta, v, one)
        want = o.query(delta, 1, 10, v)
        assert (want["counts"] > 0).any()
        assert_same(G.query(delta, (1, 10), v, one_pass=one), want)
    A = np.zeros((128, 128), np.int64)
    A[i, j] = A[j, i] = 1
    assert G.stats()["triangles"] == int((A @ A * A).sum()) // 6


@pytest.mark.parametrize("delta", [folty.DELTA_INF, 100])
def test_cached_list_takes_its_chunks_at_once(delta):
    """A cached list of 10.6 million triangles (165,000 chunks, past the 65,536 that are
    always allocated): everything kept by the first query, and next to nothing."""
    g = cliques(1, 400, 10**6, 62)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build(cache_triangles=True)
    H = folty.Graph(g.n, g.src, g.dst, g.t).build()
    for v in (0, 5):
        say("cached list", delta, v)
        got, want = G.query(delta, (1, 400), v), H.query(delta, (1, 400), v)
        assert np.array_equal(got.counts(), want.counts()) and got.pairs() == want.pairs()
        assert got.stats["tests"] == want.stats["tests"]
        a, b = G.triad_query(delta, v, triples=False), H.triad_query(delta, v, triples=False)
        assert a.triads()["n_instances"] == b.triads()["n_instances"]
        assert a.triads()["n_solutions"] == b.triads()["n_solutions"]
