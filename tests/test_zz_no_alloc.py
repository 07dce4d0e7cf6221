"""The entry point that allocates nothing (folty_run_fol_query_noalloc) against
the ordinary query entry point: identical per-edge counts, pairs, certificate
counts and |Sol|, on two calls in a row (the second on a smaller graph), and a
clear error when the fixed scratch is too small."""
import numpy as np
import pytest
import torch

from paper_2507_17215_amd import folty, synth

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


def outputs(G, cap):
    dev = torch.device("cuda:0")
    z = lambda k: torch.full((k,), -7, dtype=torch.int32, device=dev)
    return dict(pair_u=z(cap), pair_v=z(cap), n_cert=z(cap), edge_count=z(G.m))


def same_as_query(G, delta, theta, variant, universe=0, smaller_side=False):
    want = G.query(delta, theta, variant, universe, smaller_side=smaller_side)
    out = outputs(G, max(1, want.pair_u.size + 5))
    got = G.query_noalloc(delta, theta, variant, universe, smaller_side=smaller_side, **out)
    torch.cuda.synchronize()
    assert got["n_pairs"] == want.pair_u.size
    assert got["n_certificates"] == want.n_certificates
    assert np.array_equal(got["pair_u"].cpu().numpy(), want.pair_u)
    assert np.array_equal(got["pair_v"].cpu().numpy(), want.pair_v)
    assert np.array_equal(got["n_cert"].cpu().numpy().view(np.uint32), want.n_cert)
    assert np.array_equal(got["edge_count"].cpu().numpy().view(np.uint32), want.counts())
    return got


def test_noalloc_equals_query_two_calls_then_smaller():
    torch.cuda.set_device(0)
    big = synth.tiny(seed=41)
    small = synth.bruteforce_size(seed=42)
    Gb = folty.Graph(big.n, big.src, big.dst, big.t).build()
    Gs = folty.Graph(small.n, small.src, small.dst, small.t).build()
    for delta, theta, variant in ((200_000, (1, 4), 0), (10**6, (1, 2), 3), (3600, (0, 1), 6)):
        say("noalloc", delta, theta, variant)
        same_as_query(Gb, delta, theta, variant)   # first call
        same_as_query(Gs, delta, theta, variant)   # second call, smaller input
    same_as_query(Gb, 10**6, (1, 4), 0, smaller_side=True)
    # the universe N(a) & N(b) once its per-edge triangle counts exist
    Gb.query(10**6, (1, 4), 0, folty.UNIVERSE_COMMON)
    same_as_query(Gb, 10**6, (1, 4), 0, folty.UNIVERSE_COMMON)
    with pytest.raises(folty.FoltyError) as ei:
        Gs.query_noalloc(10**6, (1, 4), 0, folty.UNIVERSE_COMMON, **outputs(Gs, 4096))
    assert ei.value.code == folty.EINVAL


def test_noalloc_pair_capacity_and_scratch_limit():
    g = synth.tiny(seed=43)
    G = folty.Graph(g.n, g.src, g.dst, g.t).build()
    want = G.query(10**6, (0, 1), 0)  # theta = 0: every pair is a solution
    out = outputs(G, 3)
    with pytest.raises(folty.FoltyError) as ei:
        G.query_noalloc(10**6, (0, 1), 0, **out)
    assert ei.value.code == folty.EOVERFLOW
    assert str(want.pair_u.size) in str(ei.value)
    big = synth.c1_family(4_000_000, seed=44)
    Gbig = folty.Graph(big.n, big.src, big.dst, big.t).build()
    with pytest.raises(folty.FoltyError) as ei:
        Gbig.query_noalloc(10**6, (1, 2), 0, **outputs(Gbig, 16))
    assert ei.value.code == folty.ENOMEM
    assert "scratch" in str(ei.value)
    # the scratch is still fine for the next call
    same_as_query(G, 10**6, (1, 4), 3)


def spread_ids(n, ids, m, seed):
    """m edges between ids of n vertices, the others without any."""
    rng = np.random.default_rng(seed)
    label = rng.choice(n, ids, replace=False).astype(np.int32)
    return label[rng.integers(0, ids, m)], label[rng.integers(0, ids, m)], np.sort(rng.integers(0, 10**6, m))


def test_noalloc_takes_few_edges_on_many_ids():
    """The scratch is shared by what the edges need, whatever the number of vertices:
    the first call on the index, which counts its triangles, and later ones."""
    src, dst, t = spread_ids(4_000_000, 20_000, 500_000, 45)
    G = folty.Graph(4_000_000, src, dst, t).build()
    say("many ids, first call")
    out = outputs(G, G.m)
    got = G.query_noalloc(10**6, (1, 100), 0, **out)
    want = G.query(10**6, (1, 100), 0)
    assert got["n_pairs"] == want.pair_u.size and got["n_certificates"] == want.n_certificates
    assert np.array_equal(got["edge_count"].cpu().numpy().view(np.uint32), want.counts())
    for delta, variant in ((10**6, 0), (20_000, 6)):
        say("many ids", delta, variant)
        got = same_as_query(G, delta, (1, 100), variant)
        assert got["n_pairs"] > 0


@pytest.mark.parametrize("cached", [False, True])
def test_noalloc_tests_triangles_in_parts(cached):
    """All triangles of a 400-vertex clique (10.6 million, 127 MB as a list) are kept:
    several times the scratch, so they are tested in parts, on a fresh index (which
    counts them) and later ones, from items and from the cached list."""
    k = 400
    a, b = np.triu_indices(k, 1)
    rng = np.random.default_rng(46)
    flip = rng.random(a.size) < 0.5
    src = np.where(flip, b, a).astype(np.int32)
    dst = np.where(flip, a, b).astype(np.int32)
    t = np.sort(rng.integers(0, 10**6, a.size))
    G = folty.Graph(k, src, dst, t).build(cache_triangles=cached)
    H = folty.Graph(k, src, dst, t).build(cache_triangles=cached)  # queried without a prior count
    for delta, variant, side in ((10**6, 0, False), (10**6, 5, False), (10**6, 0, True)):
        say("clique in parts", cached, delta, variant, side)
        same_as_query(G, delta, (1, 4), variant, smaller_side=side)
        want = G.query(delta, (1, 4), variant)
        out = outputs(H, want.pair_u.size + 1)
        got = H.query_noalloc(delta, (1, 4), variant, smaller_side=side, **out)
        assert got["n_certificates"] == want.n_certificates
        assert np.array_equal(got["edge_count"].cpu().numpy().view(np.uint32), want.counts())
    assert H.stats()["triangles"] == k * (k - 1) * (k - 2) // 6
