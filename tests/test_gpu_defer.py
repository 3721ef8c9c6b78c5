"""Sets of small graphs (visited marks in LDS, up to 32768 vertices) that move
to the grid-wide phase, and mixes of small and larger graphs in one workspace:
every RR set equals the oracle's."""
import numpy as np
import pytest

import hypergen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hy():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_01911_amd as hy
    hy.load_library()
    return hy


def _graph(n, seed, largest=90):
    """Two hyperedges per vertex of 2 to `largest` members and a few hubs."""
    rng = np.random.Generator(np.random.PCG64(seed))
    sizes = np.minimum(2 + (rng.pareto(1.2, size=2 * n)).astype(np.int64), min(largest, n))
    edges = [rng.choice(n, size=int(s), replace=False).tolist() for s in sizes]
    for h in range(3):
        for e in rng.choice(len(edges), size=n // 3, replace=False):
            if h not in edges[e]:
                edges[e].append(h)
    return hypergen.from_lists(n, edges)


def _check(hy, g, o, pools, ids):
    for tag, pool in pools:
        off, mem, roots = pool.read()
        roff, rmem, rroots = o.generate(5, 1, tag, 0, ids)
        assert np.array_equal(roots, rroots)
        assert np.array_equal(off, roff)
        assert np.array_equal(mem, rmem)


# model, p, (heavy, budget, chunk, seg): every set deferred at once, by a hub,
# by its budget after a while, never
@pytest.mark.parametrize("model,p", [(0, 0.05), (1, 0.0), (5, 0.05), (6, 0.0)])
@pytest.mark.parametrize("tune", [(1, 1, 16, 16), (20, 1 << 30, 64, 64), (1 << 30, 300, 16, 128),
                                  (1 << 30, 1 << 30, 256, 512)])
def test_small_graph_deferral(hy, model, p, tune):
    print(f"[gpu] defer model={model} tune={tune}", flush=True)
    hg = _graph(900, 4)
    g, o = hy.build_graph(hg.n, hg.he_off, hg.he_mem, model, p), oracle.Graph(hg, model, p)
    g.stratify()
    o.stratify()
    g.set_tuning(heavy=tune[0], budget=tune[1], chunk=tune[2], seg=tune[3])
    pools = [(tag, hy.Pool(g)) for tag in (0, 1)]
    for tag, pool in pools:
        hy.generate_rr(g, 5, 1, tag, 0, 100, pool)
        hy.generate_rr(g, 5, 1, tag, 100, 700, pool)
    _check(hy, g, o, pools, 700)


def test_small_and_larger_graphs_share_a_workspace(hy):
    """32768 vertices (marks in LDS), 33000 (marks in memory), 40, in turn."""
    print("[gpu] defer: mixed sizes", flush=True)
    for n, seed in ((40, 1), (33000, 2), (32768, 3), (40, 1), (33000, 2)):
        hg = _graph(n, seed)
        g, o = hy.build_graph(n, hg.he_off, hg.he_mem, 1, 0.0), oracle.Graph(hg, 1, 0.0)
        g.stratify()
        o.stratify()
        g.set_tuning(heavy=64, budget=2000, chunk=16, seg=64)
        pool = hy.Pool(g)
        hy.generate_rr(g, 5, 1, 0, 0, 300, pool)
        _check(hy, g, o, [(0, pool)], 300)


@pytest.mark.parametrize("chunk,seg", [(16, 16), (256, 512)])
def test_long_hyperedges_weigh_by_their_members(hy, chunk, seg):
    """Vertices in few, long hyperedges: items are cut by member positions."""
    print(f"[gpu] defer: long hyperedges chunk={chunk}", flush=True)
    hg = _graph(2500, 9, largest=2000)
    extra = [list(range(0, 2500, 2)), list(range(1, 2400)), list(range(5, 2500, 3))]
    hg = hypergen.from_lists(hg.n, [hg.he_mem[a:b].tolist() for a, b in zip(hg.he_off[:-1], hg.he_off[1:])] + extra)
    for model, p in ((0, 0.002), (1, 0.0)):
        g, o = hy.build_graph(hg.n, hg.he_off, hg.he_mem, model, p), oracle.Graph(hg, model, p)
        g.stratify()
        o.stratify()
        g.set_tuning(heavy=4, budget=500, chunk=chunk, seg=seg)
        pool = hy.Pool(g)
        hy.generate_rr(g, 5, 1, 0, 0, 200, pool)
        _check(hy, g, o, [(0, pool)], 200)


@pytest.mark.parametrize("first", [(1 << 32) - 100, (1 << 33) - 64, (1 << 32) + 5])
@pytest.mark.parametrize("chunk", [16, 4096])
def test_bundles_at_multiples_of_2_32(hy, first, chunk):
    """Bundled generation across a multiple of 2^32, where the ids' upper word
    changes: every entry heavy (chunk 16) or light (4096)."""
    print(f"[gpu] bundles at {first} chunk={chunk}", flush=True)
    hg = _graph(600, 6)
    for model, p in ((0, 0.05), (1, 0.0), (0, 1.0)):
        g, o = hy.build_graph(hg.n, hg.he_off, hg.he_mem, model, p), oracle.Graph(hg, model, p)
        g.stratify()
        o.stratify()
        for filt in (1, 65):
            g.set_tuning(ms_min=1, chunk=chunk, seg=4096, ms_filter=filt)
            pool = hy.Pool(g)
            hy.generate_rr(g, 5, 1, 1, first, first + 300, pool)
            off, mem, roots = pool.read()
            roff, rmem, rroots = o.generate(5, 1, 1, first, first + 300)
            assert np.array_equal(roots, rroots)
            assert np.array_equal(off, roff)
            assert np.array_equal(mem, rmem)
