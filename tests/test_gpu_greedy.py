"""Greedy and coverage at the edges of their set classes: sets of up to 4096
members go through an inverted index, larger ones through searches in their
members and, on graphs of up to 4194304 vertices, through ranges of 8192
vertices.  Channels of probability 1 make every RR set a connected component,
so the components' sizes set the sets' sizes.  Whole numbers, equal to the
oracle's."""
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


def _stars(n, sizes, seed):
    """Star components of the given sizes over shuffled ids (a centre and one
    hyperedge per leaf); the other vertices are alone."""
    ids = np.random.Generator(np.random.PCG64(seed)).permutation(n).astype(np.uint32)
    mem, at = [], 0
    for size in sizes:
        part = ids[at:at + size]
        at += size
        mem.append(np.stack([np.full(size - 1, part[0], np.uint32), part[1:]], 1).reshape(-1))
    mem = np.concatenate(mem)
    return hypergen.Hypergraph(n, np.arange(0, mem.size + 1, 2, dtype=np.uint32), mem)


# vertices, component sizes, RR sets, seeds
CASES = {
    "small_only": (9000, [4096, 1500, 700, 16, 17, 2], 1000, 12),
    "edge": (14000, [4097, 4096, 3000, 900], 1000, 8),
    "big_only": (8192, [8192], 300, 3),
    "many_big": (33000, [5000, 6000, 7000, 4500, 4200, 5500], 2000, 9),
    "no_ranges": (4194305, [1500000, 600000, 4000], 256, 6),
    "few_counts": (50000, [2, 3, 2], 40, 60),
    "shared_members": (600, [300, 200], 1500, 5),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_greedy_and_coverage_by_set_class(hy, case):
    print(f"[gpu] greedy case={case}", flush=True)
    n, sizes, theta, k = CASES[case]
    hg = _stars(n, sizes, len(case))
    g = hy.build_graph(n, hg.he_off, hg.he_mem, 0, 1.0)
    g.stratify()
    pool = hy.Pool(g)
    hy.generate_rr(g, 3, 0, 0, 0, theta, pool)
    off, mem, _ = pool.read()
    for th in (theta, theta // 2 + 1):
        seeds, gains = hy.greedy(g, pool, th, k)
        ws, wg = oracle.greedy(n, off, mem, k, theta=th)
        assert np.array_equal(seeds, ws), th
        assert np.array_equal(gains, wg), th
        for s in (seeds, seeds[1:3], np.arange(0, n, max(1, n // 300), dtype=np.uint32)):
            assert hy.coverage(g, pool, th, s) == oracle.coverage(n, off, mem, s, theta=th)


@pytest.mark.parametrize("case", ["small_only", "many_big", "few_counts"])
def test_upper_bound_by_set_class(hy, case):
    """lambda_u (the smallest of greedy's prefix bounds) against the oracle's
    on the same sets."""
    print(f"[gpu] upper bound case={case}", flush=True)
    n, sizes, theta, k = CASES[case]
    hg = _stars(n, sizes, len(case))
    g = hy.build_graph(n, hg.he_off, hg.he_mem, 0, 1.0)
    g.stratify()
    r = hy.select_seeds(g, k, 0.1, 1.0, seed=3, theta_fixed=theta)
    pool = hy.Pool(g)
    hy.generate_rr(g, 3, 0, 0, 0, theta, pool)
    off, mem, _ = pool.read()
    ws, wg = oracle.greedy(n, off, mem, k, theta=theta)
    assert np.array_equal(r["seeds"], ws) and np.array_equal(r["gains"], wg)
    assert r["lambda_u"] == oracle.upper_eq8(n, off, mem, ws, theta=theta)
