"""Greedy over big sets where the way their members leave the counts changes:
shares of sets up to about 2^22 members a round, vertex ranges counted in LDS
above, ranges that none of the sets touches, one set and thousands.  Channels
of probability 1 make every RR set a connected component.  Whole numbers, equal
to the oracle's."""
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


def _stars(n, sizes, first):
    """Star components of neighbouring ids from `first` on; the other vertices
    are alone."""
    mem, at = [], first
    for size in sizes:
        part = np.arange(at, at + size, dtype=np.uint32)
        at += size
        mem.append(np.stack([np.full(size - 1, part[0], np.uint32), part[1:]], 1).reshape(-1))
    mem = np.concatenate(mem)
    return hypergen.Hypergraph(n, np.arange(0, mem.size + 1, 2, dtype=np.uint32), mem)


# vertices, component sizes, id of the first, RR sets, seeds
CASES = {
    "one_set": (8192, [8192], 0, 1, 2),
    "two_sets": (9000, [8999], 1, 2, 2),
    "below_the_line": (8192, [8192], 0, 511, 2),       # 511 * 8192 members in the first round
    "at_the_line": (8192, [8192], 0, 512, 2),
    "thousands": (5000, [4999], 1, 3001, 3),           # one range, many workgroups
    "two_ranges": (8193, [8193], 0, 1100, 2),
    "empty_ranges": (100000, [30000, 9000, 4097], 40000, 2500, 5),   # most ranges untouched, a few sets or none each
    "no_ranges": (4200000, [1200000, 900000], 3, 90, 4),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_big_sets_leave_the_counts(hy, case):
    print(f"[gpu] greedy of big sets: {case}", flush=True)
    n, sizes, first, theta, k = CASES[case]
    hg = _stars(n, sizes, first)
    g = hy.build_graph(n, hg.he_off, hg.he_mem, 0, 1.0)
    g.stratify()
    pool = hy.Pool(g)
    hy.generate_rr(g, 3, 0, 0, 0, theta, pool)
    off, mem, _ = pool.read()
    seeds, gains = hy.greedy(g, pool, theta, k)
    ws, wg = oracle.greedy(n, off, mem, k, theta=theta)
    assert np.array_equal(seeds, ws)
    assert np.array_equal(gains, wg)
    r = hy.select_seeds(g, k, 0.1, 1.0, seed=3, theta_fixed=theta)
    assert np.array_equal(r["seeds"], ws)
    assert r["lambda_u"] == oracle.upper_eq8(n, off, mem, ws, theta=theta)
