"""Equation (8)'s sums of the k largest counts where many vertices share a
count, where counts lie on both sides of the window that is listed once per
value, and where there are fewer than k.  Channels of probability 1 make every
RR set a connected component.  Whole numbers, equal to the oracle's."""
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


def _components(n, sizes):
    """Star components of neighbouring ids (a hyperedge of two per leaf); the
    other vertices are alone."""
    edges, at = [], 0
    for s in sizes:
        edges += [[at, at + i] for i in range(1, s)]
        at += s
    assert at <= n
    return hypergen.from_lists(n, edges)


# vertices, component sizes, RR sets, seeds
CASES = {
    "pairs": (30000, [2] * 15000, 20000, 40),
    "tens": (30001, [10] * 3000, 4000, 60),
    "tens_many_sets": (20002, [10] * 2000, 100000, 30),       # counts about 50
    "all_equal": (4099, [4096], 3000, 5),                       # one count, then none
    "far_apart": (30003, [15000] + [7] * 2000, 30000, 50),      # 15000 and 7 per vertex: 256 and more between them
    "window_edge": (600, [200] * 3, 1500, 250),                 # about 500 each; k reaches into the second
    "steps": (9000, [1000, 500, 250, 125, 60, 30, 15, 8, 4, 2], 9000, 70),
    "fewer_than_k": (2000, [3, 2], 20, 100),
    "one_vertex": (1, [1], 50, 1),
    "all_seeds": (37, [5, 4, 3, 2], 300, 37),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_upper_bound_of_shared_counts(hy, case):
    print(f"[gpu] upper bound: {case}", flush=True)
    n, sizes, theta, k = CASES[case]
    hg = _components(n, sizes)
    g = hy.build_graph(n, hg.he_off, hg.he_mem, 0, 1.0)
    g.stratify()
    r = hy.select_seeds(g, k, 0.1, 1.0, seed=3, theta_fixed=theta)
    pool = hy.Pool(g)
    hy.generate_rr(g, 3, 0, 0, 0, theta, pool)
    off, mem, _ = pool.read()
    ws, wg = oracle.greedy(n, off, mem, k, theta=theta)
    assert np.array_equal(r["seeds"], ws) and np.array_equal(r["gains"], wg)
    assert r["lambda_u"] == oracle.upper_eq8(n, off, mem, ws, theta=theta)
