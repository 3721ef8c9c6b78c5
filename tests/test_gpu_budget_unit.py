"""The incidence budget of the per-set phase counts incidences: a set is handed
over once it has read more of them, or more member positions than the larger
of the budget and 262144."""
import numpy as np
import pytest

import hypergen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hy():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_01911_amd as hy
    hy.load_library()
    return hy


# Disjoint hyperedges with p = 1: a set is its root's hyperedge, reads `size`
# incidences and size * size positions, 64 vertices at a time after the root.
@pytest.mark.parametrize("size,budget,over", [
    (100, 1000, False),      # 100 incidences, 10000 positions
    (100, 100, False),
    (100, 64, True),         # 65 after the second batch, more to come
    (600, 262144, True),     # 600 incidences; 269400 positions when 151 vertices are left
    (600, 400000, False),    # 346200 before the last batch
    (600, 1 << 30, False)])
@pytest.mark.parametrize("model", [0, 5])
def test_budget_counts_incidences(hy, model, size, budget, over):
    print(f"[gpu] budget unit model={model} size={size} budget={budget}", flush=True)
    count = 40000 // size
    hg = hypergen.from_lists(size * count, [list(range(i * size, (i + 1) * size)) for i in range(count)])
    g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, model, 1.0)
    g.stratify()
    g.set_tuning(budget=budget)
    theta = 512
    r = hy.select_seeds(g, 3, 0.5, 1.0, seed=2, theta_fixed=theta)
    assert r["entries1"] == r["entries2"] == theta * size
    assert r["deferred"] == (2 * theta if over else 0)
