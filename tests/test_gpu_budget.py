"""Sessions with a small budget: queries on small graphs are answered as they
are alone, with RR slots laid out in less memory, and after another graph's
preparation has left gigabytes of scratch in the workspace."""
import numpy as np
import pytest

import hypergen

pytestmark = pytest.mark.gpu

GIB = 1 << 30


@pytest.fixture(scope="module")
def hy():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_01911_amd as hy
    hy.load_library()
    return hy


def _graph(hy, n, seed, model=1):
    """Two hyperedges per vertex of 2 to 60 members and a few hubs."""
    rng = np.random.Generator(np.random.PCG64(seed))
    sizes = np.minimum(2 + (rng.pareto(1.3, size=2 * n)).astype(np.int64), 60)
    edges = [rng.choice(n, size=int(s), replace=False).tolist() for s in sizes]
    for h in range(2):
        for e in rng.choice(len(edges), size=n // 2, replace=False):
            if h not in edges[e]:
                edges[e].append(h)
    hg = hypergen.from_lists(n, edges)
    g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, model, 0.0)
    g.stratify()
    return g


def _answers(hy, graphs, budget):
    s = hy.Session(hbm_budget=budget)
    tickets = [s.submit(g, 7 + i, 0.4, 1.0, 5, i) for i, g in enumerate(graphs)]
    out = [None] * len(graphs)
    for _ in range(100):
        st = s.step()
        assert st["bytes_resident"] <= budget
        out = [r if r is not None else s.poll(t) for r, t in zip(out, tickets)]
        if all(r is not None for r in out):
            break
    s.close()
    return out


def _check(hy, graphs, got):
    for i, (g, r) in enumerate(zip(graphs, got)):
        a = hy.select_seeds(g, 7 + i, 0.4, 1.0, seed=5, instance=i)
        assert np.array_equal(a["seeds"], r["seeds"]) and np.array_equal(a["gains"], r["gains"])
        for key in ("theta", "rounds", "lambda1", "lambda2", "entries1", "entries2"):
            assert a[key] == r[key], (i, key)


@pytest.mark.parametrize("warm", [False, True])
def test_small_graphs_within_one_gibibyte(hy, warm):
    print(f"[gpu] budget warm={warm}", flush=True)
    graphs = [_graph(hy, 30000, 1), _graph(hy, 4000, 2), _graph(hy, 30000, 3, model=6)]
    hy.workspace_release()
    if warm:   # the usual layout, more than the budget
        hy.select_seeds(graphs[0], 3, 0.5, 1.0, seed=1)
        assert hy.workspace_bytes() > GIB
    got = _answers(hy, graphs, GIB)
    assert hy.workspace_bytes() < GIB
    _check(hy, graphs, got)
    assert hy.workspace_bytes() > GIB   # calls without a budget take the usual layout again


def test_scratch_of_another_graph_is_given_back(hy):
    print("[gpu] budget after a stratified-setting graph", flush=True)
    hy.workspace_release()
    rng = np.random.Generator(np.random.PCG64(4))
    big = hypergen.from_lists(3000, [rng.choice(3000, size=1000, replace=False).tolist() for _ in range(150)])
    layered = hy.build_graph(big.n, big.he_off, big.he_mem, 4, 0.0)
    layered.stratify()
    assert hy.workspace_bytes() > 2 * GIB
    graphs = [_graph(hy, 3000, 5), _graph(hy, 2000, 6)]
    _check(hy, graphs, _answers(hy, graphs, 2 * GIB))
