"""How waves share a launch group's work: launch indices handed out several at
a time (from 16 sets per wave on) with room in the stage to go with them, moved
sets of every mean size, and superstep batches of every length.  RR sets are
fixed by their ids, so any other way to the same ids has to give the same
bytes."""
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


def _sets(hy, g, bounds):
    """Members, sizes and roots of the ids between consecutive bounds."""
    pool = hy.Pool(g)
    for lo, hi in zip(bounds, bounds[1:]):
        hy.generate_rr(g, 11, 2, 0, lo, hi, pool)
    return [np.asarray(x).copy() for x in pool.read()]


@pytest.mark.parametrize("workload", ["tiny", "mid_lt", "tiny_layered"])
@pytest.mark.parametrize("ids", [70000, 300001])
def test_indices_handed_out_several_at_a_time(hy, workload, ids):
    print(f"[gpu] shares {workload} ids={ids}", flush=True)
    w = hypergen.workload(workload)
    hg = w.build()
    g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, w.model, w.p)
    g.stratify()
    if workload == "tiny":
        ids //= 10   # large sets: the pool would take gigabytes
    whole = _sets(hy, g, [0, ids])
    pieces = _sets(hy, g, list(range(0, ids, 9973)) + [ids])   # less than one per wave and turn
    assert all(np.array_equal(a, b) for a, b in zip(whole, pieces))


@pytest.mark.parametrize("steps", [1, 2, 7, 8, 9, 16, 64])
def test_superstep_batches_of_every_length(hy, steps):
    print(f"[gpu] steps_per_sync={steps}", flush=True)
    w = hypergen.workload("mid")
    hg = w.build()
    g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, w.model, w.p)
    g.stratify()
    want = _sets(hy, g, [0, 1500])
    g.set_tuning(**{**g.tuning(), "steps_per_sync": steps, "budget": 64})
    for _ in range(2):   # captured, then replayed
        got = _sets(hy, g, [0, 1500])
        assert all(np.array_equal(a, b) for a, b in zip(want, got))
