"""Against the oracle: launch indices handed out several at a time, superstep
batches of every length, and blocks of freed handles that serve again on
several threads."""
import threading

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


def _both(hy, name):
    w = hypergen.workload(name)
    hg = w.build()
    g, o = hy.build_graph(hg.n, hg.he_off, hg.he_mem, w.model, w.p), oracle.Graph(hg, w.model, w.p)
    g.stratify()
    o.stratify()
    return g, o


def _same(o, read, lo, parts, seed, instance):
    """The sets of the id ranges `parts` within a pool that starts at id lo."""
    off, mem, roots = read
    for a, b in parts:
        woff, wmem, wroots = o.generate(seed, instance, 0, a, b)
        i, j = a - lo, b - lo
        assert np.array_equal(roots[i:j], wroots)
        assert np.array_equal(off[i:j + 1] - off[i], woff)
        assert np.array_equal(mem[int(off[i]):int(off[j])], wmem)


@pytest.mark.parametrize("workload,ids", [("tiny", 30000), ("mid_lt", 300001), ("tiny_layered", 120000)])
def test_indices_handed_out_several_at_a_time(hy, workload, ids):
    print(f"[gpu] several indices at a time: {workload}", flush=True)
    g, o = _both(hy, workload)
    pool = hy.Pool(g)
    hy.generate_rr(g, 11, 2, 0, 0, ids, pool)
    # the first grabs, which go by wave number, some of those after them, the last ones
    _same(o, pool.read(), 0, [(0, 400), (ids // 2, ids // 2 + 400), (ids - 400, ids)], 11, 2)


@pytest.mark.parametrize("steps", [1, 2, 7, 8, 9, 16, 64])
def test_superstep_batches_of_every_length(hy, steps):
    print(f"[gpu] supersteps per wait: {steps}", flush=True)
    g, o = _both(hy, "mid")
    g.set_tuning(**{**g.tuning(), "steps_per_sync": steps, "budget": 8})
    for _ in range(2):   # captured, then replayed
        pool = hy.Pool(g)
        hy.generate_rr(g, 11, 2, 0, 0, 1200, pool)
        _same(o, pool.read(), 0, [(0, 1200)], 11, 2)


def test_blocks_of_freed_handles(hy):
    import torch
    jobs = []
    for name, ids in (("tiny", 500), ("mid", 900), ("tiny_layered", 700)):
        w = hypergen.workload(name)
        hg = w.build()
        o = oracle.Graph(hg, w.model, w.p)
        o.stratify()
        jobs.append((w, hg, o.generate(6, 1, 0, 0, ids), ids))
    hy.workspace_release()
    wrong = []

    def work(t):
        print(f"[gpu] freed blocks, thread {t}", flush=True)
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(6):
                w, hg, want, ids = jobs[(i + t) % len(jobs)]
                g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, w.model, w.p)
                g.stratify()
                pool = hy.Pool(g)
                hy.generate_rr(g, 6, 1, 0, 0, ids, pool)
                if not all(np.array_equal(a, b) for a, b in zip(pool.read(), want)):
                    wrong.append((t, i))
                del pool, g

    ts = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not wrong
