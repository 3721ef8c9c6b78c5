"""Device blocks that outlive the handles they belonged to: graphs and pools
built, queried and freed again and again, on several threads with a stream
each, give the bytes that the first ones gave, also after a release in
between."""
import threading

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


def _once(hy, hg, w, seed, ids):
    g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, w.model, w.p)
    g.stratify()
    r = hy.select_seeds(g, 5, 0.5, 1.0, seed=seed)
    pool = hy.Pool(g)
    hy.generate_rr(g, seed, 1, 0, 0, ids, pool)
    off, mem, roots = pool.read()
    out = [np.asarray(r["seeds"]).copy(), np.asarray(off).copy(), np.asarray(mem).copy(), np.asarray(roots).copy()]
    del pool, g
    return out


@pytest.mark.parametrize("threads", [1, 4])
def test_blocks_of_freed_handles_serve_again(hy, threads):
    import torch
    print(f"[gpu] blocks threads={threads}", flush=True)
    jobs = []
    for name, seed, ids in (("tiny", 3, 700), ("mid", 4, 1500)):
        w = hypergen.workload(name)
        hg = w.build()
        jobs.append((hg, w, seed, ids))
    hy.workspace_release()
    want = [_once(hy, *j) for j in jobs]
    wrong = []

    def work(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(4):
                k = (i + t) % len(jobs)
                got = _once(hy, *jobs[k])
                if not all(np.array_equal(a, b) for a, b in zip(want[k], got)):
                    wrong.append((t, i, k))

    ts = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not wrong
    hy.workspace_release()
    for j, w in zip(jobs, want):
        assert all(np.array_equal(a, b) for a, b in zip(w, _once(hy, *j)))
