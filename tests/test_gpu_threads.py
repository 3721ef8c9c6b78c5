"""Generation on several threads with a stream each: the sets of every thread
equal the oracle's, those that a workgroup moves into the pool (above 4096
members) among them."""
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


def _hypergraph(n, seed):
    """A dense half, whose sets hold thousands, and a half of pairs."""
    rng = np.random.Generator(np.random.PCG64(seed))
    half = n // 2
    edges = [rng.choice(half, size=6, replace=False).tolist() for _ in range(half)]
    edges += [[v, v + 1] for v in range(half, n - 1, 2)]
    return hypergen.from_lists(n, edges)


def test_generation_on_streams_equals_the_oracle(hy):
    import torch
    threads, ids, step = 4, 240, 60
    jobs = []
    for t in range(threads):
        hg = _hypergraph(12000 + 500 * t, t)
        o = oracle.Graph(hg, 0, 0.3)
        o.stratify()
        jobs.append((hg, o.generate(9, t, 0, 0, ids)))
        sizes = np.diff(jobs[-1][1][0].astype(np.int64))
        assert (sizes > 4096).any() and (sizes < 64).any()
    wrong = []

    def work(t):
        print(f"[gpu] generation on stream {t}", flush=True)
        hg, want = jobs[t]
        with torch.cuda.stream(torch.cuda.Stream()):
            g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, 0, 0.3)
            g.stratify()
            for _ in range(3):
                pool = hy.Pool(g)
                for j in range(0, ids, step):
                    hy.generate_rr(g, 9, t, 0, j, j + step, pool)
                if not all(np.array_equal(a, b) for a, b in zip(pool.read(), want)):
                    wrong.append(t)

    ts = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not wrong
