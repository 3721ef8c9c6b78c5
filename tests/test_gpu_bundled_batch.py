"""Instances of the 64-instance workload grown in bundles from their first set
on, in one batched call: ids drawn from every instance, its largest sets among
them, equal the oracle's."""
import numpy as np
import pytest

import hypergen
import oracle

pytestmark = pytest.mark.gpu

# index -> vertices, mean live in-edges: 1 (109845, 0.54), 31 (150193, 4.53), 22 (10021, 4.40)
PICK = (1, 31, 22)


@pytest.fixture(scope="module")
def hy():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_01911_amd as hy
    hy.load_library()
    return hy


def test_bundled_instances_in_one_batch(hy):
    ws = hypergen.multi_instance_workloads(64)
    inst, tasks = [], []
    for i in PICK:
        print(f"[gpu] bundled instance {i}", flush=True)
        w, hg = ws[i], ws[i].build()
        g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, w.model, w.p)
        g.stratify()
        g.set_tuning(ms_min=1, ms_filter=8, chunk=2048, seg=2048)
        o = oracle.Graph(hg, w.model, w.p)
        o.stratify()
        pools = [hy.Pool(g), hy.Pool(g)]
        inst.append((i, w, o, pools))
        tasks += [dict(graph=g, pool=p, seed=w.philox_seed, instance=i, pool_tag=t, id_begin=0, id_end=300 - 100 * t)
                  for t, p in enumerate(pools)]
    hy.generate_rr_batch(tasks, form=0)
    rng = np.random.default_rng(5)
    for i, w, o, pools in inst:
        for tag, pool in enumerate(pools):
            off, mem, roots = pool.read()
            sizes = np.diff(off.astype(np.int64))
            ids = set(np.argsort(sizes, kind="stable")[-2:].tolist()) | set(rng.choice(sizes.size, 4).tolist())
            for j in sorted(ids):
                _, m, r = o.generate(w.philox_seed, i, tag, j, j + 1)
                assert r[0] == roots[j], (i, tag, j)
                assert np.array_equal(mem[int(off[j]):int(off[j + 1])], m), (i, tag, j)
