"""Stage room: a range of RR sets that the sets seen before foretell badly is
generated again in a larger stage, whatever the sizes of its sets, and comes
out right."""
import numpy as np
import pytest

import hypergen
import oracle

pytestmark = pytest.mark.gpu

BLOCK = 1 << 20   # ids of one ladder block: [BLOCK, 2 * BLOCK)


@pytest.fixture(scope="module")
def hy():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_01911_amd as hy
    hy.load_library()
    return hy


# Components of `large` vertices, and of two: with p = 1 a set is its root's
# component.  A hyperedge of two puts its vertices in the same stratum as one of
# many, so a block's first ids have roots in the pairs (small ids), its last
# ones in the large components.
def _hypergraph(large, comps=40):
    half = large * comps
    edges = [[2 * i, 2 * i + 1] for i in range(half // 2)]
    edges += [list(range(half + i * large, half + (i + 1) * large)) for i in range(comps)]
    return hypergen.from_lists(2 * half, edges), half


@pytest.mark.parametrize("large,ids", [(60, 400000), (100, 300000), (140, 330000), (180, 400000), (250, 300000)])
def test_more_members_than_foretold(hy, large, ids):
    print(f"[gpu] stage large={large} ids={ids}", flush=True)
    hg, half = _hypergraph(large)
    g = hy.build_graph(hg.n, hg.he_off, hg.he_mem, 0, 1.0)
    g.stratify()
    hy.workspace_release()
    small = hy.Pool(g)
    hy.generate_rr(g, 3, 0, 0, BLOCK, BLOCK + 3000, small)
    off, _, _ = small.read()
    assert np.all(np.diff(off.astype(np.int64)) == 2)
    first = 2 * BLOCK - ids
    pool = hy.Pool(g)
    hy.generate_rr(g, 3, 0, 0, first, 2 * BLOCK, pool)
    off, mem, roots = pool.read()
    assert roots.size == ids
    # every set is the component of its root
    top = roots >= half
    want_size = np.where(top, large, 2)
    begin = np.where(top, half + (roots.astype(np.int64) - half) // large * large, roots // 2 * 2)
    assert top.sum() > ids // 2
    assert np.array_equal(np.diff(off.astype(np.int64)), want_size)
    at = np.repeat(begin - off[:-1].astype(np.int64), want_size) + np.arange(mem.size)
    assert np.array_equal(mem, at)
    # and its root the oracle's
    o = oracle.Graph(hg, 0, 1.0)
    o.stratify()
    assert np.array_equal(o.generate(3, 0, 0, first, first + 500)[2], roots[:500])
