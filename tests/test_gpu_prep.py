"""Graph preparation at the edges of its classes: vertices are counted by one
of five routes depending on their co-member occurrences c(v) (64, 512 and
3072 are the last of three; the hubs begin above 12288, n / 48 or 131072), and segments of more than 4096 hyperedges are
sorted through bitmaps.  Everything is whole numbers and has to equal the
oracle's."""
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


def _vertex(rng, v, n, occurrences, size, pool):
    """Hyperedges of `size` (the last one smaller) that give v exactly
    `occurrences` co-member occurrences among the first `pool` ids."""
    out, left = [], occurrences
    while left:
        k = min(size - 1, left)
        others = rng.choice(pool, size=k, replace=False)
        others = np.where(others == v, n - 1, others)
        out.append([int(v)] + [int(x) for x in others])
        left -= k
    return out


# c(v), members per hyperedge, ids the co-members come from
VERTICES = {
    "registers": [(c, s, p) for c in (1, 63, 64) for s, p in ((2, 5), (9, 40), (64, 400))],
    "wave": [(c, s, p) for c in (65, 511, 512) for s, p in ((3, 7), (33, 600))],
    "block": [(c, s, p) for c in (513, 3072, 3073) for s, p in ((4, 11), (60, 3500))],
    "block_passes": [(12288, 64, 30000), (30000, 50, 39000), (131072, 400, 139000), (131072, 9, 30)],
    "hub": [(131073, 33, 39000), (150000, 31, 39000), (140000, 21, 25)],
    "last_before_hubs": [(12288, 31, 39000), (12289, 31, 39000)],
}


@pytest.mark.parametrize("case", sorted(VERTICES))
def test_layer_counts_at_class_edges(hy, case):
    print(f"[gpu] prep case={case}", flush=True)
    # hubs begin above 131072 occurrences on 6.3 million vertices or more
    n = {"block_passes": 6300000, "last_before_hubs": 150000}.get(case, 140000)
    rng = np.random.Generator(np.random.PCG64(sorted(VERTICES).index(case)))
    edges = []
    for i, (c, size, pool) in enumerate(VERTICES[case]):
        edges += _vertex(rng, 139500 + i, n, c, size, pool)
    edges += [[139500]] * 100   # singletons: more hyperedges than occurrences
    hg = hypergen.from_lists(n, [edges[i] for i in rng.permutation(len(edges))])
    g, o = hy.build_graph(n, hg.he_off, hg.he_mem, 1, 0.0), oracle.Graph(hg, 1, 0.0)
    info, st = g.stratify(), o.stratify()
    a, b = g.read(), o.arrays()
    for k in ("v_off", "v_he", "thr", "c"):
        assert np.array_equal(a[k], b[k]), k
    for i, (c, _, _) in enumerate(VERTICES[case]):
        assert a["c"][139500 + i] == c
    for k in ("l", "deg", "top", "stratum", "P"):
        assert np.array_equal(a[k], st[k]), k
    assert np.array_equal(info["B"], st["B"])


@pytest.mark.parametrize("d", [4096, 4097, 9000])
@pytest.mark.parametrize("duplicate", [False, True])
def test_long_segments(hy, d, duplicate):
    """A vertex in d hyperedges (and one beside it in more than 2048 words of
    marks); one hyperedge naming it twice is refused."""
    print(f"[gpu] long segments d={d} duplicate={duplicate}", flush=True)
    n, m = 500, 140000
    rng = np.random.Generator(np.random.PCG64(d))
    edges = [[int(x)] for x in rng.integers(2, n, size=m)]
    for v in (0, 1):
        for e in rng.choice(m, size=d, replace=False):
            edges[e] = edges[e] + [v]
    if duplicate:
        e = next(i for i in range(m - 1, -1, -1) if 1 in edges[i])
        edges[e] = edges[e] + [1]
    hg = hypergen.from_lists(n, edges)
    if duplicate:
        with pytest.raises(hy.HyperIMError) as err:
            hy.build_graph(n, hg.he_off, hg.he_mem, 0, 0.1)
        assert err.value.status == hy.EINVAL
        return
    g, o = hy.build_graph(n, hg.he_off, hg.he_mem, 0, 0.1), oracle.Graph(hg, 0, 0.1)
    a, b = g.read(strata=False), o.arrays()
    for k in ("v_off", "v_he", "thr", "c"):
        assert np.array_equal(a[k], b[k]), k


def _layers_of(co):
    """l, deg and top of a vertex with these co-member occurrences."""
    w = np.unique(co, return_counts=True)[1]
    return len(np.unique(w)), len(w), int((w == w.max()).sum())


def test_hubs_in_several_batches(hy):
    """Every vertex a hub and 1.4e9 occurrences together: more than one batch
    of hubs holds (2 GiB, two bytes each)."""
    print("[gpu] prep hub batches", flush=True)
    n = 24000
    half = n // 2
    rng = np.random.Generator(np.random.PCG64(3))
    edges = [rng.permutation(n), rng.permutation(n), rng.permutation(half), rng.permutation(half)]
    hg = hypergen.from_lists(n, [e.tolist() for e in edges])
    g = hy.build_graph(n, hg.he_off, hg.he_mem, 1, 0.0)
    g.stratify()
    a = g.read()
    first = np.arange(n) < half   # in four hyperedges: weight 4 inside the half, 2 outside
    assert np.array_equal(a["l"], np.where(first, 2, 1))
    assert np.array_equal(a["deg"], np.full(n, n - 1))
    assert np.array_equal(a["top"], np.where(first, half - 1, n - 1))


@pytest.mark.parametrize("n", [(1 << 24) - 1, (1 << 24) + 1, (1 << 24) + 40000])
def test_hubs_over_wide_ids(hy, n):
    """Ids on both sides of 2^24, the ids one pass over a hub's members takes."""
    print(f"[gpu] prep wide hub n={n}", flush=True)
    rng = np.random.Generator(np.random.PCG64(n))
    hub = n - 1
    edges = []
    for i in range(400):
        near = rng.integers(n - 3000, n - 1, size=200)   # weights up to dozens, at the far end of the ids
        m = np.unique(np.concatenate([near, rng.integers(0, n - 1, size=300)]))
        edges.append([hub] + m.tolist())
    hg = hypergen.from_lists(n, edges)
    co = np.concatenate([np.asarray(e[1:]) for e in edges])
    assert len(co) > 131072
    g = hy.build_graph(n, hg.he_off, hg.he_mem, 1, 0.0)
    g.stratify()
    a = g.read()
    assert a["c"][hub] == len(co)
    assert (a["l"][hub], a["deg"][hub], a["top"][hub]) == _layers_of(co)
