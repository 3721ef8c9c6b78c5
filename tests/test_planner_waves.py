"""A planning wave's share of a superstep, on the CPU: several batches of 64
frontier entries per reservation, chunks by members as well as incidences, and
what happens when the item buffer is full.  Supersteps are run over the host
model until every entry is planned; each live entry's incidences must come up
exactly once, in items of bounded weight, and every superstep that starts with
an empty buffer must get on."""
import ctypes as C
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2406_01911_amd", "libhyperim.so")
CAP = 1 << 22
SKIP = 0xFFFFFFFF


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2406_01911_amd import build
        build.build()
    import torch  # noqa: F401  (binds the HIP runtime first, as the binding does)
    L = C.CDLL(LIB)
    vp = C.c_void_p
    L.hyperim_model_plan_wave.argtypes = [C.c_uint32, C.c_uint32, vp, vp, vp, vp, vp, C.c_uint32, C.c_uint32,
                                          C.c_uint32, vp, C.POINTER(C.c_uint64), C.POINTER(C.c_uint32)]
    return L


class Frontier:
    """Entries of one set (mode 0) or of a level (mode 1), all still to plan."""

    def __init__(self, deg, quads=None, sets=None, expanded=None):
        n = len(deg)
        self.deg = np.ascontiguousarray(deg, np.uint32)
        self.quads = np.ascontiguousarray(deg if quads is None else quads, np.uint32)
        self.sets = np.ascontiguousarray(np.ones(n) if sets is None else sets, np.uint32)
        self.done = np.ascontiguousarray(np.zeros(n) if expanded is None else expanded, np.uint8)
        self.e0 = (np.arange(n, dtype=np.uint64) * 1000 % (1 << 20)).astype(np.uint32)
        self.head = 0
        self.marks = np.zeros((n + 63) // 64, np.uint8)
        self.covered = [[] for _ in range(n)]   # ranges of incidences per entry

    def left(self, mode):
        return self.head < len(self.deg) if mode == 0 else not self.marks.all()


def plan(lib, mode, f, items, counter, chunk, seg, cap):
    h = f.head if mode == 0 else 0
    taken = C.c_uint32(0)
    deg, quads, e0, sets = (np.ascontiguousarray(x[h:]) for x in (f.deg, f.quads, f.e0, f.sets))
    marks = np.ascontiguousarray(f.done[h:]) if mode == 0 else f.marks
    rc = lib.hyperim_model_plan_wave(mode, len(deg), deg.ctypes.data, quads.ctypes.data, e0.ctypes.data,
                                     sets.ctypes.data, marks.ctypes.data, chunk, seg, cap, items.ctypes.data,
                                     C.byref(counter), C.byref(taken))
    assert rc == 0
    if mode == 0:
        f.head += taken.value
    return h, taken.value


def chunk_of(mode, f, i, chunk):
    """Length of entry i's chunks and whether it is cut, from the rule."""
    d, q, s = int(f.deg[i]), int(f.quads[i]), int(f.sets[i])
    if mode == 0:
        c = chunk if q <= 8 * d else max(1, chunk * 8 * d // q)
        return max(c, -(-d // (1 << 20))), d > c
    c = max(1, chunk // max(s, 1), -(-d // (CAP // 128)))
    return c, d > c


def weight(mode, f, i, chunk):
    if (mode == 0 and f.done[i]) or chunk_of(mode, f, i, chunk)[1]:
        return 0
    return max(int(f.deg[i]), -(-int(f.quads[i]) // 8)) if mode == 0 else int(f.deg[i]) * int(f.sets[i])


def run(lib, mode, fs, chunk, seg, cap=CAP, most=10000):
    seg = max(seg, chunk)
    items = np.zeros((cap, 4), np.uint32)
    steps = 0
    while any(f.left(mode) for f in fs):
        steps += 1
        assert steps <= most
        counter, progress = C.c_uint64(0), 0
        for f in fs:
            if not f.left(mode):
                continue
            at = min(counter.value, cap)
            items[at:] = 0x7FFFFFFF   # unwritten
            h, taken = plan(lib, mode, f, items, counter, chunk, seg, cap)
            progress += taken
            for x, a, b, _ in items[at:min(counter.value, cap)]:
                assert x != 0x7FFFFFFF
                if x == SKIP:
                    continue
                if x & 0x80000000:
                    i = h + int(x & 0x7FFFFFFF)
                    length, cut = chunk_of(mode, f, i, chunk)
                    assert cut and 0 < b - a <= length
                    f.covered[i].append((int(a), int(b)))
                else:
                    i0 = h + int(x)
                    assert 1 <= a <= 64
                    ws = [weight(mode, f, i, chunk) for i in range(i0, i0 + int(a))]
                    last = max((k for k, w in enumerate(ws) if w), default=0)
                    assert sum(ws[:last]) < seg
                    for i in range(i0, i0 + int(a)):
                        if weight(mode, f, i, chunk):
                            f.covered[i].append((int(f.e0[i]), int(f.e0[i]) + int(f.deg[i])))
        assert progress > 0
    for f in fs:
        for i, rs in enumerate(f.covered):
            want = [] if (mode == 0 and f.done[i]) or f.deg[i] == 0 else [(int(f.e0[i]), int(f.e0[i]) + int(f.deg[i]))]
            if want:
                rs.sort()
                assert all(p[1] == q[0] for p, q in zip(rs, rs[1:])), i
                assert [(rs[0][0], rs[-1][1])] == want, i
            else:
                assert rs == [], i
    return steps


def frontiers(rng, mode, count, chunk, n_max):
    out = []
    for _ in range(count):
        n = int(rng.integers(1, n_max))
        kind = rng.integers(0, 5, n)
        deg = np.select([kind == 0, kind == 1, kind == 2], [np.zeros(n), rng.integers(1, chunk + 1, n),
                                                            rng.integers(1, 4, n)],
                        rng.integers(chunk, 6 * chunk, n))
        long = rng.integers(1, 400, n)   # runs per incidence: hyperedges of up to 1600 members
        quads = np.where(kind == 4, deg * long, deg + rng.integers(0, 8, n) * deg)
        out.append(Frontier(deg, quads, rng.integers(1, 65, n), rng.random(n) < 0.3 if mode == 0 else None))
    return out


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("chunk,seg", [(1, 1), (16, 64), (256, 512), (1024, 16)])
def test_every_incidence_is_planned_once(lib, mode, chunk, seg):
    rng = np.random.default_rng(1000 * mode + chunk)
    for _ in range(6):
        assert run(lib, mode, frontiers(rng, mode, 5, chunk, 1500 if chunk < 1024 else 700), chunk, seg) == 1


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("cap", [160, 700, 5000])
def test_full_item_buffer(lib, mode, cap):
    # reservations for eight batches, for one, for one entry (mode 0), and none at all
    rng = np.random.default_rng(7 + cap)
    chunk = 16 if mode == 0 else 512
    fs = frontiers(rng, mode, 6, chunk, 1200)
    if mode == 1:   # a batch has to fit by itself: at most 64 chunks and 64 segments
        for f in fs:
            f.sets[:] = 1
            f.deg = np.minimum(f.deg, chunk).astype(np.uint32)
            f.deg[::64] = 30 * chunk
    else:           # and an entry: at most cap - 1 chunks
        for f in fs:
            big = f.quads > 8 * (cap - 2) * chunk
            f.quads[big] = f.deg[big]
    steps = run(lib, mode, fs, chunk, 64, cap)
    assert steps > 1 or cap == 5000


def test_long_hyperedges(lib):
    # one incidence in a hyperedge of a million members: light, heavier than any
    # segment; two of them: a chunk each
    f = Frontier([1, 1, 2, 5, 1], quads=[250000, 1, 500000, 5, 250000])
    assert [weight(0, f, i, 256) for i in range(5)] == [31250, 1, 0, 5, 31250]
    assert run(lib, 0, [f], 256, 512) == 1
    assert [len(r) for r in f.covered] == [1, 1, 2, 1, 1]


def test_arguments(lib):
    z = np.zeros(64, np.uint32)
    b = np.zeros(64, np.uint8)
    c, t = C.c_uint64(0), C.c_uint32(0)
    p = z.ctypes.data
    assert lib.hyperim_model_plan_wave(2, 1, p, p, p, p, b.ctypes.data, 1, 1, 4, p, C.byref(c), C.byref(t)) == -1
    assert lib.hyperim_model_plan_wave(0, 1, p, None, p, p, b.ctypes.data, 1, 1, 4, p, C.byref(c), C.byref(t)) == -1
    assert lib.hyperim_model_plan_wave(0, 1, p, p, p, p, b.ctypes.data, 0, 1, 4, p, C.byref(c), C.byref(t)) == -1
