"""GPU star-join counts over every form a hash table takes (bitmap, bitmap with
repeated keys, counts, hash, hash with repeated keys), against the CPU oracle,
at the edges between the forms and of the build's two range passes."""
import numpy as np
import pytest

from oracle import join as oj
from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu

LO, HI = -2**31, 2**31 - 1


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    return esc.Context(0)


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def _slots(n):
    s = 64
    while s < 2 * n:
        s *= 2
    return s


def _dense(rng, n, span, base=0):
    """n distinct keys whose extremes are `span` apart."""
    pool = rng.choice(span + 1, n, replace=False).astype(np.int64)
    pool[0] = 0
    if n > 1:
        pool[1] = span
    pool = np.unique(pool)
    return (pool + base).astype(np.int64)


def _builds(rng):
    yield "one key", np.array([5])
    yield "the key that marks empty slots", np.array([LO])
    yield "extremes", np.array([LO, HI, LO, 0, -1, HI, HI])
    yield "empty marker among spread keys", np.concatenate([rng.integers(LO, HI, 3000), [LO] * 3])
    for n in (31, 1000, 40_000):
        s = _slots(n)
        # the widest range a bitmap takes, and one value more (hash)
        yield "bitmap at its limit", _dense(rng, n, 32 * s - 1, -7)
        yield "hash just beyond", _dense(rng, n, 32 * s, -7)
        d = _dense(rng, n - n // 3, 2 * n, LO)
        yield "bitmap, repeated keys", np.concatenate([d, rng.choice(d, n // 3), np.repeat(d[:1], 40)])
        yield "as many keys as values", np.concatenate([np.arange(n - 1), [0]])
        yield "counts", rng.integers(0, max(1, n // 4), n) + HI - n
        h = rng.integers(LO, HI + 1, n)
        yield "hash", h
        yield "hash, repeated keys", np.concatenate([h, rng.choice(h, n // 2), np.repeat(h[:1], 70)])
    for n in (262_143, 262_144, 262_145, 400_001):
        yield "range passes", _dense(rng, n, 3 * n, 11)


@pytest.mark.parametrize("n", [1_048_575, 1_048_576, 1_600_003])
def test_bitmap_built_in_parts(ctx, n):
    """Dense keys in numbers from which the bitmap is built part by part, with
    rows of one key in one slice of the keys and in several, and a probe long
    enough for a filter of the first side."""
    rng = np.random.default_rng(n)
    span = 9 * n // 2   # no whole number of 2^20-bit parts
    for repeated in (False, True):
        keys = _dense(rng, n - (2003 if repeated else 0), span, -1_000_000).astype(np.int32)
        rng.shuffle(keys)
        if repeated:
            keys = np.concatenate([np.repeat(keys[:1], 1001), keys, rng.choice(keys, 1002)])
        probe = rng.integers(-1_000_100, span - 999_000, 5_000_011).astype(np.int32)
        small = rng.permutation(3000)[:700].astype(np.int32)
        spread = rng.choice(np.arange(LO, HI, 65_537), 500, replace=False).astype(np.int32)
        other = rng.integers(-5, 3005, len(probe)).astype(np.int32)
        third = np.where(rng.random(len(probe)) < 0.5, rng.choice(spread, len(probe)), 17).astype(np.int32)
        tabs = [ctx.hash_table(_dev(b)) for b in (keys, small, spread)]
        for cols, sides, refs in (([probe], [0], [keys]), ([other, probe], [1, 0], [small, keys]),
                                  ([third, probe, other], [2, 0, 1], [spread, keys, small])):
            t = esc.Table(len(probe), [esc.INT32] * len(cols), [_dev(c) for c in cols])
            got = ctx.join_count(t, list(range(len(cols))), [tabs[j] for j in sides])
            assert got == oj.count(cols, refs), (repeated, sides)


def test_every_form(ctx):
    rng = np.random.default_rng(5)
    for name, keys in _builds(rng):
        keys = np.asarray(keys, np.int64).astype(np.int32)
        k64 = keys.astype(np.int64)
        near = np.concatenate([k64, k64 + 1, k64 - 1, [k64.min() - 1, k64.max() + 1, LO, HI, 0]])
        near = near[(near >= LO) & (near <= HI)]
        for nprobe in (511, 60_003):
            probe = rng.choice(near, nprobe).astype(np.int32)
            t = esc.Table(nprobe, [esc.INT32], [_dev(probe)])
            assert ctx.join_count(t, [0], [ctx.hash_table(_dev(keys))]) == oj.count([probe], [keys]), (name, len(keys))


@pytest.mark.parametrize("k", [2, 3, 4])
def test_forms_together(ctx, k):
    """Sides of different forms in one join, with and without repeated keys."""
    rng = np.random.default_rng(20 + k)
    n = 20_011
    for repeated in (False, True):
        sides = [rng.permutation(4000)[:900], rng.choice(np.arange(LO, HI, 65_537), 3000, replace=False),
                 rng.permutation(64) - 32, rng.choice(np.arange(LO, HI, 99_991), 64, replace=False)][:k]
        if repeated:
            sides[0] = np.concatenate([sides[0], sides[0][:50], sides[0][:7]])
            sides[1] = np.concatenate([sides[1], sides[1][:60]])
            if k > 2:
                sides[2] = rng.integers(-5, 5, 500)
        builds = [np.asarray(s, np.int64).astype(np.int32) for s in sides]
        probe = [np.where(rng.random(n) < 0.7, rng.choice(b, n), rng.integers(LO, HI, n)).astype(np.int32) for b in builds]
        t = esc.Table(n, [esc.INT32] * k, [_dev(p) for p in probe])
        tabs = [ctx.hash_table(_dev(b)) for b in builds]
        assert ctx.join_count(t, list(range(k)), tabs) == oj.count(probe, builds)


def test_rebuild_in_another_form(ctx):
    """A table rebuilt in place with keys of another form forgets the old ones."""
    import ctypes
    rng = np.random.default_rng(9)
    n = 5000
    probe = np.concatenate([np.arange(-100, 12_000), rng.integers(LO, HI, 5000)]).astype(np.int32)
    t = esc.Table(len(probe), [esc.INT32], [_dev(probe)])
    forms = [rng.permutation(10_000)[:n], rng.integers(LO, HI, n), rng.integers(0, 700, n),
             np.concatenate([np.arange(n - 10), np.arange(10)])]
    tab = ctx.hash_table(_dev(forms[0]))
    for a in (0, 1, 2, 3, 1, 0, 2, 0):
        keys = np.asarray(forms[a], np.int64).astype(np.int32)
        d = _dev(keys)
        esc.check(esc.lib().esc_hash_build(ctx.h, ctypes.c_void_p(d.data_ptr()), n, ctypes.c_void_p(tab.data_ptr()),
                                           tab.numel(), None))
        assert ctx.join_count(t, [0], [tab]) == oj.count([probe], [keys]), a


def test_build_under_capture(ctx):
    """Builds captured into a graph and replayed on changed keys, with eager
    work between the replays."""
    import torch
    rng = np.random.default_rng(3)
    n = 1_200_000
    sets = [rng.permutation(4 * n)[:n], rng.integers(LO, HI, n), rng.integers(0, n // 3, n)]
    sets = [np.asarray(k, np.int64).astype(np.int32) for k in sets]
    probe = np.concatenate([rng.choice(k, 40_000) for k in sets] + [rng.integers(LO, HI, 40_000)]).astype(np.int32)
    t = esc.Table(len(probe), [esc.INT32], [_dev(probe)])
    keys = _dev(sets[0])
    tab = ctx.hash_table(keys)
    import ctypes
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        esc.check(esc.lib().esc_hash_build(ctx.h, ctypes.c_void_p(keys.data_ptr()), n, ctypes.c_void_p(tab.data_ptr()),
                                           tab.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    for a in (0, 1, 2, 1, 0):
        keys.copy_(_dev(sets[a]))
        g.replay()
        torch.zeros(1 << 20, device="cuda").add_(1)
        assert ctx.join_count(t, [0], [tab]) == oj.count([probe], [sets[a]]), a
