"""Materializations at the edges of the write pass: units of 1,024 rows, tiles
of 2,048 (up to six columns) and 1,024 rows, blocks of several tiles, the most
tiles for which every block finds its own offset and one more, every number of
projected columns, selections from nothing to everything, clustered and
spread, with a capacity below the count; row ids and values bit for bit
against torch's own selection of the same rows."""
import numpy as np
import pytest

from paper_1901_01488_amd import datagen as dg
from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu

OWN_PREFIX_TILES = 40960


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    return esc.Context(0)


def _check(ctx, dt, spec, mask, proj, capacity=None, count_first=False):
    import torch
    p = esc.Pred(dt, spec)
    want = mask.nonzero()[:, 0]
    c = want.numel()
    cap = c if capacity is None else capacity
    ids = torch.full((cap + 3,), -7, dtype=torch.int32, device="cuda")
    outs = [torch.full((cap + 3,), -7, dtype=torch.int32, device="cuda").view(dt.cols[j].dtype) for j in proj]
    if count_first:
        assert ctx.count(dt, p, ws=ctx.workspace(dt, True)) == c
    assert ctx.materialize(dt, p, proj, ids, outs, cap, allow_overflow=cap < c) == c
    k = min(c, cap)
    assert torch.equal(ids[:k], want[:k].to(torch.int32)) and bool((ids[k:] == -7).all())
    for j, o in zip(proj, outs):
        o = o.view(torch.int32)
        assert torch.equal(o[:k], dt.cols[j].view(torch.int32)[want[:k]]) and bool((o[k:] == -7).all())


@pytest.mark.parametrize("rows", [1, 63, 1023, 1024, 1025, 2047, 2048, 2049, 4097, 70_001, 1_048_577, 20_000_003])
def test_units_and_projections(ctx, rows):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    perm = torch.randperm(rows, generator=g, device="cuda").to(torch.int32)
    seq = torch.arange(rows, device="cuda", dtype=torch.int32)
    cols = [perm, seq] + [torch.randint(-2**31, 2**31 - 1, (rows,), generator=g, device="cuda", dtype=torch.int32)
                          for _ in range(5)]
    cols.append(torch.randn(rows, generator=g, device="cuda"))
    dt = esc.Table(rows, [esc.INT32] * 7 + [esc.FLOAT32], cols)
    rng = np.random.default_rng(rows)
    for nproj in range(9):
        proj = [int(j) for j in rng.permutation(8)[:nproj]]
        k = int(rows * rng.choice([0.0, 0.002, 0.05, 0.4, 1.0]))
        a = int(rng.integers(0, max(1, rows - k + 1)))
        _check(ctx, dt, ("lt", 0, k), perm < k, proj)                                            # spread
        _check(ctx, dt, ("between", 1, a, a + k), (seq >= a) & (seq <= a + k), proj, count_first=True)   # clustered
        _check(ctx, dt, ("lt", 0, rows), perm < rows, proj, capacity=rows // 3)
    # seven columns: tiles of 1,024 rows
    wide = ("and", [("lt", 0, rows // 2)] + [("gt", c, -2_000_000_000) for c in range(2, 7)] + [("gt", 7, np.float32(-1.5))])
    m = (perm < rows // 2) & (cols[7] > -1.5)
    for c in range(2, 7):
        m &= cols[c] > -2_000_000_000
    _check(ctx, dt, wide, m, [7, 0, 3, 2], count_first=rows % 2 == 0)


@pytest.mark.parametrize("tiles,extra", [(OWN_PREFIX_TILES, 0), (OWN_PREFIX_TILES, 1), (16384, 1)])
def test_offsets_by_blocks_and_by_scan(ctx, tiles, extra):
    import torch
    rows = tiles * 2048 + extra
    x = torch.arange(rows, device="cuda", dtype=torch.int32)
    x = (x * 1_103_515_245 + 12_345) % 1000   # int32 wrap-around: values spread over (-1000, 1000)
    dt = esc.Table(rows, [esc.INT32], [x])
    _check(ctx, dt, ("between", 0, 7, 11), (x >= 7) & (x <= 11), [0])
    _check(ctx, dt, ("lt", 0, 400), x < 400, [0], capacity=1_000_003, count_first=True)
