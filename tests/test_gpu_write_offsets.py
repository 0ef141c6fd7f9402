"""Materializations of as many tiles as find their own offsets, of one fewer
and one more (those take the scan's), in tiles of 2,048 rows and of 1,024
(seven columns), after a count and without one, with a capacity below the
count; row ids and values bit for bit against torch's own selection."""
import pytest

from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu

OWN_PREFIX_TILES = 12288


def _check(ctx, dt, spec, mask, proj, capacity, count_first):
    import torch
    want = mask.nonzero()[:, 0].to(torch.int32)
    c = want.numel()
    k = min(c, capacity)
    ids = torch.full((capacity + 3,), -7, dtype=torch.int32, device="cuda")
    outs = [torch.full((capacity + 3,), -7, dtype=torch.int32, device="cuda") for _ in proj]
    p = esc.Pred(dt, spec)
    if count_first:
        assert ctx.count(dt, p, ws=ctx.workspace(dt, True)) == c
    assert ctx.materialize(dt, p, proj, ids, outs, capacity, allow_overflow=True) == c
    assert torch.equal(ids[:k], want[:k]) and bool((ids[k:] == -7).all())
    for j, o in zip(proj, outs):
        assert torch.equal(o[:k], dt.cols[j][want[:k].long()]) and bool((o[k:] == -7).all())


@pytest.mark.parametrize("tiles,extra", [(OWN_PREFIX_TILES - 1, 1000), (OWN_PREFIX_TILES, 0), (OWN_PREFIX_TILES, 1),
                                         (OWN_PREFIX_TILES, 1025), (OWN_PREFIX_TILES + 3, 1)])
@pytest.mark.parametrize("wide", [False, True])
def test_offsets(tiles, extra, wide):
    import torch
    rows = tiles * (1024 if wide else 2048) + extra
    ctx = esc.Context(0)
    x = (torch.arange(rows, device="cuda", dtype=torch.int32) * 1_103_515_245 + 12_345) % 1000
    ncols = 7 if wide else 1
    cols = [x] + [x + c for c in range(1, ncols)]
    dt = esc.Table(rows, [esc.INT32] * ncols, cols)
    for k in (-990, 100, 800):
        spec = ("and", [("lt", 0, k)] + [("gt", c, -5000) for c in range(1, ncols)]) if wide else ("lt", 0, k)
        mask = x < k
        c = int(mask.sum())
        for capacity in (c, c // 2 + 1):
            for count_first in (False, True):
                _check(ctx, dt, spec, mask, [0] if not wide else [3, 0], capacity, count_first)
