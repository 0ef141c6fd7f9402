"""Outputs with room for fewer than a 64th of the rows, and for just that many,
on tables whose write pass then takes fewer blocks than units: few rows, rows in
one place, more rows than the room; row ids and values bit for bit against
torch's own selection."""
import pytest

from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [26_000_003, 40_000_000])
def test_little_room(rows):
    import torch
    ctx = esc.Context(0)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    x = torch.randperm(rows, generator=g, device="cuda").to(torch.int32)
    z = torch.arange(rows, device="cuda", dtype=torch.int32)
    dt = esc.Table(rows, [esc.INT32] * 2, [x, z])
    edge = rows // 64
    for spec, mask in ((("lt", 0, 1000), x < 1000), (("between", 1, 7_000_001, 7_300_000), (z >= 7_000_001) & (z <= 7_300_000)),
                       (("lt", 0, rows // 2), x < rows // 2), (("eq", 1, rows - 1), z == rows - 1)):
        want = mask.nonzero()[:, 0].to(torch.int32)
        c = want.numel()
        p = esc.Pred(dt, spec)
        for cap in (edge - 1, edge, min(c, edge - 1)):
            k = min(c, cap)
            ids = torch.full((cap + 3,), -7, dtype=torch.int32, device="cuda")
            out = torch.full((cap + 3,), -7, dtype=torch.int32, device="cuda")
            assert ctx.materialize(dt, p, [0], ids, [out], cap, allow_overflow=True) == c
            assert torch.equal(ids[:k], want[:k]) and bool((ids[k:] == -7).all())
            assert torch.equal(out[:k], x[want[:k].long()]) and bool((out[k:] == -7).all())
