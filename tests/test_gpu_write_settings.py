"""The write pass under its settings (ESC_MAT_BLOCKS_PER_CU: fewer blocks, which
go on to further units; ESC_DENSE_SHIFT: another line between the two ways of
writing a unit), sparse, dense and mixed units; row ids and values bit
for bit against torch's own selection."""
import pytest

from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,value", [("ESC_MAT_BLOCKS_PER_CU", "1"), ("ESC_MAT_BLOCKS_PER_CU", "3"), ("ESC_DENSE_SHIFT", "0"),
                                        ("ESC_DENSE_SHIFT", "7"), ("ESC_DENSE_SHIFT", "12")])
@pytest.mark.parametrize("rows", [1, 2049, 70_001, 3_000_007])
def test_settings(monkeypatch, rows, name, value):
    import torch
    monkeypatch.setenv(name, value)
    ctx = esc.Context(0)
    monkeypatch.delenv(name)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    x = torch.randint(0, 1000, (rows,), generator=g, device="cuda", dtype=torch.int32)
    y = torch.randint(-2**31, 2**31 - 1, (rows,), generator=g, device="cuda", dtype=torch.int32)
    z = torch.arange(rows, device="cuda", dtype=torch.int32)
    dt = esc.Table(rows, [esc.INT32] * 3, [x, y, z])
    for spec, mask in ((("lt", 0, 1), x < 1), (("lt", 0, 100), x < 100), (("lt", 0, 126), x < 126), (("lt", 0, 700), x < 700),
                       (("gt", 0, -1), x > -1), (("or", [("lt", 0, 3), ("between", 2, 5000, 60_000)]), (x < 3) | ((z >= 5000) & (z <= 60_000)))):
        want = mask.nonzero()[:, 0].to(torch.int32)
        c = want.numel()
        ids = torch.full((c + 3,), -7, dtype=torch.int32, device="cuda")
        outs = [torch.full((c + 3,), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
        p = esc.Pred(dt, spec)
        assert ctx.count(dt, p) == c
        assert ctx.materialize(dt, p, [1, 2], ids, outs, c) == c
        assert torch.equal(ids[:c], want) and bool((ids[c:] == -7).all())
        for j, o in zip((1, 2), outs):
            assert torch.equal(o[:c], dt.cols[j][want.long()]) and bool((o[c:] == -7).all())
