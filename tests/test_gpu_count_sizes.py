"""Plain counts around the sizes where their launch changes: rows per lane of
8, 16 and 32 (fewer than two tiles a CU take fewer), every block's own host
word or one word for all, up to two blocks a CU at once or several tiles a
wave; short and long programs, with counts pending in the context's slots and
on a second stream; against torch's own masks."""
import numpy as np
import pytest

from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    return esc.Context(0)


def _edges():
    out = [1, 63, 64, 65, 511, 512, 513, 2047, 2049]
    for tiles in (255, 256, 257, 511, 512, 513):                 # one and two tiles a CU
        for rpt in (8, 16, 32):
            out += [tiles * 64 * rpt - 1, tiles * 64 * rpt, tiles * 64 * rpt + 1]
    for blocks in (512, 513):                                     # two blocks a CU
        for rpt in (16, 32):
            out += [blocks * 4 * 64 * rpt, blocks * 4 * 64 * rpt + 1]
    return sorted(set(out))


@pytest.mark.parametrize("part", range(4))
def test_counts_at_launch_edges(ctx, part):
    import torch
    rows = _edges()[part::4]
    top = max(rows)
    g = torch.Generator(device="cuda")
    g.manual_seed(part)
    full = [torch.randint(0, 1000, (top,), generator=g, device="cuda", dtype=torch.int32) for _ in range(4)]
    side = torch.cuda.Stream()
    for n in rows:
        a, b, c, d = (x[:n] for x in full)
        dt = esc.Table(n, [esc.INT32] * 4, [a, b, c, d])
        specs = [("lt", 0, 500),
                 ("and", [("gt", 0, 100), ("lt", 1, 700)]),
                 ("or", [("and", [("lt", 0, 300), ("gt", 1, 200), ("gt", 2, 5)]), ("between", 2, 10, 90),
                         ("and", [("gt", 2, 900), ("lt", 0, 650), ("gt", 1, 10)])]),
                 ("or", [("and", [("lt", 0, 300), ("gt", 1, 200)]), ("and", [("gt", 2, 900), ("lt", 3, 650)]),
                         ("between", 3, 10, 20)])]
        masks = [a < 500, (a > 100) & (b < 700),
                 ((a < 300) & (b > 200) & (c > 5)) | ((c >= 10) & (c <= 90)) | ((c > 900) & (a < 650) & (b > 10)),
                 ((a < 300) & (b > 200)) | ((c > 900) & (d < 650)) | ((d >= 10) & (d <= 20))]
        want = [int(m.sum()) for m in masks]
        preds = [esc.Pred(dt, s) for s in specs]
        ws = [ctx.workspace(dt, False, key=("sizes", k)) for k in range(3)]
        torch.cuda.synchronize()
        for k in (0, 1):
            ctx.count_begin(dt, preds[k], ws[k], slot=k, stream=side)
        got = [ctx.count(dt, p, ws=ws[2]) for p in preds]
        assert got == want, n
        assert [ctx.count(dt, p, ws=ws[2]) for p in reversed(preds)] == want[::-1], n
        assert [ctx.count_end(k) for k in (0, 1)] == want[:2], n
        out = torch.zeros(1, dtype=torch.int64, device="cuda")
        ctx.count_async(dt, preds[3], out, ws[0])
        assert int(out) == want[3], n
