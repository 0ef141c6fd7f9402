"""Materializations of many rows of a unit: densities around the eighth from
which a unit goes out in 16-byte groups and up to every row, spread and
clustered, outputs that begin at each word of a group, capacities that end
inside a run, tables that end inside a unit, no to eight projected columns;
row ids and values bit for bit against torch's own selection, and nothing
written beside them."""
import numpy as np
import pytest

from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    return esc.Context(0)


@pytest.mark.parametrize("rows", [1024, 2048, 2049, 4095, 4096, 4097, 6143, 300_000, 4_194_305])
def test_dense_units(ctx, rows):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    key = torch.randint(0, 1024, (rows,), generator=g, device="cuda", dtype=torch.int32)
    seq = torch.arange(rows, device="cuda", dtype=torch.int32)
    cols = [key, seq] + [torch.randint(-2**31, 2**31 - 1, (rows,), generator=g, device="cuda", dtype=torch.int32)
                         for _ in range(6)]
    dt = esc.Table(rows, [esc.INT32] * 8, cols)
    rng = np.random.default_rng(rows)
    cases = [(("lt", 0, k), key < k) for k in (100, 125, 128, 131, 256, 700, 1000, 1024)]
    a = int(rng.integers(0, rows // 2))
    cases.append((("between", 1, a, a + rows // 3), (seq >= a) & (seq <= a + rows // 3)))
    cases.append((("gt", 1, -1), seq >= 0))
    for i, (spec, mask) in enumerate(cases):
        want = mask.nonzero()[:, 0]
        c = want.numel()
        for shift in range(4):
            nproj = (2 * i + shift) % 9
            proj = [int(j) for j in rng.permutation(8)[:nproj]]
            cap = c if shift % 2 == 0 else max(0, c - 1 - int(rng.integers(0, c // 2 + 1)))
            full = [torch.full((cap + 9,), -7, dtype=torch.int32, device="cuda") for _ in range(nproj + 1)]
            at = [(shift + q) % 4 for q in range(nproj + 1)]   # words before each output
            p = esc.Pred(dt, spec)
            assert ctx.materialize(dt, p, proj, full[-1][at[-1]:], [f[o:] for f, o in zip(full, at)][:nproj], cap,
                                   allow_overflow=cap < c) == c
            k = min(c, cap)
            for f, o, v in zip(full, at, [dt.cols[j][want[:k]] for j in proj] + [want[:k].to(torch.int32)]):
                assert torch.equal(f[o:o + k], v), (spec, shift)
                assert bool((f[:o] == -7).all()) and bool((f[o + k:] == -7).all()), (spec, shift)
