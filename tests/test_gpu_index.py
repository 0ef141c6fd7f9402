"""GPU counts through the predicate index (batches of several predicates on
one table) against the CPU oracle, at the edges of a wave tile (256 rows), a
block step (2,048 rows) and the 32-predicate result words, with ORs over
several columns and float columns that hold NaN, both zeros and infinities."""
import numpy as np
import pytest

from oracle import scan
from paper_1901_01488_amd import datagen as dg
from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    return esc.Context(0)


def _table(n):
    t = dg.table_mixed(n, 6, seed=77 + n, kinds=list(dg.LEARNED_KINDS))
    f = t.cols[5]
    edges = np.array([np.nan, -np.nan, 0.0, -0.0, np.inf, -np.inf, 1e-45, -1.0], np.float32)
    f[: min(n, 8)] = edges[: min(n, 8)]
    t.cols[1][n // 2:n // 2 + 2] = np.array([-2**31, 2**31 - 1], np.int32)[: max(0, min(2, n - n // 2))]
    return t


def _preds(t, count, seed):
    ps = dg.preds_mixed(t, count, seed=seed, max_conj=4, p_or=0.4)
    special = [("between", 5, np.float32(-0.0), np.float32(0.0)), ("lt", 5, np.float32(np.inf)),
               ("gt", 5, np.float32(-np.inf)), ("in", 5, [np.float32(0.0), np.float32(np.nan), np.float32(-1.0)]),
               ("between", 1, -2**31, 5), ("gt", 1, 2**31 - 2), ("or", [("eq", 1, 2**31 - 1), ("lt", 5, np.float32(0.5))])]
    for i, p in enumerate(special[: max(0, count - 1)]):
        ps[i] = p
    return ps


@pytest.mark.parametrize("rows", [1, 3, 255, 256, 257, 2047, 2049, 70_001])
@pytest.mark.parametrize("npreds", [4, 31, 33, 64, 65, 129])
def test_indexed_counts(ctx, rows, npreds):
    t = _table(rows)
    preds = _preds(t, npreds, seed=1000 * npreds + rows)
    dt = esc.device_table(t)
    cps = [esc.Pred(dt, p) for p in preds]
    want = [scan.count(t, p) for p in preds]
    b = esc.Batch(ctx, [dt], cps, [0] * npreds)
    for _ in range(3):   # the counters start from zero on every launch
        assert b.count().tolist() == want


def test_indexed_beside_interpreted(ctx):
    """One batch whose predicates take both kernels (udfs cannot be indexed),
    then an update that leaves nothing to the interpreter and one that
    leaves nothing to an index."""
    t = _table(300_007)
    dt = esc.device_table(t)
    udf = [("and", [("udf", ("mod", ("add", ("col", 1), ("col", 2)), ("const", 5 + i)), ("gt", 2)), ("gt", 1, 100 * i)])
           for i in range(6)]
    plain = _preds(t, 60, seed=5)
    for preds in (udf + plain, plain, udf, plain[:30] + udf):
        cps = [esc.Pred(dt, p) for p in preds]
        want = [scan.count(t, p) for p in preds]
        if preds is not None and len(preds) == 66:
            b = esc.Batch(ctx, [dt], cps, [0] * len(preds))
        else:
            b.update(cps, [0] * len(preds))
        assert b.count().tolist() == want


def test_flushes_within_an_item(ctx):
    """More rows per lane than the bit-sliced counters hold (1,020): one
    block's share of a large chunk is summed several times."""
    import torch
    n = 9_000_001
    x = torch.arange(n, device="cuda", dtype=torch.int32)
    y = (x % 1000).to(torch.int32)
    dt = esc.Table(n, [esc.INT32, esc.INT32], [x, y])
    preds = [("lt", 0, 250_000 * i + 1) for i in range(1, 33)] + [("between", 1, i, 999) for i in range(1, 33)]
    cps = [esc.Pred(dt, p) for p in preds]
    b = esc.Batch(ctx, [dt], cps, [0] * len(cps), chunk_rows=1 << 23)
    want = [min(n, 250_000 * i + 1) for i in range(1, 33)]
    want += [int((y >= i).sum().item()) for i in range(1, 33)]
    assert b.count().tolist() == want
