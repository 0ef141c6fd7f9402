"""Batches whose indexes are large beside their predicates' programs: updates
from short ranges to IN-lists of many constants, in batches of few predicates,
and lists that are cut into several groups by their ORs; against the oracle."""
import numpy as np
import pytest

from oracle import scan
from paper_1901_01488_amd import datagen as dg
from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


def test_update_to_large_indexes():
    ctx = esc.Context(0)
    ts = [dg.table_mixed(n, 6, seed=n, kinds=list(dg.LEARNED_KINDS)) for n in (5_003, 100_001)]
    dts = [esc.device_table(t) for t in ts]
    owner = [0] * 4 + [1] * 4
    short = [("lt", 1, 10 * i) for i in range(8)]

    def lists(seed):
        r = np.random.default_rng(seed)
        return [("and", [("in", c, [int(v) for v in r.choice(ts[owner[i]].cols[c], 60)]) for c in (1, 2, 3)] +
                 [("gt", 0, int(r.integers(0, 500)))]) for i in range(8)]

    b = esc.Batch(ctx, dts, [esc.Pred(dts[o], p) for o, p in zip(owner, short)], owner)
    for preds in (short, lists(1), lists(2), short, lists(3)):
        b.update([esc.Pred(dts[o], p) for o, p in zip(owner, preds)], owner)
        want = [scan.count(ts[o], p) for o, p in zip(owner, preds)]
        for _ in range(2):
            assert b.count().tolist() == want


@pytest.mark.parametrize("npreds", [33, 40, 63, 64, 100])
def test_groups_cut_by_their_ors(npreds):
    ctx = esc.Context(0)
    t = dg.table_mixed(30_011, 6, seed=9, kinds=list(dg.LEARNED_KINDS))
    dt = esc.device_table(t)
    rng = np.random.default_rng(npreds)
    q = [np.sort(np.asarray(t.cols[c])) for c in range(4)]
    preds = [("and", [("or", [("lt", i, q[i][int(rng.integers(0, 30_011))].item()),
                              ("gt", (i + 1) % 4, q[(i + 1) % 4][int(rng.integers(0, 30_011))].item())])
                      for i in range(4)]) for _ in range(npreds)]
    b = esc.Batch(ctx, [dt], [esc.Pred(dt, p) for p in preds], [0] * npreds)
    assert b.count().tolist() == [scan.count(t, p) for p in preds]
