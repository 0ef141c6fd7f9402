"""Split selectivities by both ways that the conjunct programs reach the
kernel (one argument, or uploaded when they need more instructions, slot
tables or pool words than fit), with one to eight columns and 1 to 32 conjuncts, at the
edges of tiles, blocks and of the grid; against torch's own masks."""
import numpy as np
import pytest

from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    return esc.Context(0)


def _conjuncts(form, cols, rng):
    import torch

    def isin(c, keys):
        return ("in", c, keys), torch.isin(cols[c], torch.tensor(keys, device="cuda", dtype=torch.int32))

    def below(c, k):
        return ("lt", c, k), cols[c] < k

    if form == "ranges":
        return [below(c, int(rng.integers(200, 900))) for c in range(8)]
    if form == "tables":      # four bitmaps or hash tables, then lists and ranges
        return ([isin(c, [int(k) for k in rng.choice(1000, 30, replace=False)]) for c in range(4)] + [below(4, 700)])
    if form == "tables5":     # a fifth table: uploaded
        return [isin(c, [int(k) for k in rng.choice(1000, 30, replace=False)]) for c in range(5)] + [below(0, 500)]
    if form == "udf":
        return [(("udf", ("add", ("col", 0), ("col", 1)), ("gt", 600)), cols[0] + cols[1] > 600), below(1, 800),
                (("udf", ("mul", ("col", 2), ("const", 3)), ("lt", 2000)), cols[2] * 3 < 2000),
                isin(3, [int(k) for k in rng.choice(1000, 40, replace=False)])]
    if form == "thirtytwo":
        return [below(int(rng.integers(0, 8)), int(rng.integers(500, 1000))) for _ in range(32)]
    # 20 ORs of three: 60 instructions, nearly all that one argument holds
    out = []
    for _ in range(20):
        a, b, c = (int(x) for x in rng.choice(8, 3, replace=False))
        out.append((("or", [("lt", a, 400), ("gt", b, 450), ("between", c, 100, 300)]),
                    (cols[a] < 400) | (cols[b] > 450) | ((cols[c] >= 100) & (cols[c] <= 300))))
    return out


@pytest.mark.parametrize("form", ["ranges", "tables", "tables5", "udf", "thirtytwo", "many"])
@pytest.mark.parametrize("rows", [1, 1023, 1025, 4096, 4097, 512 * 4096 + 1, 2 * 512 * 4096 + 777])
def test_forms(ctx, rows, form):
    import torch
    rng = np.random.default_rng(rows + len(form))
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    cols = [torch.randint(0, 1000, (rows,), generator=g, device="cuda", dtype=torch.int32) for _ in range(8)]
    dt = esc.Table(rows, [esc.INT32] * 8, cols)
    parts = _conjuncts(form, cols, rng)
    conj = [int(m.sum()) for _, m in parts]
    prefix, run = [], torch.ones(rows, dtype=torch.bool, device="cuda")
    for _, m in parts:
        run &= m
        prefix.append(int(run.sum()))
    p = esc.Pred(dt, ("and", [s for s, _ in parts]))
    for _ in range(3):
        assert ctx.count_conjuncts(dt, p) == (conj, prefix)
    one = esc.Pred(dt, parts[0][0])
    assert ctx.count_conjuncts(dt, one) == (conj[:1], conj[:1])
