"""The estimator's kernels at the edges of their row tiles (32 and 64 rows a
block; the switch between them at 64 rows per CU) and of the weight
gradient's runs of 16 k steps, against the CPU oracle with the same rounding."""
import numpy as np
import pytest

from oracle import mlp as om
from paper_1901_01488_amd import datagen as dg
from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    return esc.Context(0)


def _inputs(n, seed):
    rng = np.random.default_rng(seed)
    x = rng.random((n, 64)).astype(np.float32)
    x[rng.random((n, 64)) < 0.4] = 0.0
    return x, (-14.0 * rng.random(n) ** 2).astype(np.float32)


@pytest.mark.parametrize("off", [-1, 0, 1, 63, 65])
def test_forward_around_the_tile_switch(ctx, off):
    """Both row tilings round alike: outputs at and beyond the switch equal,
    bit for bit, those of the same rows in a small batch, which the oracle
    checks (float32 sums of 256 products of bfloat16 against float64: 1e-4
    of the outputs' scale, as a bfloat16 step in a hidden layer moves them)."""
    import torch
    n = 64 * ctx.num_cus() + off
    x, _ = _inputs(n, 3)
    params = dg.mlp_init(11)
    m = esc.MLP(ctx, params)
    xt = torch.from_numpy(x).cuda()
    y = m.predict(xt).cpu().numpy()
    pick = np.r_[0:40, n - 70:n]
    small = m.predict(torch.from_numpy(x[pick]).cuda()).cpu().numpy()
    assert np.array_equal(y[pick], small)
    want, _ = om.forward(params, x[pick])
    assert np.max(np.abs(small - want)) <= 2.0 ** -8 * np.max(np.abs(want))


@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 257, 513, 4095, 4096])
def test_gradients_at_tile_edges(ctx, n):
    """Relative to each block's largest gradient: bfloat16 roundings that fall
    the other way move single rows' terms by 2^-8 of themselves."""
    import torch
    x, y = _inputs(n, 100 + n)
    params = dg.mlp_init(12)
    m = esc.MLP(ctx, params)
    g = m.gradients(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()).cpu().numpy()
    yhat, acts = om.forward(params, x)
    want = om.backward(params, acts, yhat, y)
    for (gw, gb), (ww, wb) in zip(esc.flat_to_params(g), want):
        for a, b in ((gw, ww), (gb, wb)):
            b = np.asarray(b).reshape(a.shape)
            assert np.max(np.abs(a - b)) <= 2.0 ** -7 * np.max(np.abs(b)) + 1e-12
