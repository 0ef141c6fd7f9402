"""The estimator's inference around 96, 128 and 160 rows for every CU, where
blocks of 32 and 64 rows take turns: outputs equal, bit for bit, those of the same rows
in a small batch."""
import numpy as np
import pytest

from paper_1901_01488_amd import datagen as dg
from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [96, 128, 160])
@pytest.mark.parametrize("off", [-33, 0, 1, 65])
def test_forward_around_the_switches(rows, off):
    import torch
    ctx = esc.Context(0)
    n = rows * ctx.num_cus() + off
    x = torch.rand((n, 64), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    m = esc.MLP(ctx, dg.mlp_init(11))
    y = m.predict(x)
    for a in (0, n // 2, n - 40):
        assert torch.equal(y[a:a + 40], m.predict(x[a:a + 40].contiguous()))
    assert np.isfinite(y.cpu().numpy()).all()
