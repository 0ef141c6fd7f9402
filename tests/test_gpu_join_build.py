"""Which of the two build kernels inserts a table's keys is said once, in the
table's header: key sets on both sides of the rule and at its edges (keys,
values of their range in 2^20-bit parts up to one for every CU and one more),
each key inserted exactly once; against torch's own counts."""
import pytest

from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu

PARTS_WORD = 6   # of the header


def _pays(n, span, cus):
    parts = (span >> 20) + 1
    return n >= 1 << 20 and parts <= cus and n / 25000.0 > 30.0 + n // (cus // parts) * 150e-6


@pytest.mark.parametrize("n,span", [(1_048_575, 1 << 21), (1_048_576, 1 << 21), (1_048_576, (1 << 24) - 1),
                                    (1_048_576, 1 << 26), (1_500_000, 100_000_000), (3_000_001, (1 << 28) - 1),
                                    (4_194_304, 1 << 28)])
def test_one_kernel_inserts(n, span):
    import ctypes
    import torch
    ctx = esc.Context(0)
    cus = ctypes.c_int()
    esc.check(esc.lib().esc_ctx_num_cus(ctx.h, ctypes.byref(cus)))
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    keys = (torch.randperm(span + 1, generator=g, device="cuda")[:n].to(torch.int64) - span // 3).to(torch.int32)
    keys[0], keys[1] = -(span // 3), span - span // 3
    keys = torch.unique(keys)
    keys = keys[torch.randperm(len(keys), generator=g, device="cuda")]
    if n % 2 == 0:   # a few keys of several rows
        keys = torch.cat([keys, keys[:1001], keys[:5]])
    tab = ctx.hash_table(keys)
    parts = int(tab[:64].view(torch.int32)[PARTS_WORD])
    # a bitmap, unless the range is beyond 32 values a slot
    if _pays(keys.numel(), span, cus.value):
        assert parts == (span >> 20) + 1
    else:
        assert parts == 0
    # every key once, as often as it has rows, and its neighbours
    probe = torch.cat([keys[:200_000], keys[-200_000:], keys[:100_000] + 1])
    k64, order = torch.sort(keys.to(torch.int64))
    p64 = probe.to(torch.int64)
    want = int((torch.searchsorted(k64, p64, right=True) - torch.searchsorted(k64, p64)).sum())
    t = esc.Table(probe.numel(), [esc.INT32], [probe.contiguous()])
    assert ctx.join_count(t, [0], [tab]) == want
