"""Hash tables that begin at a multiple of 8 bytes but not of 16, in each form;
keys that begin at each multiple of 4; nothing written beside the table."""
import numpy as np
import pytest

from oracle import join as oj
from paper_1901_01488_amd import esc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 8, 24])
def test_table_offsets(offset):
    import ctypes
    import torch
    ctx = esc.Context(0)
    rng = np.random.default_rng(offset)
    probe = np.concatenate([np.arange(-50, 9_000), rng.integers(-2**31, 2**31, 3000)]).astype(np.int32)
    t = esc.Table(len(probe), [esc.INT32], [torch.from_numpy(probe).cuda()])
    spread = rng.integers(-2**31, 2**31, 2000)
    for i, keys in enumerate((rng.permutation(8000)[:3000], np.concatenate([rng.permutation(8000)[:3000], np.arange(900)]),
                              rng.integers(0, 500, 4001), spread, np.concatenate([spread, spread[:70], spread[:9]]),
                              np.array([7]), np.array([], np.int64))):
        keys = keys.astype(np.int32)
        word = i % 4
        d = torch.zeros(len(keys) + 4, dtype=torch.int32, device="cuda")
        d[word:word + len(keys)] = torch.from_numpy(keys).cuda()
        nb = ctypes.c_size_t()
        esc.check(esc.lib().esc_hash_table_bytes(len(keys), ctypes.byref(nb)))
        room = torch.full((nb.value + 64,), 0x5A, dtype=torch.uint8, device="cuda")
        tab = room[offset:offset + nb.value]
        assert tab.data_ptr() % 16 == offset % 16
        esc.check(esc.lib().esc_hash_build(ctx.h, ctypes.c_void_p(d.data_ptr() + 4 * word), len(keys),
                                           ctypes.c_void_p(tab.data_ptr()), nb.value, None))
        assert ctx.join_count(t, [0], [tab]) == oj.count([probe], [keys]), i
        assert bool((room[:offset] == 0x5A).all()) and bool((room[offset + nb.value:] == 0x5A).all())
