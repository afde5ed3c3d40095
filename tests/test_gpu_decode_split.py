"""Decode attention over heads that are cut into segments: lengths at the edges of
blocks and segments, next to caches that stay whole or are empty, over whole caches
and over kept lists; a NaN key must reach the output from any segment."""

import numpy as np
import pytest

from oracle import decode_oracle as do
from test_gpu_decode import ATOL, RTOL, _setup

pytestmark = pytest.mark.gpu

# segments of 16 blocks here (a few heads on any chip): 256 tokens
LENS = [[511], [512], [513, 0, 1, 256, 257], [2049, 255, 700, 16, 4096], [32768, 5]]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens", LENS, ids=lambda v: str(v[0]))
def test_split_attention(lens, d):
    import torch
    from paper_2503_08461_amd import fastcache as fc
    s, wl = _setup(lens, d=d, n_heads=2, n_layers=1)
    try:
        rng = np.random.default_rng(3)
        q = rng.standard_normal((len(lens), 1, 2, d)).astype(np.float16)
        q_dev = torch.from_numpy(q).to(s.dev)
        got = fc.fc_decode_attention(s.pool, s.bt_dev, s.lens_g, q_dev).cpu().numpy()
        want = do.decode_attention(s.kv_host, s.bt_host, s.lens_o, q)
        assert (np.abs(got - want) <= RTOL * np.abs(want) + ATOL).all()
        # every token kept but every third
        keep = [[np.flatnonzero(np.arange(n) % 3 != 1) for _ in range(2)] for n in lens]
        budgets = np.array([k[0].size for k in keep], np.int32)
        kept = torch.from_numpy(np.concatenate([x for k in keep for x in k]).astype(np.int32)).to(s.dev)
        got = fc.fc_decode_attention_kept(s.pool, s.bt_dev, s.lens_g, budgets, kept, q_dev).cpu().numpy()
        want = do.decode_attention_kept(s.kv_host, s.bt_host, s.lens_o, [np.array(k).reshape(1, 2, -1) for k in keep], q)
        assert (np.abs(got - want) <= RTOL * np.abs(want) + ATOL).all()
    finally:
        s.close()


@pytest.mark.parametrize("at", [0, 255, 256, 1024])
def test_nan_key_reaches_the_output(at):
    import torch
    from paper_2503_08461_amd import fastcache as fc
    s, wl = _setup([1025, 1025], n_heads=1, n_layers=1)
    try:
        blk = int(s.bt_dev[1, at // 16])
        s.kv_dev[0, blk, 0, 0, at % 16, 3] = float("nan")
        q = torch.ones((2, 1, 1, 128), dtype=torch.float16, device=s.dev)
        got = fc.fc_decode_attention(s.pool, s.bt_dev, s.lens_g, q)
        assert torch.isnan(got[1]).all() and not torch.isnan(got[0]).any()
    finally:
        s.close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("blocks", [23, 24, 32, 39, 40, 41, 56, 57])
def test_even_segments(blocks, d):
    """Both sides of the block counts at which a head gets one segment more, next to a head
    of twice 16 blocks that makes the call cut: one to four segments of 16 to 23 blocks,
    whose wavefronts have an even or an odd number of blocks, down to one."""
    import torch
    from paper_2503_08461_amd import fastcache as fc
    lens = [blocks * 16 - 7, 512, 16 * blocks, 3]
    s, wl = _setup(lens, d=d, n_heads=2, n_layers=1)
    try:
        q = np.random.default_rng(blocks).standard_normal((len(lens), 1, 2, d)).astype(np.float16)
        got = fc.fc_decode_attention(s.pool, s.bt_dev, s.lens_g, torch.from_numpy(q).to(s.dev)).cpu().numpy()
        want = do.decode_attention(s.kv_host, s.bt_host, s.lens_o, q)
        assert (np.abs(got - want) <= RTOL * np.abs(want) + ATOL).all()
    finally:
        s.close()
