"""Descriptors as kernel arguments: calls whose descriptors just fit one launch's
arguments, just do not, need several launches, and go through pinned memory, one
after the other on the same pool (each may only see its own)."""

import numpy as np
import pytest

from oracle import decode_oracle as do
from oracle import fastcache_oracle as fo
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_req", [1, 34, 35, 36, 37, 107, 108, 143, 144, 300])
def test_compression(n_req):
    """96 bytes a request and 4 per entry of a work list: 35 requests fill 3584 bytes, 107 three times as much."""
    from parity_util import SideBySide
    lens = [17 + (37 * i) % 90 for i in range(n_req)]
    methods = [(fo.METHOD_SNAPKV, fo.METHOD_KNORM, fo.METHOD_STREAMING)[i % 3] for i in range(n_req)]
    s = SideBySide(_custom(lens, [max(16, n // 2) for n in lens], methods, W=16, d=64, n_heads=1))
    try:
        s.compress_and_compare()
        # again, with the shorter caches and fewer of them taking part
        methods = np.array([m if i % 2 else fo.METHOD_NONE for i, m in enumerate(methods)], np.int32)
        s.compress_and_compare(methods, np.full(n_req, 16, np.int32))
    finally:
        s.close()


@pytest.mark.parametrize("n_req", [1, 112, 113, 148, 149, 150, 460, 640])
def test_decode_step(n_req):
    """24 bytes a request: 149 fill the arguments of the kernels themselves (3584 bytes), more go
    through pinned memory."""
    import torch
    from paper_2503_08461_amd import fastcache as fc
    from test_gpu_decode import ATOL, RTOL, _setup
    lens = [(29 * i) % 70 for i in range(n_req)]
    s, wl = _setup(lens, d=64, n_heads=1, n_layers=1, spare=n_req)
    try:
        rng = np.random.default_rng(4)
        for _ in range(2):
            new = rng.standard_normal((n_req, 1, 2, 1, 64)).astype(np.float16)
            fc.fc_append_batch(s.pool, s.bt_dev, s.lens_g, torch.from_numpy(new).to(s.dev))
            q = rng.standard_normal((n_req, 1, 1, 64)).astype(np.float16)
            got = fc.fc_decode_attention(s.pool, s.bt_dev, s.lens_g, torch.from_numpy(q).to(s.dev)).cpu().numpy()
            assert do.append_batch(s.kv_host, s.stack, s.bt_host, s.lens_o, new, np.ones(n_req, np.int32)) is None
            want = do.decode_attention(s.kv_host, s.bt_host, s.lens_o, q)
            assert (np.abs(got - want) <= RTOL * np.abs(want) + ATOL).all()
        torch.cuda.synchronize()
        s.compare_state()
    finally:
        s.close()


@pytest.mark.parametrize("n_req", [149, 200])
def test_captured_decode_step(n_req):
    """Every replay works on the requests of the capture, whatever other steps did in between."""
    import torch
    from paper_2503_08461_amd import fastcache as fc
    from test_gpu_decode import _setup
    lens = [(29 * i) % 70 + 1 for i in range(n_req)]
    s, wl = _setup(lens, d=64, n_heads=1, n_layers=1, spare=n_req)
    try:
        q = torch.randn((n_req, 1, 1, 64), device=s.dev).half()
        want = fc.fc_decode_attention(s.pool, s.bt_dev, s.lens_g, q).clone()
        out = torch.zeros_like(want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fc.fc_decode_attention(s.pool, s.bt_dev, s.lens_g, q, out)
        other = s.lens_g[::-1].copy() // 2
        for _ in range(3):
            out.zero_()
            fc.fc_decode_attention(s.pool, s.bt_dev, other, q)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
    finally:
        s.close()


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("L,B,method,n_heads", [
    (16, 16, fo.METHOD_SNAPKV, 1),       # everything kept, one block
    (300, 77, fo.METHOD_SNAPKV, 4),      # narrow workgroups, two passes
    (700, 300, fo.METHOD_SNAPKV, 300),   # more than one head a CU
    (700, 300, fo.METHOD_KNORM, 5),      # wide
    (1500, 400, fo.METHOD_SNAPKV, 140),  # wide
    (6000, 2176, fo.METHOD_SNAPKV, 136),  # 375 + 136 ids: fits
    (6000, 2192, fo.METHOD_SNAPKV, 136),  # 512 ids: just
    (6000, 2193, fo.METHOD_SNAPKV, 136),  # 513: has a plan_alloc
    (700, 300, fo.METHOD_STREAMING, 3),  # has one
])
def test_one_request(L, B, method, n_heads, in_place):
    """A call of one request reads table and stack itself and writes both at its end, whichever row
    of the table it has; call after call on one pool, also between calls of several requests."""
    from parity_util import SideBySide
    lens = [40, L, 33]
    s = SideBySide(_custom(lens, [20, B, 20], [method] * 3, W=16, d=64, n_heads=n_heads), in_place=in_place)
    try:
        for only in (1, 1, None, 0, 2):
            methods = np.full(3, fo.METHOD_NONE, np.int32)
            methods[slice(None) if only is None else only] = method
            budgets = np.maximum(16, np.minimum(s.lens_o, [20, B, 20]) - (only is None)).astype(np.int32)
            s.compress_and_compare(methods, budgets)
    finally:
        s.close()
