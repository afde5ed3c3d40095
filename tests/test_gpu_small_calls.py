"""Descriptors as kernel arguments: calls whose descriptors just fit one launch's
arguments, just do not, need several launches, and go through pinned memory, one
after the other on the same pool (each may only see its own)."""

import numpy as np
import pytest

import launch_shapes
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


def _one_request(L, B, method, n_heads, d, W, in_place=False):
    """A side-by-side pool whose second of three requests is the one under test."""
    from parity_util import SideBySide
    wl = _custom([40 + W, L, 33 + W], [20 + W, B, 20 + W], [method] * 3, W=W, d=d, n_heads=n_heads)
    return wl, SideBySide(wl, in_place=in_place)


def _only(method, r):
    methods = np.full(3, fo.METHOD_NONE, np.int32)
    methods[slice(None) if r is None else r] = method
    return methods


SNAP = fo.METHOD_SNAPKV


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("L,B,method,n_heads,d,W,scores,shape,pruned,alone", [
    (16, 16, SNAP, 1, 64, 16, False, "narrow", False, True),        # everything kept, one block
    (300, 77, SNAP, 4, 64, 16, False, "narrow", False, True),       # two passes
    (300, 77, SNAP, 4, 64, 16, True, "narrow", False, False),       # asks for the scores
    (450, 140, SNAP, 129, 128, 64, False, "narrow", False, True),
    (700, 300, SNAP, 300, 64, 16, False, "narrow", False, False),   # many short heads
    (900, 300, SNAP, 300, 64, 33, False, "narrow", False, True),    # more than one head a CU
    (800, 300, SNAP, 300, 128, 32, False, "narrow", True, True),
    (640, 160, SNAP, 520, 128, 32, False, "narrow", True, True),    # more than two, each number of query tiles
    (530, 150, SNAP, 515, 128, 16, False, "narrow", True, True),
    (600, 150, SNAP, 515, 128, 48, False, "narrow", True, True),
    (700, 300, SNAP, 515, 128, 64, False, "narrow", True, True),
    (880, 300, SNAP, 520, 64, 16, False, "narrow", True, True),
    (1000, 400, SNAP, 140, 64, 32, False, "wide", False, True),
    (2100, 400, SNAP, 140, 128, 16, False, "wide", True, True),
    (2100, 400, SNAP, 140, 128, 64, False, "wide", True, True),
    (5200, 900, SNAP, 136, 64, 32, False, "wide", True, True),
    (6000, 2176, SNAP, 136, 64, 16, False, "wide", True, True),     # 375 + 136 ids: fits
    (6000, 2192, SNAP, 136, 64, 16, False, "wide", True, True),     # 512 ids: just
    (6000, 2193, SNAP, 136, 64, 16, False, "wide", True, False),    # 513: has a plan_alloc
    (6000, 2193, SNAP, 136, 64, 16, True, "wide", True, False),
    (200, 90, fo.METHOD_KNORM, 5, 64, 16, False, "narrow", False, True),
    (700, 300, fo.METHOD_KNORM, 5, 64, 16, True, "wide", False, True),
    (450, 300, fo.METHOD_KNORM, 515, 128, 16, False, "narrow", False, True),
    (700, 300, fo.METHOD_STREAMING, 3, 64, 16, False, "wide", False, False),
])
def test_one_request(L, B, method, n_heads, d, W, scores, shape, pruned, alone, in_place):
    """A call of one request reads table and stack itself and writes both at its end, whichever row
    of the table it has; call after call on one pool, also between calls of several requests.
    `alone`: the library's planner says that it takes that way (in place no ids are new); `pruned`:
    that a call without scores prunes it."""
    wl, s = _one_request(L, B, method, n_heads, d, W, in_place)
    if in_place and B == 2193:
        alone = not scores
    assert launch_shapes.planned(wl, methods=_only(method, 1), in_place=in_place)[1] == shape
    assert launch_shapes.without_plan_alloc(wl, scores, methods=_only(method, 1), in_place=in_place) == alone
    assert launch_shapes.pruned(wl, methods=_only(method, 1), in_place=in_place)[1] == pruned
    try:
        for r in (1, 1, None, 0, 2):
            budgets = np.maximum(W, np.minimum(s.lens_o, [20 + W, B, 20 + W]) - (r is None)).astype(np.int32)
            s.compress_and_compare(_only(method, r), budgets, scores=scores)
    finally:
        s.close()


@pytest.mark.parametrize("L,B,method,n_heads,d,W,shape", [
    (300, 77, SNAP, 4, 64, 16, "narrow"),
    (640, 160, SNAP, 520, 128, 32, "narrow"),
    (2100, 400, SNAP, 140, 128, 64, "wide"),
    (700, 300, fo.METHOD_KNORM, 5, 64, 16, "wide"),
])
def test_captured_call_of_one_request(L, B, method, n_heads, d, W, shape):
    """Replays between eager calls on the same pool: each leaves cache, table, free list and kept
    list as the eager call does."""
    import torch
    from paper_2503_08461_amd import fastcache as fc
    wl, s = _one_request(L, B, method, n_heads, d, W)
    try:
        methods = _only(method, 1)
        assert launch_shapes.planned(wl, methods=methods)[1] == shape
        assert launch_shapes.without_plan_alloc(wl, False, methods=methods)
        kv0, bt0 = s.kv_dev.clone(), s.bt_dev.clone()
        stack, top = fc.fc_pool_export_state(s.pool)
        stack0 = torch.from_numpy(stack).to(s.dev)
        kept = torch.zeros(int(B) * wl.n_layers * wl.n_heads, dtype=torch.int32, device=s.dev)

        def rewind():
            fc.fc_pool_import_state_dev(s.pool, stack0, top)
            s.kv_dev.copy_(kv0)
            s.bt_dev.copy_(bt0)
            kept.fill_(-7)
            torch.cuda.synchronize()

        def call(m, out=None):
            lens = wl.seq_lens.copy()
            fc.fc_compress_batch(s.pool, s.bt_dev, lens, s.q_dev, W, m, wl.budgets, wl.pool_kernel, 0.0, None, out)
            return lens

        def state():
            torch.cuda.synchronize()
            return [s.kv_dev.view(torch.int16).clone(), s.bt_dev.clone(),
                    torch.from_numpy(fc.fc_pool_export_state(s.pool)[0]), kept.clone()]

        rewind()
        call(methods, kept)
        want = state()
        assert fc.fc_pool_export_state(s.pool)[1] == top + (L + 15) // 16 - (B + 15) // 16
        rewind()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call(methods, kept)
        for other in (1, None, 0):
            rewind()
            call(_only(method, other))     # (the library's own state, in between)
            rewind()
            graph.replay()
            for got, exact in zip(state(), want):
                assert torch.equal(got, exact)
    finally:
        s.close()
