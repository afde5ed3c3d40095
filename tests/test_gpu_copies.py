"""The copy of kept rows by itself: calls whose heads are not scored (streaming), in each
workgroup shape, and the copy that is a kernel of its own (separate scheduling, split heads),
whose wavefronts take four blocks at a time and the ids of sixty-four."""

import numpy as np
import pytest

import launch_shapes
from oracle import fastcache_oracle as fo
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu


def _run(wl, **kw):
    from parity_util import SideBySide
    s = SideBySide(wl, **kw)
    try:
        s.compress_and_compare(scores=False)
    finally:
        s.close()


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,n_heads,n_layers,shape", [
    ([1, 16, 17, 250], 3, 1, "narrow"),
    ([33, 900, 767], 40, 2, "wide"),               # more than a tile for some of 16 wavefronts
    ([9000, 20, 1], 2, 1, "wide"),                 # more blocks than a narrow workgroup keeps ids of
    ([250, 1, 77, 16] * 4, 32, 4, "narrow"),       # 2048 heads: two workgroups a CU
    ([9000] + [40] * 63, 9, 1, "narrow"),          # ids in LDS and not
])
def test_calls_of_streaming_requests(lens, n_heads, n_layers, shape, d, in_place):
    budgets = [max(1, (n * (30 + 7 * (i % 10))) // 100) for i, n in enumerate(lens)]
    wl = _custom(lens, budgets, [fo.METHOD_STREAMING] * len(lens), d=d, n_heads=n_heads, n_layers=n_layers)
    assert launch_shapes.planned(wl, in_place=in_place) == [shape] * len(lens)
    _run(wl, in_place=in_place)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("blocks", [1, 3, 4, 5, 13, 16, 17, 21, 255, 256, 257, 261, 273])
def test_blocks_of_a_copy_of_its_own(blocks, d):
    """Four wavefronts: up to 69 blocks each."""
    from paper_2503_08461_amd import fastcache as fc
    B = 16 * blocks - 5
    _run(_custom([B + 900, B], [B, B], [fo.METHOD_KNORM, fo.METHOD_STREAMING], d=d, n_heads=2),
         score_mode=fc.FC_SCORE_TWO_PASS)


@pytest.mark.parametrize("d", [64, 128])
def test_copies_of_split_heads(d):
    """Segments without a block, with a single one, and with several rounds of four."""
    lens, budgets = [4000, 2048, 30000, 700], [1, 150, 21000, 650]
    wl = _custom(lens, budgets, [fo.METHOD_KNORM, fo.METHOD_KNORM, fo.METHOD_STREAMING, fo.METHOD_KNORM], d=d, n_heads=2)
    assert launch_shapes.planned(wl) == ["split"] * 4
    _run(wl)
