"""Selection and classification on the four-tokens-per-lane layout: competing
token counts at the edges of a lane's four tokens, of a wavefront's 256-token
chunk and of its segment, crossed with pooling widths that stay inside, reach
and cross the neighbouring lanes' tokens.  With scores the kept list must be
the exact top budget of the GPU's own scores; without, the oracle's."""

import numpy as np
import pytest

import launch_shapes
from oracle import fastcache_oracle as fo
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [1, 3, 5, 7, 9, 11, 17, 63])
@pytest.mark.parametrize("scores,shape", [(True, "few"), (False, "few"), (False, "wide"), (False, "narrow")])
def test_token_counts_at_layout_edges(width, scores, shape):
    """(Without the scores, classification of the heads that are long enough to be pruned.)"""
    from parity_util import SideBySide
    W = 16
    # competing tokens: 1..5, around 256 (one chunk), 1024 (a segment per wavefront), 2048
    n_sel = [1, 2, 3, 4, 5, 31, 63, 255, 256, 257, 511, 513, 1023, 1024, 1025, 1027, 2047, 2049]
    if shape == "wide":  # a segment per wavefront of sixteen
        n_sel += [1407, 1535, 1537, 4095, 4096, 4097]
    lens = [n + W for n in n_sel]
    budgets = [W + max(1, n // 3) for n in n_sel]
    d = 64 if scores else 128
    wl = launch_shapes.in_shape(_custom(lens, budgets, [fo.METHOD_SNAPKV] * len(lens), W=W, d=d, n_heads=2), shape)
    if shape != "few":
        assert launch_shapes.planned(wl) == [shape] * wl.n_req
        assert sum(launch_shapes.pruned(wl)) >= 7
    s = SideBySide(wl)
    try:
        s.compress_and_compare(scores=scores, pool_kernel=width)
    finally:
        s.close()


def test_key_norm_counts_at_layout_edges():
    from parity_util import SideBySide
    lens = [1, 3, 4, 5, 255, 256, 257, 1023, 1025, 2048, 8191, 8192, 8193]
    s = SideBySide(_custom(lens, [max(1, n // 2) for n in lens], [fo.METHOD_KNORM] * len(lens), d=64, n_heads=2))
    try:
        s.compress_and_compare()
    finally:
        s.close()
