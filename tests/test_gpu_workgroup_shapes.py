"""Both workgroup shapes of the fused kernels against the oracle: narrow ones
(a launch with more heads than fit the chip as wide workgroups) and wide ones
(few heads, or heads of more than 8192 tokens), with the pruned second pass,
with the scores asked for, and in place."""

import numpy as np
import pytest

from oracle import fastcache_oracle as fo
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

SNAP, KNORM, STREAM = fo.METHOD_SNAPKV, fo.METHOD_KNORM, fo.METHOD_STREAMING


def _run(lens, budgets, methods, W, d, scores, fillers=0, n_heads=2, in_place=False, **kw):
    from paper_2503_08461_amd import fastcache as fc
    from parity_util import SideBySide
    lens = list(lens) + [9] * fillers        # key-norm requests of nine tokens that only add heads
    budgets = list(budgets) + [4] * fillers
    methods = list(methods) + [KNORM] * fillers
    s = SideBySide(_custom(lens, budgets, methods, W=W, d=d, n_heads=n_heads))
    try:
        if in_place:
            fc.fc_set_compaction_mode(s.pool, fc.FC_COMPACT_IN_PLACE)
            s.in_place = True
        return s.compress_and_compare(scores=scores, **kw)
    finally:
        s.close()


@pytest.mark.parametrize("scores", [True, False])
@pytest.mark.parametrize("W,d", [(16, 128), (32, 128), (48, 128), (64, 128), (32, 64), (48, 64), (64, 64)])
def test_narrow_workgroups(W, d, scores):
    # (2 heads x more than 256 requests: more heads than two per compute unit)
    lens = [W, 511, 512, 700, 2047, 2049, 4100, 8192]
    _run(lens, [max(W, n // 4) for n in lens], [SNAP] * len(lens), W, d, scores, fillers=300)


@pytest.mark.parametrize("scores", [True, False])
@pytest.mark.parametrize("W,d", [(16, 128), (32, 128), (48, 128), (64, 128), (32, 64), (48, 64), (64, 64)])
def test_wide_workgroups(W, d, scores):
    # both sides of the pruning limit of wide workgroups, of the narrow ones' longest head, of the
    # longer epochs and of a wavefront's last chunk; the longest head of all
    lens = [W, 300, 2047, 2048 + W, 8192, 8193, 16384, 16385, 32768]
    _run(lens, [max(W, n // 5) for n in lens], [SNAP] * len(lens), W, d, scores, n_heads=1)


def test_long_heads_of_every_method_in_one_batch():
    lens = [9000, 20000, 12345, 32768, 8200, 600]
    methods = [SNAP, KNORM, STREAM, KNORM, SNAP, SNAP]
    for scores in (True, False):
        _run(lens, [1800, 19999, 4000, 5, 8200, 300], methods, 32, 128, scores, n_heads=2)
        _run(lens, [1800, 19999, 4000, 5, 8200, 300], methods, 32, 128, scores, fillers=300)
