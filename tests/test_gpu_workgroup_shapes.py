"""The three ways a head is spread over the chip, against the oracle: narrow
workgroups (a launch with more heads than fit the chip as wide workgroups, or short
ones), wide ones (fewer heads, or heads of more than 8192 tokens), heads split over
several workgroups (very few long heads); with the pruned second pass (narrow and
wide) and with the scores asked for."""

import pytest

import launch_shapes
from oracle import fastcache_oracle as fo
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

SNAP, KNORM, STREAM = fo.METHOD_SNAPKV, fo.METHOD_KNORM, fo.METHOD_STREAMING


# requests of nine tokens, two heads each, that bring a batch to more than 128 and to more than
# 512 heads: half of a chip's 256 compute units, and two per compute unit
WIDE, NARROW = 70, 300


def _run(lens, budgets, methods, W, d, scores, fillers=0, n_heads=2, in_place=False, shape=None, half=None, limit=None, **kw):
    from parity_util import SideBySide
    lens = list(lens) + [9] * fillers        # key-norm requests of nine tokens that only add heads
    budgets = list(budgets) + [4] * fillers
    methods = list(methods) + [KNORM] * fillers
    wl = _custom(lens, budgets, methods, W=W, d=d, n_heads=n_heads)
    if shape:
        assert set(launch_shapes.planned(wl)) == {shape}
    if limit:
        assert launch_shapes.pruned(wl) == [m == SNAP and n >= limit for n, m in zip(lens, methods)]
    if half is not None:
        assert launch_shapes.leaves_half(wl) == half
    s = SideBySide(wl, in_place=in_place)
    try:
        return s.compress_and_compare(scores=scores, **kw)
    finally:
        s.close()


SHAPES = [(16, 128), (32, 128), (48, 128), (64, 128), (32, 64), (48, 64), (64, 64)]


@pytest.mark.parametrize("scores", [True, False])
@pytest.mark.parametrize("W,d", SHAPES)
def test_narrow_workgroups(W, d, scores):
    limit = {128: [512, 512, 576, 576], 64: [864, 864, 1024, 1152]}[d][W // 16 - 1]
    lens = [W, limit - 1, limit, 700, 2047, 2049, 4100, 8192]
    _run(lens, [max(W, n // 4) for n in lens], [SNAP] * len(lens), W, d, scores, NARROW, shape="narrow",
         limit=limit)


@pytest.mark.parametrize("scores", [True, False])
@pytest.mark.parametrize("W,d", SHAPES)
def test_wide_workgroups(W, d, scores):
    # both sides of the pruning limit of wide workgroups, of the narrow ones' longest head, of the
    # longer epochs and of a wavefront's last chunk; the longest head of all
    limit = {128: [1408, 1664, 1664, 1664], 64: [3584, 5120, 5632, 7168]}[d][W // 16 - 1]
    lens = [W, 300, limit - 1, limit, limit + W, 8192, 8193, 16384, 16385, 32768]
    _run(lens, [max(W, n // 5) for n in lens], [SNAP] * len(lens), W, d, scores, 2 * WIDE, n_heads=1, shape="wide",
         limit=limit)


@pytest.mark.parametrize("scores", [True, False])
@pytest.mark.parametrize("W,d", SHAPES)
def test_split_heads(W, d, scores):
    # segments that end inside the window, heads with fewer blocks than segments, empty prefixes
    lens = [W, W + 1, 100, 2047, 2048, 4097, 16384, 32768]
    _run(lens, [max(W, n // 5) for n in lens], [SNAP] * len(lens), W, d, scores, n_heads=1, shape="split")


@pytest.mark.parametrize("fillers", [0, WIDE, NARROW])
def test_every_method_in_one_batch(fillers):
    lens = [9000, 20000, 12345, 32768, 8200, 600]
    budgets = [1800, 19999, 4000, 5, 8200, 300]
    methods = [SNAP, KNORM, STREAM, KNORM, SNAP, SNAP]
    for scores in (True, False):
        _run(lens, budgets, methods, 32, 128, scores, fillers)
    _run(lens, budgets, methods, 32, 128, False, fillers, in_place=True)


@pytest.mark.parametrize("fillers", [0, WIDE, NARROW])
def test_log_sum_exp_handed_in(fillers):
    lens = [2500, 9000, 700]
    _run(lens, [500, 1800, 300], [SNAP] * 3, 32, 128, True, fillers, lse="library")


@pytest.mark.parametrize("W,d", SHAPES)
def test_single_pass_of_narrow_workgroups(W, d):
    # prefixes that end anywhere in a block, in a wavefront's first and later ones; the keys come in whole lines
    lens = [W, W + 1, W + 15, W + 16, W + 17, W + 64, 500, 1037, 2050]
    _run(lens, [max(W, n // 4) for n in lens], [SNAP] * len(lens), W, d, True, NARROW, shape="narrow", lse="library")


@pytest.mark.parametrize("W", [16, 32, 48, 64])
@pytest.mark.parametrize("lens,half", [([513, 640, 2303, 2303, 2303], False),  # mean (weighted) below 2304: all keys cached
                                       ([600, 2500, 2519, 2593, 2400], True),   # above: half of them
                                       ([2304 + 17, 527, 528, 4097 + 63], True),
                                       ([7820, 2321], True), ([7821, 2321], None)])  # three workgroups per CU, with W up to 32
def test_narrow_pruned_first_pass(W, lens, half):
    _run(lens, [max(W, n // 4) for n in lens], [SNAP] * len(lens), W, 128, False, NARROW, shape="narrow",
         half=W <= 32 if half is None else half)
