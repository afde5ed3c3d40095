"""Chunk-MLP kernel at the edges of its tiles (128 or 256 rows, two rows a chunk
here), and with more tiles than workgroups are resident, jobs of both modalities in
turn: every workgroup walks several, with the next one's rows requested ahead."""

import pytest

from test_gpu_mlp import run_case

pytestmark = pytest.mark.gpu

SHAPES = [(64, 128), (64, 256), (128, 128), (128, 256)]


@pytest.mark.parametrize("d,hidden", SHAPES)
def test_tile_edges(d, hidden):
    chunks = [63, 64, 65, 127, 128, 129]
    lens = [2 * c + 5 for c in chunks]           # five text tokens in front
    run_case(lens, [5] * 6, lens, [1] * 6, d=d, k=2, hidden=hidden, n_heads=1, seed=3)


@pytest.mark.parametrize("d,hidden", SHAPES)
def test_more_tiles_than_workgroups(d, hidden):
    n = 420                                      # 840 jobs of one tile, at most 768 workgroups
    lens = [2 + i % 5 for i in range(n)]
    run_case(lens, [1] * n, lens, [1] * n, d=d, k=3, hidden=hidden, n_heads=1, seed=4)
