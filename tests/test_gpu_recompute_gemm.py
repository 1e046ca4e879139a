"""GPU parity of the projection kernels at the edges of their tiles: the layer of test_gpu_recompute.run_case (same
oracle, same bars) at row counts around the streamed / tiled boundary and around the row blocks per workgroup, at
widths that fill no column tile, and at K that is no multiple of a stage, of a step, or shorter than one.  Layers this
small are all tiled by three row blocks; the other tiles, which wide layers take, are asked for through the
environment."""
import numpy as np
import pytest

from test_gpu_recompute import run_case

pytestmark = pytest.mark.gpu


def some(n, of, seed):
    return sorted(np.random.default_rng(seed).choice(of, size=n, replace=False).tolist())


@pytest.mark.parametrize("case", [
    # L, Hkv, Hq, D, N, T, d_model, d_ff, layer, missing
    (1, 1, 1, 64, 64, 8, 8, 8, 0, [3]),                          # 8 rows, K = 8: half a step
    (1, 1, 2, 64, 128, 8, 24, 40, 0, [1, 3, 4, 7, 15]),          # 40 rows: two row blocks, the last of 8; K = 24 and 40
    (1, 2, 2, 64, 256, 16, 312, 264, 0, [0, 5, 9, 14]),          # 64 rows: the last streamed size
    (1, 2, 2, 64, 256, 8, 1000, 520, 0, some(9, 32, 1)),         # 72 rows: tiled, three row blocks; K = 1000 divided
    (1, 1, 2, 64, 256, 8, 520, 1000, 0, some(13, 32, 2)),        # 104 rows: two row tiles, the second one block of 8
    (1, 1, 2, 128, 512, 16, 264, 712, 0, some(17, 32, 3)),       # 272 rows: three row tiles, the last block of 16
    (1, 2, 4, 64, 1024, 16, 136, 1032, 0, some(46, 64, 4)),      # 736 rows; too short a K to divide: gate and up gated in one
    (1, 1, 2, 64, 512, 8, 56, 136, 0, some(29, 64, 5)),          # 232 rows, gated: three blocks and two, the last of 8
    (1, 1, 1, 64, 256, 8, 64, 8, 0, some(12, 32, 6)),            # 96 rows, gated: one piece of columns
    (1, 1, 2, 64, 256, 8, 2568, 1288, 0, some(20, 32, 7)),       # 160 rows, K divided over 11 column tiles: XCDs shared by splits
])
def test_projection_edges(case):
    run_case(*case, seed=71)


@pytest.mark.parametrize("row_blocks", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("splits", [1, 4])
@pytest.mark.parametrize("case", [
    # 264 rows, the last block of 8 (eight blocks and one; five and four; ...).  K = 392, 128, 520: 6, 2 and 8 whole
    # stages, two of them with a half step behind; gate | up gated, the others in up to three splits
    (1, 1, 2, 64, 512, 8, 392, 520, 0, some(33, 64, 8)),
    # 360 rows: twelve blocks, the last of 8.  K = 264, 192, 1288: 4, 3 and 20 whole stages; gated
    (1, 1, 3, 64, 512, 8, 264, 1288, 0, some(45, 64, 9)),
    # 136 rows: five blocks, the last of 8.  K = 200, 128, 96: 3, 2 and 1 whole stages; nothing to divide
    (1, 1, 2, 64, 512, 8, 200, 96, 0, some(17, 64, 10)),
    # 264 rows.  K = 1032, 512, 264: divided in four (gate | up too: not gated then), the last of 4 to 20 steps
    (1, 2, 8, 64, 512, 8, 1032, 264, 0, some(33, 64, 11)),
])
def test_every_tile(case, splits, row_blocks, monkeypatch):
    monkeypatch.setenv("KVSWITCH_GEMM_TILE", f"{row_blocks},{splits}")
    run_case(*case, seed=79)


def test_more_rows_than_the_library_limit(monkeypatch):
    """2080 rows on the library's own kernels, GEMM library switched off: 22 row tiles of three blocks, the last of two."""
    monkeypatch.setenv("KVSWITCH_OWN_GEMM", "1")
    run_case(1, 1, 1, 64, 2080, 16, 72, 136, 0, list(range(130)), seed=73)
