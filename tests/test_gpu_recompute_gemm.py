"""GPU parity of the projection kernels at the edges of their tiles: the layer of test_gpu_recompute.run_case (same
oracle, same bars) at row counts around the streamed / tiled boundary and the row blocks per workgroup, at widths that
fill no column tile, and at K that is no multiple of a stage, of a step, or shorter than one."""
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
    (1, 1, 2, 64, 256, 8, 520, 1000, 0, some(13, 32, 2)),        # 104 rows: four row blocks, the last of 8
    (1, 1, 2, 128, 512, 16, 264, 712, 0, some(17, 32, 3)),       # 272 rows: two row tiles, the last block of 16
    (1, 2, 4, 64, 1024, 16, 136, 1032, 0, some(46, 64, 4)),      # 736 rows; too short a K to divide: gate and up gated in one
    (1, 1, 2, 64, 512, 8, 56, 136, 0, some(29, 64, 5)),          # 232 rows, gated: an odd number of row blocks, the last of 8
    (1, 1, 1, 64, 256, 8, 64, 8, 0, some(12, 32, 6)),            # 96 rows, gated: one piece of columns
    (1, 1, 2, 64, 256, 8, 2568, 1288, 0, some(20, 32, 7)),       # 160 rows, K divided over 11 column tiles: XCDs shared by splits
])
def test_projection_edges(case):
    run_case(*case, seed=71)


def test_more_rows_than_the_library_limit(monkeypatch):
    """2080 rows on the library's own kernels, GEMM library switched off: nine row tiles, the last with one block."""
    monkeypatch.setenv("KVSWITCH_OWN_GEMM", "1")
    run_case(1, 1, 1, 64, 2080, 16, 72, 136, 0, list(range(130)), seed=73)
