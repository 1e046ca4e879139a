"""How scoring divides a head's tiles into runs where the longest runs leave CUs idle: the number of runs, read off the
workspace a shape asks for, goes with the lengths that were measured to be fast there.  CPU only."""
import random

import pytest

import paper_2403_11805_amd as kvs


def planes(L, Hkv, Hq, D, N, T, R):
    """Bytes of the planes per tile and sub-block, and of one run's."""
    rows = (R + 31) // 32 * 32
    return 4 * L * Hq * rows * (N // 32 + N // min(T, 32)), 12 * L * Hq * rows


def runs_of(*shape):
    L, Hkv, Hq, D, N, T, R = shape
    tiles, run = planes(*shape)
    return (kvs.kv_score_workspace_bytes(kvs.Shape(L, Hkv, Hq, D, N, T, 64), R) - tiles) // run


@pytest.mark.parametrize("shape,lengths", [
    # an odd number of row blocks per kv head: two workgroups of a CU hide each other's waits
    ((28, 4, 28, 128, 2048, 16, 32), range(16, 18)),     # 46.2 us; runs of 33 tiles 57.7
    ((6, 1, 71, 64, 4096, 16, 32), range(8, 16)),        # 36.7 to 44; 33 tiles 55.1
    ((14, 2, 10, 128, 8192, 16, 32), range(14, 18)),     # 39.8; 29 tiles 50.6
    ((4, 2, 6, 128, 4096, 16, 32), range(4, 8)),         # 18; 9 tiles 22.5
    # all wavefronts with two row blocks: one workgroup per CU is as good as two
    ((4, 1, 4, 256, 32768, 16, 64), range(33, 36)),      # 37 to 38; 17 tiles 42
    ((18, 1, 8, 256, 4096, 16, 23), range(19, 21)),      # 29 to 30; 10 tiles 31.6
    ((22, 2, 8, 64, 4736, 16, 59), range(15, 17)),       # 30.5; 30 tiles 35.1
    # the last run, which reaches the diagonal, shorter than the others: 15 runs of 18 tiles and one of four, not 15 of 17 and
    # one of one
    ((4, 4, 16, 128, 8192, 32, 64), range(18, 19)),      # 25.6; 28.3
    # launches that fill no CU twice: runs of fewer than nine tiles
    ((16, 2, 8, 128, 512, 16, 32), range(4, 8)),         # 14; 9 tiles 17.6
    ((4, 1, 8, 128, 1024, 16, 32), range(4, 8)),         # 17.2; 9 tiles 18.2
])
def test_run_lengths(shape, lengths):
    tiles = shape[4] // 32
    assert runs_of(*shape) in {-(-tiles // n) for n in lengths}


def test_the_planes_of_shorter_runs_stay_within_their_bound():
    """At most 1.5 MiB more than the longest runs need, which a workspace may do without."""
    rng = random.Random(5)
    shorter = 0
    for _ in range(3000):
        Hkv = rng.choice((1, 2, 3, 4, 8, 12))
        shape = (rng.choice((1, 2, 7, 32, 80)), Hkv, Hkv * rng.choice((1, 2, 3, 4, 7, 8, 16)), rng.choice((64, 128, 256)),
                 32 * round(2 ** rng.uniform(0, 13)), rng.choice((8, 16, 32)), rng.randint(1, 256))
        if shape[6] > shape[4]:
            continue
        L, Hkv, Hq, D, N, T, R = shape
        tiles, run = planes(*shape)
        blocks = Hq // Hkv * ((R + 31) // 32)
        longest = -(-N // 32 // (8 if blocks <= 2 else 64))
        more = kvs.kv_score_workspace_bytes(kvs.Shape(L, Hkv, Hq, D, N, T, 64), R) - (tiles + longest * run + 255) // 256 * 256
        assert 0 <= more <= 3 << 19, shape
        shorter += more > 0
    assert shorter > 500
