"""The rules that divide launches, compiled for the CPU: at the sizes below the choice is one that was measured to be
fast, and where a former choice was not, not that one."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("rules") / "librules.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2403_11805_amd", "csrc"),
                    os.path.join(ROOT, "tests", "launch_rules_driver.cpp"), "-o", lib], check=True)
    handle = ctypes.CDLL(lib)
    handle.stream_splits.restype = ctypes.c_int64
    handle.stream_splits.argtypes = [ctypes.c_int64] * 3
    handle.attention_shares.restype = ctypes.c_int64
    handle.attention_shares.argtypes = [ctypes.c_int64] * 4
    return handle


@pytest.mark.parametrize("tiles,K,good", [
    # more than 256 column tiles, not divided: a second workgroup on a few CUs and none beside the others
    (264, 4096, range(2, 9)),      # gate | up of d_ff 16896: 137.3 us a layer divided in two, 148.9 undivided
    (288, 4096, range(2, 9)),      # d_ff 18432: 141.5, 152.8
    (320, 4096, range(2, 9)),      # d_ff 20480: 146.3, 156.3
    (272, 5120, range(2, 9)),      # 184.7, 199.7
    (288, 12288, range(2, 9)),     # q | k | v of d_model 12288: 551.6, 584.2
    # a few workgroups more than one or two to a CU
    (40, 13824, (5, 6)),           # down of d_model 5120: 148.7 in six, 157.3 in eight
    (172, 4096, (1,)),             # gate | up of d_ff 11008: 113.0, 116.5 in two
    (96, 4096, (2,)),              # q | k | v: 115.0, 116.4 in five
    (88, 2048, (2,)),              # 65.4, 67.6 in five
    (48, 2048, (3, 4, 5)),         # 65.1 in five, 67.3 in eight
    # short of 256 however it is divided
    (32, 11008, (7, 8)),
    (8, 2816, (6, 7, 8)),
])
def test_splits_of_the_streamed_gemm(rules, tiles, K, good):
    assert rules.stream_splits(tiles, (K + 15) // 16, 16) in good


def test_splits_of_the_streamed_gemm_stay_in_their_limits(rules):
    """At least one split; at most eight, as many as there is room for, and 256 of K for each."""
    for tiles in (1, 2, 3, 31, 64, 100, 255, 256, 257, 300, 511, 513, 3000):
        for steps in (1, 15, 16, 31, 32, 33, 128, 257, 1792):
            for most in (0, 1, 2, 3, 8, 16):
                s = rules.stream_splits(tiles, steps, most)
                assert 1 <= s <= max(1, min(8, most, steps // 16))


@pytest.mark.parametrize("pairs,kv_heads,tokens,good", [
    (1, 16, 512, (1,)),            # 51.2 us undivided, 53.4 in two shares
    (2, 16, 512, (1,)),            # 63.7, 65.3
    (2, 4, 512, (1,)),             # 42.0, 43.9
    (2, 16, 640, (1,)),            # 50.5, 52.9
    (1, 8, 1024, (8,)),            # 49.5 in eight, 50.2 in four, 52.8 undivided
    (2, 16, 1024, (4,)),           # 66.2 in four, 66.5 in eight, 67.5 undivided
    (1, 32, 4096, (8,)),
    (2, 32, 4096, (4,)),
    (2, 1, 4096, (16,)),
    (3, 32, 4096, (8,)),           # a wavefront per pair
    (64, 32, 4096, (1,)),
])
def test_shares_of_the_attention(rules, pairs, kv_heads, tokens, good):
    assert rules.attention_shares(pairs, kv_heads, tokens // 32, 100) in good
    assert rules.attention_shares(pairs, kv_heads, tokens // 32, 3) <= 3
    assert rules.attention_shares(pairs, kv_heads, tokens // 32, 0) == 1
