"""The rule for the score kernel's tiles per wave (csrc/score_rules.h), compiled for the host: batches measured with one
and with two tiles take the faster."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_17077_amd", "csrc")


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    d = tmp_path_factory.mktemp("score_rules")
    src = d / "harness.c"
    src.write_text('#include "score_rules.h"\nint tiles(int b, int t, int m, int h, int g, int r) '
                   '{ return dllm_rule_score_tiles(b, t, m, h, g, r); }\n')
    lib = d / "librules.so"
    subprocess.run(["gcc", "-std=c99", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)],
                   check=True)
    return ctypes.CDLL(str(lib)).tiles


@pytest.mark.parametrize("batch,total_kv,max_kv,hkv,group,row_bytes,want", [
    (17, 9146, 567, 16, 1, 256, 1), (10, 8530, 853, 32, 1, 256, 1), (7, 6790, 1310, 32, 1, 256, 1),   # a second round nearly empty
    (13, 31153, 2710, 8, 4, 256, 1), (9, 4761, 529, 40, 1, 256, 1), (25, 7471, 516, 40, 1, 256, 1),
    (1, 1024, 1024, 32, 1, 256, 1), (7, 14501, 2517, 8, 4, 256, 1),                                   # all resident
    (3, 6639, 2213, 32, 1, 256, 2), (9, 4370, 722, 32, 1, 256, 2), (1, 8000, 8000, 32, 1, 256, 2),    # one round of two
    (12, 22847, 2806, 16, 1, 128, 2), (4, 5345, 2348, 40, 1, 256, 2),
    (7, 8392, 1287, 40, 1, 256, 2), (16, 34500, 4096, 32, 1, 256, 2),                                 # three rounds and more
    (24, 24 * 8192, 8192, 8, 4, 256, 4)])
def test_score_tiles_per_wave(tiles, batch, total_kv, max_kv, hkv, group, row_bytes, want):
    assert tiles(batch, total_kv, max_kv, hkv, group, row_bytes) == want
