"""The split of the row kernels of small layers (csrc/small_split.h), on the host: the rounds it plans with are those of the XCD that
gets the most workgroups."""
import ctypes
import os
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2308_14352_amd", "csrc")


@pytest.fixture(scope="module")
def rows_of_wg(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    src = d / "split.cc"
    src.write_text('#include "small_split.h"\nextern "C" int rows_of_wg(int rows, int cols, long long items) { return moeq::small_rows_of_wg(rows, cols, items); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(d / "split.so")], check=True)
    f = ctypes.CDLL(str(d / "split.so")).rows_of_wg
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    return f


def rounds(rows, R, items):
    """Of the busiest XCD: workgroup (b, item) of a grid whose first dimension is a multiple of eight runs on XCD b % 8, two on each of
    its 32 compute units."""
    blocks = (rows + R - 1) // R
    most = max(sum(1 for b in range(blocks) if b % 8 == x) for x in range(8))
    return -(-most * items // 64)


@pytest.mark.parametrize("rows,cols", [(1024, 1024), (2048, 512), (512, 2048), (512, 512), (512, 1024), (3072, 768), (768, 3072), (96, 32),
                                       (8192, 2048), (2048, 8192)])
def test_no_other_split_is_shorter_on_the_busiest_xcd(rows, cols, rows_of_wg):
    steps = lambda R: -(-R // max(1, 512 * 32 // cols))
    for items in list(range(1, 40)) + [64, 65, 84, 128, 200, 1000, 33203]:
        R = rows_of_wg(rows, cols, items)
        assert R % 4 == 0 and 4 <= R <= 256
        cost = {r: rounds(rows, r, items) * (6 + steps(r)) for r in range(4, 257, 4)}
        assert cost[R] <= 1.02 * min(cost.values()), (items, R, cost[R], min(cost.values()))
