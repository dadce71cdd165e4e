"""csrc/split.h, compiled for the host: how work is divided between workgroups."""
from __future__ import annotations

import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "split.h"
using namespace tdt;
extern "C" void pred_share_c(int deep, int nt_a, int nt_b, int h_pred, int C, int rank, int *out)
{
    const PredShare s = pred_share(deep != 0, nt_a, nt_b, h_pred, C, rank);
    const int v[6] = {s.qt0, s.na, s.r0, s.nr, s.u0, s.U};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    src, lib = str(d / "split.cpp"), str(d / "libsplit.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2406_06220_amd", "csrc"), src, "-o", lib], check=True)
    return C.CDLL(lib)


@pytest.mark.parametrize("deep", [0, 1])
@pytest.mark.parametrize("H,Hp", [(8, 8), (16, 40), (48, 40), (640, 640), (24, 1024), (1024, 8), (264, 200)])
def test_predictor_side_is_dealt_out_whole(split, deep, H, Hp):
    """Every column tile and hidden unit has one owner, and no workgroup points at a unit the model does
    not have: all of them request the per-label table from their first unit on."""
    nt_a, nt_b = -(-H // 16), -(-Hp // 4)
    out = (C.c_int * 6)()
    for n in (1, 2, 3, 7, 16, 51, 85, 128, 255, 256):
        tiles_a, tiles_b, units = [], [], []
        for rank in range(n):
            split.pred_share_c(deep, nt_a, nt_b, Hp, n, rank, out)
            qt0, na, r0, nr, u0, U = out
            assert na >= 0 and nr >= 0 and U >= 0
            tiles_a += range(qt0, qt0 + na)
            tiles_b += range(r0, r0 + nr)
            units += range(u0, u0 + U)
            assert 0 <= u0 and u0 + max(U, 1) <= Hp, (n, rank)
        assert tiles_a == list(range(nt_a)) and tiles_b == list(range(nt_b)) and units == list(range(Hp))


def test_stateless_predictor_has_no_share(split):
    out = (C.c_int * 6)()
    split.pred_share_c(0, 40, 0, 640, 9, 4, out)
    assert list(out) == [0] * 6
