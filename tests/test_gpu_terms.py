"""csrc/terms.h: what the split of a float32 into bfloat16 terms leaves, by one dot-product instruction, bit for
bit the subtraction of the number with its lower 16 bits masked away."""
from __future__ import annotations

import ctypes as C
import os

import numpy as np
import pytest

import parity
from paper_2406_06220_amd import build

pytestmark = pytest.mark.gpu


def patterns():
    """Finite float32 bit patterns: every exponent with every kind of lower half, subnormal numbers, zeros, the
    largest, and random ones."""
    rng = np.random.default_rng(17)
    exponents = np.arange(0, 255, dtype=np.uint32) << np.uint32(23)
    low = np.array([0, 1, 2, 0x7fff, 0x8000, 0x8001, 0xfffe, 0xffff], np.uint32)
    top = np.array([0, 1 << 16, 0x3f << 16, 0x40 << 16, 0x7f << 16], np.uint32)
    edges = (exponents[:, None, None] | top[None, :, None] | low[None, None, :]).ravel()
    edges = np.concatenate([edges, edges | np.uint32(1 << 31)])
    drawn = rng.integers(0, 2 ** 32, 1 << 20, dtype=np.uint32)
    small = rng.integers(0, 2 ** 24, 1 << 18, dtype=np.uint32) | (rng.integers(0, 2, 1 << 18, dtype=np.uint32) << np.uint32(31))
    bits = np.concatenate([edges, drawn, small])
    return bits[(bits >> np.uint32(23)) & np.uint32(255) != 255]


@pytest.mark.parametrize("partner", ["itself", "zero", "edge", "drawn"])
def test_what_a_term_leaves(partner):
    import torch
    if not os.path.exists(build.TERMS_TEST_LIB):
        build.build_terms_test_library()
    lib = C.CDLL(build.TERMS_TEST_LIB)
    x = patterns()
    rng = np.random.default_rng(3)
    y = {"itself": x, "zero": np.zeros_like(x), "edge": np.roll(x[:20400].repeat(len(x) // 20400 + 1)[:len(x)], 7),
         "drawn": rng.permutation(x)}[partner]
    want = [v.view(np.float32) - (v & np.uint32(0xffff0000)).view(np.float32) for v in (x, y)]
    parity.announce(f"less_term of {len(x)} pairs, partner {partner}")
    dx, dy = (torch.from_numpy(v.view(np.int32).copy()).to("cuda:0") for v in (x, y))
    rx, ry = torch.empty_like(dx), torch.empty_like(dy)
    assert lib.run_less_terms(C.c_void_p(dx.data_ptr()), C.c_void_p(dy.data_ptr()), C.c_void_p(rx.data_ptr()), C.c_void_p(ry.data_ptr()),
                              len(x), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    for got, w, v in ((rx, want[0], x), (ry, want[1], y)):
        got = got.cpu().numpy().view(np.uint32)
        w = w.view(np.uint32)
        off = np.flatnonzero(got != w)
        assert off.size == 0, (off.size, [hex(int(q)) for q in (v[off[0]], got[off[0]], w[off[0]])])
