"""The order in which the label loop's float32 products of one LSTM layer are summed up, sixteen rows at a time and four
(label_loop.hip, products_of and few_products), formed on the CPU: how far each is from 64 bits."""
from __future__ import annotations

import numpy as np

WAVES, STEPS, QUARTERS, INPUTS = 4, 10, 4, 4   # 640 inputs: of a wavefront, of a step, of a lane


def chain(x, w):
    """Multiply and add with one rounding each, along the first axis."""
    c = np.zeros(x.shape[1:], np.float32)
    for a, b in zip(x, w):
        c = (a.astype(np.float64) * b + c).astype(np.float32)
    return c


def added(parts):
    total = parts[0]
    for p in parts[1:]:
        total = total + p
    return total


def sixteen_rows(x, w):
    """Two chains a wavefront, of even and of odd steps, a product of four inputs at a time."""
    def in_turn(v, odd):
        return v[odd::2].transpose(0, 2, 1, 3).reshape(-1, v.shape[-1])
    return added([chain(in_turn(x[i], 0), in_turn(w[i], 0)) + chain(in_turn(x[i], 1), in_turn(w[i], 1)) for i in range(WAVES)])


def four_rows(x, w):
    """A chain a quarter of a step's inputs, quarters in pairs, then wavefronts, then the two pairs."""
    def quarter(i, q):
        return chain(x[i, :, q].reshape(-1, x.shape[-1]), w[i, :, q].reshape(-1, x.shape[-1]))
    return added([added([quarter(i, q) + quarter(i, q + 2) for i in range(WAVES)]) for q in (0, 1)])


def test_few_rows_are_summed_no_less_exactly():
    """For a result of 1 rms.  A rounding is at most 2^-24 of what is rounded, so errors of independent inputs are, rms, no more than
    that times the root of the sum of the partial sums' squares: n chains of m inputs n m (m + 1) / 2 of 640, 40.5 and 20.5."""
    rng = np.random.default_rng(7)
    shape = (WAVES, STEPS, QUARTERS, INPUTS, 20000)
    x = rng.standard_normal(shape).astype(np.float32)
    w = (rng.standard_normal(shape) / np.sqrt(640)).astype(np.float32)
    exact = (x.astype(np.float64) * w).sum((0, 1, 2, 3))
    sixteen, four = (np.sqrt(((f(x, w) - exact) ** 2).mean()) / exact.std() for f in (sixteen_rows, four_rows))
    assert four < sixteen
    assert sixteen < 2.0 ** -24 * 40.5 ** 0.5 and four < 2.0 ** -24 * 20.5 ** 0.5
