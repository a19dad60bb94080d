"""CPU check that the bounds of the trainer's accuracy tests tell apart products of
operands held as three bf16 terms (six products kept) from less: the split is
emulated in 64-bit sums, and leaving products out has to break the bounds."""
import numpy as np
import pytest

import oracle
from train_split import FORWARD_TOL, GRADIENT_TOL, SIZES, fixed_masks, inputs, predictions, rms


def _bf16(v):
    u = np.ascontiguousarray(v, np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) >> 16 << 16
    return u.astype(np.uint32).view(np.float32)


def _terms(v):
    v = np.asarray(v, np.float32)
    h = _bf16(v)
    m = _bf16(v - h)
    return [t.astype(np.float64) for t in (h, m, _bf16(v - h - m))]


def _product(a, b, kept):
    """a @ b from the `kept` largest products of the terms."""
    ta, tb = _terms(a), _terms(b)
    pairs = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)][:kept]
    return sum(ta[i] @ tb[j] for i, j in pairs)


@pytest.mark.parametrize("kept,holds", [(6, True), (5, False), (4, False), (3, False)])
def test_forward_bound(kept, holds):
    for m, d, hidden in SIZES:
        x, _, p = inputs(m, d, hidden)
        y = predictions(x, p).astype(np.float32)
        h = np.maximum(_product(x, p["W1"].T, kept) + p["b1"], 0)
        err = rms(h @ p["W2"].T.astype(np.float64) + p["b2"] - y)
        assert (err <= FORWARD_TOL / 10) if holds else (err > 1.5 * FORWARD_TOL), (m, d, hidden, err)


@pytest.mark.parametrize("kept,holds", [(6, True), (4, False), (3, False)])
def test_gradient_bound(kept, holds):
    for m, d, hidden in SIZES[:4]:
        x, y, p = inputs(m, d, hidden)
        p["b1"] = fixed_masks(x, p["W1"])
        _, g, _, _ = oracle.mlp_train_step(x, y, p, "sgd", lr=1.0)
        dp = 2 * (predictions(x, p) - y) / m
        on = np.arange(hidden) % 2 == 0
        dz = np.where(on, dp @ p["W2"].astype(np.float64), 0).astype(np.float32)
        err = np.linalg.norm(_product(dz.T, x, kept) - g["W1"]) / np.linalg.norm(g["W1"])
        assert (err <= GRADIENT_TOL / 10) if holds else (err > 2 * GRADIENT_TOL), (m, d, hidden, err)
