"""Inputs and bounds that pin the trainer's products to fp32 accuracy, shared by
the GPU tests and by the CPU test that shows what the bounds tell apart.

fp32 operands kept to 24 bits with fp32 sums leave
  * an error of the prediction of about 2^-24 of the layer-1 sums, 7e-8 RMS at
    the sizes here (predictions of 0.2): FORWARD_TOL = 2e-7;
  * an error of dW1 of a few 2^-24 (sums over short runs of rows): with masks
    that no rounding flips (b1 beyond the largest |W1 x|), GRADIENT_TOL = 1e-6.
Operands short of the third bf16 term of one side give 4e-7 and more of the first
and 3e-6 and more of the second.
"""
import numpy as np

from paper_2504_19417_amd import synth

KEYS = ("W1", "b1", "W2", "b2")
FORWARD_TOL, GRADIENT_TOL = 2e-7, 1e-6
# (with the 70000 rows of the last, dW1 is large beside its terms' rounding)
SIZES = [(64, 16, 64), (300, 40, 448), (640, 65, 128), (2049, 256, 512), (70000, 24, 64)]


def fixed_masks(x, W1):
    """b1 that keeps even units on and odd units off whatever rounding does."""
    z = np.abs(x.astype(np.float64) @ W1.astype(np.float64).T).max()
    return (1.25 * z * np.where(np.arange(len(W1)) % 2 == 0, 1.0, -1.0)).astype(np.float32)


def inputs(m, d, hidden):
    rng = np.random.Generator(np.random.PCG64(7700 + m))
    x = rng.uniform(-1, 1, (m, 2 * d)).astype(np.float32)
    y = rng.normal(0, 1.5, (m, 2)).astype(np.float32)
    return x, y, dict(zip(KEYS, synth.init_mlp(d, hidden)))


def predictions(x, p):
    """In 64 bits."""
    q = {k: v.astype(np.float64) for k, v in p.items()}
    return np.maximum(x.astype(np.float64) @ q["W1"].T + q["b1"], 0) @ q["W2"].T + q["b2"]


def rms(e):
    return float(np.sqrt((np.asarray(e, np.float64) ** 2).sum(1).mean()))
