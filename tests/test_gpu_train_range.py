"""GPU checks of the trainer's fp32 arithmetic over the whole range of fp32: values
that three bf16 terms do not carry (below 2^-110 their last bits fall under bf16's
smallest number, from 2^127 on they may round to infinity) in the inputs and in W1,
against the FP64 oracle.

Half of the units are on and half off whatever rounding does (b1 is beyond the
largest |W1 x|), so no ReLU can flip and a step's change of the weights is a
smooth function of its operands: fp32 sums over m rows in partial sums of 16 are
good to about 2^-24 sqrt(m / 16) of it, 1e-6 leaves a factor of four at the sizes
here; rounding the new weights costs 2^-24 of them.
"""
import sys

import numpy as np
import pytest

import oracle
from paper_2504_19417_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
KEYS = ("W1", "b1", "W2", "b2")
TOL = 1e-6


@pytest.fixture(scope="module")
def vk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19417_amd import veckm
    return veckm


def _fixed_masks(x, W1):
    """b1 that keeps even units on and odd units off."""
    z = np.abs(x.astype(np.float64) @ W1.astype(np.float64).T).max()
    sign = np.where(np.arange(len(W1)) % 2 == 0, 1.0, -1.0)
    return (1.25 * z * sign).astype(np.float32)


def _step(vk, x, y, p, lr):
    m, k2 = x.shape
    print("case: trainer step m=%d d=%d hidden=%d |x| <= %.2g |W1| <= %.2g lr=%.2g" % (
        m, k2 // 2, len(p["b1"]), np.abs(x).max(), np.abs(p["W1"]).max(), lr), file=sys.stderr, flush=True)
    tr = vk.Trainer(k2 // 2, len(p["b1"]), m, *(p[k] for k in KEYS))
    loss = torch.zeros(1, device="cuda")
    tr.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), "sgd", lr, loss)
    got = dict(zip(KEYS, tr.weights()))
    tr.close()
    L, _, new, _ = oracle.mlp_train_step(x, y, p, "sgd", lr=lr)
    return float(loss.cpu()[0]), got, L, new


def _check(got, new, p, keys, axis=None):
    for k in keys:
        ref = new[k] - p[k].astype(np.float64)
        err = np.linalg.norm(got[k].astype(np.float64) - p[k] - ref, axis=axis if k == "W1" else None)
        size = np.linalg.norm(ref, axis=axis if k == "W1" else None)
        kept = np.linalg.norm(new[k], axis=axis if k == "W1" else None)
        assert (size > 0).all() and (err <= TOL * size + 1e-7 * kept).all(), (k, (err / size).max())


def _inputs(seed, m, d, hidden):
    rng = np.random.Generator(np.random.PCG64(seed))
    x = rng.uniform(-1, 1, (m, 2 * d))
    y = rng.normal(0, 1.5, (m, 2)).astype(np.float32)
    return x, y, dict(zip(KEYS, synth.init_mlp(d, hidden)))


@pytest.mark.parametrize("m,d,hidden", [(40, 16, 64), (300, 65, 320)])
def test_tiny_inputs_in_the_gradient(vk, m, d, hidden):
    x, y, p = _inputs(7400 + m, m, d, hidden)
    x = (x * 2.0 ** -116).astype(np.float32)
    p["b1"] = _fixed_masks(np.ones_like(x), p["W1"])
    _, got, _, new = _step(vk, x, y, p, 2.0 ** 116)
    _check(got, new, p, ("W1",))


@pytest.mark.parametrize("m,d,hidden", [(40, 16, 64), (2049, 64, 256)])
def test_tiny_inputs_in_the_forward_pass(vk, m, d, hidden):
    x, y, p = _inputs(7500 + m, m, d, hidden)
    x = (x * 2.0 ** -122).astype(np.float32)
    p["W1"] = (p["W1"] * 2.0 ** 100).astype(np.float32)
    p["b1"] = _fixed_masks(x, p["W1"])
    p["b2"] = np.zeros(2, np.float32)
    y = np.zeros_like(y)
    loss, got, L, new = _step(vk, x, y, p, 2.0 ** 40)
    assert abs(loss - L) <= TOL * L
    _check(got, new, p, ("W2", "b2"))


@pytest.mark.parametrize("m,d,hidden", [(4, 16, 64), (40, 65, 320)])
def test_tiny_weights(vk, m, d, hidden):
    x, y, p = _inputs(7600 + m, m, d, hidden)
    x = x.astype(np.float32)
    p["W1"] = (p["W1"] * 2.0 ** -122).astype(np.float32)
    p["b1"] = _fixed_masks(x, p["W1"])
    _, got, _, new = _step(vk, x, y, p, 2.0 ** 122)
    _check(got, new, p, ("W2",))


def test_device_memory_of_a_small_batch_trainer(vk):
    """The partial sums of W1 are sized for the row splits a step takes: 64 of 1 MB
    at D = 256 and 512 units (4 tiles of 256 x 256), beside 42 MB for the rows."""
    d, hidden, rows = 256, 512, 20_000
    torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    tr = vk.Trainer(d, hidden, rows, *synth.init_mlp(d, hidden))
    used = before - torch.cuda.mem_get_info()[0]
    tr.close()
    need = 64 * hidden * 2 * d * 4 + 79 * 256 * hidden * 4
    assert used <= need + (32 << 20), (used, need)
