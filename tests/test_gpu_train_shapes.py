"""GPU checks of the trainer at the edges of its kernels' tiles (row blocks of
64, 128 and 256 rows, 16-feature steps, one or two unit halves, one to four
feature tiles of dW1), on unaligned inputs and on values beyond the range of
the bf16 terms, against the FP64 oracle.

Tolerance: operands keep 24 bits and sums are fp32, so a step's change of the
weights is good to a few 2^-24 sqrt(rows) of it, and rounding the new weights
to fp32 costs 2^-24 |w| / |change|; 1e-4 covers both at these sizes (as the
trainer's other tests).
"""
import sys

import numpy as np
import pytest

import oracle
from paper_2504_19417_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
KEYS = ("W1", "b1", "W2", "b2")


@pytest.fixture(scope="module")
def vk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19417_amd import veckm
    return veckm


def _check(vk, x, y, p, d, hidden, offset=0):
    m = len(x)
    print("case: trainer step m=%d d=%d hidden=%d offset=%d" % (m, d, hidden, offset), file=sys.stderr,
          flush=True)
    buf = torch.zeros(m * 2 * d + offset, device="cuda")
    xt = buf[offset:].view(m, 2 * d)  # `offset` floats past an aligned address
    xt.copy_(torch.from_numpy(x))
    tr = vk.Trainer(d, hidden, m, *(p[k] for k in KEYS))
    loss = torch.zeros(1, device="cuda")
    tr.step(xt, torch.from_numpy(y).cuda(), "sgd", 1.0, loss)
    got = tr.weights()
    tr.close()
    L, _, new, _ = oracle.mlp_train_step(x, y, p, "sgd", lr=1.0)
    assert abs(float(loss.cpu()[0]) - L) <= 1e-5 * L
    for k, g in zip(KEYS, got):
        ref = new[k] - p[k]
        err = np.linalg.norm(g.astype(np.float64) - p[k] - ref)
        assert err <= 1e-4 * np.linalg.norm(ref) + 1e-7 * np.linalg.norm(new[k]), k


@pytest.mark.parametrize("m,d,hidden,offset", [
    (1, 1, 64, 0), (31, 3, 64, 0), (65, 9, 192, 1), (257, 129, 320, 0), (640, 65, 128, 2),
    (2049, 256, 512, 0), (300, 40, 448, 3), (32769, 16, 384, 0), (66001, 24, 64, 0),
    (65537, 64, 256, 1),
])
def test_step_at_tile_edges(vk, m, d, hidden, offset):
    rng = np.random.Generator(np.random.PCG64(7100 + m))
    x = rng.uniform(-1, 1, (m, 2 * d)).astype(np.float32)
    y = rng.normal(0, 1.5, (m, 2)).astype(np.float32)
    _check(vk, x, y, dict(zip(KEYS, synth.init_mlp(d, hidden))), d, hidden, offset)


@pytest.mark.parametrize("m", [100, 70000])
def test_values_beyond_the_split(vk, m):
    """The largest fp32 numbers (they round to infinity in bf16) in the rows of
    one block: W2 = 0 keeps everything finite, and the step matches."""
    d, hidden = 16, 64
    rng = np.random.Generator(np.random.PCG64(7200))
    x = rng.uniform(-1, 1, (m, 2 * d)).astype(np.float32)
    x[3, 5] = np.finfo(np.float32).max
    y = rng.normal(0, 1.5, (m, 2)).astype(np.float32)
    p = dict(zip(KEYS, synth.init_mlp(d, hidden)))
    p["W2"] = np.zeros_like(p["W2"])
    p["W1"] = (p["W1"] * 2.0 ** -20).astype(np.float32)
    _check(vk, x, y, p, d, hidden)


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_non_finite_inputs_show(vk, value):
    d, hidden, m = 16, 64, 100
    rng = np.random.Generator(np.random.PCG64(7300))
    x = rng.uniform(-1, 1, (m, 2 * d)).astype(np.float32)
    x[40, 7] = value
    y = rng.normal(0, 1.5, (m, 2)).astype(np.float32)
    tr = vk.Trainer(d, hidden, m, *synth.init_mlp(d, hidden))
    loss = torch.zeros(1, device="cuda")
    tr.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), "sgd", 0.1, loss)
    W1 = tr.weights()[0]
    assert not np.isfinite(W1[:, 7]).any()
    if value == np.inf:  # relu(+inf) reaches the loss
        assert not np.isfinite(float(loss.cpu()[0]))
    else:  # relu(nan) = 0: the other columns see a finite step
        assert np.isfinite(np.delete(W1, 7, 1)).all()
    tr.close()
