"""GPU checks that the trainer's products are fp32 products: the error of the
predictions and of dW1 against the FP64 oracle within bounds that operands of
fewer bits break (train_split), and the steps that run on the fp32 matrix cores
(values that three bf16 terms do not carry) column by column.
"""
import sys

import numpy as np
import pytest

import oracle
from train_split import FORWARD_TOL, GRADIENT_TOL, KEYS, SIZES, fixed_masks, inputs, predictions

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
HUGE = float(np.finfo(np.float32).max)


@pytest.fixture(scope="module")
def vk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19417_amd import veckm
    return veckm


def _step(tr, x, y, lr):
    loss = torch.zeros(1, device="cuda")
    tr.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), "sgd", lr, loss)
    return float(loss.cpu()[0]), dict(zip(KEYS, tr.weights()))


def _one(vk, what, x, y, p, lr):
    m, k2 = x.shape
    print("case: trainer %s m=%d d=%d hidden=%d" % (what, m, k2 // 2, len(p["b1"])), file=sys.stderr,
          flush=True)
    tr = vk.Trainer(k2 // 2, len(p["b1"]), m, *(p[k] for k in KEYS))
    loss, got = _step(tr, x, y, lr)
    tr.close()
    return loss, got


def _check_gradient(got, new, old):
    """The change of W1 as a whole, to GRADIENT_TOL and the rounding of the new weights."""
    ref = new - old.astype(np.float64)
    err = np.linalg.norm(got.astype(np.float64) - old - ref)
    assert err <= GRADIENT_TOL * np.linalg.norm(ref) + 1e-7 * np.linalg.norm(new)


def _check_columns(got, new, x, y, p, lr, cols):
    """Every column of W1's change (`cols`): an fp32 sum over rows is good to a few
    2^-24 of the sum of its terms' magnitudes, whatever cancels in it."""
    q = {k: v.astype(np.float64) for k, v in p.items()}
    on = x.astype(np.float64) @ q["W1"].T + q["b1"] > 0
    dz = np.where(on, (2 * (predictions(x, p) - y) / len(x)) @ q["W2"], 0)
    terms = lr * np.linalg.norm(np.abs(dz).T @ np.abs(x.astype(np.float64)), axis=0)
    ref = new["W1"] - q["W1"]
    err = np.linalg.norm(got["W1"].astype(np.float64) - q["W1"] - ref, axis=0)
    bound = GRADIENT_TOL * terms + 1e-7 * np.linalg.norm(new["W1"], axis=0)
    assert (np.linalg.norm(ref, axis=0) > 100 * bound)[cols].all()  # (the bound says something)
    assert (err <= bound)[cols].all(), (err / bound)[cols].max()


@pytest.mark.parametrize("m,d,hidden", SIZES)
def test_predictions(vk, m, d, hidden):
    x, _, p = inputs(m, d, hidden)
    loss, _ = _one(vk, "forward", x, predictions(x, p).astype(np.float32), p, 1.0)
    assert np.sqrt(loss) <= FORWARD_TOL


@pytest.mark.parametrize("m,d,hidden", SIZES[:4])
def test_gradient(vk, m, d, hidden):
    x, y, p = inputs(m, d, hidden)
    p["b1"] = fixed_masks(x, p["W1"])
    _, got = _one(vk, "gradient", x, y, p, 64.0)
    new = oracle.mlp_train_step(x, y, p, "sgd", lr=64.0)[2]
    _check_gradient(got["W1"], new["W1"], p["W1"])


@pytest.mark.parametrize("m,d,hidden", [(300, 40, 448), (2100, 16, 64), (700, 130, 512)])
def test_huge_inputs(vk, m, d, hidden):
    """The largest fp32 numbers in rows and columns of several tiles; small weights
    keep everything finite, and every column of dW1 is that of the oracle."""
    x, y, p = inputs(m, d, hidden)
    p["W1"] = (p["W1"] * 2.0 ** -60).astype(np.float32)
    p["W2"] = (p["W2"] * 2.0 ** -60).astype(np.float32)
    p["b1"] = fixed_masks(x, p["W1"])
    on = np.where(np.arange(hidden) % 2 == 0, 1, -1)
    for i, r in enumerate((3, 47, m // 2, m - 1)):
        c = (7 + 29 * i) % (2 * d)
        x[r, c] = HUGE * (-1) ** i  # (the units it would flip take its sign)
        p["W1"][:, c] = np.abs(p["W1"][:, c]) * on * (-1) ** i
    loss, got = _one(vk, "huge inputs", x, y, p, 64.0)
    L, _, new, _ = oracle.mlp_train_step(x, y, p, "sgd", lr=64.0)
    assert abs(loss - L) <= GRADIENT_TOL * L
    _check_columns(got, new, x, y, p, 64.0, np.arange(2 * d))


@pytest.mark.parametrize("m,d,hidden", [(100, 16, 64), (700, 65, 320)])
def test_huge_weight(vk, m, d, hidden):
    """One weight near the largest fp32 number, on a feature small enough."""
    x, y, p = inputs(m, d, hidden)
    u, c = hidden - 2, 5
    p["b1"] = fixed_masks(x, p["W1"])
    x[:, c] = np.random.Generator(np.random.PCG64(m)).uniform(0.25, 1, m) * 2.0 ** -107
    p["W1"][u, c] = 0.9 * HUGE
    p["W2"][:, u] *= 2.0 ** -20
    loss, got = _one(vk, "huge weight", x, y, p, 64.0)
    L, _, new, _ = oracle.mlp_train_step(x, y, p, "sgd", lr=64.0)
    assert abs(loss - L) <= GRADIENT_TOL * L
    _check_columns(got, new, x, y, p, 64.0, np.delete(np.arange(2 * d), c))


def test_weight_that_becomes_huge(vk):
    """A step takes one weight to -2^127; the next runs with it."""
    d, hidden, u, c, m = 16, 64, 40, 9, 40
    p = {"W1": np.zeros((hidden, 2 * d), np.float32), "b1": np.zeros(hidden, np.float32),
         "W2": np.zeros((2, hidden), np.float32), "b2": np.zeros(2, np.float32)}
    p["b1"][u] = p["W2"][0, u] = 1
    x1 = np.zeros((2, 2 * d), np.float32)
    x1[:, c] = 1, -1
    print("case: trainer weight grows to -2^127", file=sys.stderr, flush=True)
    tr = vk.Trainer(d, hidden, m, *(p[k] for k in KEYS))
    loss, now = _step(tr, x1, np.array([[0, 0], [2, 0]], np.float32), 2.0 ** 126)
    assert loss == 1 and now["W1"][u, c] == -2.0 ** 127
    x, y, _ = inputs(m, d, hidden)
    x[:, c] = -np.random.Generator(np.random.PCG64(m)).uniform(0.25, 1, m) * 2.0 ** -107
    loss, got = _step(tr, x, y, 1.0)
    tr.close()
    L, _, new, _ = oracle.mlp_train_step(x, y, now, "sgd", lr=1.0)
    assert abs(loss - L) <= GRADIENT_TOL * L
    rest = np.delete(np.arange(2 * d), c)
    _check_gradient(got["W1"][u, rest], new["W1"][u, rest], now["W1"][u, rest])
