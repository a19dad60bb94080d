"""GPU checks of the encoder's single rows (bricks with few query voxels, whose
windows are collected as bits per voxel and from the pair grid) against the
FP64 oracle: windows that leave the slice on every side, bricks of 32, 16 and 8
columns, even and odd radii, voxels with 1 to 6 events (two bits hold counts up
to 2), slices of one bin, query subsets, several slices of different sensors,
and calls whose rows fill items only partly.

Tolerance: the FP32 form's table entries keep 22 bits and sums are fp32, so
encodings are good to about 2^-22 relative L2; 1e-6 leaves a factor of four.
"""
import sys

import numpy as np
import pytest

import oracle
from paper_2504_19417_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def vk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19417_amd import veckm
    return veckm


def _events(seed, W, H, T, n, t0=1000):
    """Events on the faces, in a dense spot, scattered, and repeated in a voxel."""
    rng = np.random.Generator(np.random.PCG64(seed))
    ev = np.stack([rng.integers(0, W, n), rng.integers(0, H, n), rng.integers(0, T, n),
                   rng.choice([-1, 1], n)], 1)
    k = n // 4
    ev[:k, 0] = rng.choice([0, 1, W - 2, W - 1], k).clip(0, W - 1)
    ev[k:2 * k, :2] = np.stack([rng.integers(0, min(W, 9), k), rng.integers(0, min(H, 7), k)], 1)
    ev[2 * k:2 * k + k // 2] = ev[rng.integers(0, max(1, k // 8), k // 2)]
    ev[:, 2] += t0
    return ev[np.argsort(ev[:, 2], kind="stable")].astype(np.int32), t0


def _rel(a, b):
    return np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b)


@pytest.mark.parametrize("W,H,T,rx,ry,rt,d,n", [
    (40, 30, 1, 5, 5, 3, 128, 300), (70, 50, 9, 4, 6, 2, 64, 2000), (33, 17, 20, 3, 2, 1, 16, 800),
    (64, 48, 12, 6, 6, 3, 256, 1500), (100, 9, 6, 2, 2, 0, 32, 500), (346, 260, 50, 5, 5, 3, 128, 3000),
    (20, 20, 20, 9, 9, 2, 48, 400), (1, 1, 3, 1, 1, 1, 16, 7),
])
def test_rows_match_oracle(vk, W, H, T, rx, ry, rt, d, n):
    print("case: single rows %dx%dx%d r=%d,%d,%d d=%d n=%d" % (W, H, T, rx, ry, rt, d, n),
          file=sys.stderr, flush=True)
    ev, t0 = _events(8100 + n, W, H, T, n)
    A = synth.draw_frequencies(d, rx, ry, max(rt, 1), nbins=T)
    c = vk.Context(W, H, rx, ry, rt, A, T, n, "fp32")
    evt = torch.from_numpy(ev).cuda()
    ref, _ = oracle.encode(ev, A, rx, ry, rt)
    got = c.encode(evt, t0, T).cpu().numpy()
    assert _rel(got, ref) <= 1e-6
    q = np.random.Generator(np.random.PCG64(n)).integers(0, n, max(1, n // 9)).astype(np.int32)
    sub = c.encode(evt, t0, T, queries=torch.from_numpy(q).cuda()).cpu().numpy()
    assert np.array_equal(sub, got[q])
    assert c.status() == vk.VECKM_OK
    c.close()


def test_batch_rows_match_single_calls(vk):
    """Slices of three sensors in one call: bit-identical to each slice alone."""
    rx, ry, rt, d = 5, 4, 2, 64
    A = synth.draw_frequencies(d, rx, ry, rt)
    shapes = [(40, 30, 1, 250), (96, 64, 10, 1200), (33, 70, 7, 40), (96, 64, 3, 1)]
    evs = [_events(8200 + i, W, H, T, n, t0=50 * i)[0] for i, (W, H, T, n) in enumerate(shapes)]
    specs = [(W, H, 50 * i, T, n) for i, (W, H, T, n) in enumerate(shapes)]
    mlp = synth.init_mlp(d, 128)
    c = vk.Context(96, 70, rx, ry, rt, A, 10, 2000, "fp32", max_slices=4)
    c.set_mlp(*mlp)
    got = c.flow_batch(specs, torch.from_numpy(np.concatenate(evs)).cuda()).cpu().numpy()
    off = 0
    for (W, H, T, n), ev, sp in zip(shapes, evs, specs):
        one = vk.Context(W, H, rx, ry, rt, A, T, n, "fp32")
        one.set_mlp(*mlp)
        alone = one.flow(torch.from_numpy(ev).cuda(), sp[2], T).cpu().numpy()
        assert np.array_equal(alone, got[off:off + n])
        off += n
        one.close()
    c.close()


def test_window_rows_match_a_slice(vk):
    """A sliding window (ring planes wrap, voxels of 3 and more events in wrapped
    planes, the tiling changed mid-stream) gives the rows of a slice that holds
    the window's events, bit for bit."""
    W, H, T, rx, ry, rt, d, n = 75, 40, 7, 5, 4, 3, 128, 900
    A = synth.draw_frequencies(d, rx, ry, rt)
    win = vk.Window(W, H, rx, ry, rt, A, T, n, "fp32")
    one = vk.Context(W, H, rx, ry, rt, A, T, T * n, "fp32")
    bins = []
    for k in range(2 * T + 3):
        ev, _ = _events(8300 + k, W, H, 1, n, t0=100 + k)
        bins.append(ev)
        win.push(torch.from_numpy(ev).cuda(), 100 + k, 1)
        if k == T + 2:
            win.select_tiling(len(win.tilings()) - 1)
        if k < T:
            continue
        q = torch.from_numpy(bins[k - rt]).cuda()
        got = win.encode_window(q).cpu().numpy()
        held = np.concatenate(bins[k - T + 1:k + 1])
        m = sum(len(b) for b in bins[k - T + 1:k - rt])
        one.select_tiling(win.tiling())
        ref = one.encode(torch.from_numpy(held).cuda(), 100 + k - T + 1, T).cpu().numpy()
        assert np.array_equal(got, ref[m:m + n])
    win.close()
    one.close()
