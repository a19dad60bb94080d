"""GPU checks of the encoder's work list at the sizes where its scan, its list of
single rows and the dealing of items change: one brick, one tile of bricks (up to
2048, up to 8192) and several, rows in the first and last brick of a tile, slices
that share a tile, fewer items than blocks and more.

Encodings are compared with the FP64 oracle on sampled events (the FP32 form's
table keeps 22 bits and sums are fp32: 1e-6 leaves a factor of four) and, whole,
bit for bit with those of a tiling of other bricks.
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


def _events(seed, W, H, T, n, t0):
    """Scattered events, the corners of the grid, and a dense column (whole bricks
    beside the single rows)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    ev = np.stack([rng.integers(0, W, n), rng.integers(0, H, n), t0 + rng.integers(0, T, n),
                   rng.choice([-1, 1], n)], 1)
    k = n // 4
    ev[:k, :2] = np.stack([rng.integers(0, min(W, 40), k), rng.integers(0, min(H, 30), k)], 1)
    for i in range(min(n, 8)):
        ev[i, :3] = [(W - 1) * (i & 1), (H - 1) * (i >> 1 & 1), t0 + (T - 1) * (i >> 2)]
    return ev.astype(np.int32)


def _rel(a, b):
    return np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b)


@pytest.mark.parametrize("W,H,T,d,n", [
    (20, 10, 4, 16, 1), (346, 260, 50, 16, 900), (640, 480, 50, 128, 4000), (1280, 720, 15, 16, 2000),
    (1280, 720, 60, 32, 5000), (1280, 720, 60, 16, 200_000), (346, 260, 50, 64, 120_000),
    (300, 200, 400, 48, 30_000),
])
def test_one_slice(vk, W, H, T, d, n):
    print("case: work list %dx%dx%d d=%d n=%d" % (W, H, T, d, n), file=sys.stderr, flush=True)
    rx, ry, rt, t0 = 3, 2, 1, 77
    ev = _events(8700 + n, W, H, T, n, t0)
    A = synth.draw_frequencies(d, rx, ry, rt, nbins=T)
    c = vk.Context(W, H, rx, ry, rt, A, T, n, "fp32")
    evt = torch.from_numpy(ev).cuda()
    got = c.encode(evt, t0, T)
    q = np.unique(np.r_[0:min(n, 8), np.random.Generator(np.random.PCG64(n)).integers(0, n, 1500)])
    ref, _ = oracle.encode(ev, A, rx, ry, rt, queries=q.astype(np.int32))
    assert _rel(got.cpu().numpy()[q], ref) <= 1e-6
    tl = c.tilings()
    for i in [i for i, t in enumerate(tl) if t[4] in (0, 3) and i][:3]:
        c.select_tiling(i)
        assert torch.equal(c.encode(evt, t0, T), got), tl[i]
    assert c.status() == vk.VECKM_OK
    c.close()


@pytest.mark.parametrize("count,n", [(3, 40), (90, 300), (40, 6000)])
def test_slices_that_share_tiles(vk, count, n):
    print("case: work list of %d slices of about %d events" % (count, n), file=sys.stderr, flush=True)
    rx, ry, rt, d = 2, 3, 2, 32
    A = synth.draw_frequencies(d, rx, ry, rt)
    rng = np.random.Generator(np.random.PCG64(8800 + count))
    specs, evs = [], []
    for k in range(count):
        W, H, T = int(rng.integers(1, 640)), int(rng.integers(1, 480)), int(rng.integers(1, 30))
        m = 0 if k % 7 == 3 else int(rng.integers(1, 2 * n))
        specs.append((W, H, 100 * k, T, m))
        evs.append(_events(8900 + k, W, H, T, m, 100 * k) if m else np.zeros((0, 4), np.int32))
    ev = np.concatenate(evs)
    c = vk.Context(640, 480, rx, ry, rt, A, 30, len(ev), "fp32", max_slices=count)
    got = c.encode_batch(specs, torch.from_numpy(ev).cuda()).cpu().numpy()
    off = 0
    for sp, e in zip(specs, evs):
        if len(e):
            ref, _ = oracle.encode(e, A, rx, ry, rt, queries=np.arange(min(len(e), 60), dtype=np.int32))
            assert _rel(got[off:off + len(ref)], ref) <= 1e-6, sp
        off += len(e)
    assert c.status() == vk.VECKM_OK
    c.close()


@pytest.mark.parametrize("W,H,T,n", [
    (346, 260, 1, 3000), (346, 260, 2, 900), (346, 260, 2, 2500), (346, 260, 10, 2000),
    (346, 260, 10, 3000), (346, 260, 50, 33_000), (346, 260, 50, 38_000), (640, 480, 50, 360_000),
    (640, 480, 50, 380_000), (1280, 720, 60, 30_000), (100, 60, 300, 20_000), (640, 480, 6, 8000),
])
def test_ranking_and_clearing_routes(vk, W, H, T, n):
    """Both sides of the rules that choose how bricks are ranked (a wave or a block
    each, of 4 or 8 waves) and how the count grid is cleared (with the flows, in one
    pass, by events): a call after another on the same context gives what a fresh
    context gives, and sampled encodings match the oracle."""
    print("case: routes %dx%dx%d n=%d" % (W, H, T, n), file=sys.stderr, flush=True)
    rx, ry, rt, d, t0 = 3, 3, 1, 64, 5
    A = synth.draw_frequencies(d, rx, ry, rt, nbins=T)
    mlp = synth.init_mlp(d, 128)
    evs = [_events(9100 + n + k, W, H, T, n, t0) for k in range(2)]
    q = np.random.Generator(np.random.PCG64(n)).integers(0, n, 500).astype(np.int32)

    def calls(c, e):
        out = [c.flow(e, t0, T), c.encode(e, t0, T), c.flow(e, t0, T, queries=torch.from_numpy(q).cuda())]
        assert c.status() == vk.VECKM_OK
        return out

    def context():
        c = vk.Context(W, H, rx, ry, rt, A, T, n, "fp32")
        c.set_mlp(*mlp)
        return c

    dev = [torch.from_numpy(e).cuda() for e in evs]
    used, fresh = context(), context()
    first = calls(used, dev[0])
    second = calls(used, dev[1])
    for a, b in zip(second, calls(fresh, dev[1])):
        assert torch.equal(a, b)
    for a, b in zip(first, calls(used, dev[0])):
        assert torch.equal(a, b)
    assert torch.equal(first[2], first[0][torch.from_numpy(q).cuda().long()])
    ref, _ = oracle.encode(evs[0], A, rx, ry, rt, queries=q)
    assert _rel(first[1].cpu().numpy()[q], ref) <= 1e-6
    used.close()
    fresh.close()
