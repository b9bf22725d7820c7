"""The failing-pixel counts of on-device verification: frames changed between
their compression and the check, counted here in float64 from the definition
(a pixel in a window fails when its bits differ, any other when it lies further
than eb + |y| 2^-23 + |mean| 2^-40 from the mean of its bin's pixels that enter
the bin).  Widths that load four columns at a time and widths that do not,
blocks of raw rows cut by the panel's edge, bins cut by both edges."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz, synth

pytestmark = pytest.mark.gpu


def _count(x, y, peaks, w, b, mode, eb):
    P, H, W = x.shape
    roi = np.zeros(x.shape, bool)
    for p, i, j in peaks:
        i0, j0 = i - w // 2, j - w // 2
        roi[p, max(i0, 0):max(i0 + w, 0), max(j0, 0):max(j0 + w, 0)] = True
    Hb, Wb = -(-H // b), -(-W // b)
    S, n = np.zeros((P, Hb, Wb)), np.zeros((P, Hb, Wb))
    for di in range(b):
        for dj in range(b):
            v = x[:, di::b, dj::b].astype(np.float64)
            on = np.ones(v.shape, bool) if mode else ~roi[:, di::b, dj::b]
            S[:, :v.shape[1], :v.shape[2]] += np.where(on, v, 0.0)
            n[:, :v.shape[1], :v.shape[2]] += on
    mean = np.where(n > 0, S / np.maximum(n, 1), 0.0)
    m = np.repeat(np.repeat(mean, b, 1), b, 2)[:, :H, :W]
    yd = y.astype(np.float64)
    off = ~(np.abs(yd - m) <= eb + np.abs(yd) * 2.0 ** -23 + np.abs(m) * 2.0 ** -40)
    return int(np.where(roi, x.view(np.uint32) != y.view(np.uint32), off).sum())


def test_counts_of_changed_frames():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    cases, prm = [], []
    for k, (shape, b) in enumerate([((2, 33, 256), 1), ((3, 65, 520), 2), ((1, 30, 4), 2),
                                    ((2, 70, 132), 4), ((2, 31, 30), 2), ((2, 67, 61), 3),
                                    ((1, 35, 44), 8), ((1, 64, 2048), 1)]):
        cases.append(synth.tiny_case(820 + k, shape, 5, "normal", scale=30.0))
        prm.append((7, b, 2.0, k % 2))
    frames = [torch.from_numpy(f).cuda() for f, _ in cases]
    B = rsz.Batch(frames, [torch.from_numpy(p).cuda() for _, p in cases], prm)
    B.prepare()
    V = rsz.Verify(B)
    B.launch()
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    for (f, _), g in zip(cases, frames):
        at = rng.random(f.shape) < 0.05
        f[at] += rng.choice([-40.0, -1.0, 1e-3, 40.0], int(at.sum())).astype(np.float32)
        g.copy_(torch.from_numpy(f))
    V.launch()
    torch.cuda.synchronize()
    want = [_count(f, y.cpu().numpy(), pk, t[0], t[1], t[3], t[2])
            for (f, pk), y, t in zip(cases, V.frames, prm)]
    assert min(want[:2]) > 0
    assert V.bad_counts() == want
