"""On-device verification of panels with few bins a row, in small calls (blocks
of 32 raw rows) and in calls of many blocks (of more rows): the failing-pixel
counts of changed frames against the definition in float64; and narrow panels
checked in not much more time than the same pixels in wide ones."""
import numpy as np
import pytest

from paper_2206_11297_amd import rsz
from tests.test_gpu_verify_counts import _count

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return torch


def _frame(shape, seed):
    rng = np.random.default_rng(seed)
    f = rng.normal(0.0, 30.0, shape).astype(np.float32)
    pk = np.stack([rng.integers(0, shape[k], 6) for k in range(3)], 1).astype(np.int32)
    return f, pk


@pytest.mark.parametrize("panels", [2, 500])
def test_counts_on_narrow_panels(panels):
    torch = _gpu()
    cases, prm = [], []
    for k, (h, w, b) in enumerate([(70, 20, 6), (129, 23, 6), (33, 5, 1), (65, 64, 2), (64, 63, 1),
                                   (40, 130, 2), (97, 257, 1), (31, 9, 8), (257, 4, 4),
                                   (35, 1, 3), (300, 100, 5)]):
        cases.append(_frame((panels if k % 3 else 7, h, w), 500 + k))
        prm.append((7, b, 2.0, k % 2))
    frames = [torch.from_numpy(f).cuda() for f, _ in cases]
    B = rsz.Batch(frames, [torch.from_numpy(p).cuda() for _, p in cases], prm)
    B.prepare()
    V = rsz.Verify(B)
    B.launch()
    V.launch()
    torch.cuda.synchronize()
    assert V.bad_counts() == [0] * len(cases)
    rng = np.random.default_rng(6)
    for (f, _), g in zip(cases, frames):
        at = rng.random(f.shape) < 0.03
        f[at] += rng.choice([-40.0, -1.0, 1e-3, 40.0], int(at.sum())).astype(np.float32)
        g.copy_(torch.from_numpy(f))
    V.launch()
    torch.cuda.synchronize()
    want = [_count(f, y.cpu().numpy(), pk, t[0], t[1], t[3], t[2])
            for (f, pk), y, t in zip(cases, V.frames, prm)]
    assert V.bad_counts() == want


def _verify_ms(shape, n):
    torch = _gpu()
    f, pk = _frame(shape, 4)
    g, p = torch.from_numpy(f).cuda(), torch.from_numpy(pk).cuda()
    B = rsz.Batch([g] * n, [p] * n, (7, 6, 2.0))
    B.prepare()
    V = rsz.Verify(B)
    B.launch()
    best = None
    for _ in range(6):
        rsz.rsz_profile_enable(1)
        V.launch()
        torch.cuda.synchronize()
        t = rsz.rsz_profile_read()
        rsz.rsz_profile_enable(0)
        ms = t["k_verify"][1]
        best = ms if best is None else min(best, ms)
    assert V.bad_counts() == [0] * n
    return best


def test_narrow_panels_take_not_much_longer():
    """With a wave a bin row, four bins of it, 300 frames took 189 us."""
    narrow, wide = _verify_ms((5, 127, 20), 300), _verify_ms((5, 127, 400), 15)
    print(f"300 of 5x127x20: {1e3 * narrow:.1f} us, 15 of 5x127x400: {1e3 * wide:.1f}", flush=True)
    assert narrow < 2 * wide
