"""On-device verification of panels wider than one block of columns (2048):
the failing-pixel counts of frames changed after their compression against the
definition in float64, with windows across the blocks' edges; the widths that
are refused; and a wide panel checked about as fast as a narrow one."""
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
    P, H, W = shape
    cols = [c for c in (0, 2015, 2016, 2017, 2046, 2048, 2049, 4095, 4096, W - 1) if c < W]
    pk = np.array([[k % P, (7 * k) % H, c] for k, c in enumerate(cols)], np.int32)
    return f, pk


def test_counts_on_wide_panels():
    torch = _gpu()
    cases, prm = [], []
    for k, (shape, b) in enumerate([((1, 33, 2048), 2), ((1, 33, 2049), 2), ((2, 9, 2052), 1),
                                    ((1, 40, 4100), 4), ((1, 35, 4033), 3), ((1, 8, 6001), 7),
                                    ((2, 5, 4096), 8), ((1, 16, 65535), 2), ((1, 70, 4097), 5),
                                    ((1, 3, 8192), 1)]):
        cases.append(_frame(shape, 300 + k))
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
    assert min(want) > 0
    assert V.bad_counts() == want


@pytest.mark.parametrize("b,verified", [(4, True), (5, False), (8, False)])
def test_refused_widths_stay_refused(b, verified):
    torch = _gpu()
    f, pk = _frame((1, 9, 65535), 9)
    B = rsz.Batch([torch.from_numpy(f).cuda()], [torch.from_numpy(pk).cuda()], (7, b, 2.0))
    B.prepare()
    V = rsz.Verify(B)
    B.launch()
    V.launch()
    torch.cuda.synchronize()
    assert int(B.status[0]) == 0
    assert V.bad_counts() == [0 if verified else 0xFFFFFFFF]


def _verify_ms(shape):
    torch = _gpu()
    f, pk = _frame(shape, 4)
    B = rsz.Batch([torch.from_numpy(f).cuda()], [torch.from_numpy(pk).cuda()], (7, 2, 2.0))
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
    assert V.bad_counts() == [0]
    return best


def test_wide_panels_take_no_longer():
    """Blocks of whole rows left one of 16 x 65535 to four workgroups: 1016 us,
    40 times as long as the same pixels in a narrow panel."""
    wide, narrow = _verify_ms((1, 16, 65535)), _verify_ms((1, 1024, 1023))
    print(f"16 x 65535: {1e3 * wide:.1f} us, 1024 x 1023: {1e3 * narrow:.1f}", flush=True)
    assert wide < 5 * narrow
