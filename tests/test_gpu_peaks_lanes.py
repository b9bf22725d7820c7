"""GPU peak finding where one lane holds a pixel at amax_min in the first half
of its 64 pixels and a lower spot, which passes every other cut, in the second:
only the first is a candidate."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz

pytestmark = pytest.mark.gpu


def _pixel(bit, thread):
    """(row, column) in a 128 x 128 panel of a lane's pixel: load bit / 4 of 4 pixels."""
    return divmod(((bit >> 2) * 256 + thread) * 4 + (bit & 3), 128)


def _frame(first, second, thread):
    rng = np.random.default_rng(first * 64 + second)
    f = rng.normal(0.0, 2.0, (1, 128, 128)).astype(np.float32)
    for bit, amp in ((first, 2000.0), (second, 264.0)):
        i, j = _pixel(bit, thread)
        u, v = np.mgrid[:128, :128]
        f[0] += (amp * np.exp(-((u - i) ** 2 + (v - j) ** 2) / 1.4)).astype(np.float32)
    return f


@pytest.mark.parametrize("first", [0, 15, 31])
def test_candidates_of_one_lane(first):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    seconds = (32, 41, 47, 50, 63)
    frames = [_frame(first, s, 16 + s // 4) for s in seconds]
    B = rsz.PeakBatch([torch.from_numpy(f).cuda() for f in frames])
    B.run()
    torch.cuda.synchronize()
    for k, f in enumerate(frames):
        pk, n = O.find_peaks(O.peak_params(), f)
        low, n_low = O.find_peaks(O.peak_params(amax_min=200.0), f)
        assert n == 1 and n_low == 2   # the lower spot fails amax_min alone
        assert int(B.counts[k]) == n
        np.testing.assert_array_equal(B.peaks(k).cpu().numpy(), pk)
