"""GPU parity of the binning kernel over every bin factor and panel width around
its loads, bit for bit against the oracle: widths one bin wide, cut last bins of
every length, rows that start at every 4-byte alignment, strips of 64 bins and
the columns of a short last strip, several column groups, windows across bins
and words of the ROI bitmap, NaN and infinities inside windows; both bin modes
and every Lorenzo dimension."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz, synth

pytestmark = pytest.mark.gpu


def _widths(b):
    ws = {b, b + 1, 2 * b + 1, 31, 33, 64 * b - 1, 64 * b, 64 * b + 1, 64 * b + b - 1,
          64 * b + 2 * b, 130 * b - 1, 200 * b + 1, 270 * b - b // 2}
    return sorted(w for w in ws if w >= b)


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("b", range(1, 9))
def test_widths(b, dim):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    cases = []
    for k, W in enumerate(_widths(b)):
        H = (b * 5 + 1, 37, b * 20)[k % 3]
        f, pk = synth.tiny_case(1000 + 17 * b + k, (1 + k % 2, H, W), 4 + k % 3, "normal", scale=40.0)
        if k % 2 == 0:   # a window's pixels may hold anything
            f[pk[0, 0], pk[0, 1], pk[0, 2]] = (np.nan, np.inf, -np.inf)[k % 3]
        cases.append((f, pk))
    for mode in (0, 1):
        use = [(f, pk) for f, pk in cases if mode == 0 or np.isfinite(f).all()]
        B = rsz.Batch([torch.from_numpy(f).cuda() for f, _ in use],
                      [torch.from_numpy(p).cuda() for _, p in use], (7, b, 1.0, mode, dim))
        B.run()
        torch.cuda.synchronize()
        assert B.status.cpu().tolist() == [0] * len(use)
        for i, (f, pk) in enumerate(use):
            st, ref, _ = O.compress(O.params(*f.shape, 7, b, 1.0, mode, dim), f, pk)
            assert st == O.OK
            np.testing.assert_array_equal(B.stream(i).cpu().numpy(), ref,
                                          err_msg=f"b {b} {f.shape} mode {mode}")


@pytest.mark.parametrize("panels", [1, 63, 65, 255, 257, 1025])
def test_peak_bands(panels):
    """Peaks sorted by (panel, segment) band: 256, 1024 and more bands, below and
    above each."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    f, pk = synth.tiny_case(1300 + panels, (panels, 17, 9), 300, "normal", scale=40.0)
    st, ref, _ = O.compress(O.params(*f.shape, 3, 2, 1.0), f, pk)
    assert st == O.OK
    got = rsz.compress(torch.from_numpy(f).cuda(), torch.from_numpy(pk).cuda(), 3, 2, 1.0)
    np.testing.assert_array_equal(got.cpu().numpy(), ref)
