"""GPU peak lists of frames full of candidates (a hundredth of the pixels at
amax_min, and every pixel of a frame on a pedestal), against the oracle, with
rings whose pixels a wave loads once (up to 128 of them, ring_out 5) and
rings that it loads again."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,ring_in,ring_out", [(1, 2, 2), (3, 4, 4), (3, 4, 5), (2, 3, 6),
                                                   (3, 7, 8), (3, 8, 15)])
@pytest.mark.parametrize("pedestal", [0.0, 1000.0])
def test_dense_candidates(rank, ring_in, ring_out, pedestal):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    rng = np.random.default_rng(ring_out)
    kw = dict(rank=rank, ring_in=ring_in, ring_out=ring_out, npix_min=1, snr_min=2.0,
              pix_nsigma=1.0)
    frames = [rng.normal(pedestal, 130.0, s).astype(np.float32)
              for s in ((2, 90, 131), (1, 40, 40), (3, 7, 300))]
    B = rsz.PeakBatch([torch.from_numpy(f).cuda() for f in frames], rsz.peak_params(**kw))
    B.run()
    torch.cuda.synchronize()
    total = 0
    for k, f in enumerate(frames):
        pk, n = O.find_peaks(O.peak_params(**kw), f)
        total += n
        assert int(B.status[k]) == 0 and int(B.counts[k]) == n
        np.testing.assert_array_equal(B.peaks(k).cpu().numpy(), pk)
    assert total > 20
