"""Counts beyond what a first pass over them covers, bit for bit against the
oracle: panels of more than 2048 bin rows (more than 8 bands a segment of
column sums), by shared bands and by whole ones, and calls of more than 4096
frames or streams (a third step of the search for a workgroup's frame)."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return torch


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("shape,b,copies", [((1, 2065, 70), 1, 1), ((1, 2065, 70), 1, 9),
                                            ((2, 4801, 9), 2, 1), ((1, 9000, 12), 3, 8),
                                            ((1, 4130, 1030), 2, 1)])
def test_tall_panels(shape, b, copies, dim):
    torch = _gpu()
    rng = np.random.default_rng(shape[1] + dim)
    f = rng.normal(0.0, 20.0, shape).astype(np.float32)
    f[rng.random(shape) < 0.001] += 900.0
    st, s, _ = O.compress(O.params(*shape, 3, b, 0.5, 0, dim), f, np.array([[0, 7, 2]], np.int32))
    assert st == O.OK
    y = O.decompress(s)[1].view(np.uint32)
    D = rsz.DecodeBatch([torch.from_numpy(s).cuda() for _ in range(copies)])
    D.run()
    torch.cuda.synchronize()
    assert int(D.status.abs().max()) == 0
    for g in D.frames:
        np.testing.assert_array_equal(g.cpu().numpy().view(np.uint32), y)


@pytest.mark.parametrize("n", [4096, 4097, 4300])
def test_calls_of_many_frames(n):
    torch = _gpu()
    rng = np.random.default_rng(n)
    shapes = [(1, 5, 7), (2, 9, 33), (1, 18, 20), (3, 4, 4)]
    opts = [(3, 1, 0.5, 0, 1, 0, 0), (3, 2, 1.0, 1, 2, 1, 1), (5, 3, 2.0, 0, 3, 0, 1),
            (1, 2, 0.5, 0, 2, 0, 0), (3, 1, 1.0, 0, 3, 1, 0)]
    kinds = []   # a few kinds of frame, in a mixed order
    for k in range(20):
        sh = shapes[k % 4]
        f = rng.normal(0.0, 30.0, sh).astype(np.float32)
        f[0, sh[1] // 2, sh[2] // 2] += 5000.0
        pk = np.array([[0, sh[1] // 2, sh[2] // 2]], np.int32)
        st, s, _ = O.compress(O.params(*sh, *opts[k % 5]), f, pk)
        assert st == O.OK
        kinds.append((torch.from_numpy(f).cuda(), torch.from_numpy(pk).cuda(), opts[k % 5],
                      s, O.decompress(s)[1].view(np.uint32),
                      O.find_peaks(O.peak_params(snr_min=1.0, npix_min=1), f)[1]))
    pick = [kinds[int(k)] for k in rng.integers(0, 20, n)]
    B = rsz.Batch([k[0] for k in pick], [k[1] for k in pick], [k[2] for k in pick])
    B.run()
    torch.cuda.synchronize()
    assert int(B.status.abs().max()) == 0
    sizes, out = B.sizes.cpu().tolist(), B.out.cpu().numpy()
    for i, k in enumerate(pick):
        assert sizes[i] == k[3].size
        np.testing.assert_array_equal(out[B.offsets[i]:B.offsets[i] + sizes[i]], k[3])
    D = rsz.DecodeBatch([B.stream(i, sizes) for i in range(n)])
    D.run()
    torch.cuda.synchronize()
    assert int(D.status.abs().max()) == 0
    got = torch.cat([f.reshape(-1) for f in D.frames]).cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got, np.concatenate([k[4].reshape(-1) for k in pick]))
    P = rsz.PeakBatch([k[0] for k in pick], rsz.peak_params(snr_min=1.0, npix_min=1), 16)
    P.run()
    torch.cuda.synchronize()
    assert int(P.status.abs().max()) == 0
    assert P.counts.cpu().tolist() == [k[5] for k in pick]
