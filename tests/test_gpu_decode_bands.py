"""GPU parity of the decoder's inverse Lorenzo and pixel kernels at the sizes
where they change course, bit for bit against the oracle: bin rows around a
band (16) and a segment of bands (128), bin columns around a wave's strip (64
bins a lane group, 2 or 4 bins a lane for b = 2 and 1), bins cut by the panel's
edge, every bin factor and Lorenzo dimension, and residuals that mostly need
the escape form (bounds far below the noise), outliers among them."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    rsz.lib()
    return t


# (bin, bin rows, bin columns); the raw size is cut by 0 .. b - 1 pixels
SHAPES = [(1, 16, 255), (1, 17, 256), (1, 1, 257), (1, 129, 5), (1, 300, 3), (2, 15, 127),
          (2, 16, 128), (2, 33, 129), (2, 128, 1), (2, 257, 70), (3, 17, 63), (3, 31, 64),
          (3, 48, 65), (4, 16, 64), (4, 18, 130), (5, 17, 66), (6, 5, 64), (7, 16, 9),
          (8, 33, 65), (8, 1, 1)]


def _streams(dim):
    out = []
    for k, (b, hb, wb) in enumerate(SHAPES):
        P = 1 + (k + dim) % 3 + (9 if k % 7 == 0 else 0)
        H, W = b * hb - (k % b), b * wb - ((k // 2) % b)
        f, pk = synth.tiny_case(700 + k, (P, H, W), k % 4, "normal", scale=30.0)
        # k % 3: residuals of a few codes, of the escape form, and outliers
        eb = (20.0, 0.06, 0.01)[k % 3]
        st, s, _ = O.compress(O.params(P, H, W, 5, b, eb, k & 1, dim, 0, (k >> 1) & 1), f, pk)
        assert st == O.OK
        out.append(s)
    return out


@pytest.mark.parametrize("dim", [1, 2, 3])
def test_band_and_strip_edges(torch, dim):
    host = _streams(dim)
    D = rsz.DecodeBatch([torch.from_numpy(s).cuda() for s in host])
    for f in D.frames:
        f.fill_(float("nan"))
    D.run()
    torch.cuda.synchronize()
    assert D.status.cpu().tolist() == [0] * len(host)
    for k, s in enumerate(host):
        st, y = O.decompress(s)
        np.testing.assert_array_equal(D.frames[k].cpu().numpy().view(np.uint32),
                                      y.view(np.uint32), err_msg=f"{SHAPES[k]} dim {dim}")
