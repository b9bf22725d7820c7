"""GPU parity of the run and ROI decoders at the sizes where they change
course, bit for bit against the oracle: chunks of few and many Huffman and run
bits (past the words a wave keeps in LDS), residuals 0 alone (no run code at
all) and long zero runs (quotients of many words), a partial last chunk;
windows around the largest that LDS holds (48), one lane's worth of windows
and one more, and no window."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz, synth

pytestmark = pytest.mark.gpu


def _decode(host):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    D = rsz.DecodeBatch([torch.from_numpy(s).cuda() for s in host])
    D.run()
    torch.cuda.synchronize()
    status = D.status.cpu().tolist()
    for k, s in enumerate(host):
        st, y = O.decompress(s)
        assert status[k] == st, k
        if st == 0:
            np.testing.assert_array_equal(D.frames[k].cpu().numpy().view(np.uint32),
                                          y.view(np.uint32), err_msg=str(k))


def _spread(shape, codes, seed):
    """A frame at b = 1, eb = 0.5 whose residuals take about `codes` values."""
    rng = np.random.default_rng(seed)
    f = np.zeros(shape, np.float32)
    f[:, :, ::2] = rng.integers(-codes // 2, codes // 2 + 1, f[:, :, ::2].shape)
    return f


def _run_streams():
    frames = [np.zeros((1, 64, 128), np.float32), np.zeros((1, 64, 64), np.float32)]
    frames[1][0, 40, 3] = 9.0                      # one run of thousands of zeros
    lone = np.zeros((1, 300, 100), np.float32)     # long runs, k = 0 and larger
    lone[0, ::37, ::31] = 4.0
    frames.append(lone)
    frames += [_spread((1, 65, 64), 2, 1), _spread((2, 64, 96), 30, 2),
               _spread((1, 128, 97), 900, 3), _spread((1, 90, 91), 100000, 4)]
    out = []
    for f in frames:
        for dim in (1, 2, 3):
            st, s, _ = O.compress(O.params(*f.shape, 3, 1, 0.5, 0, dim, 0, 1), f,
                                  np.zeros((0, 3), np.int32))
            assert st == O.OK
            out.append(s)
    return out


def test_run_chunks():
    _decode(_run_streams())


def test_run_chunks_corrupt():
    rng = np.random.default_rng(17)
    host = []
    for s in _run_streams():
        for t in range(4):
            c = s.copy()
            for _ in range(1 + t):
                c[int(rng.integers(80, c.size))] ^= np.uint8(1 << int(rng.integers(0, 8)))
            host.append(c)
    _decode(host)


@pytest.mark.parametrize("codes", [16, 24, 36, 42, 48, 64, 180])
def test_dense_chunks(codes):
    """Chunks of about 6 to 9 bits a symbol, below and above the 928 words of
    them that a wave keeps in LDS, and a short last chunk; valid and corrupt."""
    rng = np.random.default_rng(codes)
    host = []
    for p, h, w in ((1, 256, 80), (3, 97, 131)):
        f = rng.integers(0, codes, (p, h, w)).astype(np.float32)
        f[:, 1::2, 1::2] = f[:, :-1:2, :-1:2][:, :h // 2, :w // 2]
        st, s, _ = O.compress(O.params(p, h, w, 3, 1, 0.5), f, np.zeros((0, 3), np.int32))
        assert st == O.OK
        host.append(s)
        for _ in range(3):
            c = s.copy()
            c[int(rng.integers(80, c.size))] ^= np.uint8(1 << int(rng.integers(0, 8)))
            host.append(c)
    _decode(host)


@pytest.mark.parametrize("w,n", [(1, 40), (17, 0), (17, 8), (17, 33), (25, 5), (31, 3), (33, 9),
                                 (48, 2), (49, 2), (70, 9)])
def test_roi_windows(w, n):
    f, pk = synth.tiny_case(900 + w + n, (2, 90, 120), n, "normal", scale=50.0)
    st, s, _ = O.compress(O.params(2, 90, 120, w, 2, 1.0, 0, 2, 1, 0), f, pk)
    assert st == O.OK
    host = [s]
    rng = np.random.default_rng(w * 100 + n)
    for t in range(6):
        c = s.copy()
        c[int(rng.integers(80, c.size))] ^= np.uint8(1 << int(rng.integers(0, 8)))
        host.append(c)
    _decode(host)


@pytest.mark.parametrize("n,w", [(20, 5), (65, 9), (512, 5), (513, 5), (4096, 3), (4097, 3)])
def test_windows_must_agree_on_shared_pixels(n, w):
    """One payload word changed at a time (in a shared pixel, in a pixel of one
    window alone, in one outside the frame): the oracle's status, and its frame
    where the stream is still valid.  512 windows is the most that are
    compared with each other instead of with the frame."""
    f, _ = synth.tiny_case(990 + w, (2, 60, 70), 0, "normal", scale=50.0)
    rng = np.random.default_rng(n)
    pk = np.stack([rng.integers(0, 2, n), rng.integers(0, 60, n), rng.integers(0, 70, n)],
                  axis=1).astype(np.int32)
    pk[n // 2] = pk[n // 3]
    st, s, _ = O.compress(O.params(2, 60, 70, w, 2, 1.0), f, pk)
    assert st == O.OK
    off = 80 + (6 * n + 3) // 4 * 4
    host = [s]
    for t in range(24 if n < 1000 else 6):
        c = s.copy()
        k = (n // 2, 0, n - 1, int(rng.integers(0, n)))[t % 4]
        c[off + 4 * (k * w * w + int(rng.integers(0, w * w))) + t % 4] ^= np.uint8(1 << (t % 8))
        host.append(c)
    _decode(host)
