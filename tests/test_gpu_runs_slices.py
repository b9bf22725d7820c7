"""The run decoder where a chunk's bits make few slices (1 to 64, of a few codes
each): frames from no one bit to a few hundred a chunk, their runs of equal
and of very different lengths, bit for bit against the oracle, valid and with
bits of the run section flipped."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz
from tests import streamfmt as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("ones", [0, 1, 2, 5, 20, 60, 130, 260, 500, 1500])
def test_sparse_chunks(ones, dim):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    rng = np.random.default_rng(ones * 3 + dim)
    host = []
    for even in (True, False):
        f = np.zeros(3 * 4096 + 1024, np.float32)
        if ones:
            at = (np.arange(ones) * (f.size // ones) if even
                  else np.sort((f.size * rng.random(ones) ** 4).astype(int)))
            f[at] = rng.choice([1.0, -1.0, 2.0], ones)
            if dim == 1:
                f = np.cumsum(f, dtype=np.float32)
        f = np.ascontiguousarray(f.reshape(1, 16, -1) if dim != 3 else f.reshape(4, 8, -1))
        st, s, _ = O.compress(O.params(*f.shape, 1, 1, 0.5, 0, dim, 0, 1), f,
                              np.zeros((0, 3), np.int32))
        assert st == O.OK
        host.append(s)
        start = F.parse(s)["off"]["run"]
        for _ in range(6):
            c = s.copy()
            c[int(rng.integers(start, c.size))] ^= np.uint8(1 << int(rng.integers(0, 8)))
            host.append(c)
    D = rsz.DecodeBatch([torch.from_numpy(s).cuda() for s in host])
    D.run()
    torch.cuda.synchronize()
    seen = 0
    for k, s in enumerate(host):
        st, y = O.decompress(s)
        assert int(D.status[k]) == st, k
        if st == 0:
            seen += 1
            np.testing.assert_array_equal(D.frames[k].cpu().numpy().view(np.uint32),
                                          y.view(np.uint32), err_msg=str(k))
    assert seen >= 2
