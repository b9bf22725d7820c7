"""Batches on both sides of the size (256 MiB of frames) above which k_bin reads
whole-line rows past the caches: every stream equals the one that the frame
gives alone, and the oracle's for one of each kind; also from a graph, with the
frames changed between replays."""
import numpy as np
import pytest

from oracle import rsz_oracle as O
from paper_2206_11297_amd import rsz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,dim", [(2, 1), (2, 2), (2, 3), (4, 2)])
@pytest.mark.parametrize("n", [15, 16, 17])
def test_sizes_around_the_cache(n, b, dim):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    shape, prm = (8, 512, 1024), (11, b, 3.0, n & 1, dim)   # 16 MiB a frame
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n * 10 + b)
    frames = [torch.randn(shape, generator=gen, device="cuda") * 4.0 for _ in range(n)]
    rng = np.random.default_rng(n)
    peaks = [torch.from_numpy(np.stack([rng.integers(0, s, 30) for s in shape], 1)
                              .astype(np.int32)).cuda() for _ in range(n)]
    B = rsz.Batch(frames, peaks, prm)
    B.prepare()
    B.graph()
    for rep in range(2):
        if rep:
            for f in frames:
                f += torch.randn(shape, generator=gen, device="cuda")
        B.replay()
        torch.cuda.synchronize()
        assert int(B.status.abs().max()) == 0
        for i in range(n):
            one = rsz.compress(frames[i], peaks[i], *prm[:4], dim=dim)
            assert torch.equal(one, B.stream(i)), i
    st, ref, _ = O.compress(O.params(*shape, *prm), frames[n - 1].cpu().numpy(),
                            peaks[n - 1].cpu().numpy())
    assert st == O.OK
    np.testing.assert_array_equal(B.stream(n - 1).cpu().numpy(), ref)
