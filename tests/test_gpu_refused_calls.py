"""A single-frame call that is refused for its workspace makes no HIP call."""
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


def test_refused_calls_leave_a_capture_alone(torch):
    """A workspace too small is found before any HIP call: the stream's capture
    goes on, and its graph replays."""
    frame, peaks = synth.tiny_case(9, (2, 40, 60), 4, "normal", scale=30.0)
    f, pk = torch.from_numpy(frame).cuda(), torch.from_numpy(peaks).cuda()
    p = rsz.params(2, 40, 60, 5, 2, 1.0)
    st, wsb = rsz.rsz_workspace_bytes(p, len(peaks))
    ws, out = rsz.workspace(wsb), torch.zeros(1 << 16, dtype=torch.uint8, device="cuda")
    x = torch.arange(64, device="cuda", dtype=torch.float32)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = x * 2
        got = [rsz.rsz_compress(p, rsz._ptr(f), rsz._ptr(pk), len(peaks), rsz._ptr(out),
                                out.numel(), rsz._ptr(ws), n, rsz._stream())[0]
               for n in (0, 255, wsb - 1)]
        z = y + 1
    assert got == [rsz.RSZ_ERR_WORKSPACE] * 3
    for k in range(3):
        x.fill_(float(k))
        g.replay()
        torch.cuda.synchronize()
        assert bool((z == 2 * k + 1).all())
    s = rsz.compress(f, pk, window=5, bin=2, eb=1.0)
    np.testing.assert_array_equal(s.cpu().numpy(),
                                  O.compress(O.params(2, 40, 60, 5, 2, 1.0), frame, peaks)[1])
