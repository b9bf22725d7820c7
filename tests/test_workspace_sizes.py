"""Workspace sizes (host-only queries) of frames at bin factor 3 whose binning
tiles of three strips would take more memory than single strips do: no more
than single strips take, so that the frames which the static scratch of the
allocation-free entry point holds stay in it."""
import pytest

from paper_2206_11297_amd import rsz

# (panels, height, width, dim, roi_coding, run_coding), bytes with single strips
SIZES = [((56, 214, 3679, 1, 0, 0), 62716160), ((28, 6925, 208, 2, 1, 0), 60351744),
         ((37, 5252, 206, 1, 0, 0), 60141824), ((39, 233, 5234, 2, 1, 0), 65595136),
         ((63, 215, 3300, 1, 1, 0), 63333888), ((6, 32692, 233, 1, 0, 0), 66037760),
         ((4, 48996, 248, 1, 0, 0), 68957184), ((38, 2292, 934, 2, 1, 1), 140552960)]


@pytest.mark.parametrize("case,bytes_", SIZES)
@pytest.mark.parametrize("npeaks", [0, 200])
def test_bin_3_takes_no_more_than_single_strips(case, bytes_, npeaks):
    P, H, W, dim, roi, run = case
    st, n = rsz.rsz_workspace_bytes(rsz.params(P, H, W, 17, 3, 1.0, 0, dim, roi, run), npeaks)
    assert st == 0
    assert n <= bytes_ + 16384   # (the window and peak tables differ by npeaks)
    if bytes_ < rsz.NOALLOC_SCRATCH_BYTES - 16384:
        assert n <= rsz.NOALLOC_SCRATCH_BYTES
