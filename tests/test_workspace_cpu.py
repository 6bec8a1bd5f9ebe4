"""What callers are asked for (CPU; the sizes are computed on the host)."""
import pytest

from paper_2511_16298_amd import _abi


def frame(w, h, n):
    f = _abi.ss_frame()
    f.width, f.height, f.tile_px, f.num_gaussians = w, h, 16, n
    f.gaussians = 256 if n else None
    return f


@pytest.mark.parametrize("n", [1, 511, 5000, 16_384])
@pytest.mark.parametrize("capacity", [0, 1000, 131_072, 4_000_000])
def test_small_frames_ask_for_no_more_than_the_passes(n, capacity):
    """The one-kernel path of small frames uses two words; the size is that of
    the passes, which the next larger Gaussian count takes."""
    st, small = _abi.ss_workspace_bytes(frame(256, 256, n), capacity)
    assert st == _abi.SS_OK
    st, passes = _abi.ss_workspace_bytes(frame(256, 256, 16_385), capacity)
    assert st == _abi.SS_OK
    assert 256 <= small <= passes
