"""Frames around the number of Gaussians per tile from which the image-only
kernel is taken, and lists around the length from which a tile's first batch is half a batch, of
faint entries (the whole list counts) and of opaque ones (the tile ends within
its first batch, or just past it): the image-only kernel against the counting
kernel, bit for bit (tolerance 0)."""
import numpy as np
import pytest

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_render_tiles import both, scene  # noqa: E402


@pytest.mark.parametrize("n", [127, 128, 129, 1535, 1536, 1537, 1663, 1664, 1665, 1793, 4000])
@pytest.mark.parametrize("opacity", [(0.004, 0.006), (0.02, 0.1), (0.9, 0.99)], ids=["faint", "middling", "opaque"])
def test_long_lists(n, opacity):
    rec, co, cl = scene(16, 16, n, n, ratio=(0.8, 1.0), opacity=opacity)
    rec["mean_x"], rec["mean_y"] = np.random.default_rng(n).integers(0, 256, (2, n))
    rec["radius"] = 24
    co[:, 0], co[:, 1], co[:, 2] = 1 / 64.0, 0, 1 / 64.0
    print(f"list of {n}", flush=True)
    both(16, 16, rec, co, cl)


@pytest.mark.parametrize("W,H,tiles", [(640, 360, 920), (50, 40, 12), (16, 16, 1)])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_sparse_frames(W, H, tiles, extra):
    n = 4 * tiles + extra
    print(f"{W}x{H} n={n}", flush=True)
    both(W, H, *scene(W, H, n, n))
