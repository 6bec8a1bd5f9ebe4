"""The one-kernel path of small frames where it can go wrong: tile lists
around the sizes at which the ordering changes its way, Gaussian counts around
a workgroup's loads, means and radii too large for 32-bit sums.  Against the
oracle, bit for bit (tolerance 0)."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_16298_amd as ss  # noqa: E402


def check(W, H, rec):
    ref = oracle.sort_frame(W, H, rec, stages=False)
    assert ref.status == 0
    s = ss.FrameSorter(W, H, len(rec), ref.num_pairs)
    out = s(ss.records_to_device(rec))
    st, m = out.result()
    assert st == 0 and m == ref.num_pairs
    assert np.array_equal(out.keys.cpu().numpy().view(np.uint64)[:m], ref.keys)
    assert np.array_equal(out.values.cpu().numpy().view(np.uint32)[:m], ref.values)
    assert np.array_equal(out.tile_ranges.cpu().numpy().view(np.uint32).reshape(-1, 2), ref.ranges)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 8191, 8193, 16383, 16384])
def test_lists(n):
    """One tile whose list is the whole frame, beside tiles with less of it;
    ties in depth."""
    print(f"list of {n}", flush=True)
    rs = np.random.default_rng(n)
    rec = np.zeros(n, synth.RECORD_DTYPE)
    rec["mean_x"], rec["mean_y"] = 256 * 3 + 128, 256 * 2 + 128
    rec["radius"] = np.where(rs.random(n) < 0.3, rs.integers(9, 60, n), 1)
    rec["depth"] = rs.choice(np.exp(rs.uniform(-3, 6, max(1, n // 3))).astype(np.float32), n)
    check(100, 90, rec)


@pytest.mark.parametrize("W,H", [(1, 1), (16, 4096), (4096, 16), (250, 250)])
def test_wide_values(W, H):
    """Means and radii at the ends of their types beside ordinary ones, some
    wavefronts with them and some without."""
    n = 3000
    rs = np.random.default_rng(W)
    rec = synth.make_frame(synth.FrameSpec(W, H, n), 5)
    k = rs.integers(0, 400, n)
    k[:1024] = 99
    rec["radius"][k == 0] = 0xFFFFFFFF
    rec["radius"][k == 1] = 1 << 25
    rec["radius"][k == 2] = (1 << 25) - 1
    rec["mean_x"][k == 3] = 2**31 - 1
    rec["mean_x"][k == 4] = -(2**31)
    rec["mean_y"][k == 5] = 1 << 29
    rec["mean_y"][k == 6] = -(1 << 29)
    far = k == 7
    rec["mean_x"][far], rec["radius"][far] = 2**31 - 1, 1 << 27
    check(W, H, rec)
