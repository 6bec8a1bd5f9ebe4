"""Which passes a call takes, read from the timer's kernel kinds (the digit
passes have a launch for the ranges, the spread passes none), and that its
result is the oracle's either way (tolerance 0)."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_16298_amd as ss  # noqa: E402
from paper_2511_16298_amd import _abi  # noqa: E402


def u64(t):
    return t.cpu().numpy().view(np.uint64)


def u32(t):
    return t.cpu().numpy().view(np.uint32)


def route(sorter, records):
    """Sorts, and tells "spread", "digits" or "small" (the one-kernel path)."""
    t = ss.Timer()
    sorter(records, timer=t)
    torch.cuda.synchronize()
    depth, ranges = t.read(_abi.SS_KERNEL_DEPTH_PASS)[1], t.read(_abi.SS_KERNEL_RANGES)[1]
    t.close()
    return "small" if depth == 0 else "digits" if ranges else "spread"


def check_frame(sorter, o):
    st, m = sorter.out.result()
    assert st == 0 and m == o.num_pairs
    assert np.array_equal(u64(sorter.out.keys)[:m], o.keys)
    assert np.array_equal(u32(sorter.out.values)[:m], o.values)
    assert np.array_equal(u32(sorter.out.tile_ranges).reshape(-1, 2), o.ranges)


@pytest.mark.parametrize("tx,ty,n,want", [
    (120, 68, 30_000, "spread"), (160, 8, 30_000, "spread"), (8, 160, 30_000, "spread"), (40, 23, 20_000, "spread"),
    (161, 8, 30_000, "digits"), (8, 161, 30_000, "digits"), (40, 7, 30_000, "digits"), (7, 40, 30_000, "digits"),
    (16, 16, 20_000, "spread"), (32, 8, 200_000, "digits"), (256, 1, 30_000, "digits"), (1, 1, 20_000, "digits"),
    (240, 135, 50_000, "digits"), (16, 16, 16_384, "small")])
def test_frames(tx, ty, n, want):
    W, H = 16 * tx, 16 * ty
    print(f"{tx}x{ty} n={n}", flush=True)
    rec = synth.make_frame(synth.FrameSpec(W, H, n, sigma_mu=0.7), 9500 + tx)
    o = oracle.sort_frame(W, H, rec, stages=False)
    s = ss.FrameSorter(W, H, n, o.num_pairs + o.num_pairs // 8)
    assert route(s, ss.records_to_device(rec)) == want
    check_frame(s, o)


@pytest.mark.parametrize("room", [1, 3, 12])
@pytest.mark.parametrize("frames,n,want", [(64, 5000, "digits"), (10, 20_000, "spread")])
def test_spare_capacity_does_not_change_the_route(frames, n, want, room):
    """Full-HD frames in buffers of one, three and twelve times their pairs."""
    batch = [(1920, 1080, synth.make_frame(synth.FrameSpec(1920, 1080, n), 9600 + i)) for i in range(frames)]
    o = oracle.sort_batch(batch)
    m0 = int(o.num_pairs.sum())
    s = ss.BatchSorter([(w, h, len(r)) for (w, h, r) in batch], room * m0)
    assert route(s, [ss.records_to_device(r) for (_, _, r) in batch]) == want
    st, m = s.result()
    assert st == 0 and m == m0
    assert np.array_equal(u64(s.keys)[:m], o.keys)
    assert np.array_equal(u32(s.values)[:m], o.values)
    assert np.array_equal(u32(s.tile_ranges).reshape(-1, 2), o.ranges)
