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
import test_gpu_parity as parity  # noqa: E402  (its cases)
import test_gpu_spread as spread  # noqa: E402  (its records)
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


# ------------------------------------------------------------- digit passes
# (items_per_thread = 8 asks for them where the default takes the spread passes)

@pytest.mark.parametrize("case", parity.PACKED_CASES, ids=lambda c: f"{c[0]}x{c[1]}-n{c[2]}-{c[5]}")
def test_digit_passes_both_depth_fields(case):
    """Packed pairs with the trimmed depth field and with the depth-order
    position, expanded and unpacked by the digit passes."""
    tx, ty, n, lo, hi, mode = case
    W, H = 16 * tx, 16 * ty
    rec = synth.make_frame(synth.FrameSpec(W, H, n, depth_lo=lo, depth_hi=hi), 7100 + tx)
    cnt, _ = oracle.count(W, H, rec)
    assert parity.depth_field_mode(int(np.ceil(np.log2(tx * ty))), n, rec["depth"][cnt > 0]) == mode
    print(f"{tx}x{ty} N={n} depth [{lo}, {hi}] -> {mode}", flush=True)
    o = oracle.sort_frame(W, H, rec, stages=False)
    s = ss.FrameSorter(W, H, n, o.num_pairs, items_per_thread=8)
    assert route(s, ss.records_to_device(rec)) == "digits"
    check_frame(s, o)


@pytest.mark.parametrize("lo,hi,mode", [(0.5, 50.0, "trimmed"), (1e-6, 1e6, "position")])
def test_digit_passes_of_16_items(lo, hi, mode):
    """2^23 pairs and more on a grid beyond the spread passes: packed passes
    of 8,192 pairs, one workgroup per tile of them."""
    tx, ty, n = 257, 135, 1_500_000
    W, H = 16 * tx, 16 * ty
    rec = synth.make_frame(synth.FrameSpec(W, H, n, sigma_mu=1.5, depth_lo=lo, depth_hi=hi), 9700)
    cnt, _ = oracle.count(W, H, rec)
    assert parity.depth_field_mode(int(np.ceil(np.log2(tx * ty))), n, rec["depth"][cnt > 0]) == mode
    o = oracle.sort_frame(W, H, rec, stages=False)
    assert o.num_pairs >= 1 << 23
    s = ss.FrameSorter(W, H, n, o.num_pairs)
    assert route(s, ss.records_to_device(rec)) == "digits"
    check_frame(s, o)


@pytest.mark.parametrize("case", parity.DEPTH_RANGE_CASES, ids=lambda c: f"{c[0]}-{c[1]}")
@pytest.mark.parametrize("drop", [False, True])
def test_digit_passes_depth_ranges(case, drop):
    lo, hi, span = case
    W, H, n = 1920, 1080, 300_000
    rec = synth.make_frame(synth.FrameSpec(W, H, n, depth_lo=lo, depth_hi=hi), 7300 + span)
    rec["radius"][::4] = 0
    o = oracle.sort_frame(W, H, rec, stages=False)
    s = ss.FrameSorter(W, H, n, o.num_pairs, items_per_thread=8, drop_culled=drop)
    assert route(s, ss.records_to_device(rec)) == "digits"
    check_frame(s, o)


@pytest.mark.parametrize("frames", [1, 5])
@pytest.mark.parametrize("shape,want", [({}, "spread"), ({"items_per_thread": 8}, "digits")], ids=["spread", "digits"])
def test_timeouts(shape, want, frames):
    """Counts (spread passes) or digit bases (digit passes, one workgroup per
    tile) withheld: every kernel ends and the status says so; then exact."""
    batch = [(1280, 720, synth.make_frame(synth.FrameSpec(1280, 720, 60_000), 9800 + i)) for i in range(frames)]
    o = oracle.sort_batch(batch)
    m0 = int(o.num_pairs.sum())
    d = [ss.records_to_device(r) for (_, _, r) in batch]
    shapes = [(w, h, len(r)) for (w, h, r) in batch]
    bad = ss.BatchSorter(shapes, m0, spin_limit=32, fault=_abi.SS_FAULT_WITHHOLD_BASES, **shape)
    assert route(bad, d) == want
    assert bad.result()[0] == _abi.SS_ERR_TIMEOUT
    good = ss.BatchSorter(shapes, m0, **shape)
    assert route(good, d) == want
    st, m = good.result()
    assert st == 0 and m == m0
    assert np.array_equal(u64(good.keys)[:m], o.keys)
    assert np.array_equal(u32(good.values)[:m], o.values)
    assert np.array_equal(u32(good.tile_ranges).reshape(-1, 2), o.ranges)


# ------------------------------------------------------------- spread passes

def spread_frame(tx, ty, rec):
    W, H = 16 * tx, 16 * ty
    o = oracle.sort_frame(W, H, rec, stages=False)
    s = ss.FrameSorter(W, H, len(rec), o.num_pairs + spread.ROOM)
    assert route(s, ss.records_to_device(rec)) == "spread"
    check_frame(s, o)


@pytest.mark.parametrize("tx,ty,n", [
    (8, 33, 9000), (33, 8, 9000), (16, 17, 6000), (17, 16, 2049), (65, 64, 6000), (80, 80, 3000), (81, 80, 3000),
    (80, 81, 3000), (127, 129, 2500), (8, 160, 6000), (160, 8, 6000), (160, 160, 2500)])
def test_spread_grids(tx, ty, n):
    print(f"grid {tx}x{ty} n={n}", flush=True)
    spread_frame(tx, ty, spread.records(tx, ty, n, 1000 * tx + ty, big=0.05 if tx * ty < 20_000 else 0.01))


@pytest.mark.parametrize("ty,items", [(64, 4096), (81, 2048)])
@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("workgroups", [1, 2, 3])
def test_spread_items_around_a_workgroup(ty, items, extra, workgroups):
    """A tile column whose items just miss, fill or overflow whole workgroups
    of the row pass, in a grid with empty columns beside it."""
    n = items * workgroups + extra
    rec = spread.records(1, ty, n, n, big=0.0, few_depths=False)
    rs = np.random.default_rng(n)
    rec["mean_x"], rec["mean_y"] = 256 * 17 + 128, rs.integers(0, 256 * ty, n)
    rec["radius"] = rs.integers(1, 8, n)
    tall = rs.random(n) < 0.5          # off the column's side, reaching just into it, and high
    rec["radius"][tall] = rs.integers(20, 120, int(tall.sum()))
    rec["mean_x"][tall] = -16 * rec["radius"][tall].astype(np.int32) + 5
    rec["mean_x"][~tall] -= 256 * 17
    print(f"column of {n} items, {ty} rows", flush=True)
    spread_frame(20, ty, rec)


@pytest.mark.parametrize("wide", [0, 4])
def test_spread_uneven_batch(wide):
    """Frames of one Gaussian, none, all culled, one tile, tall and wide; with
    full-HD frames beside them the columns are many and thinly filled, and the
    row pass takes its smallest workgroups, one column just past one of them."""
    frames = [(1920, 1080, spread.records(120, 68, 3000, 90 + i, big=0.0)) for i in range(wide)]
    if wide:
        one = spread.records(1, 30, 1025, 99, big=0.0)
        one["mean_x"], one["radius"] = 128, np.maximum(one["radius"], 1)
        frames.append((16, 480, one))
    for i, (tx, ty, n) in enumerate([(40, 23, 9000), (1, 1, 300), (7, 2, 0), (120, 68, 20_000), (2, 80, 5000),
                                     (150, 3, 5000), (16, 16, 1), (9, 9, 2048), (30, 70, 4097)]):
        rec = spread.records(tx, ty, n, 50 + i, big=0.02, few_depths=i % 2 == 0)
        if i == 7:
            rec["radius"] = 0
        frames.append((16 * tx, 16 * ty, rec))
    o = oracle.sort_batch(frames)
    m0 = int(o.num_pairs.sum())
    s = ss.BatchSorter([(w, h, len(r)) for (w, h, r) in frames], m0 + 4 * spread.ROOM)
    assert route(s, [ss.records_to_device(r) for (_, _, r) in frames]) == "spread"
    st, m = s.result()
    assert st == 0 and m == m0
    assert np.array_equal(u64(s.keys)[:m], o.keys)
    assert np.array_equal(u32(s.values)[:m], o.values)
    assert np.array_equal(u32(s.tile_ranges).reshape(-1, 2), o.ranges)
    assert np.array_equal(u32(s.frame_pairs), o.num_pairs.astype(np.uint32))
    assert np.array_equal(u32(s.frame_pair_base), o.pair_base.astype(np.uint32))


# ------------------------------------------------------------- small frames

@pytest.mark.parametrize("n", [0, 1, 3000, 16_384])
def test_small_frames_without_status_and_count(n):
    """Without the caller's words for them, the status and the pair count lie
    in the workspace's first two; an exact workspace serves."""
    rec = synth.make_frame(synth.FrameSpec(256, 256, max(n, 1)), 9900)[:n]
    o = oracle.sort_frame(256, 256, rec, stages=False)
    s = ss.FrameSorter(256, 256, n, o.num_pairs)
    s._cout.status = s._cout.num_pairs = None
    s.workspace = torch.full((s.workspace_bytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    assert route(s, ss.records_to_device(rec)) == "small"
    words = s.workspace[:8].cpu().numpy().view(np.uint32)
    assert words[0] == 0 and words[1] == o.num_pairs
    assert bool((s.workspace[s.workspace_bytes:] == 0x5A).all().item())
    assert np.array_equal(u64(s.out.keys)[:o.num_pairs], o.keys)
    assert np.array_equal(u32(s.out.values)[:o.num_pairs], o.values)
    assert np.array_equal(u32(s.out.tile_ranges).reshape(-1, 2), o.ranges)
