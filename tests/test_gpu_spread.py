"""The spread passes (column pass, row pass) where they can go wrong: grids of
one tile to 256 tiles per axis and just past it, columns of items around the
workgroup sizes, lists longer than a workgroup holds, empty columns and rows,
culled Gaussians, uneven batches.  Against the oracle and against the digit
passes (asked for by their shape), bit for bit (tolerance 0)."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_16298_amd as ss  # noqa: E402

#: spare pair capacity: the spread passes serve a frame only inside the digit
#: passes' workspace, which is the larger one where pairs outnumber the grid
ROOM = 300_000


def u64(t):
    return t.cpu().numpy().view(np.uint64)


def u32(t):
    return t.cpu().numpy().view(np.uint32)


def check(W, H, rec, **kw):
    ref = oracle.sort_frame(W, H, rec)
    assert ref.status == 0
    d = ss.records_to_device(rec)
    # stages: asking for the per-Gaussian outputs keeps small frames off the small-frame kernels
    for shape in ({}, {"items_per_thread": 8}):
        s = ss.FrameSorter(W, H, len(rec), ref.num_pairs + ROOM, stages=True, **shape, **kw)
        out = s(d)
        st, m = out.result()
        assert st == 0 and m == ref.num_pairs, (shape, st, m, ref.num_pairs)
        assert np.array_equal(u64(out.keys)[:m], ref.keys), shape
        assert np.array_equal(u32(out.values)[:m], ref.values), shape
        assert np.array_equal(u32(out.tile_ranges).reshape(-1, 2), ref.ranges), shape
        assert np.array_equal(u32(out.tiles_touched)[:len(rec)], ref.tiles_touched), shape


def records(tx, ty, n, seed, big=0.05, few_depths=True):
    """Gaussians of mixed size on a tx x ty grid: mostly a few tiles, some off
    the image, a share `big` covering much of it; ties in depth."""
    rs = np.random.default_rng(seed)
    rec = np.zeros(n, synth.RECORD_DTYPE)
    rec["mean_x"] = rs.integers(-400, 256 * tx + 400, n)
    rec["mean_y"] = rs.integers(-400, 256 * ty + 400, n)
    rec["radius"] = rs.integers(0, 40, n)
    k = rs.random(n) < big
    rec["radius"][k] = rs.integers(1, 16 * max(tx, ty) + 1, int(k.sum()))
    rec["depth"] = rs.choice(np.float32([0.25, 1.0, 1.5, 7.0, 300.0]), n) if few_depths \
        else np.exp(rs.uniform(-2, 5, n)).astype(np.float32)
    return rec


@pytest.mark.parametrize("tx,ty,n", [
    (1, 1, 5000), (2, 1, 5000), (1, 2, 5000), (1, 16, 4097), (16, 17, 6000), (17, 16, 2049), (33, 3, 6000),
    (3, 33, 6000), (80, 80, 3000), (81, 80, 3000), (80, 81, 3000), (120, 68, 9000), (129, 127, 2500),
    (255, 256, 700), (256, 255, 700), (256, 256, 900), (257, 5, 2500), (5, 257, 2500)])
def test_grids(tx, ty, n):
    print(f"grid {tx}x{ty} n={n}", flush=True)
    check(16 * tx, 16 * ty, records(tx, ty, n, 1000 * tx + ty, big=0.05 if tx * ty < 20_000 else 0.01))


@pytest.mark.parametrize("ty,items", [(64, 4096), (81, 2048)])
@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("workgroups", [1, 2, 3])
def test_items_around_a_workgroup(ty, items, extra, workgroups):
    """One tile column whose items just miss, fill or overflow whole
    workgroups of the row pass (and of the column pass)."""
    n = items * workgroups + extra
    print(f"column of {n} items, {ty} rows", flush=True)
    rec = records(1, ty, n, n, big=0.01, few_depths=False)
    rec["mean_x"] = 128
    rec["mean_y"] = np.random.default_rng(n).integers(0, 256 * ty, n)
    rec["radius"] = np.maximum(rec["radius"], 1)
    check(16, 16 * ty, rec)


@pytest.mark.parametrize("n", [1, 2047, 3000])
def test_long_lists(n):
    """Every Gaussian covers the whole grid: lists many times longer than a
    workgroup's, digits with more outputs than one round holds."""
    print(f"covering n={n}", flush=True)
    rec = records(24, 20, n, n, few_depths=False)
    rec["mean_x"], rec["mean_y"], rec["radius"] = 128 * 24, 128 * 20, 10_000
    check(16 * 24, 16 * 20, rec)


@pytest.mark.parametrize("where", ["first", "last", "middle", "two", "none"])
def test_empty_columns_and_rows(where):
    tx, ty, n = 40, 30, 6000
    rec = records(tx, ty, n, 7, big=0.0, few_depths=False)
    rec["radius"] = 3
    rs = np.random.default_rng(5)
    col = {"first": [0], "last": [tx - 1], "middle": [17], "two": [3, 36], "none": [-5]}[where]
    rec["mean_x"] = 256 * rs.choice(col, n) + 128
    rec["mean_y"] = 256 * rs.choice([4, 25], n) + 128
    check(16 * tx, 16 * ty, rec)


@pytest.mark.parametrize("drop", [False, True])
@pytest.mark.parametrize("share", [0.0, 0.5, 0.999])
def test_culled(share, drop):
    rec = records(50, 40, 30_000, 11, big=0.01, few_depths=False)
    k = np.random.default_rng(3).random(len(rec)) < share
    rec["radius"][k] = 0
    check(800, 640, rec, drop_culled=drop)


@pytest.mark.parametrize("wide", [0, 4])
def test_uneven_batch(wide):
    """Frames of one Gaussian, none, all culled, one tile, tall and wide, in
    one segmented sort; with full-HD frames beside them the columns are many
    and thinly filled, and the row pass takes its smallest workgroups, one
    column just past one of them."""
    frames = [(1920, 1080, records(120, 68, 3000, 90 + i, big=0.0)) for i in range(wide)]
    if wide:
        one = records(1, 30, 1025, 99, big=0.0)
        one["mean_x"], one["radius"] = 128, np.maximum(one["radius"], 1)
        frames.append((16, 480, one))
    for i, (tx, ty, n) in enumerate([(40, 23, 9000), (1, 1, 300), (7, 2, 0), (120, 68, 20_000), (2, 80, 5000),
                                     (200, 3, 5000), (16, 16, 1), (9, 9, 2048), (30, 70, 4097)]):
        rec = records(tx, ty, n, 50 + i, big=0.02, few_depths=i % 2 == 0)
        if i == 7:
            rec["radius"] = 0
        frames.append((16 * tx, 16 * ty, rec))
    ref = oracle.sort_batch(frames)
    m0 = int(ref.num_pairs.sum())
    for shape in ({}, {"items_per_thread": 8}):
        b = ss.BatchSorter([(w, h, len(r)) for (w, h, r) in frames], m0 + 4 * ROOM, **shape)
        b([ss.records_to_device(r) for (_, _, r) in frames])
        st, m = b.result()
        assert st == 0 and m == m0
        assert np.array_equal(u64(b.keys)[:m], ref.keys)
        assert np.array_equal(u32(b.values)[:m], ref.values)
        assert np.array_equal(u32(b.tile_ranges).reshape(-1, 2), ref.ranges)
        assert np.array_equal(u32(b.frame_pairs), ref.num_pairs.astype(np.uint32))
        assert np.array_equal(u32(b.frame_pair_base), ref.pair_base.astype(np.uint32))
