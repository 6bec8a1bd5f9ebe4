"""Passes whose workgroups look back in tiers of sixteen: workgroup counts
around whole tiers, and around the launch sizes up to which the tiers are
taken.  Stable order against numpy's, bit for bit (tolerance 0)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_16298_amd as ss  # noqa: E402
import synth  # noqa: E402


@pytest.mark.parametrize("workgroups", [1, 15, 16, 17, 31, 32, 33, 48, 511, 512, 513])
@pytest.mark.parametrize("items", [8, 16])
@pytest.mark.parametrize("extra", [0, 1])
def test_pairs(workgroups, items, extra):
    """Key + value passes of 4,096- and 8,192-pair workgroups, asked for and
    (on both sides of 1.25M pairs) taken by default; few distinct keys, so
    that stability shows."""
    n = 512 * items * workgroups - (1 - extra) * 5
    print(f"{workgroups} workgroups, n={n}", flush=True)
    rs = np.random.default_rng(n)
    keys = rs.integers(0, 1 << 45, 97, dtype=np.int64)[rs.integers(0, 97, n)]
    k, v = ss.sort_pairs(torch.from_numpy(keys).cuda(), torch.arange(n, dtype=torch.int32, device="cuda"), 45,
                         items_per_thread=items if extra else 0)
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(v.cpu().numpy(), order.astype(np.int32))
    assert np.array_equal(k.cpu().numpy(), keys[order])


@pytest.mark.parametrize("workgroups", [1, 15, 16, 17, 33, 255, 256, 257])
def test_depth_sort(workgroups):
    """Depth passes of 4,096-Gaussian workgroups: one tile, so that the frame's
    order is the Gaussians' stable depth order."""
    n = 4096 * workgroups - 3
    print(f"{workgroups} workgroups, n={n}", flush=True)
    rs = np.random.default_rng(n)
    rec = np.zeros(n, synth.RECORD_DTYPE)
    rec["mean_x"] = rec["mean_y"] = 128
    rec["radius"] = 1
    rec["depth"] = rs.choice(np.exp(rs.uniform(-3, 6, 500)).astype(np.float32), n)
    s = ss.FrameSorter(16, 16, n, n, stages=True)
    out = s(ss.records_to_device(rec))
    st, m = out.result()
    assert st == 0 and m == n
    assert np.array_equal(out.values.cpu().numpy()[:n], np.argsort(rec["depth"], kind="stable").astype(np.int32))
