"""The image-only rendering kernel, which leaves list entries out of the 8 x 8
blocks that they cannot reach, against the counting kernel, which evaluates
every entry at every pixel and is itself checked against the render oracle:
colour and T bit for bit, at image edges and with conics, opacities and list
lengths at the edges of the reach bound (tolerance 0: the same arithmetic on
every entry that changes a pixel)."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2511_16298_amd as ss  # noqa: E402


def both(W, H, rec, co, cl, bg=(0.1, 0.2, 0.3)):
    d = ss.records_to_device(rec)
    out = ss.sort_frame(d, W, H)
    assert out.result()[0] == 0
    cod, cld = ss.render_attrs_to_device(co, cl)
    got = []
    for counting in (False, True):
        r = ss.Renderer(W, H, want_T=True, want_contrib=counting)
        r.out.color.fill_(-7.0)
        o = r(d, cod, cld, out.values, out.tile_ranges, out.status, bg)
        torch.cuda.synchronize()
        got.append((o.color.cpu().numpy().view(np.uint32), o.T.cpu().numpy().view(np.uint32)))
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])


def scene(W, H, n, seed, ratio=(0.25, 1.0), opacity=(0.02, 0.99), shrink=(0.3, 1.0)):
    """Gaussians of mixed size; conics with the given ratio of deviations."""
    rs = np.random.default_rng(seed)
    rec = np.zeros(n, synth.RECORD_DTYPE)
    rec["mean_x"] = rs.integers(-200, 16 * W + 200, n)
    rec["mean_y"] = rs.integers(-200, 16 * H + 200, n)
    rec["radius"] = np.maximum(1, np.exp(rs.uniform(0, np.log(max(W, H)), n))).astype(np.uint32)
    rec["depth"] = np.exp(rs.uniform(-1, 4, n)).astype(np.float32)
    s1 = rec["radius"] / 3.0 * rs.uniform(*shrink, n)
    s2 = s1 * np.exp(rs.uniform(np.log(ratio[0]), np.log(ratio[1]), n))
    th = rs.uniform(0, np.pi, n)
    c, s = np.cos(th), np.sin(th)
    xx, yy, xy = (s1 * c) ** 2 + (s2 * s) ** 2, (s1 * s) ** 2 + (s2 * c) ** 2, (s1 ** 2 - s2 ** 2) * s * c
    det = (s1 * s2) ** 2
    co = np.stack([yy / det, -xy / det, xx / det, rs.uniform(*opacity, n)], 1).astype(np.float32)
    cl = np.concatenate([rs.random((n, 3)), np.zeros((n, 1))], 1).astype(np.float32)
    return rec, co, cl


@pytest.mark.parametrize("W,H,n", [(1, 1, 40), (8, 8, 300), (9, 7, 300), (17, 33, 1000), (100, 60, 5000),
                                   (250, 131, 20_000), (16, 2048, 3000), (640, 360, 50_000),
                                   (640, 360, 3679), (640, 360, 3680)])
def test_sizes(W, H, n):
    print(f"{W}x{H} n={n}", flush=True)
    both(W, H, *scene(W, H, n, n + W))


@pytest.mark.parametrize("n", [255, 256, 257, 511, 513, 1024])
def test_list_lengths_around_a_batch(n):
    """One tile whose list fills batches of 256 entries just so."""
    rec, co, cl = scene(16, 16, n, n, opacity=(0.004, 0.03))
    rec["mean_x"], rec["mean_y"] = np.random.default_rng(n).integers(0, 256, (2, n))
    both(16, 16, rec, co, cl)


@pytest.mark.parametrize("ratio", [(0.9, 1.0), (0.01, 0.02), (0.001, 0.011), (1e-4, 1e-3)])
def test_elongated(ratio):
    """Narrow footprints, on both sides of the ratio up to which the bound is
    trusted."""
    both(200, 120, *scene(200, 120, 4000, 17, ratio=ratio, shrink=(1.0, 4.0)))


@pytest.mark.parametrize("opacity", [(0.0039, 0.00393), (0.00392157, 0.0040), (0.98, 1.0), (1.0, 50.0)])
def test_opacities(opacity):
    both(120, 90, *scene(120, 90, 3000, 23, opacity=opacity))


def test_degenerate_conics():
    """Conics that are not positive definite, zero, infinite or NaN, and
    opacities of 0: evaluated as they are or without effect, never bounded."""
    rec, co, cl = scene(120, 90, 4000, 29)
    rs = np.random.default_rng(31)
    k = rs.integers(0, 12, len(rec))
    co[k == 1, 0] *= -1
    co[k == 2, 2] = 0
    co[k == 3, 1] = 10 * np.abs(co[k == 3, 0]) + 1
    co[k == 4, 0] = np.inf
    co[k == 5, 1] = np.nan
    co[k == 6, 3] = 0
    co[k == 7, :3] = 0
    co[k == 8, 3] = np.nan
    co[k == 9, :3] *= 1e30
    co[k == 10, :3] *= 1e-30
    both(120, 90, rec, co, cl)
