"""The depth order of the entries at the edges of its sort: one block, the
row and column counts of 256 buckets, 1024 buckets, LDS buckets of every size
and buckets sorted in global memory (many equal depths beside others).  The
sorted pairs must hold every entry once per bin it touches, bins ascending,
depths ascending in a bin, ids ascending on ties."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


def depths(kind, n, rng):
    z = rng.uniform(-1.0, 1.0, n)
    if kind == "equal":
        z[:] = 0.25
    elif kind == "few":
        z = rng.integers(0, 5, n) * 0.25 - 0.5
    elif kind == "duplicates":      # most at one depth, the rest next to it: one bucket over the LDS capacity
        z = np.where(rng.uniform(size=n) < 0.9, 0.5, 0.5 + rng.uniform(-1e-4, 1e-4, n))
    elif kind == "outlier":
        z = 0.1 + rng.uniform(0, 1e-3, n)
        z[n // 2] = 1e6
    elif kind == "ascending":
        z = np.sort(z)
    elif kind == "descending":
        z = np.sort(z)[::-1].copy()
    elif kind == "behind":          # half of the entries behind the camera
        z = rng.uniform(-9.0, 1.0, n)
    return z.astype(np.float32)


def check(n, kind, views=1, bin_tile=16):
    rng = np.random.default_rng(n + len(kind))
    g = api.Gaussians.empty(n, 0)
    xy = rng.uniform(-1.2, 1.2, (2, n)).astype(np.float32)
    g.means.copy_(torch.from_numpy(np.stack([xy[0], xy[1], depths(kind, n, rng)])))
    g.log_scales.fill_(-6.0)
    g.quats[0] = 1.0
    ctx = api.Context(0)
    api.set_tuning(ctx, bin_tile=bin_tile)
    cam = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), 200, 150, 60.0)
    frame = api.BatchFrame.for_views(ctx, n, [cam] * views, key_cap=8 * n * views + 1024)
    api.render_batch(ctx, g, [cam] * views, frame)
    st = frame.host_state(n)
    ne = n * views
    v0 = frame.view(0)
    depth = frame._dev(v0.depth_key, 4 * ne).view(np.uint32)
    nt = frame._dev(v0.ntiles, 4 * ne).view(np.uint32)
    vals, tk = st["vals"].astype(np.int64), st["tile_keys"].astype(np.int64)
    assert st["n_keys"] == int(nt.sum()) == len(vals)
    np.testing.assert_array_equal(np.bincount(vals, minlength=ne), nt)
    key = np.stack([tk, depth[vals].astype(np.int64), vals])
    step = np.diff(key, axis=1)
    ok = (step[0] > 0) | ((step[0] == 0) & ((step[1] > 0) | ((step[1] == 0) & (step[2] > 0))))
    assert ok.all(), int((~ok).sum())


@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1025, 2049, 4096, 4097, 8193, 131_072, 131_073, 524_288,
                               524_289, 1_310_720, 1_310_721])
def test_depth_order_at_size_edges(n):
    check(n, "random")


@pytest.mark.parametrize("n", [5000, 60_000, 600_000])
@pytest.mark.parametrize("kind", ["equal", "few", "duplicates", "outlier", "ascending", "descending", "behind"])
def test_depth_order_of_distributions(n, kind):
    check(n, kind)


@pytest.mark.parametrize("n,views,kind", [(3000, 5, "random"), (350_000, 8, "random"), (400_000, 8, "duplicates"),
                                          (330_000, 16, "few"), (2_621_441, 1, "random")])
def test_depth_order_of_many_entries(n, views, kind):
    check(n, kind, views, bin_tile=32)
