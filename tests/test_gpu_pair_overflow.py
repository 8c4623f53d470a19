"""Renders that need 2^32 pairs or more, binned in two levels: the prefix that
fits is written, the count saturates, and a growing frame says so."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402

W, H, BINS = 1920, 1080, 8160


def covering(n):
    """n Gaussians that each cover the whole view."""
    rng = np.random.default_rng(n)
    g = api.Gaussians.empty(n, 0)
    xyz = np.stack([rng.uniform(-0.1, 0.1, n), rng.uniform(-0.1, 0.1, n), rng.uniform(-1.0, 1.0, n)])
    g.means.copy_(torch.from_numpy(xyz.astype(np.float32)))
    g.log_scales.fill_(2.0)
    g.quats[0] = 1.0
    return g, synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), W, H, 60.0)


@pytest.mark.parametrize("n,cap", [(600_000, 1 << 22), (600_000, 514 * BINS + (1 << 20)), (4_300_000, 1 << 22)])
def test_the_prefix_that_fits_is_written(n, cap):
    ctx = api.Context(0)
    g, cam = covering(n)
    frame = api.Frame(ctx, n, W, H, key_cap=cap, auto_grow=False, forward_only=True)
    api.render(ctx, g, cam, frame)
    v = frame.view(0)
    nt = frame._dev(v.ntiles, 4 * n).view(np.uint32)
    assert (nt == BINS).all()
    fit = cap // BINS
    assert frame.n_keys() == api.MAX_PAIRS and frame.n_emitted() == fit * BINS
    first = np.argsort(frame._dev(v.depth_key, 4 * n).view(np.uint32), kind="stable")[:fit].astype(np.uint32)
    vals = frame._dev(v.vals, 4 * fit * BINS).view(np.uint32).reshape(BINS, fit)
    assert (vals == first).all()
    keys = frame._dev(v.keys, 4 * fit * BINS).view(np.uint32).reshape(BINS, fit)
    assert (keys == np.arange(BINS, dtype=np.uint32)[:, None]).all()
    r = frame._dev(v.ranges, 8 * BINS).view(np.uint32).reshape(BINS, 2)
    np.testing.assert_array_equal(r[:, 0], np.arange(BINS) * fit)
    np.testing.assert_array_equal(r[:, 1], (np.arange(BINS) + 1) * fit)


def test_a_growing_frame_says_that_no_capacity_is_enough():
    n = 600_000
    ctx = api.Context(0)
    g, cam = covering(n)
    frame = api.Frame(ctx, n, W, H, key_cap=1 << 22)
    with pytest.raises(api.AdpSplitError) as e:
        api.render(ctx, g, cam, frame)
    assert e.value.status == api.AS_ERR_CAPACITY and frame.key_cap == 1 << 22
