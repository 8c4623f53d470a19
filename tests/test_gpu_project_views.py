"""Projection of several views of one set (a thread per Gaussian walking the
views) against the single-view kernel: depth keys, records, boxes and tile
counts bit for bit, for every SH degree, row counts off the block size, sets
shared by some views only, uneven sets, and both row addressings."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


def projected(frame, view, n):
    v = frame.view(view)
    return [frame._dev(v.depth_key, 4 * n), frame._dev(v.rec, 48 * n), frame._dev(v.box, 8 * n), frame._dev(v.ntiles, 4 * n)]


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("ns,shown,addr64", [
    ([120_001, 1_000], [0, 0, 0, 1, 0, 0, 0, 0, 0, 0, 1], False),   # walked in twos; the small set's views too
    ([400_003], [0, 0, 0, 0], True),
    ([300_000, 255, 1], [0, 1, 2], False),                          # nothing shared, sizes far apart
    ([2_000], [0, 0, 0], False)])                                   # too few blocks to walk views
def test_views_of_one_set_match_single_views(deg, ns, shown, addr64):
    rng = np.random.default_rng(deg)
    sets = []
    for k, n in enumerate(ns):
        g = torch.Generator(device="cuda").manual_seed(10 * deg + k)
        randn = lambda *s: torch.randn(*s, generator=g, device="cuda")
        means = randn(3, n) * 1.5          # some behind the cameras, some outside the images
        sets.append(api.Gaussians(means, randn(3, n) * 0.8 - 4, randn(4, n), randn(n) * 3, randn((deg + 1) ** 2, 3, n) * 0.3, deg))
    cams = [synth.random_pose_camera(rng, 3.0, 200 + 16 * k, 150) for k in range(len(shown))]
    ctx = api.Context(0)
    api.debug_row_addressing(ctx, addr64)
    scenes = [sets[k] for k in shown]
    frame = api.BatchFrame.for_views(ctx, [s.n for s in scenes], cams, key_cap=8 * sum(s.n for s in scenes))
    api.render_batch(ctx, scenes, cams, frame)
    for v, (s, cam) in enumerate(zip(scenes, cams)):
        one = api.Frame(ctx, s.n, cam.width, cam.height, key_cap=8 * s.n + 64)
        api.render(ctx, s, cam, one)
        for a, b in zip(projected(frame, v, s.n), projected(one, 0, s.n)):
            assert np.array_equal(a, b)
        one.close()
