"""Which forward renders are dispatched longest list first: batch depths and
persistent grids around the tiles from which on they are (two, three and five
a CU, 256 CUs), images bit-identical to those in tile order; and the time of
a render whose long lists come last in tile order."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


def render(g, cam, reps=1, **tuning):
    ctx = api.Context(0)
    api.set_tuning(ctx, **tuning)
    frame = api.Frame(ctx, g.n, cam.width, cam.height, key_cap=1 << 21, auto_grow=False, forward_only=True)
    times = []
    for _ in range(reps):
        api.timing_enable(ctx, True)
        image = api.render(ctx, g, cam, frame)
        torch.cuda.synchronize()
        times.append(api.timing_read(ctx)["blend_fwd"][0])
    return image, min(times)


@pytest.mark.parametrize("tiles", [(32, 16), (513, 1), (32, 24), (769, 1), (40, 32), (61, 21)])   # 512, 768, 1280 and one more
@pytest.mark.parametrize("batch,persistent", [(256, False), (512, False), (1024, False), (256, True), (1024, True)])
@pytest.mark.parametrize("bin_tile", [16, 32])
def test_images_do_not_depend_on_the_order(tiles, batch, persistent, bin_tile):
    g = api.Gaussians.from_scene(synth.scene_uniform_sh0(2000, seed=5, log_scale_mu=-3.0))
    cam = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), 16 * tiles[0], 16 * tiles[1], 60.0)
    want, _ = render(g, cam, longest_first=False)
    got, _ = render(g, cam, longest_first=True, lds_batch=batch, persistent=persistent, bin_tile=bin_tile)
    assert torch.equal(got, want)


def test_long_lists_do_not_start_last():
    # long transparent lists in the last rows of tiles, short ones before them
    rng = np.random.default_rng(1)
    n = 60_000
    y = np.where(np.arange(n) < 50_000, rng.uniform(1.45, 1.7, n), rng.uniform(-1.7, 1.45, n))
    g = api.Gaussians.empty(n, 0)
    g.means.copy_(torch.from_numpy(np.stack([rng.uniform(-2.9, 2.9, n), y, rng.uniform(-0.1, 0.1, n)]).astype(np.float32)))
    g.log_scales.fill_(-3.5)
    g.quats[0] = 1.0
    g.opacity_logits.fill_(-4.0)
    cam = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), 640, 480, 60.0)
    _, ordered = render(g, cam, 6, longest_first=True, lds_batch=1024)
    _, plain = render(g, cam, 6, longest_first=False, lds_batch=1024)
    assert ordered <= 0.9 * plain   # 97 us against 120
