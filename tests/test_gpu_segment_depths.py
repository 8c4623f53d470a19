"""Checkpoint spacing of the reverse pass at batch depths of 512 and 1024: the
gradients of lists around the segments' boundaries are those at a depth of 256
(both walk the same contributors; T is divided back over at most 4100 of
a few ulp each, 1e-4 relative), and a deeper batch keeps its wider segments."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


def gradients(g, sizes, batch, dL):
    ctx = api.Context(0)
    api.set_tuning(ctx, lds_batch=batch)
    cams = [synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0 if k == 0 else -9.0), w, h, 30.0)
            for k, (w, h) in enumerate(sizes)]   # the second looks away
    frame = api.BatchFrame.for_views(ctx, g.n, cams, key_cap=16 * g.n + 1024)
    image = api.render_batch(ctx, g, cams, frame)[0]
    dLs = [dL] + [torch.zeros(3, h, w, device="cuda") for w, h in sizes[1:]]
    return image, api.render_backward_batch(ctx, g, frame, dLs).tensors()


@pytest.mark.parametrize("batch", [512, 1024])
@pytest.mark.parametrize("sizes", [[(40, 24)], [(40, 24), (640, 640)]])   # few tiles, many
@pytest.mark.parametrize("n", [64, 257, 511, 513, 1023, 1025, 1537, 2049, 3072, 4100])
def test_gradients_do_not_depend_on_the_depth(n, sizes, batch):
    rng = np.random.default_rng(n)
    g = api.Gaussians.empty(n, 0)
    g.means.copy_(torch.from_numpy(rng.uniform(-0.5, 0.5, (3, n)).astype(np.float32)))
    g.log_scales.fill_(-0.5)   # wider than the image: every tile lists them all
    g.quats[0] = 1.0
    g.opacity_logits.fill_(-5.4)
    g.sh.copy_(torch.from_numpy(rng.uniform(-1, 1, tuple(g.sh.shape)).astype(np.float32)))
    dL = torch.from_numpy(rng.uniform(-1, 1, (3, 24, 40)).astype(np.float32)).cuda()
    want, got = gradients(g, sizes, 256, dL), gradients(g, sizes, batch, dL)
    assert torch.equal(want[0], got[0])
    a, b = (torch.cat([t.flatten() for t in r[1]]).double() for r in (got, want))
    assert torch.isfinite(a).all()
    assert (a - b).norm() <= 1e-4 * b.norm()


def test_deep_batches_keep_wide_segments():
    W, H, n = 1256, 828, 500_000
    g = api.Gaussians.from_scene(synth.scene_uniform_sh0(n, seed=5, log_scale_mu=-4.5))
    g.opacity_logits.fill_(-3.0)
    cam = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), W, H, 60.0)
    dL = torch.ones(3, H, W, device="cuda")
    ms = {}
    for batch in (256, 512):
        ctx = api.Context(0)
        api.set_tuning(ctx, lds_batch=batch)
        frame = api.Frame(ctx, n, W, H, key_cap=8 * n, auto_grow=False)
        times = []
        for _ in range(5):
            api.timing_enable(ctx, True)
            api.render(ctx, g, cam, frame)
            api.render_backward(ctx, g, cam, frame, dL)
            torch.cuda.synchronize()
            times.append(api.timing_read(ctx)["blend_bwd"][0])
        ms[batch] = min(times[1:])
    # segments of 256 at both depths: 1.09 times as long at 512; of 512 there: 0.72 times
    assert ms[512] <= 0.9 * ms[256]
