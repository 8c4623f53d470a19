"""DensifyStep's scratch for the error statistics: a caller that allows fewer
pixels at a time reserves less and gets the same step."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api, densify  # noqa: E402


def test_fewer_pixels_at_a_time():
    n, W, H, V = 6000, 131, 93, 5
    scene = synth.scene_clusters(n, 3, 1, log_scale_mu=-3.0, log_scale_sd=0.6)
    g, zero = api.Gaussians.from_scene(scene), api.Gaussians.empty(n, 1)
    for t in zero.tensors():
        t.zero_()
    rng = np.random.default_rng(3)
    accum = torch.from_numpy(rng.exponential(1.0, n).astype(np.float32)).cuda()
    vis = torch.ones(n, dtype=torch.int32, device="cuda")
    views = synth.sphere_cameras(V, 4.0, [(W, H)], seed=3)
    gts = [torch.from_numpy(synth.smooth_image(H, W, k)).cuda() for k in range(V)]
    px = (W * H + 3) // 4 * 4
    results = []
    for kw, together in ((dict(), V), (dict(stat_pixels=1), 1), (dict(stat_pixels=3 * px - 1), 2)):
        ctx = api.Context(0)
        step = densify.DensifyStep(ctx, n, 1, "adpsplit", api.SplitParams(), views, gts, api.RegionBuffer(V * W * H // 5), **kw)
        assert step.stat_views == together and ctx.reserved()["max_pixels"] == together * px
        step.noise.copy_(torch.from_numpy(synth.vanilla_noise(step.cc, 5, step.noise_n)).view_as(step.noise))
        step.run(g, zero, zero, accum, vis, 1.5, 0.05, 0.005, 0.5)
        k = int(step.n_out.item())
        assert k > n and int(step.regions.count.item()) > 0
        results.append([t[..., :k].cpu() for t in step.out.tensors()] + [step.attr.cpu(), step.st3[:k].cpu()])
    for r in results[1:]:
        for a, b in zip(r, results[0]):
            assert torch.equal(a, b)
