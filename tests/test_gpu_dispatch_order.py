"""Dispatch orders of the blends at the edges of their counting sort: tile
counts around one ordering block, around the count up to which every block
counts all tiles, and above it; bins of 16 and 32; several views; longest
first and tile order.  Each render and its gradients against the same frame
size rendered view by view in tile order: images bit-identical (every tile must be
dispatched exactly once), gradients within FP32 summation order."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


def render(sizes, g, bin_tile, longest, dLs, split):
    ctx = api.Context(0)
    api.set_tuning(ctx, bin_tile=bin_tile, longest_first=longest)
    rng = np.random.default_rng(3)
    cams = [synth.random_pose_camera(rng, 4.0, W, H) for W, H in sizes]
    frame = api.BatchFrame.for_views(ctx, g.n, cams, key_cap=64 * g.n * len(cams))
    images, grads = [], [torch.zeros_like(t) for t in g.tensors()]
    for part in ([[k] for k in range(len(cams))] if split else [list(range(len(cams)))]):
        images += api.render_batch(ctx, g, [cams[k] for k in part], frame)
        out = api.render_backward_batch(ctx, g, frame, [dLs[k] for k in part])
        again = api.render_backward_batch(ctx, g, frame, [dLs[k] for k in part])
        for a, b, c in zip(grads, out.tensors(), again.tensors()):
            torch.testing.assert_close(b, c, rtol=1e-3, atol=1e-3 * float(b.abs().mean()) + 1e-12)
            a += b
    torch.cuda.synchronize()
    return images, grads


@pytest.mark.parametrize("sizes", [[(16, 16)], [(1, 1), (33, 40)], [(16 * 32, 16 * 32)], [(16 * 41, 16 * 25 + 1)],
                                   [(16 * 64, 16 * 80)], [(16 * 64, 16 * 80 + 1)], [(700, 500), (1256, 828), (31, 900)]])
@pytest.mark.parametrize("bin_tile,longest", [(16, True), (32, True), (16, False), (32, False)])
def test_every_tile_is_dispatched_once(sizes, bin_tile, longest):
    g = api.Gaussians.from_scene(synth.scene_uniform_sh0(3000, seed=5, log_scale_mu=-3.0))
    dLs = [torch.from_numpy(np.random.default_rng(k).normal(size=(3, H, W)).astype(np.float32)).cuda()
           for k, (W, H) in enumerate(sizes)]
    want = render(sizes, g, 16, False, dLs, True)
    got = render(sizes, g, bin_tile, longest, dLs, False)
    for a, b in zip(got[0], want[0]):
        assert torch.equal(a, b)
    for a, b in zip(got[1], want[1]):
        rel = float((a.double() - b.double()).norm() / b.double().norm().clamp(min=1e-30))
        assert rel <= 1e-4, rel
