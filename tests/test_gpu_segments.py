"""Checkpoint spacing of the reverse pass: lists that end at, before and after
the boundaries of its segments, in a small render (spacing from 64 entries,
doubled as the list goes on) and beside a view that makes the render large
(256 entries).  Both walk the same contributors, so the gradients differ only
by the rounding of the restored states: T is divided back over at most 1500
contributors of a few ulp each, 1e-4 relative."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


@pytest.mark.parametrize("opacity", [-5.3, -1.0])   # nothing saturates; saturation within the list
@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 129, 192, 193, 255, 257, 320, 513, 768, 769, 1025, 1500])
def test_gradients_do_not_depend_on_the_spacing(n, opacity):
    rng = np.random.default_rng(n)
    g = api.Gaussians.empty(n, 0)
    xyz = np.stack([rng.uniform(-0.5, 0.5, n), rng.uniform(-0.5, 0.5, n), rng.uniform(-0.5, 0.5, n)])
    g.means.copy_(torch.from_numpy(xyz.astype(np.float32)))
    g.log_scales.fill_(-0.5)   # wider than the image: every tile lists them all
    g.quats[0] = 1.0
    g.opacity_logits.fill_(opacity)
    g.sh.copy_(torch.from_numpy(rng.uniform(-1, 1, tuple(g.sh.shape)).astype(np.float32)))
    ctx = api.Context(0)
    small = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), 40, 24, 30.0)
    large = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, -9.0), 640, 640, 30.0)   # looks away: nothing visible
    dL = torch.from_numpy(rng.uniform(-1, 1, (3, 24, 40)).astype(np.float32)).cuda()
    got, images = [], []
    for cams in ([small], [small, large]):
        frame = api.BatchFrame.for_views(ctx, n, cams, key_cap=16 * n + 1024)
        images.append(api.render_batch(ctx, g, cams, frame)[0])
        dLs = [dL] + [torch.zeros(3, 640, 640, device="cuda")] * (len(cams) - 1)
        got.append(api.render_backward_batch(ctx, g, frame, dLs).tensors())
    assert torch.equal(images[0], images[1])
    for a, b in zip(*got):
        assert torch.isfinite(a).all()
        assert (a - b).norm() <= 1e-4 * b.norm() + 1e-12
