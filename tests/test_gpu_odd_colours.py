"""Records whose colour is infinite or NaN, behind saturated pixels: no pixel
takes them, so image, counts and the other Gaussians' gradients are those of the same
records with finite colours.  In front, the pixels they cover take them and no others do."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402

CAM = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), 40, 24, 30.0)


def scene(n, opaque, seed=1):
    """n Gaussians wider than the view, one behind the other; the first `opaque` saturate every pixel."""
    rng = np.random.default_rng(seed)
    g = api.Gaussians.empty(n, 0)
    xyz = np.stack([rng.uniform(-0.2, 0.2, n), rng.uniform(-0.2, 0.2, n), np.linspace(-1.0, 1.0, n)])
    g.means.copy_(torch.from_numpy(xyz.astype(np.float32)))
    g.log_scales.fill_(1.5)
    g.quats[0] = 1.0
    g.opacity_logits.fill_(-4.0)
    g.opacity_logits[:opaque] = 12.0
    g.sh.copy_(torch.from_numpy(rng.uniform(-1, 1, tuple(g.sh.shape)).astype(np.float32)))
    return g


def render(g, batch, odd=None, value=0.0):
    h = api.Gaussians(*[t.clone() for t in g.tensors()], g.sh_degree)
    if odd is not None:
        h.sh.reshape(-1, g.n)[:, odd] = value
    ctx = api.Context(0)
    api.set_tuning(ctx, lds_batch=batch)
    frame = api.Frame(ctx, h.n, 40, 24, key_cap=16 * h.n)
    image = api.render(ctx, h, CAM, frame)
    dL = torch.from_numpy(np.random.default_rng(0).normal(size=(3, 24, 40)).astype(np.float32)).cuda()
    grads = api.render_backward(ctx, h, CAM, frame, dL).tensors()
    torch.cuda.synchronize()
    return image, frame.host_state(h.n)["n_contrib"], [t.reshape(-1, h.n) for t in grads]


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("batch", [256, 512])
@pytest.mark.parametrize("opaque,at,n", [(3, 3, 4), (3, 4, 5), (4, 4, 6), (4, 5, 6), (5, 64, 70), (5, 65, 70), (3, 255, 300),
                                         (4, 256, 300), (4, 257, 600), (3, 550, 600)])
def test_behind_saturated_pixels(opaque, at, n, batch, value):
    g = scene(n, opaque)
    want, got = render(g, batch), render(g, batch, at, value)
    assert torch.equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    others = torch.arange(n, device="cuda") != at
    # the gradients together (the quaternions' is zero here but for rounding): float atomics in another order
    a, b = (torch.cat([t[:, others].flatten() for t in r[2]]).double() for r in (got, want))
    assert torch.isfinite(a).all()
    assert (a - b).norm() <= 1e-4 * b.norm()


@pytest.mark.parametrize("n,at", [(5, 2), (90, 70), (300, 280)])
def test_pixels_outside_the_box_keep_their_colour(n, at):
    g = scene(n, 0)
    g.log_scales[:, at] = -4.0   # a few pixels
    g.opacity_logits[at] = 3.0
    want, got = render(g, 256), render(g, 256, at, float("inf"))
    np.testing.assert_array_equal(got[1], want[1])
    g.opacity_logits[at] = -30.0
    free = render(g, 256)
    taken = want[1] != free[1]   # the pixels that take the record
    assert 0 < taken.sum() < taken.size // 4
    image = got[0].cpu().numpy()
    assert np.isinf(image[:, taken]).all()
    np.testing.assert_array_equal(image[:, ~taken], want[0].cpu().numpy()[:, ~taken])
