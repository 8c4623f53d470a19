"""Two-level binning of long coarse lists (many entries behind one another), at
the lengths where the groups of their work items change, several of them and
beside ordinary lists.  Pairs are compared bit for bit with a stable sort by bin on the
host, and the placing may not take longer than that of as many spread entries."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402

GROUP = 64 * 1536   # pairs of a group of work items


def prepare(sizes, W, H, spread=30_000):
    """sizes[k] tiny Gaussians at the k-th of a few places, and some everywhere."""
    rng = np.random.default_rng(sum(sizes))
    n = sum(sizes) + spread
    xyz = rng.uniform(-1.0, 1.0, (3, n))
    at = 0
    for k, m in enumerate(sizes):
        xyz[0, at:at + m], xyz[1, at:at + m] = 0.4 * k - 0.31 + rng.uniform(-0.01, 0.01, m), 0.21 * k - 0.4
        at += m
    g = api.Gaussians.empty(n, 0)
    g.means.copy_(torch.from_numpy(xyz[:, rng.permutation(n)].astype(np.float32)))
    g.log_scales.fill_(-7.0)
    g.quats[0] = 1.0
    g.opacity_logits.fill_(5.0)
    cam = synth.look_at((0.0, 0.0, -40.0), (0.0, 0.0, 0.0), W, H, 4.0)
    ctx = api.Context(0)
    return ctx, g, cam, api.Frame(ctx, n, W, H, key_cap=max(1 << 22, 4 * n), auto_grow=False, forward_only=True)


# coarse bins of 2 x 2 bins, of 4 x 4
@pytest.mark.parametrize("W,H", [(640, 480), (1040, 1024)])
@pytest.mark.parametrize("sizes", [[GROUP - 1], [GROUP], [GROUP + 1], [2 * GROUP + 700, 3 * GROUP], [GROUP, GROUP + 1536, 100, 2 * GROUP - 1],
                                   [1_400_000]])
def test_pairs_of_long_lists(W, H, sizes):
    ctx, g, cam, frame = prepare(sizes, W, H)
    api.render(ctx, g, cam, frame)
    n, v = g.n, frame.view(0)
    depth = frame._dev(v.depth_key, 4 * n).view(np.uint32)
    nt = frame._dev(v.ntiles, 4 * n).view(np.uint32).astype(np.int64)
    box = frame._dev(v.box, 8 * n).view(np.int16).reshape(n, 4).astype(np.int64) // 16
    e = np.argsort(depth, kind="stable")
    e = e[nt[e] > 0]
    ent = np.repeat(e, nt[e])
    q = np.arange(len(ent)) - np.repeat(np.cumsum(nt[e]) - nt[e], nt[e])
    wd = box[ent, 2] - box[ent, 0] + 1
    key = (box[ent, 1] + q // wd) * v.tiles_x + box[ent, 0] + q % wd
    o = np.argsort(key, kind="stable")
    assert frame.n_keys() == frame.n_emitted() == len(o)
    np.testing.assert_array_equal(frame._dev(v.keys, 4 * len(o)).view(np.uint32), key[o])
    np.testing.assert_array_equal(frame._dev(v.vals, 4 * len(o)).view(np.uint32), ent[o])


def ranges_ms(sizes, spread):
    ctx, g, cam, frame = prepare(sizes, 1920, 1080, spread)
    times = []
    for _ in range(4):
        api.timing_enable(ctx, True)
        api.render(ctx, g, cam, frame)
        torch.cuda.synchronize()
        times.append(api.timing_read(ctx)["ranges"][0])
    return min(times[1:])


def test_time_does_not_follow_the_lists():
    long, short = ranges_ms([4_000_000, 4_000_000], 30_000), ranges_ms([], 8_030_000)
    print("ranges of two long lists %.4f ms, of spread entries %.4f ms" % (long, short))
    assert long <= 2.0 * short
