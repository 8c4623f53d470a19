"""Two-level binning at its edges: the smallest set and capacity it takes, coarse bins of
2 x 2 and 4 x 4 bins, ragged borders, bins of 32, several views, sets above
the bucketed depth sort, renders over the pair capacity, nothing visible.
Pairs and ranges are compared bit for bit with the boxes' bins listed in depth
order and sorted stably on the bin, on the host."""
import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


def expected(depth, box, nt, view, bin_base, bins_x, bin_size, cap):
    """Bin keys and entry ids of the pairs that fit in cap, sorted."""
    e = np.argsort(depth, kind="stable")
    e = e[nt[e] > 0]
    e = e[np.cumsum(nt[e].astype(np.int64)) <= cap]
    b = box[e].astype(np.int64) // bin_size
    cnt = nt[e].astype(np.int64)
    first = np.concatenate([[0], np.cumsum(cnt)[:-1]]) if len(e) else cnt
    q = np.arange(int(cnt.sum())) - np.repeat(first, cnt)
    wd = np.repeat(b[:, 2] - b[:, 0] + 1, cnt)
    key = np.repeat(bin_base[view[e]] + b[:, 1] * bins_x[view[e]] + b[:, 0], cnt)
    key = key + (q // wd) * np.repeat(bins_x[view[e]], cnt) + q % wd
    o = np.argsort(key, kind="stable")
    return key[o], np.repeat(e, cnt)[o]


LEAST = 1 << 22   # the smallest pair capacity that takes this path


@pytest.mark.parametrize("n,sizes,bin_tile,cap,grow,where", [
    (32_768, [(615, 437)], 16, LEAST, 0.0, "front"),
    (300_000, [(615, 437)], 16, LEAST, 0.0, "front"),
    (400_000, [(1031, 1029)], 16, None, 0.0, "front"),
    (400_000, [(1031, 1029)], 16, LEAST, 2.5, "front"),
    (300_000, [(1031, 1029)], 32, None, 0.0, "front"),
    (150_000, [(640, 333), (517, 300), (16, 16)], 16, None, 0.0, "front"),
    (150_000, [(1040, 700), (800, 600), (16, 16)], 32, LEAST + 1, 3.5, "front"),
    (1_048_577, [(1040, 1024)], 16, None, 0.0, "half"),
    (1_400_000, [(1040, 1024)], 16, LEAST, 2.5, "half"),
    (2_200_000, [(1000, 403)] * 2, 16, None, 0.0, "half"),
    (320_000, [(640, 480)], 16, LEAST, 0.0, "behind"),
    (200_000, [(2048, 1024)], 16, LEAST, 0.0, "front"),    # 8,192 bins, scanned by one block
    (200_000, [(2049, 1024)], 16, LEAST, 0.0, "front"),    # 8,256
])
def test_pairs_match_a_stable_sort_by_bin(n, sizes, bin_tile, cap, grow, where):
    rng = np.random.default_rng(n + bin_tile)
    g = api.Gaussians.empty(n, 0)
    z = {"front": (-1.0, 1.0), "half": (-8.0, 1.0), "behind": (-9.0, -5.0)}[where]
    xyz = np.stack([rng.uniform(-1.3, 1.3, n), rng.uniform(-1.3, 1.3, n), rng.uniform(z[0], z[1], n)])
    g.means.copy_(torch.from_numpy(xyz.astype(np.float32)))
    # mostly a bin or two across, one in a thousand over many coarse bins
    s = np.where(rng.uniform(size=n) < 1e-3, rng.uniform(-3.0, -1.0, n), rng.uniform(-7.0, -4.6, n) + grow)
    g.log_scales.copy_(torch.from_numpy(np.stack([s] * 3).astype(np.float32)))
    g.quats[0] = 1.0
    ctx = api.Context(0)
    api.set_tuning(ctx, bin_tile=bin_tile)
    cams = [synth.look_at((0.3 * k, 0.0, -4.0), (0.0, 0.0, 0.0), w, h, 60.0) for k, (w, h) in enumerate(sizes)]
    V, ne = len(cams), n * len(cams)
    probe = api.BatchFrame.for_views(ctx, n, cams, key_cap=1, auto_grow=False, forward_only=True)
    api.render_batch(ctx, g, cams, probe)
    demand = probe.n_keys()
    if cap is None:
        cap = max(LEAST, demand)
    assert grow == 0.0 or cap < demand   # the cut renders are cut
    frame = api.BatchFrame.for_views(ctx, n, cams, key_cap=cap, auto_grow=False, forward_only=True)
    api.render_batch(ctx, g, cams, frame)
    vs = [frame.view(k) for k in range(V)]
    depth = frame._dev(vs[0].depth_key, 4 * ne).view(np.uint32)
    box = frame._dev(vs[0].box, 8 * ne).view(np.int16).reshape(ne, 4)
    nt = frame._dev(vs[0].ntiles, 4 * ne).view(np.uint32)
    base, bx = np.array([v.bin_base for v in vs]), np.array([v.bins_x for v in vs])
    key, val = expected(depth, box, nt, np.repeat(np.arange(V), n), base, bx, bin_tile, cap)
    assert frame.n_keys() == demand == int(nt.astype(np.int64).sum())
    assert frame.n_emitted() == len(key)
    K = len(key)
    np.testing.assert_array_equal(frame._dev(vs[0].keys, 4 * K).view(np.uint32), key)
    np.testing.assert_array_equal(frame._dev(vs[0].vals, 4 * K).view(np.uint32), val)
    f = bin_tile // 16
    for v in vs:
        r = frame._dev(v.ranges, 8 * v.tiles_x * v.tiles_y).view(np.uint32).reshape(v.tiles_y, v.tiles_x, 2)
        ty, tx = np.mgrid[:v.tiles_y, :v.tiles_x]
        b = v.bin_base + (ty // f) * v.bins_x + tx // f
        lo, hi = np.searchsorted(key, b), np.searchsorted(key, b, side="right")
        np.testing.assert_array_equal(r[..., 0], np.where(hi > lo, lo, 0))
        np.testing.assert_array_equal(r[..., 1], np.where(hi > lo, hi, 0))
