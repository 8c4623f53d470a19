"""The split's per-region kernels at the edges of their waves: candidates with
none, one, and up to several waves of regions, regions handed over in any
order, every SH degree (whole and partial row chunks) and up to more children
than a candidate has child lanes.  Oracle and bars as the other split tests:
modes, counts, offsets and row order bit-exact, children relative 1e-5."""
import numpy as np
import pytest

import oracle
from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402
from test_gpu_split import compare_split, gparams  # noqa: E402

COUNTS = (0, 1, 2, 7, 63, 64, 65, 130)


def make_regions(scene, cand, views, counts, seed):
    """Random regions around each candidate's projection, in shuffled order."""
    rng = np.random.default_rng(seed)
    total = int(sum(counts))
    recs = np.zeros(total, api.REGION_DTYPE)
    k = 0
    for c, m in zip(cand, counts):
        for j in range(m):
            v = int(rng.integers(len(views)))
            cam = views[v]
            p = np.asarray(cam.R, np.float64) @ scene.means[:, c].astype(np.float64) + np.asarray(cam.t, np.float64)
            r = recs[k]
            r["cand"], r["view"], r["label"], r["area"], r["band"] = c, v, j, 10, 0
            spread = 2.0 if j % 2 else 25.0      # some groups merge, some stay apart
            r["cx"] = cam.fx * p[0] / p[2] + cam.cx + rng.normal(0, spread)
            r["cy"] = cam.fy * p[1] / p[2] + cam.cy + rng.normal(0, spread)
            th = rng.uniform(-1.5, 1.5)
            r["e1"] = (np.cos(th), np.sin(th))
            r["sigma1"], r["sigma2"] = rng.uniform(1.0, 3.0), rng.uniform(0.3, 1.0)
            r["rgb"] = rng.uniform(0, 0.3 if j % 2 else 1.0, 3)
            k += 1
    return recs[rng.permutation(total)]


@pytest.mark.parametrize("deg,n_max,variant,flags", [
    (0, 19, oracle.VARIANT_ADPSPLIT, 0), (1, 3, oracle.VARIANT_ADPSPLIT, 0), (2, 100, oracle.VARIANT_ADPSPLIT, 0),
    (3, 19, oracle.VARIANT_ADPSPLIT, oracle.FLAG_SHARE_OPACITY), (3, 8, oracle.VARIANT_CHILD_INIT, oracle.FLAG_EXTENT_MAX)])
def test_split_at_wave_edges(deg, n_max, variant, flags):
    seed = 900 + deg * 10 + n_max
    scene = synth.scene_clusters(300, seed, deg, log_scale_mu=-2.5, log_scale_sd=0.4)
    views = synth.sphere_cameras(3, 4.0, [(640, 480)], seed=seed)
    rng = np.random.default_rng(seed)
    cand = np.sort(rng.choice(scene.n, 3 * len(COUNTS), replace=False)).astype(np.int32)
    counts = np.array(COUNTS * 3)[rng.permutation(3 * len(COUNTS))]
    recs = make_regions(scene, cand, views, counts, seed)
    attr = np.zeros(scene.n, np.int32)
    attr[cand[rng.uniform(size=len(cand)) < 0.8]] = 4
    prm = oracle.SplitParams(n_max=n_max, variant=variant, flags=flags)
    noise = synth.vanilla_noise(len(cand), seed)
    regs = np.zeros(len(recs), oracle.REGION_DTYPE)
    for f in regs.dtype.names:
        if f in recs.dtype.names:
            regs[f] = recs[f]
    want = oracle.adaptive_split(scene, cand, regs, views, attr, prm, noise)
    assert (want["mode"] == 2).any() and want["count"].max() > min(n_max, 8)
    ctx = api.Context(0, max_gaussians=scene.n, max_candidates=len(cand), max_regions=len(recs) + 100, max_views=3)
    rb = api.RegionBuffer(len(recs) + 100)
    rb.records[: recs.nbytes] = torch.from_numpy(recs.view(np.uint8).copy()).cuda()
    rb.count.fill_(len(recs))
    out, mode, count, offset, n_out = api.adaptive_split(
        ctx, api.Gaussians.from_scene(scene), torch.from_numpy(cand).cuda(), rb, views, torch.from_numpy(attr).cuda(),
        gparams(prm), torch.from_numpy(noise).cuda())
    torch.cuda.synchronize()
    compare_split(want, (out, mode.cpu().numpy(), count.cpu().numpy(), offset.cpu().numpy(), int(n_out.item())))
