"""Error statistics of noisy views: regions of a few pixels, tens of them
among a wave's 64 and thousands in a chunk, at odd sizes and next to large
regions, against the CPU oracle (whole numbers and records bit-exact)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402
from test_gpu_split import compare_regions, gparams  # noqa: E402


@pytest.mark.parametrize("W,H,m_min", [(1, 4099, 1), (17, 61, 1), (33, 31, 2), (64, 64, 1), (65, 63, 1), (128, 97, 3), (1031, 8, 1)])
@pytest.mark.parametrize("noisy", ["all", "half", "none"])
def test_noisy_views_match_the_oracle(W, H, m_min, noisy):
    r = np.random.default_rng(W * 1000 + H)
    n = 5
    img = r.uniform(0, 1, (3, H, W)).astype(np.float32)
    gt = np.zeros((3, H, W), np.float32)
    y, x = np.mgrid[0:H, 0:W]
    dom = r.integers(-1, n, (H, W)).astype(np.int32)
    large = (x * n // W).astype(np.int32)
    if noisy != "all":
        keep = (x < W // 2) if noisy == "half" else np.ones((H, W), bool)
        img = np.where(keep, np.float32(0.9), img)
        dom = np.where(keep, large, dom).astype(np.int32)
        img[:, 0, 0] = 0.0                       # an error range to normalise by
    is_cand = np.array([1, 1, 0, 1, 1], np.uint8)
    prm = oracle.SplitParams(r_erode=0, m_min=m_min, tau_l1=0.2)
    attr_o = np.zeros(n, np.int32)
    want, _ = oracle.error_stats(img, gt, dom, is_cand, 7, prm, attr_o)
    if noisy == "all" and m_min == 1:
        assert len(want) > W * H // 12           # regions of a few pixels
    ctx = api.Context(0, max_pixels=W * H)
    regions = api.RegionBuffer(W * H)
    attr = torch.zeros(n, dtype=torch.int32, device="cuda")
    gtt, domt, cand = torch.from_numpy(gt).cuda(), torch.from_numpy(dom).cuda(), torch.from_numpy(is_cand).cuda()
    err, mm = api.error_map(ctx, torch.from_numpy(img).cuda(), gtt)
    api.accumulate_error_stats(ctx, W, H, err, mm, domt, gtt, 7, cand, gparams(prm), regions, attr)
    torch.cuda.synchronize()
    compare_regions(regions.host(), want)
    np.testing.assert_array_equal(attr.cpu().numpy(), attr_o)
