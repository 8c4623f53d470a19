"""Error statistics of several views in one call against the CPU oracle view
by view (bit-exact, as the single call), at the edges of the 16x16 tiles, the
pixel chunks and the four-pixel alignment of a batch; and the halo's error
threshold against the classification it stands for, at errors within a few
ulps of it and on ranges that have no threshold."""
import numpy as np
import pytest

import oracle
from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402
from test_gpu_split import compare_regions, gparams, stripes_fixture  # noqa: E402


@pytest.mark.parametrize("sizes,r", [([(1, 1), (17, 16), (63, 65), (64, 64)], 0), ([(333, 201), (16, 257), (130, 127)], 2),
                                     ([(90, 91)] * 16, 1), ([(129, 97), (45, 300)], 9)])
def test_batch_matches_the_oracle_view_by_view(sizes, r):
    prm = oracle.SplitParams(r_erode=r, m_min=2)
    n = 4
    attr_o = np.full(n, 3, np.int32)
    maps, want = [], []
    for k, (W, H) in enumerate(sizes):
        img, gt, dom, is_cand = stripes_fixture(H, W, seed=70 + k, widen=r)
        is_cand[1] = 0
        rec, _ = oracle.error_stats(img, gt, dom, is_cand, 20 - k, prm, attr_o)
        want.append(rec)
        maps.append((img, gt, dom))
    want = np.concatenate(want)
    pad = sum((W * H + 3) // 4 * 4 for W, H in sizes)
    ctx = api.Context(0, max_pixels=pad)
    regions = api.RegionBuffer(pad)
    attr = torch.full((n,), 3, dtype=torch.int32, device="cuda")
    views = []
    for k, ((W, H), (img, gt, dom)) in enumerate(zip(sizes, maps)):
        gtt = torch.from_numpy(gt).cuda()
        err, mm = api.error_map(ctx, torch.from_numpy(img).cuda(), gtt)
        views.append((W, H, err, mm, torch.from_numpy(dom).cuda(), gtt, 20 - k))
    for _ in range(2):      # the second call starts from the first one's count
        api.accumulate_error_stats_batch(ctx, views, torch.from_numpy(is_cand).cuda(), gparams(prm), regions, attr)
    torch.cuda.synchronize()
    got = regions.host()
    assert len(got) == 2 * len(want)
    compare_regions(got[: len(want)], want)
    compare_regions(got[len(want):], want)
    np.testing.assert_array_equal(attr.cpu().numpy() - 3, 2 * (attr_o - 3))


@pytest.mark.parametrize("W,H", [(1, 1), (16, 16), (17, 15), (63, 65), (64, 64), (91, 90), (4097, 1)])
def test_one_view_matches_the_oracle_through_both_calls(W, H):
    """The single call and a batch of one view have the same kernels with a
    table of one view: bit-exact, at the edges of tiles and chunks."""
    prm = oracle.SplitParams(r_erode=1, m_min=1)
    img, gt, dom, is_cand = stripes_fixture(H, W, seed=7, widen=1)
    attr_o = np.full(4, 3, np.int32)
    want, _ = oracle.error_stats(img, gt, dom, is_cand, 5, prm, attr_o)
    ctx = api.Context(0, max_pixels=W * H)
    gtt, cand, domt = torch.from_numpy(gt).cuda(), torch.from_numpy(is_cand).cuda(), torch.from_numpy(dom).cuda()
    err, mm = api.error_map(ctx, torch.from_numpy(img).cuda(), gtt)
    for batch in (False, True):
        regions = api.RegionBuffer(W * H)
        attr = torch.full((4,), 3, dtype=torch.int32, device="cuda")
        if batch:
            api.accumulate_error_stats_batch(ctx, [(W, H, err, mm, domt, gtt, 5)], cand, gparams(prm), regions, attr)
        else:
            api.accumulate_error_stats(ctx, W, H, err, mm, domt, gtt, 5, cand, gparams(prm), regions, attr)
        torch.cuda.synchronize()
        compare_regions(regions.host(), want)
        np.testing.assert_array_equal(attr.cpu().numpy(), attr_o)


def test_batch_refuses_what_does_not_fit():
    ctx = api.Context(0, max_pixels=100)
    z = lambda *s, d=torch.float32: torch.zeros(*s, dtype=d, device="cuda")
    view = (10, 9, z(9, 10, d=torch.float64), z(2, d=torch.int64), z(9, 10, d=torch.int32), z(3, 9, 10), 0)
    rest = (z(5, d=torch.uint8), api.SplitParams(), api.RegionBuffer(10), z(5, d=torch.int32))
    api.accumulate_error_stats_batch(ctx, [view], *rest)
    for views, status in (([view] * 2, api.AS_ERR_CAPACITY), ([view] * 17, api.AS_ERR_ARG), ([], api.AS_ERR_ARG)):
        with pytest.raises(api.AdpSplitError) as e:
            api.accumulate_error_stats_batch(ctx, views, *rest)
        assert e.value.status == status
    torch.cuda.synchronize()


@pytest.mark.parametrize("tau", [0.0, 0.1, 1.0 / 3.0, 0.999])
@pytest.mark.parametrize("emin,emax", [(0.0, 1.7), (0.0, 5e-324), (1e-300, 3e-300), (0.25, 0.2500000001), (1e6, 1e6 + 1e-9),
                                       (2.0, 1.0), (0.5, 0.5), (0.0, np.inf), (0.0, np.nan), (-1.0, 2.0)])
def test_halo_threshold_is_the_classification(tau, emin, emax):
    """Each pixel its own candidate, no erosion: a pixel is a region (through
    the halo's test) exactly when it is attributed (through the division)."""
    W, H = 32, 16
    P = W * H
    rng = np.random.default_rng(5)
    with np.errstate(all="ignore"):
        c = np.float64(emin) + np.float64(tau) * (np.float64(emax) - np.float64(emin))
    err = rng.uniform(min(emin, 0.0), 2.0, P)
    if np.isfinite(c):
        x, y = np.full(40, c), np.full(40, c)
        for k in range(1, 40):
            x[k], y[k] = np.nextafter(x[k - 1], np.inf), np.nextafter(y[k - 1], -np.inf)
        err[:80] = np.concatenate([x, y])
    err[80:84] = (np.inf, np.nan, 0.0, emin)
    err = torch.from_numpy(err.reshape(H, W)).cuda()
    mm = torch.from_numpy(np.array([emin, emax]).view(np.int64)).cuda()
    dom = torch.arange(P, dtype=torch.int32, device="cuda").view(H, W)
    ctx = api.Context(0, max_pixels=P)
    regions = api.RegionBuffer(P)
    attr = torch.zeros(P, dtype=torch.int32, device="cuda")
    api.accumulate_error_stats(ctx, W, H, err, mm, dom, torch.zeros(3, H, W, device="cuda"), 0,
                               torch.ones(P, dtype=torch.uint8, device="cuda"),
                               api.SplitParams(tau_l1=tau, r_erode=0, m_min=1), regions, attr)
    torch.cuda.synchronize()
    hit = np.nonzero(attr.cpu().numpy())[0]
    np.testing.assert_array_equal(regions.host()["label"], hit)
