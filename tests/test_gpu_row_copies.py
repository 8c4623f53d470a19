"""Row copies and flag scans of the optimisation loop at the edges of their
blocks: clone and prune, and the row gather, against the same selections in torch."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 15, 17, 255, 257, 4095, 4097, 70_001])
def test_clone_prune_and_gather(n, deg):
    gen = torch.Generator(device="cuda").manual_seed(n + deg)
    g = api.Gaussians.empty(n, deg)
    for t in g.tensors():
        t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
    clone = (torch.rand(n, generator=gen, device="cuda") < 0.3).to(torch.uint8)
    out = api.Gaussians.empty(2 * n, deg)
    ctx = api.Context(0, max_gaussians=2 * n)
    n_out = torch.zeros(1, dtype=torch.int64, device="cuda")
    src = torch.empty(2 * n, dtype=torch.int32, device="cuda")
    api.clone_prune(ctx, g, clone, None, 0.3, 0.0, out, src, n_out)
    keep = torch.sigmoid(g.opacity_logits.double()) >= 0.3
    kept = torch.nonzero(keep).flatten()
    rows = torch.cat([kept, torch.nonzero(keep & clone.bool()).flatten()])
    m = int(n_out)
    assert m == len(rows)
    want = torch.cat([kept, torch.full((m - len(kept),), -1, dtype=kept.dtype, device="cuda")])
    assert torch.equal(src[:m], want.int())
    for a, b in zip(out.tensors(), g.tensors()):
        assert torch.equal(a[..., :m], b[..., rows])
    back = api.Gaussians.empty(n, deg)
    pick = torch.randint(-1, n + 1, (n,), generator=gen, device="cuda", dtype=torch.int32)
    api.gather_rows(ctx, g, pick, n, back)
    ok = (pick >= 0) & (pick < n)
    for a, b in zip(back.tensors(), g.tensors()):
        assert torch.equal(a, torch.where(ok, b[..., pick.clamp(0, n - 1).long()], torch.zeros((), device="cuda")))
