"""Digit widths of the radix sort: key widths that split into digits of seven
to nine bits and unevenly, each aimed width, both tile sizes and their
remainders, against numpy's stable sort of the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


@pytest.mark.parametrize("n", [1, 2047, 2049, 300_001, 2_097_152, 2_101_249])
@pytest.mark.parametrize("lo,hi,aim", [(0, 9, 8), (0, 17, 8), (0, 18, 8), (0, 13, 6), (0, 13, 8), (3, 10, 4),
                                       (0, 27, 8), (5, 32, 8), (0, 32, 7), (0, 11, 5), (31, 32, 8)])
def test_digits_sort_stably(n, lo, hi, aim):
    rng = np.random.default_rng(n + 100 * lo + hi)
    k = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    if aim == 6:   # few distinct digits: long runs of equal keys
        k &= np.uint32(0xFFFF1C07)
    v = np.arange(n, dtype=np.uint32)
    kt, vt = torch.from_numpy(k.view(np.int32)).cuda(), torch.from_numpy(v.view(np.int32)).cuda()
    api.debug_sort_u32(api.Context(0), kt, vt, lo, hi, aim, single_pass=False)
    o = np.argsort((k.astype(np.uint64) >> np.uint64(lo)) & np.uint64((1 << (hi - lo)) - 1), kind="stable")
    np.testing.assert_array_equal(vt.cpu().numpy().view(np.uint32), v[o])
    np.testing.assert_array_equal(kt.cpu().numpy().view(np.uint32), k[o])
