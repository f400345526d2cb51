"""Boxcar search of so many rows that beams x widths x rows passes 2^28, where
16 lanes each are more threads than one launch takes: every result of rows of
one sample, whose sums of any width are that sample."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402


def test_more_results_than_threads_of_a_launch():
    batch, nd, m = 3000, 8150, 10
    assert batch * nd * (m + 1) > 2 ** 28
    y = torch.randn(batch, nd, 1, device="cuda")
    res = F.boxcar_search(y, m)
    want = y.view(batch, 1, nd)
    for k in ("peak", "mean"):
        assert bool((res[k] == want).all()), k
    for k in ("t", "stdev", "snr"):
        assert bool((res[k] == 0).all()), k
