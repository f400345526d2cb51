"""Boxcar search of rows that hold NaNs and infinities only in places: a NaN is
never a peak, and a row, or a tile of 2048 samples, whose running sums are all
NaN has none: peak -inf at time 2^31 - 1. Against the definition in NumPy;
the samples are whole numbers, so every running sum is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)
NO_PEAK = 2 ** 31 - 1


def _peaks(y, m):
    """Peak and first time per width and row, by the definition."""
    b = y.astype(np.float64)
    peak, at = [], []
    for j in range(m + 1):
        if j > 0:
            w = 1 << (j - 1)
            with np.errstate(invalid="ignore"):
                b = b + np.pad(b, ((0, 0), (w, 0)))[:, : b.shape[1]]
        ok = ~np.isnan(b)
        top = np.where(ok, b, -np.inf).max(axis=1)
        hit = ok & (b == top[:, None])
        peak.append(top)
        at.append(np.where(hit.any(axis=1), hit.argmax(axis=1), NO_PEAK))
    return np.array(peak), np.array(at)


def _check(y, m):
    res = F.boxcar_search(torch.from_numpy(y).to(DEV), m)
    peak, at = _peaks(y, m)
    np.testing.assert_array_equal(res["peak"].cpu().numpy(), peak.astype(np.float32))
    np.testing.assert_array_equal(res["t"].cpu().numpy(), at)


def _rows(nt, tail):
    """All NaN; NaN but for -inf at the end, in the middle of the last `tail`
    samples and throughout them; NaN but for one finite sample."""
    y = np.full((5, nt), np.nan, np.float32)
    y[1, -1] = -np.inf
    y[2, nt - 1 - tail // 2] = -np.inf
    y[3, nt - tail:] = -np.inf
    y[4, nt - 1 - tail // 3] = 3.0
    return y


@pytest.mark.parametrize("m", (0, 3, 8))
@pytest.mark.parametrize("nt", (1, 3, 255, 1000, 2047))
def test_rows_shorter_than_a_tile(nt, m):
    _check(_rows(nt, nt), m)
