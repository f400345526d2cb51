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


@pytest.mark.parametrize("m", (0, 3, 10))
@pytest.mark.parametrize("nt,tail", ((2048, 2048), (2049, 1), (6000, 1904), (6000, 5000), (8192, 300)))
def test_rows_of_several_tiles(nt, tail, m):
    y = _rows(nt, tail)
    y[4, :] = np.nan
    y[4, 2047] = 3.0
    _check(y, m)


@pytest.mark.parametrize("search_rows", (0, 1, 2))
def test_no_candidates_in_tiles_without_a_peak(search_rows):
    """A record whose first 5000 samples are NaN, in and after the last pass of
    the transform: its NaN tiles hold no candidate, whatever the threshold, and
    both searches find the same."""
    nf, nt, nd, m = 64, 9000, 40, 4
    plan = F.Plan(nf, nt, nd, 1.2, 1.6, search_rows=search_rows)
    rng = np.random.default_rng(5)
    x = rng.integers(0, 4, (nf, nt)).astype(np.float32)
    x[:, :5000] = np.nan
    y, res, cands, n = plan.forward_search(torch.from_numpy(x).to(DEV), m, threshold=-1.0)
    alone = F.boxcar_search(y, m)
    for k in ("peak", "t"):
        assert torch.equal(res[k], alone[k]), k
    peak, at = _peaks(y.cpu().numpy(), m)
    np.testing.assert_array_equal(res["t"].cpu().numpy(), at)
    cands = cands.cpu().numpy()
    # every sum of a row with NaNs in it has a NaN mean, hence S/N 0: one
    # candidate per tile (3 of 5 reach past the NaNs) at its first largest sum
    assert n == (m + 1) * nd * 3 and len(cands) == n
    assert cands[:, 2].min() >= 5000 and cands[:, 2].max() < nt
    x[:, :] = np.nan
    _, res, _, n = plan.forward_search(torch.from_numpy(x).to(DEV), m, threshold=-1.0)
    assert n == 0 and bool((res["t"] == NO_PEAK).all())
