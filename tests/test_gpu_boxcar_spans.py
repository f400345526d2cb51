"""Boxcar search over rows of several tiles (2048 samples), for every widest
width and one, two and four tiles per wave, against the oracle's binary32
evaluation of the doubling tree: peaks and their first times bit for bit,
statistics to FP64 summation (1e-12 of the row's RMS) plus binary32 output
rounding (2^-23)."""
import numpy as np
import pytest

from oracle import boxcar_search as oboxcar

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


def _check(y, m, rows):
    """Every row against the first `rows` rows' oracle: y repeats them."""
    res = {k: v.cpu().numpy() for k, v in F.boxcar_search(torch.from_numpy(y).to(DEV), m).items()}
    ref = oboxcar(y[:rows], m, acc=np.float32)
    reps = y.shape[0] // rows
    for k in ("peak", "t"):
        np.testing.assert_array_equal(res[k], np.tile(ref[k], (1, reps)).astype(res[k].dtype), err_msg=k)
    scale = np.sqrt(ref["mean"] ** 2 + ref["stdev"] ** 2)
    for k in ("mean", "stdev"):
        tol = 1e-12 * scale + 2.0 ** -23 * np.abs(ref[k])
        if k == "stdev":  # a difference of squares
            tol = tol + 1e-12 * scale ** 2 / np.maximum(ref["stdev"], 1e-30)
        assert np.all(np.abs(res[k] - np.tile(ref[k], (1, reps))) <= np.tile(tol, (1, reps))), k


@pytest.mark.parametrize("m", range(11))
def test_every_widest_width(m):
    rng = np.random.default_rng(m)
    y = (rng.standard_normal((3, 3 * 2048 + 1025)) * 16 + 3).astype(np.float32)
    _check(y, m, 3)


@pytest.mark.parametrize("reps,nt,m", [(700, 4 * 2048, 8), (700, 4 * 2048 + 1, 10), (700, 7 * 2048 + 2047, 3),
                                       (1400, 3 * 2048 + 5, 9), (2048, 2048, 2)])
def test_spans(reps, nt, m):
    """Enough rows that a wave takes several tiles."""
    rng = np.random.default_rng(nt)
    _check(np.tile((rng.standard_normal((3, nt)) + 1).astype(np.float32), (reps, 1)), m, 3)


def test_first_of_equal_peaks():
    """Ties within a lane, across lanes, chunks (256 samples) and tiles: the first time."""
    y = np.zeros((6, 5000), np.float32)
    for r, at in enumerate(([7, 6], [300, 299, 40], [511, 512], [2047, 2048], [4095, 1], [260, 4, 5])):
        y[r, at] = 2.0
    _check(y, 8, 6)


def test_nan_and_infinities():
    """A NaN is never a peak and leaves every window that misses it; infinite
    peaks keep their first time."""
    rng = np.random.default_rng(2)
    y = rng.standard_normal((4, 6000)).astype(np.float32)
    y[0, [0, 2050, 5999]] = np.nan
    y[1, 3000:3100] = np.inf
    y[2, :4000] = -np.inf
    y[3, :2048] = np.nan
    res = F.boxcar_search(torch.from_numpy(y).to(DEV), 0)
    t, peak = res["t"].cpu().numpy()[0], res["peak"].cpu().numpy()[0]
    ok = np.where(np.isnan(y), -np.inf, y)
    np.testing.assert_array_equal(peak, ok.max(axis=1))
    np.testing.assert_array_equal(t, ok.argmax(axis=1))
