"""Boxcar search of rows whose last tile (2048 samples) holds a few samples, up
to and past the two chunks of 256 that have a form of their own, alone in the
row and after whole tiles, for every widest width, as in
test_gpu_boxcar_spans."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_boxcar_spans import _check  # noqa: E402


@pytest.mark.parametrize("m", range(11))
def test_last_tile(m):
    rng = np.random.default_rng(m)
    for last in (1, 5, 255, 256, 257, 511, 512, 513):
        for tiles in (0, 1, 2):
            y = (rng.standard_normal((3, 2048 * tiles + last)) * 16 + 3).astype(np.float32)
            _check(y, m, 3)
