"""Adjoint block passes under wide sub-bands, whose ranges are split by the rows
that they read: bit for bit the one-kernel-per-iteration schedule, for one record
and for batches, at the smallest ranges too."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_adjoint_block import _check  # noqa: E402


@pytest.mark.parametrize("band", [(0.4, 0.8), (0.3, 0.9), (0.05, 1.0)])
@pytest.mark.parametrize("nf,nt,nd,batches", [(1024, 16384, 1024, (1, 3)), (1000, 3001, 900, (1, 12)), (64, 700, 1000, (1, 30)),
                                              (16, 20000, 600, (1,)), (2048, 513, 1500, (2,))])
def test_records(nf, nt, nd, batches, band):
    for batch in batches:
        _check(nf, nt, nd, batch=batch, band=band)


def test_integers():
    _check(1024, 5000, 1024, dtype=torch.int32, band=(0.3, 0.9), d_min=40)
