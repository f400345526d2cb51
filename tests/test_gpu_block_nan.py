"""NaNs and infinities through block passes, both directions: they reach the
samples that sum them and no others, also where a block computes columns that
it does not use, reads past a row's end or stands in for a missing channel.
Against the one-kernel-per-iteration schedule, NaNs in the same places."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)
INF, NAN = float("inf"), float("nan")


def _spoil(x, seed):
    """A few NaNs and infinities, among them a row's first and last samples, the
    buffer's first and last, and the ends of time tiles."""
    g = torch.Generator().manual_seed(seed)
    rows, nt = x.shape
    for value in (NAN, INF, -INF):
        for r in torch.randint(rows, (2,), generator=g).tolist():
            x[r, int(torch.randint(nt, (1,), generator=g))] = value
    x[0, 0] = x[-1, -1] = NAN
    x[rows // 2, 0] = INF
    x[rows // 3, -1] = NAN
    x[rows // 4, min(223, nt - 1)] = -INF
    return x


def _same(a, b):
    torch.testing.assert_close(a, b, rtol=0, atol=0, equal_nan=True)
    assert bool(torch.isfinite(b).any())


@pytest.mark.parametrize("nf,nt,nd", [(64, 1024, 64), (50, 1000, 100), (33, 449, 40), (257, 700, 120), (1000, 2500, 60),
                                      (4096, 900, 200)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_forward(nf, nt, nd, dtype):
    x = _spoil(torch.randn(nf, nt, generator=torch.Generator().manual_seed(nf)), nt).to(DEV, dtype)
    p, q = (F.Plan(nf, nt, nd, 1.2, 1.6, in_dtype=dtype, unfused=u) for u in (False, True))
    _same(p.forward(x), q.forward(x))
    _same(p.forward(x.expand(40, nf, nt).contiguous())[39], q.forward(x))


@pytest.mark.parametrize("nf,nt,nd,d_min", [(64, 1024, 64, 0), (50, 1000, 100, 0), (257, 700, 120, 5000),
                                            (256, 30000, 300, 0), (1024, 512, 2048, 0), (1000, 2500, 60, 0)])
def test_adjoint(nf, nt, nd, d_min):
    g = _spoil(torch.randn(nd, nt, generator=torch.Generator().manual_seed(nf)), nt).to(DEV)
    p, q = (F.Plan(nf, nt, nd, 1.2, 1.6, d_min=d_min, unfused=u) for u in (False, True))
    _same(p.adjoint(g), q.adjoint(g))
