"""Block passes of the adjoint over one record, with ranges of rows small enough
to fill the GPU, and over batches, which take larger ones from some number of
samples on, by uniform and ragged batches, step by step as well: bit for bit
the one-kernel-per-iteration schedule (both add in the same order)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402

from test_gpu_adjoint_block import _check, _grad  # noqa: E402


@pytest.mark.parametrize("nf,nt,nd,batches", [(64, 20000, 64, (1, 2, 3, 8)), (256, 500, 256, (1, 5, 6, 7, 8, 9, 30)),
                                              (1024, 1000, 1000, (1, 2, 3, 4)), (50, 1000, 100, (1, 16, 60)),
                                              (4096, 512, 2048, (1, 3)), (32, 100000, 64, (1, 2)), (100, 225, 90, (70,))])
def test_records(nf, nt, nd, batches):
    for batch in batches:
        _check(nf, nt, nd, batch=batch)


@pytest.mark.parametrize("kw", [dict(d_min=900), dict(rule=1), dict(gamma=2.0)])
@pytest.mark.parametrize("batch", (1, 40))
def test_laws(kw, batch):
    _check(200, 600, 90, batch=batch, dtype=torch.int32, **kw)


@pytest.mark.parametrize("lengths", ([700, 0, 31], [224 + 5 * b for b in range(90)], [40000, 1, 513]))
def test_ragged(lengths):
    nf, nt, nd = 128, 3000, 140
    r = F.RaggedPlan(F.Plan(nf, nt, nd, 1.2, 1.6), lengths)
    g = _grad((nd * sum(lengths),), torch.float32, 3)
    x = r.unpack(r.adjoint(g), nf)
    for n, gb, xb in list(zip(lengths, r.unpack(g, nd), x))[::9 if len(lengths) > 9 else 1]:
        if n:
            assert torch.equal(xb, F.Plan(nf, n, nd, 1.2, 1.6, unfused=True).adjoint(gb)), n


@pytest.mark.parametrize("batch", (1, 12))
def test_step_by_step(batch):
    nf, nt, nd = 256, 500, 256
    p, g, y = _check(nf, nt, nd, batch=batch)
    ws, x = p.workspace(batch), torch.empty_like(y)
    for i in range(len(p.steps(True))):
        p.run_step(True, i, g, x, ws, batch)
    assert torch.equal(x, y)
