"""Block passes over batches of short records: a batch that fills the GPU takes
whole blocks where one record takes smaller ones. Around the number of records
where the form changes, every input type, chains, channels that are missing and
a smallest delay, step by step as well, against the one-kernel-per-iteration
schedule, bit for bit (both perform the same additions)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_block import FORMS, _input, _pair  # noqa: E402


# Nf=64, Nt=1024: whole blocks from 26 records on; Nf=256, Nt=500 from 9 and 11
# in its passes; Nf=50, Nt=1000 from 15; Nf=8 from 52; Nf=4096, Nt=1000 in its second pass from 4
@pytest.mark.parametrize("nf,nt,nd,batches", [(64, 1024, 64, (25, 26, 60)), (256, 500, 256, (8, 9, 10, 11)),
                                              (50, 1000, 100, (14, 15)), (8, 1000, 30, (51, 52)), (64, 223, 40, (300,)),
                                              (33, 225, 64, (300,)), (4096, 1000, 512, (3, 4))])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_records(form, nf, nt, nd, batches):
    p, q = _pair(nf, nt, nd, form)
    for batch in batches:
        x = _input((batch, nf, nt), FORMS[form][0], batch)
        assert torch.equal(p.forward(x), q.forward(x)), batch


@pytest.mark.parametrize("kw", [dict(d_min=700), dict(rule=1), dict(gamma=2.0), dict(search_rows=2), dict(wide_planes=True)])
def test_laws(kw):
    p, q = _pair(200, 600, 90, "u8", **kw)
    x = _input((60, 200, 600), torch.uint8, 1)
    assert torch.equal(p.forward(x), q.forward(x))


def test_step_by_step():
    nf, nt, nd, batch = 256, 500, 256, 20
    p, q = _pair(nf, nt, nd, "f32")
    x = _input((batch, nf, nt), torch.float32, 1)
    ws, y = p.workspace(batch), torch.empty(batch, nd, nt, device="cuda")
    for i in range(len(p.steps())):
        p.run_step(False, i, x, y, ws)
    assert torch.equal(y, q.forward(x))


@pytest.mark.parametrize("form", ["f32", "u8"])
def test_ragged(form):
    """A ragged batch takes whole blocks by its samples, whatever the plan's Nt."""
    import paper_1411_5373_amd as F
    nf, nd = 100, 90
    p, _ = _pair(nf, 300, nd, form)
    for lengths in ([300, 0, 17], [224 + 3 * b for b in range(120)], [30000, 1, 449]):
        r = F.RaggedPlan(p, lengths)
        x = _input((nf * sum(lengths),), FORMS[form][0], 2)
        y = r.unpack(r.forward(x), nd)
        for n, xb, yb in list(zip(lengths, r.unpack(x, nf), y))[::11 if len(lengths) > 9 else 1]:
            if n:
                assert torch.equal(yb, _pair(nf, n, nd, form)[1].forward(xb)), n
