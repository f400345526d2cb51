"""Block passes of the adjoint whose blocks start at windows of their own (a
smallest delay, delays longer than the record), against the one-kernel-per-
iteration schedule, bit for bit: records shorter and longer than the delays,
blocks split because their offsets lie apart, ragged batches whose beams are
shorter and longer than the plan's Nt."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402

from test_gpu_adjoint_block import _check, _grad  # noqa: E402


@pytest.mark.parametrize("nf,nt,nd,d_min", [(1024, 1024, 64, 10000), (1024, 1024, 64, 100000), (64, 1000, 64, 100000),
                                            (64, 250, 40, 700), (50, 300, 64, 3000), (64, 20000, 64, 10000),
                                            (600, 5000, 200, 20000), (4096, 2049, 100, 1500), (1024, 512, 2048, 0),
                                            (256, 100, 1000, 0), (256, 100, 1000, 90), (2048, 304, 1884, 0)])
def test_offsets(nf, nt, nd, d_min):
    p, _, _ = _check(nf, nt, nd, d_min=d_min)
    assert p.steps(True)[0]["lds_bytes"] > 0
    _check(nf, nt, nd, batch=2, dtype=torch.int32, d_min=d_min)


@pytest.mark.parametrize("nt", (800, 1 << 17))
@pytest.mark.parametrize("nf,nd,d_min", [(256, 128, 5000), (64, 1000, 0), (128, 700, 300)])
def test_ragged(nf, nd, d_min, nt):
    lengths = [31, 0, 224, 799, 801, 1, 6007, 30000]
    p = F.Plan(nf, nt, nd, 1.2, 1.6, d_min=d_min)
    r = F.RaggedPlan(p, lengths)
    g = _grad((nd * sum(lengths),), torch.float32, 3)
    for n, gb, xb in zip(lengths, r.unpack(g, nd), r.unpack(r.adjoint(g), nf)):
        if n:
            q = F.Plan(nf, n, nd, 1.2, 1.6, d_min=d_min, unfused=True)
            assert torch.equal(xb, q.adjoint(gb)), n


@pytest.mark.parametrize("nf,nt,nd,batch", [(100, 700, 100, 40), (50, 1000, 100, 30), (64, 20000, 200, 3),
                                            (16, 1000, 100, 50), (128, 1000, 128, 33), (8, 3001, 30, 20)])
def test_blocks_that_change_places(nf, nt, nd, batch):
    """2 to 32 blocks, an even number, over more than 16 tiles and beams."""
    _check(nf, nt, nd, batch=batch)
    lengths = [nt - 17 * b for b in range(batch) if nt > 17 * b]
    r = F.RaggedPlan(F.Plan(nf, nt, nd, 1.2, 1.6), lengths)
    g = _grad((nd * sum(lengths),), torch.float32, 3)
    for n, gb, xb in list(zip(lengths, r.unpack(g, nd), r.unpack(r.adjoint(g), nf)))[::7]:
        assert torch.equal(xb, F.Plan(nf, n, nd, 1.2, 1.6, unfused=True).adjoint(gb)), n
