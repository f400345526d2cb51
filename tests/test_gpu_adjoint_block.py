"""Block passes of the adjoint, its default schedule, against the one-kernel-
per-iteration schedule (unfused, which other tests tie to the oracle), bit for
bit: both add the same terms in the same order. Sizes where a block pass can go
wrong: both windows (256 and 512 samples), tiles and records plus and minus
one, records shorter than the shifts, each split of the iterations, lag counts
up to the separate initialisation, missing channels, other laws, ragged
batches, and a large smallest delay."""
import numpy as np
import pytest

from oracle import build_tables, fdmt_adjoint as oadj

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


def _grad(shape, dtype, seed):
    g = torch.Generator(DEV).manual_seed(seed)
    if dtype == torch.int32:
        return torch.randint(-1000, 1000, shape, device=DEV, generator=g, dtype=dtype)
    return torch.randn(shape, device=DEV, generator=g)


def _check(nf, nt, nd, batch=1, dtype=torch.float32, band=(1.2, 1.6), **kw):
    print(f"adjoint block nf={nf} nt={nt} nd={nd} batch={batch} {dtype} {kw}", flush=True)
    p = F.Plan(nf, nt, nd, *band, in_dtype=dtype, acc_dtype=dtype, **kw)
    q = F.Plan(nf, nt, nd, *band, in_dtype=dtype, acc_dtype=dtype, unfused=True, **kw)
    g = _grad((batch, nd, nt), dtype, nf + nt)
    y = p.adjoint(g)
    assert torch.equal(y, q.adjoint(g))
    return p, g, y


@pytest.mark.parametrize("nf,nd", [(4, 6), (6, 20), (8, 9), (16, 16), (32, 40), (64, 64), (50, 120), (100, 90),
                                   (500, 300), (1025, 200), (4096, 300)])
@pytest.mark.parametrize("nt", [1, 100, 227, 228, 229, 1025])
def test_tiles_and_splits(nf, nd, nt):
    p, g, y = _check(nf, nt, nd)
    if nf <= 100 and nt == 229:
        ref = oadj(g[0].cpu().numpy(), 1.2, 1.6, nf, acc=np.float32)
        np.testing.assert_array_equal(y[0].cpu().numpy(), ref)


@pytest.mark.parametrize("nf,nt,nd", [(256, 70001, 300), (1000, 30000, 900), (128, 131072, 64), (2048, 20011, 1500)])
def test_wide_windows(nf, nt, nd):
    _check(nf, nt, nd)


@pytest.mark.parametrize("nd", [32 * k for k in (1, 2, 3, 4, 5, 6, 9)])
def test_lags(nd):
    _check(32, 1500, nd, batch=2)


@pytest.mark.parametrize("kw", [dict(d_min=1), dict(d_min=900), dict(d_min=5000), dict(rule=1), dict(gamma=2.0),
                                dict(gamma=-3.0, d_min=50), dict(band=(0.4, 0.8)), dict(band=(0.1, 2.0))])
@pytest.mark.parametrize("dtype", [torch.float32, torch.int32])
def test_laws_and_types(kw, dtype):
    _check(600, 1500, 310, dtype=dtype, **dict(kw))


@pytest.mark.parametrize("dtype", [torch.float32, torch.int32])
@pytest.mark.parametrize("nt", [1000, 1 << 20])
def test_ragged(dtype, nt):
    """Windows of either size (the plan's Nt picks them); every beam equals the
    uniform plan of its length."""
    nf, nd = 128, 140
    lengths = [0, 1, 130, 223, 228, 229, 447, 513, 3000, 0, 10007]
    p = F.Plan(nf, nt, nd, 1.2, 1.6, in_dtype=dtype, acc_dtype=dtype)
    r = F.RaggedPlan(p, lengths)
    g = _grad((nd * sum(lengths),), dtype, 3)
    x = r.adjoint(g)
    for n, gb, xb in zip(lengths, r.unpack(g, nd), r.unpack(x, nf)):
        if n:
            q = F.Plan(nf, n, nd, 1.2, 1.6, in_dtype=dtype, acc_dtype=dtype, unfused=True)
            assert torch.equal(xb, q.adjoint(gb)), n


def test_unaligned_gradient():
    nf, nt, nd = 64, 1027, 70
    p = F.Plan(nf, nt, nd, 1.2, 1.6)
    q = F.Plan(nf, nt, nd, 1.2, 1.6, unfused=True)
    g = _grad((3 + nd * nt,), torch.float32, 1)[3:].view(nd, nt)
    assert torch.equal(p.adjoint(g), q.adjoint(g.clone()))


@pytest.mark.parametrize("nt", [5, 255, 1024, 1300, 3001])
@pytest.mark.parametrize("nd", [30, 60, 68, 130, 250])
@pytest.mark.parametrize("dtype,d_min", [(torch.float32, 0), (torch.float32, 77), (torch.int32, 0)])
def test_long_chains(nd, nt, dtype, d_min):
    """The separate initialisation's transpose: chains around its chunk of 16
    samples, records around its waves' 256, against the oracle's order."""
    p = F.Plan(4, nt, nd, 1.2, 1.6, in_dtype=dtype, acc_dtype=dtype, d_min=d_min)
    g = _grad((2, nd, nt), dtype, nd + nt)
    y = p.adjoint(g)
    t = build_tables(4, nd, 1.2, 1.6, d_min=d_min)
    for b in range(2):
        ref = oadj(g[b].cpu().numpy(), 1.2, 1.6, 4, tables=t, acc=np.int32 if dtype == torch.int32 else np.float32)
        np.testing.assert_array_equal(y[b].cpu().numpy(), ref)
    lengths = [nt, 0, 700, 1 + nt // 2]
    r = F.RaggedPlan(p, lengths)
    packed = torch.cat([_grad((nd, n), dtype, n).flatten() for n in lengths])
    for n, gb, xb in zip(lengths, r.unpack(packed, nd), r.unpack(r.adjoint(packed), 4)):
        ref = oadj(gb.cpu().numpy(), 1.2, 1.6, 4, tables=t, acc=np.int32 if dtype == torch.int32 else np.float32)
        np.testing.assert_array_equal(xb.cpu().numpy(), ref)
