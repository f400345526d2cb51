"""Block passes, the default forward schedule: up to six iterations per launch
through LDS (Sec. 4, Algorithm 1). Every form is compared bit for bit with the
one-kernel-per-iteration schedule (unfused), which other tests tie to the
oracle, at the sizes where a block pass can go wrong: time tiles (224 samples
and two of them) plus and minus one, records shorter than a tile or than the
delays, each split of the iterations, chains at the limit a first pass adds up
itself, missing channel positions, unaligned buffers and ragged batches.
Exact equality: both schedules perform the same additions."""
import numpy as np
import pytest

from oracle import fdmt as ofdmt

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1411_5373_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)
FORMS = {"f32": (torch.float32, torch.float32), "f16": (torch.float16, torch.float32),
         "u8": (torch.uint8, torch.float32), "u8i": (torch.uint8, torch.int32), "i32": (torch.int32, torch.int32)}


def _input(shape, dtype, seed):
    g = torch.Generator(DEV).manual_seed(seed)
    if dtype in (torch.uint8, torch.int32):
        return torch.randint(0, 256, shape, device=DEV, generator=g, dtype=torch.int32).to(dtype)
    return torch.randn(shape, device=DEV, generator=g).to(dtype)


def _pair(nf, nt, nd, form, **kw):
    ind, acc = FORMS[form]
    band = kw.pop("band", (1.2, 1.6))
    print(f"block nf={nf} nt={nt} nd={nd} {form} {kw}", flush=True)
    p = F.Plan(nf, nt, nd, *band, in_dtype=ind, acc_dtype=acc, **kw)
    q = F.Plan(nf, nt, nd, *band, in_dtype=ind, acc_dtype=acc, unfused=True, **kw)
    return p, q


# 3 to 6 iterations in one pass, 4 + 3, 5 + 5, 6 + 6, 5 + 4 + 4; the channel
# counts below a power of two leave positions without a channel
@pytest.mark.parametrize("nf,nd", [(8, 9), (13, 40), (32, 33), (64, 64), (50, 200), (100, 90), (1000, 300),
                                   (4096, 200), (5000, 60)])
@pytest.mark.parametrize("nt", [1, 223, 224, 225, 449, 1000])
def test_tiles_and_splits(nf, nd, nt):
    p, q = _pair(nf, nt, nd, "f32")
    assert len(p.steps()) <= 3 + (nd / nf > 4)
    x = _input((nf, nt), torch.float32, nf + nt)
    assert torch.equal(p.forward(x), q.forward(x))


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("nf,nt,nd,batch", [(64, 700, 64, 1), (300, 2500, 301, 3), (2048, 1111, 700, 1)])
def test_types(form, nf, nt, nd, batch):
    p, q = _pair(nf, nt, nd, form)
    x = _input((batch, nf, nt), FORMS[form][0], nf)
    y = p.forward(x)
    assert torch.equal(y, q.forward(x))
    if form in ("u8", "i32") and nf == 64:
        np.testing.assert_array_equal(y[0].cpu().numpy().astype(np.int64),
                                      ofdmt(x[0].cpu().numpy().astype(np.int64), 1.2, 1.6, nd))


@pytest.mark.parametrize("form", ["f32", "u8", "f16"])
@pytest.mark.parametrize("nd", [32 * k for k in (1, 3, 4, 5, 6, 9)])
def test_chains(form, nd):
    """Chains of 0 to 4 samples are added by the first pass, longer ones by a
    separate initialisation."""
    p, q = _pair(32, 900, nd, form)
    x = _input((32, 900), FORMS[form][0], nd)
    assert torch.equal(p.forward(x), q.forward(x))


@pytest.mark.parametrize("form,off", [("u8", 1), ("u8", 2), ("u8", 3), ("f16", 1), ("f32", 1), ("f32", 3)])
def test_unaligned_input(form, off):
    """An input that starts off a word (or off 16 bytes): a slice of a larger buffer."""
    nf, nt, nd = 64, 1027, 70
    p, q = _pair(nf, nt, nd, form)
    x = _input((off + nf * nt,), FORMS[form][0], off)[off:].view(nf, nt)
    assert torch.equal(p.forward(x), q.forward(x.clone()))


@pytest.mark.parametrize("form", ["f32", "u8"])
@pytest.mark.parametrize("kw", [dict(d_min=1), dict(d_min=777), dict(rule=1), dict(gamma=2.0), dict(gamma=-3.0, d_min=50),
                                dict(band=(0.4, 0.8)), dict(band=(0.1, 2.0)), dict(wide_planes=True), dict(search_rows=2)])
def test_laws_and_options(form, kw):
    p, q = _pair(600, 1500, 310, form, **dict(kw))
    x = _input((600, 1500), FORMS[form][0], 5)
    assert torch.equal(p.forward(x), q.forward(x))


def test_search_pass_stays_fused():
    p = F.Plan(256, 3000, 100, 1.2, 1.6, search_rows=1)
    assert p.search_fused(8)
    assert not F.Plan(256, 3000, 100, 1.2, 1.6).search_fused(8)


@pytest.mark.parametrize("form", ["f32", "u8", "i32"])
def test_ragged(form):
    """Beams around the tile widths, empty ones among them, and many tiles per
    workgroup; each equals the uniform plan of its length."""
    nf, nd, ind = 128, 140, FORMS[form][0]
    lengths = [0, 1, 223, 224, 225, 447, 448, 449, 3000, 0, 10007]
    p = F.Plan(nf, 1 << 20, nd, 1.2, 1.6, in_dtype=ind, acc_dtype=FORMS[form][1])
    r = F.RaggedPlan(p, lengths)
    x = _input((nf * sum(lengths),), ind, 3)
    y = r.forward(x)
    for n, xb, yb in zip(lengths, r.unpack(x, nf), r.unpack(y, nd)):
        if n:
            q = F.Plan(nf, n, nd, 1.2, 1.6, in_dtype=ind, acc_dtype=FORMS[form][1], unfused=True)
            assert torch.equal(yb, q.forward(xb)), n


def test_graph_replays():
    """Captured once, replayed on new inputs with eager work in between."""
    p, _ = _pair(1000, 3000, 200, "u8")
    x = _input((1000, 3000), torch.uint8, 1)
    ws, y = p.workspace(), torch.empty(200, 3000, device=DEV)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        p.forward(x, out=y, ws=ws)
        with torch.cuda.graph(graph, stream=s):
            p.forward(x, out=y, ws=ws)
    torch.cuda.synchronize()
    for k in range(4):
        x.copy_(_input((1000, 3000), torch.uint8, 10 + k))
        ref = p.forward(x)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)


@pytest.mark.parametrize("form", ["u8", "u8i"])
@pytest.mark.parametrize("nf,nt,nd,off", [(8, 300001, 20, 0), (16, 262144, 30, 1), (32, 200003, 128, 2), (64, 131075, 64, 3),
                                          (128, 131000, 200, 0), (500, 70001, 120, 1), (1000, 60000, 1000, 0),
                                          (2048, 50007, 400, 3)])
def test_packed_sums(form, nf, nt, nd, off):
    """uint8 input long enough for the first pass to pack two 16-bit sums per
    word (3 to 6 iterations, into uint16 planes or straight to the output),
    from every byte alignment; the largest input value, so that any carry
    between the halves would show."""
    p, q = _pair(nf, nt, nd, form)
    x = _input((off + nf * nt,), torch.uint8, nf)
    x[: x.numel() // 2] = 255
    x = x[off:].view(nf, nt)
    assert torch.equal(p.forward(x), q.forward(x.clone()))
