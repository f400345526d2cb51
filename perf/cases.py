"""Workloads of the dispersion measure transform, as a user's program runs them.

Each case is one call, or one differentiated step, through the package's tensor layer: forward transforms,
adjoints, gradients through autograd, ragged batches of beams, boxcar searches over an output plane, and whole
searches with a candidate list. Sizes run from a 64-channel record of a thousand samples, where launches are what
counts, to 4096 channels of 65536 samples and batches of 16 beams; channel counts that are no power of two, odd
lengths, a smallest delay, other bands and every input and accumulation type are among them. Plans are asked for
with tuned=True throughout: sizes the stored schedules know take theirs, the others the built-in default.

exact() evaluates the same transform in float64 with plain torch, from the definition alone (one C per merge at the
border frequency, t0 - t1 = floor(dt C + 0.5), the recursion over ceil(log2 Nf) iterations).
"""
import math

import numpy as np
import torch

import paper_1411_5373_amd as F

DEV = "cuda"
TYPES = {"f32": (torch.float32, torch.float32), "f16": (torch.float16, torch.float32),
         "u8": (torch.uint8, torch.float32), "u8-i32": (torch.uint8, torch.int32),
         "i32": (torch.int32, torch.int32)}
# The widest running sum of a search is 2^WIDTHS samples, its threshold THRESHOLD standard deviations.
# Candidates are kept in records of RECORD entries, the unused ones zero.
WIDTHS, THRESHOLD, RECORD = 8, 7.0, 8192


def _case(op, nf, nt, nd, dtype="f32", batch=1, band=(1.2, 1.6), d_min=0):
    return {"op": op, "nf": nf, "nt": nt, "nd": nd, "dtype": dtype, "batch": batch, "f_min": band[0],
            "f_max": band[1], "d_min": d_min}


def listed():
    low = (0.4, 0.8)
    return [
        # a short record looked at by hand, or a trigger's cut-out: the smallest call there is
        dict(_case("forward", 64, 1024, 64), name="cutout_f32"),
        # one block of a 1024-channel stream in calibrated float
        dict(_case("forward", 1024, 8192, 1024), name="block_f32"),
        # the survey block as digitised: 8 bits, 4096 channels, 65536 samples
        dict(_case("forward", 4096, 65536, 2048, "u8"), name="survey_u8"),
        # half-precision stream of a size no stored schedule knows, with a time axis that is not a multiple of 64
        dict(_case("forward", 2048, 30003, 1500, "f16"), name="stream_f16"),
        # 1000 channels of a low band, 8 bits, odd length: a filterbank file as it comes
        dict(_case("forward", 1000, 40001, 900, "u8", band=low), name="filterbank_u8"),
        # exact sums of a few beams with 336 channels, searched from a known smallest delay on
        dict(_case("forward", 336, 16384, 512, "u8-i32", batch=4, d_min=300), name="beams_u8_i32"),
        # the gradient of the survey block
        dict(_case("adjoint", 4096, 65536, 2048), name="survey_adjoint"),
        # a training step's transform and its gradient, a batch of 16 beams
        dict(_case("grad", 1024, 16384, 1024, batch=16, band=low), name="train_batch16"),
        # the same of a small model fitted to short records
        dict(_case("grad", 256, 3001, 300, batch=3), name="train_short"),
        # beams of different lengths, forward and adjoint, packed back to back
        dict(_case("ragged", 1024, 32768, 512, batch=32), name="ragged_beams"),
        # the pulse-width search over planes that a transform left in memory
        dict(_case("boxcar", 0, 32768, 1024, batch=2), name="widths"),
        # the survey's whole search: transform, widths, candidates
        dict(_case("search", 4096, 65536, 2048, "u8"), name="survey_search"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: Nf 32..4096 (half of them powers of two), Nt 512..65536, Nd 16..2048, up to
    16 beams, no larger than the survey block."""
    op = rng.choice(("forward", "forward", "forward", "adjoint", "grad", "ragged", "boxcar", "search"))
    while True:
        nf = 2 ** rng.randint(5, 12) if rng.random() < 0.5 else _log(rng, 32, 4096)
        nt = _log(rng, 512, 65536)
        if rng.random() < 0.5:
            nt = -(-nt // 64) * 64
        nd = min(_log(rng, 16, 2048), nt)
        batch = rng.choice((1, 1, 2, 4, 16)) if op != "ragged" else rng.choice((4, 12, 32))
        if batch * nt * max(nf, 2 * nd) <= 2 ** 28:
            break
    band = rng.choice(((1.2, 1.6), (0.4, 0.8), (1.1, 1.9)))
    dtype = rng.choice({"forward": ("u8", "u8", "f32", "f16", "i32", "u8-i32"), "search": ("u8", "f32", "f16")}.get(op, ("f32",)))
    d_min = rng.randint(1, 1000) if op == "forward" and rng.random() < 0.2 else 0
    if op == "boxcar":
        nf = 0
    return _case(op, nf, nt, nd, dtype, batch, band, d_min)


def _lengths(case):
    """Samples of each beam of a ragged batch: log-uniform in [Nt / 16, Nt], the same for every seed."""
    r = np.random.default_rng(case["nt"] * 64 + case["batch"])
    return [int(n) for n in np.rint(np.exp(r.uniform(math.log(case["nt"] / 16), math.log(case["nt"]), case["batch"])))]


def _pulses(x, case, seed):
    """Adds two dispersed pulses of 8 to 20 standard deviations of the band's sum to every beam of x
    [batch][nf][nt]."""
    b, nf, nt = x.shape
    r = np.random.default_rng(seed)
    centre = case["f_min"] + (np.arange(nf) + 0.5) * ((case["f_max"] - case["f_min"]) / nf)
    frac = (case["f_min"] ** -2 - centre ** -2) / (case["f_min"] ** -2 - case["f_max"] ** -2)
    for k in range(b):
        for _ in range(2):
            dt, at = case["d_min"] + int(r.integers(0, case["nd"])), int(r.integers(0, nt))
            t = np.rint(at - dt * frac).astype(np.int64)
            ch = np.nonzero(t >= 0)[0]
            x[k, torch.from_numpy(ch).to(x.device), torch.from_numpy(t[ch]).to(x.device)] += float(r.uniform(8, 20)) / math.sqrt(nf)


def _intensity(case, seed, shape):
    """Noise of unit variance with pulses, in the input type: 8 bits and integers have mean 64 and deviation 8."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randn(shape, generator=g, device=DEV)
    _pulses(x, case, seed)
    if case["dtype"] in ("u8", "u8-i32", "i32"):
        x = x.mul_(8).add_(64).round_().clamp_(0, 255)
    return x.to(TYPES[case["dtype"]][0])


def _normal(seed, shape):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device=DEV)


def _shape(case, rows):
    """One beam is a matrix, several a batch of them."""
    return (rows, case["nt"]) if case["batch"] == 1 else (case["batch"], rows, case["nt"])


def _inputs(case, seed):
    """What a pass reads: "x" the intensities, "g" the gradient at the output, "y" the plane to search."""
    nf, nt, nd, b, op = case["nf"], case["nt"], case["nd"], case["batch"], case["op"]
    s = {}
    if op == "boxcar":
        # a transform's output: row dt sums about as many samples of noise whatever its delay
        y = _normal(seed, (b, nd, nt)).mul_(16.0).add_(torch.arange(nd, device=DEV)[:, None] * 0.05)
        y[:, :: max(1, nd // 7), nt // 3] += 160.0
        s["y"] = y.view(_shape(case, nd))
    elif op == "ragged":
        x = [_intensity(case, seed + 1000 * i, (1, nf, n)) for i, n in enumerate(_lengths(case))]
        s["x"] = torch.cat([v.reshape(-1) for v in x])
        s["g"] = _normal(seed + 1, (nd * sum(_lengths(case)),))
    else:
        if op != "adjoint":
            s["x"] = _intensity(case, seed, (b, nf, nt)).view(_shape(case, nf))
        if op in ("adjoint", "grad"):
            s["g"] = _normal(seed + 1, _shape(case, nd))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["op"] != "boxcar":
        kind, acc = TYPES[case["dtype"]]
        s["plan"] = F.Plan(case["nf"], case["nt"], case["nd"], case["f_min"], case["f_max"], in_dtype=kind,
                           acc_dtype=acc, d_min=case["d_min"], tuned=True)
    if case["op"] == "ragged":
        s["beams"] = F.RaggedPlan(s["plan"], _lengths(case))
    if case["op"] == "grad":
        s["x"].requires_grad_(True)
    return s


def run(s):
    op = s["case"]["op"]
    if op == "forward":
        return s["plan"].forward(s["x"])
    if op == "adjoint":
        return s["plan"].adjoint(s["g"])
    if op == "grad":
        y = F.fdmt(s["x"], s["plan"])
        (gx,) = torch.autograd.grad(y, s["x"], s["g"])
        return y.detach(), gx
    if op == "ragged":
        return s["beams"].forward(s["x"]), s["beams"].adjoint(s["g"])
    if op == "boxcar":
        return F.boxcar_search(s["y"], WIDTHS)
    out, stats, cands, count = s["plan"].forward_search(s["x"], WIDTHS, THRESHOLD)
    # the list comes in no particular order: by beam, delay, width and time, as the clustering after it reads it
    at = cands[:, :4].to(torch.int64)
    order = torch.argsort(((at[:, 0] * 65536 + at[:, 1]) * 16 + at[:, 3]) * 2 ** 31 + at[:, 2])
    cands = cands[order][:RECORD]
    cands = torch.nn.functional.pad(cands, (0, 0, 0, RECORD - cands.shape[0]))
    return {"out": out, "stats": stats, "where": cands[:, :4], "value": cands[:, 4:].view(torch.float32), "count": count}


def work(case):
    nf, nt, nd, b, op = case["nf"], case["nt"], case["nd"], case["batch"], case["op"]
    samples = sum(_lengths(case)) if op == "ragged" else b * nt
    size = {"f32": 4, "f16": 2, "u8": 1, "u8-i32": 1, "i32": 4}[case["dtype"]]
    stats = 20 * b * (WIDTHS + 1) * nd
    if op == "boxcar":
        # per sample and width: the doubling sum, the sum of squares, the sum and the peak
        return {"bytes": 4 * nd * samples + stats, "flops": 5 * (WIDTHS + 1) * nd * samples}
    levels = max(1, math.ceil(math.log2(nf)))
    # the additions of one transform (Sec. 4.1): the initial sums and one row of Nd per iteration
    adds = (nf + nd + nd * levels) * samples
    one = size * nf * samples + 4 * nd * samples
    back = 4 * nd * samples + 4 * nf * samples
    if op == "forward":
        return {"bytes": one, "flops": adds}
    if op == "adjoint":
        return {"bytes": back, "flops": adds}
    if op == "search":
        return {"bytes": one + stats, "flops": adds + 5 * (WIDTHS + 1) * nd * samples}
    return {"bytes": one + back, "flops": 2 * adds}


# ---------------------------------------------------------------- float64 reference


def _merges(nf, nd, f_min, f_max):
    """Per iteration, last first: (lower, upper, d_lo per row) of every sub-band, as channel ranges, with the rows
    each supplies. A sub-band is a range of channels; one without an upper half is passed on as it is."""
    levels = max(0, math.ceil(math.log2(nf)))
    df = (f_max - f_min) / nf

    def edge(k):
        return f_min + k * df

    rows = {(levels, 0): nd}
    plan = []
    for level in range(levels, 0, -1):
        step, half = 2 ** level, 2 ** (level - 1)
        todo = []
        for j in range(-(-nf // step)):
            n = rows[(level, j)]
            k0, km, k1 = j * step, j * step + half, min((j + 1) * step, nf)
            if km >= nf:
                rows[(level - 1, 2 * j)] = n
                todo.append((j, None))
                continue
            f0, f1, f2 = edge(k0), edge(km), edge(k1)
            c = (1.0 / (f1 * f1) - 1.0 / (f0 * f0)) / (1.0 / (f2 * f2) - 1.0 / (f0 * f0))
            lo = [int(math.floor(dt * c + 0.5)) for dt in range(n)]
            hi = [dt - d for dt, d in enumerate(lo)]
            rows[(level - 1, 2 * j)] = max(lo) + 1
            rows[(level - 1, 2 * j + 1)] = max(hi) + 1
            todo.append((j, lo))
        plan.append((level, todo))
    return plan, rows


def _delays(case):
    """Samples by which each channel is delayed before the transform (a smallest delay searched)."""
    nf = case["nf"]
    centre = case["f_min"] + (np.arange(nf) + 0.5) * ((case["f_max"] - case["f_min"]) / nf)
    frac = (case["f_min"] ** -2 - centre ** -2) / (case["f_min"] ** -2 - case["f_max"] ** -2)
    return [int(math.floor(case["d_min"] * v + 0.5)) for v in frac]


def _shifted(x, s):
    return torch.nn.functional.pad(x[..., : max(0, x.shape[-1] - s)], (min(s, x.shape[-1]), 0))


def _forward64(case, x):
    """The transform of x [batch][nf][nt] in float64."""
    plan, rows = _merges(case["nf"], case["nd"], case["f_min"], case["f_max"])
    pre = _delays(case)
    bands = []
    for k in range(case["nf"]):
        v = _shifted(x[:, k].double(), pre[k])
        acc, chain = v.clone(), []
        for d in range(rows[(0, k)]):
            if d:
                acc = acc + _shifted(v, d)
            chain.append(acc)
        bands.append(torch.stack(chain, 1))
    for level, todo in reversed(plan):
        nxt = []
        for j, lo in todo:
            if lo is None:
                nxt.append(bands[2 * j])
                continue
            a, b = bands[2 * j], bands[2 * j + 1]
            out = a[:, lo]
            for dt, d in enumerate(lo):
                out[:, dt, d:] += b[:, dt - d, : max(0, b.shape[-1] - d)]
            nxt.append(out)
            bands[2 * j] = bands[2 * j + 1] = None
        bands = nxt
    return bands[0]


def _adjoint64(case, g):
    """The transpose of the transform, applied to g [batch][nd][nt] in float64."""
    plan, rows = _merges(case["nf"], case["nd"], case["f_min"], case["f_max"])
    nt = g.shape[-1]
    bands = [g.double()]
    for level, todo in plan:
        nxt = []
        for j, lo in todo:
            out = bands[j]
            if lo is None:
                nxt.append(out)
                continue
            a = out.new_zeros((out.shape[0], max(lo) + 1, nt))
            b = out.new_zeros((out.shape[0], max(dt - d for dt, d in enumerate(lo)) + 1, nt))
            for dt, d in enumerate(lo):
                a[:, d] += out[:, dt]
                b[:, dt - d, : max(0, nt - d)] += out[:, dt, d:]
            nxt += [a, b]
            bands[j] = None
        bands = nxt
    pre, res = _delays(case), []
    for k in range(case["nf"]):
        v = bands[k]
        acc = torch.zeros_like(v[:, 0])
        for d in range(v.shape[1]):
            for i in range(d + 1):
                s = i + pre[k]
                acc[:, : max(0, nt - s)] += v[:, d, s:]
        res.append(acc)
    return torch.stack(res, 1)


def _boxcar64(y):
    """Per beam, width and row: peak, mean, deviation and their ratio of the running sums of y [batch][nd][nt]."""
    got = {"peak": [], "mean": [], "stdev": [], "snr": []}
    total = torch.nn.functional.pad(torch.cumsum(y.double(), -1), (1, 0))
    for j in range(WIDTHS + 1):
        w = 2 ** j
        b = total[..., 1:] - torch.nn.functional.pad(total[..., :-1], (w - 1, 0))[..., : y.shape[-1]]
        peak, mean, sd = b.amax(-1), b.mean(-1), b.std(-1, unbiased=False)
        for name, v in (("peak", peak), ("mean", mean), ("stdev", sd), ("snr", (peak - mean) / sd)):
            got[name].append(v)
    res = {k: torch.stack(v, 1) for k, v in got.items()}
    res["t"] = None
    return res


def exact(case, seed):
    s, op, b = _inputs(case, seed), case["op"], case["batch"]
    one = (lambda v: v[0]) if b == 1 else (lambda v: v)  # noqa: E731
    batch = lambda v: v[None] if b == 1 else v  # noqa: E731
    if op == "boxcar":
        return {k: v if v is None else one(v) for k, v in _boxcar64(batch(s["y"])).items()}
    if op == "ragged":
        n, nf, nd = _lengths(case), case["nf"], case["nd"]
        at = np.concatenate([[0], np.cumsum(n)])
        y, gx = [None] * len(n), [None] * len(n)
        order = sorted(range(len(n)), key=lambda i: n[i])
        for part in [order[i: i + 8] for i in range(0, len(order), 8)]:
            longest = n[part[-1]]  # shorter beams end in zeros, which no sample before them sees
            x = torch.zeros((len(part), nf, longest), device=DEV)
            g = torch.zeros((len(part), nd, longest), device=DEV)
            for k, i in enumerate(part):
                x[k, :, : n[i]] = s["x"][nf * at[i]: nf * at[i + 1]].view(nf, n[i])
                g[k, :, : n[i]] = s["g"][nd * at[i]: nd * at[i + 1]].view(nd, n[i])
            yy, gg = _forward64(case, x), _adjoint64(case, g)
            for k, i in enumerate(part):
                y[i], gx[i] = yy[k, :, : n[i]].reshape(-1), gg[k, :, : n[i]].reshape(-1)
        return torch.cat(y), torch.cat(gx)
    if op == "adjoint":
        return one(_adjoint64(case, batch(s["g"])))
    y = one(_forward64(case, batch(s["x"])))
    if op == "grad":
        return y, one(_adjoint64(case, batch(s["g"])))
    if op == "search":
        return {"out": y, "stats": {k: v if v is None else one(v) for k, v in _boxcar64(batch(y)).items()},
                "where": None, "value": None, "count": None}
    return y if case["dtype"] not in ("u8-i32", "i32") else None
