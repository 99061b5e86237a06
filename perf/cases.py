"""The work that users of the correlator have it do, as measurable cases.

Every case goes through the public entry points (Correlator, Batch and
corr_xengine_noalloc), with the handle, the output buffer and the scale table
that a program keeps between integrations made in prepare().  Kinds:

  fx       voltages -> F-engine -> X-engine -> dump, one integration of
           `calls` F + X calls (the last one fused with the dump where the
           layout allows it, as a streaming program does)
  caller   X-engine on spectra that the caller has, then a dump
  noalloc  the same through the call that allocates nothing
  rect     one input range against another, on held spectra
  spectra  the F-engine alone, its spectra copied out in the public layout
  batch    many uneven sub-arrays: F-engines, one batched X-engine, dumps

Voltages are unit complex noise plus exact-bin tones, or 8-bit real samples
(8 LSB rms noise and a tone); scales put a channel's spectra at 16 LSB rms for
int8, 8 for FP8 and 1 for FP16.
"""
import math
import random

import torch

from paper_1305_5639_amd import Batch, Correlator
from paper_1305_5639_amd import corr as C_API

ELEM = {"fp32": 4, "fp16": 2, "fp8": 1, "int8": 1}
DTYPE = {"fp32": torch.float32, "fp16": torch.float16, "fp8": torch.float8_e4m3fn, "int8": torch.int8}
BLOCK = {"fp32": 16, "fp16": 32, "fp8": 64, "int8": 64}      # spectra per time block
TARGET = {"fp32": 1.0, "fp16": 1.0, "fp8": 8.0, "int8": 16.0}
TONES = ((97, 0.5), (411, 0.35), (808, 0.25))


def _fx(name, st, pols, chan, spectra, prec, src="complex", calls=1, layout="lower", order="chan"):
    return {"name": name, "kind": "fx", "stations": st, "pols": pols, "channels": chan, "spectra": spectra,
            "prec": prec, "source": src, "calls": calls, "layout": layout, "order": order}


def listed():
    return [
        # A 16-station array with a 64-point transform: latency and launches.
        _fx("fx-tiny-fp32", 16, 1, 64, 1024, "fp32"),
        # Small 8-bit-sampled array, real transform of length 256.
        _fx("fx-real8-128-int8", 128, 1, 128, 1024, "int8", src="real8"),
        # The same sampling at 2048 streams, single precision.
        _fx("fx-real8-2048-fp32", 2048, 1, 128, 1024, "fp32", src="real8"),
        # 128 dual-polarisation stations, two calls to an integration of 1000
        # spectra, dumped baseline-major as an imager reads it.
        _fx("fx-256-c1024-fp32-baseline", 128, 2, 1024, 500, "fp32", calls=2, order="baseline"),
        # 256 dual-polarisation stations, exact integer correlation.
        _fx("fx-512-c2048-int8", 256, 2, 2048, 2048, "int8"),
        # Many channels in the lowest float precision.
        _fx("fx-512-c4096-fp8", 256, 2, 4096, 512, "fp8"),
        # A large array in single precision: matrix work.
        _fx("fx-1024-c2048-fp32", 512, 2, 2048, 512, "fp32"),
        # Spectra from elsewhere (another F-engine), inputs and spectra that
        # fill no block, the full matrix wanted.
        {"name": "caller-300-fp16-full", "kind": "caller", "stations": 150, "pols": 2, "channels": 1024,
         "spectra": 777, "prec": "fp16", "layout": "full", "order": "chan"},
        # A serving loop's small call.
        {"name": "noalloc-48-int8", "kind": "noalloc", "stations": 24, "pols": 2, "channels": 256,
         "spectra": 500, "prec": "int8"},
        # One node's product in the space-division model.
        {"name": "rect-512x512-fp16", "kind": "rect", "stations": 512, "pols": 2, "channels": 512,
         "spectra": 1024, "prec": "fp16", "i0": 512, "ni": 512, "j0": 0, "nj": 512},
        # Channelised data kept for another consumer; the longest transform,
        # in two appended pieces.
        {"name": "spectra-64-c8192-fp16", "kind": "spectra", "stations": 32, "pols": 2, "channels": 8192,
         "spectra": 200, "prec": "fp16", "source": "complex", "first": 128},
        # Sub-arrays of 16 to 64 dual-polarisation stations.
        {"name": "batch-24-fp16", "kind": "batch", "arrays": 24, "shapes_seed": 6, "prec": "fp16",
         "min_stations": 16, "max_stations": 64, "max_channels_log2": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fx", "fx", "fx", "fx", "caller", "caller", "noalloc", "rect", "spectra", "batch"])
    while True:
        pols = rng.choice([1, 2])
        n = _log(rng, 8, 1024)
        st = max(1, n // pols)
        n = st * pols
        prec = rng.choice(["fp32", "fp16", "fp8", "int8"])
        chan = 1 << rng.randint(4, 13)
        spectra = _log(rng, 16, 2048)
        if kind == "batch":
            return {"kind": "batch", "arrays": rng.randint(4, 24), "shapes_seed": rng.randint(0, 1 << 20),
                    "prec": prec, "min_stations": 8, "max_stations": rng.randint(24, 64),
                    "max_channels_log2": rng.randint(8, 10)}
        samples, cmac = n * chan * spectra, n * (n + 1) // 2 * chan * spectra
        if not (1 << 20) <= samples <= (1 << 29) or cmac > 4e11 or n * (n + 1) * chan * 8 > 6e9:
            continue
        base = {"kind": kind, "stations": st, "pols": pols, "channels": chan, "spectra": spectra, "prec": prec}
        lay = rng.choice(["lower", "lower", "lower", "upper", "full"])
        order = rng.choice(["chan", "chan", "baseline"])
        if kind == "fx":
            return {**base, "source": rng.choice(["complex", "complex", "real8"]), "calls": rng.choice([1, 1, 2]),
                    "layout": lay, "order": order}
        if kind == "caller":
            return {**base, "layout": lay, "order": order}
        if kind == "noalloc":
            if n > 256 or samples > (1 << 27):
                continue
            return base
        if kind == "spectra":
            b = BLOCK[prec]
            return {**base, "source": rng.choice(["complex", "real8"]),
                    "first": b * rng.randint(0, (spectra - 1) // b)}
        if n < 16:
            continue
        ni = rng.randint(n // 4, n // 2)
        nj = rng.randint(n // 4, n - ni)
        i_first = rng.random() < 0.5                     # disjoint ranges, either one first
        return {**base, "i0": 0 if i_first else n - ni, "ni": ni, "j0": n - nj if i_first else 0, "nj": nj}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _tones(chan):
    return sorted({k % chan: a for k, a in TONES}.items())


def _voltages(n, chan, spectra, seed):
    g = _gen(seed)
    x = torch.empty((n, spectra * chan), dtype=torch.complex64, device="cuda")
    t = torch.arange(chan, device="cuda", dtype=torch.float64)
    tones = [(a * torch.exp(2j * math.pi * k * t / chan)).to(torch.complex64) for k, a in _tones(chan)]
    phases = [torch.exp(2j * math.pi * torch.rand(n, generator=g, device="cuda")) for _ in tones]
    step = max(1, (1 << 26) // (spectra * chan))
    for p in range(0, n, step):
        part = x[p:p + step]
        torch.view_as_real(part).normal_(0.0, math.sqrt(0.5), generator=g)
        v = part.view(-1, spectra, chan)
        v += sum(ph[p:p + step, None] * tone for ph, tone in zip(phases, tones))[:, None, :]
    return x


def _samples(n, chan, spectra, seed):
    g = _gen(seed)
    x = torch.empty((n, spectra * 2 * chan), dtype=torch.int8, device="cuda")
    t = torch.arange(2 * chan, device="cuda", dtype=torch.float32)
    ph = 2 * math.pi * torch.rand(n, generator=g, device="cuda")
    step = max(1, (1 << 26) // (spectra * 2 * chan))
    for p in range(0, n, step):
        part = x[p:p + step].view(-1, spectra, 2 * chan)
        tone = 6 * torch.cos(2 * math.pi * (37 % chan) * t / (2 * chan) + ph[p:p + step, None])
        f = torch.empty(part.shape, device="cuda").normal_(0.0, 8.0, generator=g)
        part.copy_((f + tone[:, None, :]).round_().clamp_(-128, 127))
    return x


def _data(case, n, chan, spectra, seed):
    return (_samples if case.get("source") == "real8" else _voltages)(n, chan, spectra, seed)


def _inv_scale(prec, chan, source):
    """The requantiser's scale: the target over a channel's rms per component."""
    if prec == "fp32":
        return None
    if source == "real8":
        var = torch.full((chan,), chan * (64.0 + 1 / 12), dtype=torch.float64)
        var[37 % chan] += (6 * chan) ** 2 / 2
    else:
        var = torch.full((chan,), chan / 2, dtype=torch.float64)
        for k, a in _tones(chan):
            var[k] += (a * chan) ** 2 / 2
    return (TARGET[prec] / var.sqrt()).float().cuda()


def _caller_spectra(prec, spectra, chan, n, seed):
    x = torch.empty((spectra, chan, n, 2), dtype=DTYPE[prec], device="cuda")
    g = _gen(seed)
    step = max(1, (1 << 26) // (chan * n * 2))
    for a in range(0, spectra, step):
        part = x[a:a + step]
        f = torch.empty(part.shape, device="cuda").normal_(0.0, TARGET[prec], generator=g)
        part.copy_(f.round_().clamp_(-127, 127) if prec == "int8" else f)
    return x


def _caller_scale(prec, chan):
    if prec not in ("fp16", "fp8"):
        return None
    return (0.5 + torch.arange(chan, dtype=torch.float32) / chan).cuda()


def _shapes(case):
    r = random.Random(case["shapes_seed"])
    return [(_log(r, case["min_stations"], case["max_stations"]), 2, 1 << r.randint(6, case["max_channels_log2"]),
             _log(r, 64, 1024)) for _ in range(case["arrays"])]


def prepare(case, seed):
    kind, prec = case["kind"], case["prec"]
    s = {"case": case}
    if kind == "batch":
        shapes = _shapes(case)
        s["batch"] = Batch(shapes, prec)
        s["in"] = [_voltages(st * p, c, a, seed * 64 + i) for i, (st, p, c, a) in enumerate(shapes)]
        s["inv"] = [_inv_scale(prec, c, "complex") for _, _, c, _ in shapes]
        s["out"] = [sub.new_visibilities() for sub in s["batch"].subs]
        s["n"] = [a for _, _, _, a in shapes]
        return s
    st, pols, chan, spectra = case["stations"], case["pols"], case["channels"], case["spectra"]
    n = st * pols
    if kind in ("caller", "noalloc"):
        s["in"] = _caller_spectra(prec, spectra, chan, n, seed)
        s["inv"] = _caller_scale(prec, chan)
        if kind == "noalloc":
            s["params"] = C_API.make_params(st, pols, chan, spectra, prec)
            s["out"] = torch.empty((chan, n * (n + 1) // 2, 2), device="cuda",
                                   dtype=torch.int32 if prec == "int8" else torch.float32)
            return s
    else:
        s["in"] = _data(case, n, chan, spectra * case.get("calls", 1), seed)
        s["inv"] = _inv_scale(prec, chan, case.get("source"))
    h = s["h"] = Correlator(st, pols, chan, spectra, prec, case.get("layout", "lower"), case.get("order", "chan"))
    if kind in ("fx", "caller"):
        s["out"] = h.new_visibilities()
    elif kind == "rect":
        h.fengine(s["in"], spectra, s["inv"])
        s["in"] = None
        s["out"] = torch.empty((chan, case["ni"], case["nj"], 2), device="cuda",
                               dtype=torch.int32 if prec == "int8" else torch.float32)
    elif kind == "spectra":
        s["out"] = torch.empty((spectra, chan, n, 2), dtype=DTYPE[prec], device="cuda")
    return s


# ------------------------------------------------------------------ a pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        b = s["batch"]
        for sub, x, a, inv in zip(b.subs, s["in"], s["n"], s["inv"]):
            sub.fengine(x, a, inv)
        b.xengine(s["n"])
        return [sub.dump(o) for sub, o in zip(b.subs, s["out"])]
    spectra, inv = case["spectra"], s["inv"]
    if kind == "noalloc":
        C_API.corr_xengine_noalloc(s["params"], s["in"], spectra, inv, s["out"])
        return s["out"]
    h, out = s["h"], s["out"]
    fused = case.get("layout") == "lower" and case.get("order") == "chan"
    if kind == "caller":
        if fused:
            return h.xengine_dump(spectra, out, s["in"], inv)
        h.xengine(spectra, s["in"], inv)
        return h.dump(out)
    if kind == "rect":
        return h.xengine_rect(case["i0"], case["ni"], case["j0"], case["nj"], spectra, out)
    x, real8 = s["in"], case["source"] == "real8"
    fengine = h.fengine_real8 if real8 else h.fengine
    block = case["channels"] * (2 if real8 else 1)       # samples of one spectrum
    if kind == "spectra":
        first = case["first"]
        if first:
            fengine(x[:, :first * block], first, inv)
        fengine(x[:, first * block:], spectra - first, inv, first_spectrum=first)
        C_API.corr_copy_spectra(h.handle, out)
        return out
    calls = case["calls"]
    for c in range(calls):
        fengine(x[:, c * spectra * block:(c + 1) * spectra * block], spectra, inv)
        if fused and c == calls - 1:
            return h.xengine_dump(spectra, out)
        h.xengine(spectra)
    return h.dump(out)


# ----------------------------------------------------------- work and truth
def work(case):
    prec = case["prec"]
    if case["kind"] == "batch":
        total = {"bytes": 0, "flops": 0}
        for st, pols, chan, spectra in _shapes(case):
            w = work({"kind": "fx", "stations": st, "pols": pols, "channels": chan, "spectra": spectra, "prec": prec,
                      "source": "complex", "calls": 1, "layout": "lower"})
            total = {k: total[k] + w[k] for k in total}
        return total
    n, chan = case["stations"] * case["pols"], case["channels"]
    a = case["spectra"] * case.get("calls", 1)
    pairs = n * (n + 1) // 2
    held = n * chan * a * 2 * ELEM[prec]                 # spectra in the X-engine's element
    stored = n * n if case.get("layout") == "full" else pairs
    ffts = n * a * 5 * chan * math.log2(chan)
    volts = n * a * chan * (2 if case.get("source") == "real8" else 8)
    if case["kind"] == "rect":
        p = case["ni"] * case["nj"]
        return {"bytes": (case["ni"] + case["nj"]) * chan * a * 2 * ELEM[prec] + p * chan * 8, "flops": 8 * p * chan * a}
    if case["kind"] == "spectra":
        return {"bytes": volts + held, "flops": ffts}
    if case["kind"] == "fx":
        return {"bytes": volts + stored * chan * 8, "flops": ffts + 8 * pairs * chan * a}
    return {"bytes": held + stored * chan * 8, "flops": 8 * pairs * chan * a}


def _spectra64(case, n, chan, spectra, seed):
    """[channels][spectra][n] complex128 transforms of the case's data."""
    x = _data(case, n, chan, spectra, seed)
    out = torch.empty((chan, spectra, n), dtype=torch.complex128, device="cuda")
    step = max(1, (1 << 26) // (spectra * chan))
    for p in range(0, n, step):
        if case.get("source") == "real8":
            f = torch.fft.rfft(x[p:p + step].view(-1, spectra, 2 * chan).double())[..., :chan]
        else:
            f = torch.fft.fft(x[p:p + step].view(-1, spectra, chan).to(torch.complex128))
        out[:, :, p:p + step] = f.permute(2, 1, 0)
    return out


def _pairs64(spec, layout, order):
    """Sum over spectra of conj(S_i) S_j, in a dump's layout and order, (re, im) last."""
    chan, _, n = spec.shape
    if layout == "full":
        i, j = (t.reshape(-1) for t in torch.meshgrid(torch.arange(n), torch.arange(n), indexing="ij"))
    else:
        i, j = torch.tril_indices(n, n) if layout == "lower" else torch.triu_indices(n, n)
    flat = (i * n + j).cuda()
    out = torch.empty((chan, flat.numel()), dtype=torch.complex128, device="cuda")
    for k in range(chan):
        out[k] = (spec[k].mH.contiguous() @ spec[k]).reshape(-1)[flat]
    return torch.view_as_real(out.T.contiguous() if order == "baseline" else out)


def exact(case, seed):
    """The visibilities (or spectra) of unquantised float64 transforms.

    Integer forms fed by the F-engine have none: their values are those of
    the requantised spectra.  A caller's spectra are taken as they are.
    """
    kind, prec = case["kind"], case["prec"]
    if kind == "batch":
        if prec == "int8":
            return None
        return [_pairs64(_spectra64({}, st * p, c, a, seed * 64 + i), "lower", "chan")
                for i, (st, p, c, a) in enumerate(_shapes(case))]
    n, chan, spectra = case["stations"] * case["pols"], case["channels"], case["spectra"]
    if kind in ("caller", "noalloc"):
        x = _caller_spectra(prec, spectra, chan, n, seed)
        spec = torch.empty((chan, spectra, n), dtype=torch.complex128, device="cuda")
        for a in range(spectra):
            spec[:, a] = torch.view_as_complex(x[a].double())
        inv = _caller_scale(prec, chan)
        if inv is not None:
            spec /= inv.double()[:, None, None]
        return _pairs64(spec, case.get("layout", "lower"), case.get("order", "chan"))
    if prec == "int8":
        return None
    spec = _spectra64(case, n, chan, spectra * case.get("calls", 1), seed)
    if kind == "spectra":
        inv = _inv_scale(prec, chan, case["source"])
        if inv is not None:
            spec *= inv.double()[:, None, None]
        return torch.view_as_real(spec.permute(1, 0, 2).contiguous())
    if kind == "rect":
        i0, ni, j0, nj = (case[k] for k in ("i0", "ni", "j0", "nj"))
        out = torch.empty((chan, ni, nj), dtype=torch.complex128, device="cuda")
        for k in range(chan):
            out[k] = spec[k, :, i0:i0 + ni].mH.contiguous() @ spec[k, :, j0:j0 + nj]
        return torch.view_as_real(out)
    return _pairs64(spec, case["layout"], case["order"])
