"""FP32 X-engine sums that the split into BF16 parts does not carry and that are
formed again with FP32 MFMAs, in each kernel that has that rule: small arrays,
blocks of 64 and 128 inputs, the rectangle and batch members.  Inputs too small for
the parts, the largest floats, infinities and NaN, from the first spectrum on, from
the middle and in the ragged last time block only, against float64."""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_5639_amd as corr
from helpers import autos, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
C, A = 16, 21 * 16 + 7
WAYS = [("small", 20), ("small", 32), ("small", 50), ("small", 64), ("64", 70), ("128", 70), ("128", 140), ("rect64", 140),
        ("rect128", 140), ("batch", 70), ("batch", 140)]


def cplx(x):
    """The pairs as they are (re + 1j * im makes NaN of an infinite im)."""
    return x.cpu().numpy().astype(np.float64).view(np.complex128)[..., 0]


def correlate(S, way):
    """Lower triangle [C][B]; the rectangle's ways: [C][ni][nj], rows N/2.. and columns ..N/2."""
    N = S.shape[2]
    dev = torch.from_numpy(S).to(DEV)
    if way == "batch":
        with corr.Batch([(N, 1, C, A), (20, 1, C, 16)], "fp32") as b:
            b.subs[0].xengine(A, dev)                  # its spectra are held from here on
            b.subs[0].dump(reset=True)
            b.xengine([A, 0])
            return cplx(b.subs[0].dump())
    with corr.Correlator(N, 1, C, A, "fp32") as c:
        c.set_tile({"small": 0, "rect64": 64, "rect128": 128}.get(way) if not way.isdigit() else int(way))
        c.xengine(A, dev)
        if way.startswith("rect"):
            return cplx(c.xengine_rect(N // 2, N - N // 2, 0, N // 2, A))
        return cplx(c.dump())


def reference(S, way):
    N = S.shape[2]
    s = S.astype(np.float64)
    ref = oracle.xengine_f64(np.ascontiguousarray(np.swapaxes(s[..., 0] + 1j * s[..., 1], 1, 2)))
    return (ref,) + places(N, way)


def places(N, way):
    """Rows and columns of the results."""
    if way.startswith("rect"):
        return np.meshgrid(np.arange(N // 2, N), np.arange(N // 2), indexing="ij")
    return np.tril_indices(N)


def bar():
    """Sums of 16 spectra from zero and one addition for each, or the products one after
    another, each within 2^-24 of the sum so far, on average half of sqrt(C_ii C_jj)."""
    return (24 + 2 * A / 2) * 2.0 ** -24


@pytest.mark.parametrize("way,N", WAYS)
@pytest.mark.parametrize("small,which", [(2.0 ** -41, "all"), (2.0 ** -50, "all"), (2.0 ** -41, "one"), (1e-30, "one"),
                                         (2.0 ** -50, "late"), (1e-30, "late")])
def test_small_inputs(way, N, small, which):
    """All inputs, one, or one that is zero up to its ragged last time block."""
    say(f"fp32 small inputs {way} N={N} {small:g} {which}")
    p = N // 3
    S = np.random.default_rng([11, N]).standard_normal((A, C, N, 2))
    if which == "late":
        S[:A - 5, :, p] = 0
    S[:, :, slice(None) if which == "all" else p] *= small
    S = S.astype(np.float32)
    ref, i, j = reference(S, way)
    got, want = correlate(S, way), ref[:, i * (i + 1) // 2 + j]
    d = autos(ref, N)
    if small < 1e-20:                                  # (that input's auto lies below the float range)
        keep = ~((i == p) & (j == p))
    else:
        keep = np.ones(i.shape, bool)
    e = np.abs(got - want) / np.sqrt(d[:, i] * d[:, j])
    assert e[:, keep].max() < bar(), e[:, keep].max()


@pytest.mark.parametrize("way,N", WAYS)
@pytest.mark.parametrize("value", [np.inf, np.nan, np.float32(3.4e38)])
@pytest.mark.parametrize("spectrum", [0, A // 2, A - 1])
def test_values_without_parts(way, N, value, spectrum):
    """One such value, alone in its input: its products are the value times the
    others' values of that spectrum, those of the other inputs are unharmed."""
    say(f"fp32 value {value} {way} N={N} spectrum {spectrum}")
    p = N // 3
    S = np.random.default_rng([12, N]).uniform(0.25, 0.5, (A, C, N, 2)).astype(np.float32)
    S[:, :, p] = 0
    clean = S.copy()
    S[spectrum, :, p, 0] = value
    ref, i, j = reference(clean, way)
    got, want = correlate(S, way), ref[:, i * (i + 1) // 2 + j]
    mine = (i == p) | (j == p)
    assert np.all(np.abs(got - want)[:, ~mine] <= bar() * np.abs(want)[:, ~mine].real.max())
    own = mine & (i == j)
    assert not got[:, own].imag.any()
    assert np.all(np.isnan(got[:, own].real) if np.isnan(value) else np.isposinf(got[:, own].real))
    for rows, sign in ((mine & (i == p) & (j != p), 1.0), (mine & (j == p) & (i != p), -1.0)):
        other = np.where(i == p, j, i)[rows]
        # conj(S_p) S_q for p = i, its conjugate for p = j
        re = float(value) * S[spectrum][:, other, 0].astype(np.float64)
        im = sign * float(value) * S[spectrum][:, other, 1].astype(np.float64)
        for part, w in ((got.real[:, rows], re), (got.imag[:, rows], im)):
            assert np.allclose(part, w, rtol=2.0 ** -22, atol=0, equal_nan=True)


def test_small_inputs_end_the_split_early():
    """Where the second sum is known to be needed from the first time block on, the
    first one ends there: both in full take more than twice as long as usual
    data, the second alone 1.4 times."""
    N, C, A = 128, 2048, 512
    say(f"fp32 time of small inputs N={N} C={C} A={A}")
    S = torch.empty((A, C, N, 2), device=DEV).normal_(generator=torch.Generator(device=DEV).manual_seed(13))
    times = []
    for scale in (1.0, 2.0 ** -46):
        with corr.Correlator(N, 1, C, A, "fp32") as c:
            c.xengine(A, S * scale)
            out = c.new_visibilities()
            t = []
            for _ in range(9):
                e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                e[0].record()
                c.xengine_dump(A, out)
                e[1].record()
                torch.cuda.synchronize()
                t.append(e[0].elapsed_time(e[1]))
            times.append(sorted(t)[4])
    say(f"  {times[0]:.3f} and {times[1]:.3f} ms")
    assert times[1] < 1.75 * times[0]
