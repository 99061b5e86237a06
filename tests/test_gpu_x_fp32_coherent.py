"""FP32 X-engine sums whose terms do not average out: sources common to all inputs
(with the phases of a quadrature and any), against FP32 sums taken one product
after another, and tones without noise over calls of many time blocks, whose
rounding errors have one sign, against a bound."""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_5639_amd as corr
from helpers import autos, cplx, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
C = 16
PIECE = 128                                            # time blocks that one running sum takes


def errors(got, ref, N):
    """(got - ref) / sqrt(C_ii C_jj), complex."""
    d = autos(ref, N)
    i, j = np.tril_indices(N)
    return (got - ref) / np.sqrt(d[:, i] * d[:, j])


def floats(x):
    """complex [A][C][N] -> float32 [A][C][N][2]."""
    return np.ascontiguousarray(x.astype(np.complex64)).view(np.float32).reshape(*x.shape, 2)


def reference(S):
    s = S.astype(np.float64)
    return oracle.xengine_f64(np.ascontiguousarray(np.swapaxes(s[..., 0] + 1j * s[..., 1], 1, 2)))


def triangle(S, tile=0):
    A, _, N, _ = S.shape
    with corr.Correlator(N, 1, C, A, "fp32") as c:
        c.set_tile(tile)
        c.xengine(A, torch.from_numpy(S).to(DEV))
        return cplx(c.dump().cpu().numpy())


@pytest.mark.parametrize("phases", ["quadrature", "any"])
@pytest.mark.parametrize("N,A,tile", [(20, 1024, 0), (48, 4096, 0), (70, 1024, 64), (70, 4096, 64), (70, 4096, 128)])
def test_common_source(N, A, tile, phases):
    """No further from float64, in the mean and at most, than FP32 sums of the products
    in turn."""
    say(f"fp32 common source {phases} N={N} A={A} tile={tile}")
    g = np.random.default_rng([3, N, A])
    n = lambda *s: g.standard_normal(s) + 1j * g.standard_normal(s)
    turn = 1j ** np.arange(N) if phases == "quadrature" else np.exp(2j * np.pi * g.random(N))
    S = floats(n(A, C, 1) * turn + 0.01 * n(A, C, N))
    ref = reference(S)
    e = errors(triangle(S, tile), ref, N)
    i, j = np.tril_indices(N)
    xr, xi = S[..., 0], S[..., 1]
    serial = np.empty(ref.shape, complex)
    for k in range(C):                                 # running sums in float32, two products a spectrum
        two = lambda p, q: np.stack([p, q], 1).reshape(2 * A, -1).cumsum(0, dtype=np.float32)[-1].astype(np.float64)
        a, b, c, d = xr[:, k, i], xr[:, k, j], xi[:, k, i], xi[:, k, j]
        serial[k] = two(a * b, c * d) + 1j * two(a * d, -(c * b))
    es = errors(serial, ref, N)
    for part in (np.real, np.imag):
        assert np.sqrt(np.mean(part(e) ** 2)) <= np.sqrt(np.mean(part(es) ** 2))
        assert np.abs(part(e)).max() <= np.abs(part(es)).max()


def tones(A, N):
    g = np.random.default_rng([5, N])
    t = np.outer(np.arange(A), g.random(C))[:, :, None]
    return floats(np.exp(2j * np.pi * (t + g.random(N))))


def check_tones(got, ref, N, A, waves):
    """A running sum takes PIECE time blocks, each an addition within 2^-24 of the sum
    so far (on average half the piece's total), then one addition per piece (and
    wave).  The real part of a block is summed from zero in 12 products of parts
    (within 2^-23 each, of the block's total), the imaginary part's 12 go straight
    into the running sum.  Products leave out 2^-24 of each, the output rounds once."""
    e = errors(got, ref, N)
    pieces = -(-A // (16 * PIECE * waves))
    rest = (pieces + waves) / 2 + 2
    assert np.abs(e.real).max() < (PIECE / 2 + 24 + rest) * 2.0 ** -24
    assert np.abs(e.imag).max() < (12 * PIECE / 2 + rest) * 2.0 ** -24


@pytest.mark.parametrize("N,A,tile,waves", [(70, 16389, 64, 1), (70, 16389, 128, 1), (20, 65541, 64, 8), (48, 32773, 64, 4)])
def test_tones_over_many_blocks(N, A, tile, waves):
    say(f"fp32 tones N={N} A={A} tile={tile}")
    S = tones(A, N)
    check_tones(triangle(S, tile), reference(S), N, A, waves)


def test_tones_over_many_blocks_rectangle_dump_and_batch():
    """The rectangle, the fused dump of a second call, and a batch member."""
    N, A = 70, 16389
    S = tones(A, N)
    ref = reference(S)
    dev = torch.from_numpy(S).to(DEV)
    say(f"fp32 tones N={N} A={A}: rectangle, dump")
    i, j = np.tril_indices(N)
    with corr.Correlator(N, 1, C, A, "fp32") as c:
        c.xengine(A, dev)
        rect = cplx(c.xengine_rect(33, 37, 0, 33, A).cpu().numpy())
        both = cplx(c.xengine_dump(A, None, dev).cpu().numpy())
    full = ref.copy()
    low = (i >= 33) & (j < 33)
    full[:, low] = rect[:, i[low] - 33, j[low]]
    check_tones(full, ref, N, A, 1)
    check_tones(both, 2 * ref, N, 2 * A, 1)
    say(f"fp32 tones N={N} A={A}: batch")
    with corr.Batch([(N, 1, C, A), (20, 1, C, 100)], "fp32") as b:
        b.subs[0].xengine(A, dev)                      # its spectra are held from here on
        b.subs[0].dump(reset=True)
        b.xengine([A, 0])
        check_tones(cplx(b.subs[0].dump().cpu().numpy()), ref, N, A, 1)
