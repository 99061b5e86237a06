"""The FP32 X-engine's sums of three BF16 parts: sizes around the blocks, time
blocks and the short-integration rule, gains far apart, and values the parts
cannot carry (infinities, the largest floats), against float64."""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_5639_amd as corr
from helpers import say, vis_errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def correlate(S, tile):
    A, C, N, _ = S.shape
    with corr.Correlator(N, 1, C, A, "fp32") as c:
        c.set_tile(tile)
        c.xengine(A, torch.from_numpy(S).to(DEV))
        return c.dump().cpu().numpy().astype(np.float64).view(np.complex128)[..., 0]


def reference(S):
    s = S.astype(np.float64)
    return oracle.xengine_f64(np.ascontiguousarray(np.swapaxes(s[..., 0] + 1j * s[..., 1], 1, 2)))


def bar(A):
    """Every sum takes at most 24 products per MFMA chain of a block of 16
    spectra and one addition per block, each within 2^-23 of sum |x_i||x_j|,
    which is at most sqrt(C_ii C_jj)."""
    return (24 + (A + 15) // 16) * 2.0 ** -23


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("N,A", [(1, 16), (31, 1), (33, 15), (64, 16), (65, 17), (97, 31), (128, 33), (129, 48),
                                 (193, 257)])
def test_edges(tile, N, A):
    say(f"fp32 split N={N} A={A} tile={tile}")
    S = np.random.default_rng([7, N, A]).standard_normal((A, 16, N, 2)).astype(np.float32)
    eF, en = vis_errors(correlate(S, tile), reference(S), N)
    assert en.max() < bar(A), en.max()


@pytest.mark.parametrize("tile", [64, 128])
def test_gains_far_apart(tile):
    """Per-input gains from 1e-36 to 1e18: parts of the smallest inputs lie
    below the normal range, their products with the others do not."""
    N, A = 130, 64
    say(f"fp32 split gains tile={tile}")
    S = np.random.default_rng(8).standard_normal((A, 16, N, 2))
    S = (S * np.logspace(-36, 18, N)[None, None, :, None]).astype(np.float32)
    got, ref = correlate(S, tile), reference(S)
    i, j = np.tril_indices(N)
    g = np.logspace(-36, 18, N)
    ok = np.outer(g, g)[i, j] > 1e-30                  # products well inside the float range
    _, en = vis_errors(got, ref, N)
    assert en[:, ok].max() < bar(A), en[:, ok].max()


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("value", [np.inf, np.float32(3.4e38)])
def test_values_past_the_parts(tile, value):
    """One value beyond BF16's finite range, alone in its input: the products
    with that input are the value times the others' (as FP32 gives them), all
    others are unharmed."""
    N, A, p = 140, 40, 70
    say(f"fp32 split value {value} tile={tile}")
    S = np.random.default_rng(9).uniform(0.25, 0.5, (A, 16, N, 2)).astype(np.float32)
    S[:, :, p] = 0
    S[5, :, p, 0] = value
    got = correlate(S, tile)
    i, j = np.tril_indices(N)
    mine = (i == p) | (j == p)
    clean = S.copy()
    clean[5, :, p, 0] = 0
    ref = reference(clean)
    assert np.all(np.abs(got - ref)[:, ~mine] <= bar(A) * np.abs(ref)[:, ~mine].real.max())
    assert np.all(np.isposinf(got[:, (i == p) & (j == p)].real))
    assert not got[:, (i == p) & (j == p)].imag.any()
    for rows, sign in (((i == p) & (j < p), 1.0), ((j == p) & (i > p), -1.0)):
        other = np.where(i == p, j, i)[rows]
        # conj(S_p) S_q for p = i, its conjugate for p = j
        want_re = float(value) * S[5][:, other, 0].astype(np.float64)
        want_im = sign * float(value) * S[5][:, other, 1].astype(np.float64)
        if np.isinf(value):
            assert np.array_equal(got.real[:, rows], want_re) and np.array_equal(got.imag[:, rows], want_im)
        else:
            assert np.allclose(got.real[:, rows], want_re, rtol=2.0 ** -22, atol=0)
            assert np.allclose(got.imag[:, rows], want_im, rtol=2.0 ** -22, atol=0)
