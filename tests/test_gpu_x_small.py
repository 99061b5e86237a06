"""The X-engine of small arrays, whose waves share out the time blocks: sizes
around its input blocks and its least number of time blocks, ragged last
blocks, a second call into the same integration, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_5639_amd as corr
from helpers import cplx, say, vis_errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TB = {"fp32": 16, "fp16": 32, "fp8": 64, "int8": 64}


@pytest.mark.parametrize("prec", ["fp32", "fp16", "fp8", "int8"])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 64])
@pytest.mark.parametrize("blocks", [3, 4, 5, 6, 9, 17])
def test_small_arrays(prec, N, blocks):
    A, C = blocks * TB[prec] - 5, 16
    say(f"small X {prec} N={N} A={A}")
    g = torch.Generator(device=DEV).manual_seed(1000 * N + blocks)
    x = torch.empty((A, C, N, 2), device=DEV).normal_(0.0, 16.0 if prec == "int8" else 1.0, generator=g)
    S = x.round().clamp(-127, 127).to(torch.int8) if prec == "int8" else x.to(corr.SPECTRA_DTYPE[corr.PRECISIONS[prec]])
    with corr.Correlator(N, 1, C, A, prec) as c:
        c.xengine(A, S)
        one = c.dump(reset=False).cpu().numpy()
        c.xengine(A, S)
        two = c.dump().cpu().numpy()
    if prec == "int8":
        ref = oracle.xengine_i8(np.ascontiguousarray(np.swapaxes(S.cpu().numpy(), 1, 2)))
        assert np.array_equal(one.astype(np.int64), ref) and np.array_equal(two.astype(np.int64), 2 * ref)
        return
    s = S.float().cpu().numpy().astype(np.float64)
    ref = oracle.xengine_f64(np.ascontiguousarray(np.swapaxes(s[..., 0] + 1j * s[..., 1], 1, 2)))
    # FP32 sums: at most 24 products an MFMA chain and one addition a block or
    # wave, each within 2^-23 of sqrt(C_ii C_jj).  FP16 products are exact, and
    # their sums round like FP32's (1e-6 as for the larger arrays, and the
    # chain above).  The FP8 matrix cores' own sums are coarser: 1e-3, far
    # below E4M3's step of 2^-4.
    bar = {"fp32": (24 + blocks + 8) * 2.0 ** -23, "fp16": (8 + blocks + 8) * 2.0 ** -23, "fp8": 1e-3}[prec]
    assert vis_errors(cplx(one), ref, N)[1].max() < bar
    assert vis_errors(cplx(two), 2 * ref, N)[1].max() < bar
