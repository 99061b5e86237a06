"""The block size of a batch's members in the persistent launch: input counts on
both sides of each step of its rule, in one batch, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_5639_amd as corr
from helpers import cplx, say, spectra_akp_to_apk, vis_errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPES = [(N, 1, 16, 130) for N in (64, 65, 128, 129, 192, 193, 256)]


@pytest.mark.parametrize("prec", ["int8", "fp16", "fp8", "fp32"])
def test_batch_block_sizes(prec):
    say(f"batch block sizes {prec}")
    g = torch.Generator(device=DEV).manual_seed(7)
    inv = None if prec == "fp32" else torch.full((16,), {"int8": 16.0, "fp16": 1.0, "fp8": 8.0}[prec] / 4.0, device=DEV)
    with corr.Batch(SHAPES, prec) as b:
        for (N, _, C, A), sub in zip(SHAPES, b.subs):
            sub.fengine(torch.view_as_complex(torch.empty((N, A * C, 2), device=DEV).normal_(generator=g)), A, inv)
        b.xengine([A for (_, _, _, A) in SHAPES])
        for (N, _, C, A), sub in zip(SHAPES, b.subs):
            S, got = sub.spectra().float().cpu().numpy(), sub.dump().cpu().numpy()
            if prec == "int8":
                assert np.array_equal(got.astype(np.int64), oracle.xengine_i8(spectra_akp_to_apk(S.astype(np.int8)))), N
                continue
            s = S.astype(np.float64) / (1.0 if inv is None else float(inv[0]))
            ref = oracle.xengine_f64(np.ascontiguousarray(np.swapaxes(s[..., 0] + 1j * s[..., 1], 1, 2)))
            # FP32 and FP16 sums: a chain of at most 24 products and of one
            # addition a 16-spectrum stage, and the scale's roundings, each within
            # 2^-23 of sqrt(C_ii C_jj); the FP8 matrix cores' own sums are coarser
            # (1e-3, far below E4M3's step of 2^-4)
            bar = 1e-3 if prec == "fp8" else (24 + (A + 15) // 16 + 8) * 2.0 ** -23
            assert vis_errors(cplx(got), ref, N)[1].max() < bar, N
