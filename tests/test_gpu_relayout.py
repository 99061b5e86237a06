"""Caller spectra into the held rows and out again, bit for bit: rows of spectra
whose columns end within a tile and within a vector, ragged time blocks, an
output that is aligned to one element only, with nothing written around it."""
import ctypes

import pytest
import torch

import paper_1305_5639_amd as corr
from paper_1305_5639_amd.corr import lib
from helpers import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TB = {"fp32": 16, "fp16": 32, "fp8": 64, "int8": 64}


@pytest.mark.parametrize("prec", ["fp32", "fp16", "fp8", "int8"])
@pytest.mark.parametrize("N", [1, 3, 31, 48, 129])
@pytest.mark.parametrize("extra", [1 - 64, -1, 0, 67])
def test_spectra_round_trip(prec, N, extra):
    C, A = 16, max(1, TB[prec] + extra)
    say(f"spectra round trip {prec} N={N} A={A}")
    es = 64 // TB[prec]
    g = torch.Generator(device=DEV).manual_seed(100 * N + A)
    raw = torch.randint(0, 256, (A * C * N * 2 * es,), dtype=torch.uint8, device=DEV, generator=g)
    S = raw.view(corr.SPECTRA_DTYPE[corr.PRECISIONS[prec]]).view(A, C, N, 2)
    want = raw.view(torch.int8).clamp(min=-127).view(torch.uint8) if prec == "int8" else raw
    with corr.Correlator(N, 1, C, A, prec) as c:
        c.xengine(A, S)
        assert torch.equal(c.spectra().view(torch.uint8).reshape(-1), want)
        # one element past a 16-byte boundary, between guards
        out = torch.full((raw.numel() + 64,), 0xA5, dtype=torch.uint8, device=DEV)
        at = 16 + es
        assert lib().corr_copy_spectra(c.handle, ctypes.c_void_p(out.data_ptr() + at), 1) == 0
        torch.cuda.synchronize()
        assert torch.equal(out[at:at + raw.numel()], want)
        assert bool((out[:at] == 0xA5).all()) and bool((out[at + raw.numel():] == 0xA5).all())
