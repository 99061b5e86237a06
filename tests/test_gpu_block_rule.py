"""The default block size of the X-engine, timed: at shapes on both sides of its rule
the default takes no more than a tenth longer than the better of 64 and 128."""
import pytest
import torch

import paper_1305_5639_amd as corr
from helpers import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(handles, run):
    t = {0: [], 64: [], 128: []}
    for _ in range(9):
        for tile in t:
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for c in handles * (1 if len(handles) > 1 else 3):
                c.set_tile(tile)
                run(c)
            e[1].record()
            torch.cuda.synchronize()
            t[tile].append(e[0].elapsed_time(e[1]))
    t = {tile: sorted(v)[4] for tile, v in t.items()}
    say("  " + ", ".join(f"{tile}: {v:.4f} ms" for tile, v in t.items()))
    assert t[0] < 1.1 * min(t[64], t[128])


def holding(N, C, A, prec):
    """A handle that holds spectra: noise, whose sums take the power that real ones take."""
    g = torch.Generator(device=DEV).manual_seed(3)
    S = torch.empty((A, C, N, 2), dtype=corr.SPECTRA_DTYPE[corr.PRECISIONS[prec]], device=DEV)
    for a in range(0, A, 64):
        x = torch.empty(S[a:a + 64].shape, device=DEV).normal_(0.0, 16.0 if prec == "int8" else 1.0, generator=g)
        S[a:a + 64] = x.to(S.dtype)
    c = corr.Correlator(N, 1, C, A, prec)
    c.xengine(A, S)
    return c


@pytest.mark.parametrize("prec,N,C,A", [
    ("int8", 80, 2048, 2560), ("fp16", 80, 2048, 1280), ("int8", 300, 512, 768), ("fp16", 256, 128, 384),
    ("fp16", 320, 256, 192), ("fp8", 200, 256, 2560), ("fp32", 200, 2048, 16), ("fp32", 200, 1024, 48),
    ("fp32", 256, 512, 1600), ("fp32", 1024, 16, 48)])
def test_default_block_size(prec, N, C, A):
    say(f"block rule {prec} N={N} C={C} A={A}")
    with holding(N, C, A, prec) as c:
        out = c.new_visibilities()
        check([c], lambda h: h.xengine_dump(A, out))


@pytest.mark.parametrize("prec,N,ni,nj,C,A,copies", [
    ("fp16", 700, 268, 422, 32, 1141, 6), ("fp16", 140, 68, 72, 512, 3200, 1), ("fp8", 260, 130, 130, 128, 2304, 1)])
def test_default_block_size_of_rectangles(prec, N, ni, nj, C, A, copies):
    """The first ni inputs against the last nj of N; with several copies (0.1 GB each)
    the spectra come from memory, not from the last-level cache."""
    say(f"block rule {prec} {ni} x {nj} of {N} C={C} A={A}")
    handles = [holding(N, C, A, prec) for _ in range(copies)]
    out = handles[0].xengine_rect(0, ni, N - nj, nj, A)
    check(handles, lambda h: h.xengine_rect(0, ni, N - nj, nj, A, out))
    for h in handles:
        h.close()
