"""The default block size of the X-engine, timed: at shapes on both sides of its rule
the default takes no more than a tenth longer than the better of 64 and 128."""
import pytest
import torch

import paper_1305_5639_amd as corr
from helpers import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(c, run):
    t = {0: [], 64: [], 128: []}
    for _ in range(9):
        for tile in t:
            c.set_tile(tile)
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(3):
                run()
            e[1].record()
            torch.cuda.synchronize()
            t[tile].append(e[0].elapsed_time(e[1]) / 3)
    t = {tile: sorted(v)[4] for tile, v in t.items()}
    say("  " + ", ".join(f"{tile}: {v * 1e3:.1f} us" for tile, v in t.items()))
    assert t[0] < 1.1 * min(t[64], t[128])


def holding(N, C, A, prec):
    """A handle that holds spectra (the low-precision forms take as long for zeros)."""
    S = torch.zeros((A, C, N, 2), dtype=corr.SPECTRA_DTYPE[corr.PRECISIONS[prec]], device=DEV)
    if prec == "fp32":
        S.normal_(generator=torch.Generator(device=DEV).manual_seed(3))
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
        check(c, lambda: c.xengine_dump(A, out))


@pytest.mark.parametrize("prec,ni,nj,C,A", [
    ("fp16", 268, 422, 32, 1141), ("fp16", 68, 72, 512, 3200), ("fp8", 130, 130, 128, 2304)])
def test_default_block_size_of_rectangles(prec, ni, nj, C, A):
    say(f"block rule {prec} {ni} x {nj} C={C} A={A}")
    with holding(ni + nj, C, A, prec) as c:
        out = c.xengine_rect(0, ni, ni, nj, A)
        check(c, lambda: c.xengine_rect(0, ni, ni, nj, A, out))
