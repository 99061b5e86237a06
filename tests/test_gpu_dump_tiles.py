"""Dump conversions in tiles of 32 inputs, 64 products and 32 channels: sizes
around the tiles, every layout and order, exact against the oracle's emission;
batch sub-arrays too, whose zero flag replaces the accumulators."""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_5639_amd as corr
from helpers import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FORMS = [(lay, order) for lay in ("lower", "upper", "full") for order in ("chan", "baseline")]


@pytest.mark.parametrize("N,C", [(1, 16), (11, 32), (31, 16), (32, 64), (33, 32), (65, 16)])
@pytest.mark.parametrize("layout,order", FORMS)
def test_dump_tiles(N, C, layout, order):
    A = 3
    say(f"dump N={N} C={C} {layout} {order}")
    S = np.random.default_rng([N, C]).integers(-127, 128, (A, C, N, 2), dtype=np.int8)
    ref = oracle.emit(oracle.xengine_i8(np.ascontiguousarray(np.swapaxes(S, 1, 2))), N, layout, order)
    dev = torch.from_numpy(S).to(DEV)
    with corr.Correlator(N, 1, C, A, "int8", layout, order) as c:
        c.xengine(A, dev)
        assert np.array_equal(c.dump(reset=True).cpu().numpy().astype(np.int64).reshape(ref.shape), ref)
        assert not c.dump().any()
    with corr.Batch([(N, 1, C, A)] * 2, "int8", layout, order) as b:
        for sub in b.subs:
            sub.xengine(A, dev)
        b.xengine([A, 0])                              # the first one again
        for sub, times in zip(b.subs, (2, 1)):
            got = sub.dump(reset=True).cpu().numpy().astype(np.int64).reshape(ref.shape)
            assert np.array_equal(got, times * ref)
            assert not sub.dump().any()
