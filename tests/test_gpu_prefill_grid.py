"""The prefill's grid: one row block per workgroup while all fit on the chip
(blocks x heads <= 512), pairs of blocks past that, at the sizes on both sides
of the line and with odd block counts, against the fp64 oracle on sampled
heads (bf16 tolerance 2e-2 on unit-scale inputs)."""
import numpy as np
import pytest
import torch

import dar_inputs as di
from oracle import oracle
from tests.dev import to_dev, to_host64, tol

pytestmark = pytest.mark.gpu

dar = pytest.importorskip("paper_2606_18587_amd")


@pytest.mark.parametrize("B,H,T", [(1, 2, 129), (4, 32, 512), (4, 32, 513), (1, 103, 640), (2, 51, 641)])
def test_row_blocks_alone_and_in_pairs(B, H, T):
    wl = di.Workload("grid", 61, B, H, H, T, 64, 16, 70, "bf16")
    inp = di.make_prefill_inputs(wl)
    o = to_host64(dar.dar_attn_prefill(to_dev(inp["q"]), to_dev(inp["k"]), to_dev(inp["v"]),
                                       to_dev(inp["wd"]), None, wl.w))
    torch.cuda.synchronize()
    for b, h in {(0, 0), (B - 1, H - 1), (B // 2, H // 2)}:
        ref = oracle.rows(inp["k"].f64[b, h], inp["v"].f64[b, h], inp["wd"].f64[h], None, wl.w,
                          list(range(T)), inp["q"].f64[b, h])
        assert np.abs(o[b, h] - ref).max() <= tol("bf16"), (b, h)
