"""The fp32 matrix-core kernels (d up to 128) at the edges of their tiles: 16
rows, keys and latent columns, head sizes padded to 64 and 128; against the
fp64 oracle at the fp32 tolerance (1e-4 on unit-scale inputs, gradients
relative to their scale), and with infinities and NaN in rows that some
queries of the same tile do not see."""
import numpy as np
import pytest
import torch

import dar_inputs as di
from oracle import oracle
from tests.dev import to_dev, to_host64, tol

pytestmark = pytest.mark.gpu

dar = pytest.importorskip("paper_2606_18587_amd")


def both(inp, w):
    q, k, v, wd, wu, dout = (to_dev(inp[n]) for n in ("q", "k", "v", "wd", "wu", "dout"))
    o, lse = dar.dar_attn_prefill(q, k, v, wd, wu, w, return_lse=True)
    g = dar.dar_attn_prefill_backward(q, k, v, wd, wu, w, o, lse, dout)
    torch.cuda.synchronize()
    return to_host64(o), [None if x is None else to_host64(x) for x in g]


@pytest.mark.parametrize("d,dd,T,w", [(64, 16, 331, 64), (64, 17, 33, 16), (64, 64, 47, 5),
                                      (63, 33, 40, 7), (1, 1, 20, 3), (65, 1, 49, 16),
                                      (128, 32, 65, 17), (127, 31, 50, 0), (128, 33, 40, 9),
                                      (64, 32, 16, 16), (64, 16, 1, 1), (20, 5, 17, 100)])
def test_tile_edges(d, dd, T, w):
    wl = di.Workload("f32_edges", 62, 2, 4, 2, T, d, dd, w, "f32")
    for untied in (False, True):
        inp = di.make_backward_inputs(wl, untied=untied)
        o, g = both(inp, w)
        wu = None if inp["wu"] is None else inp["wu"].f64
        args = (inp["q"].f64, inp["k"].f64, inp["v"].f64, inp["wd"].f64, wu, w)
        assert np.abs(o - oracle.prefill(*args)).max() <= tol("f32")
        for n, a, b in zip(("dq", "dk", "dv", "dwd", "dwu"), g, oracle.backward(*args, inp["dout"].f64)):
            if b is None:
                assert a is None
                continue
            assert np.abs(a - b).max() <= tol("f32") * max(1.0, np.abs(b).max()), n


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("w", [0, 3, 40])
def test_unseen_tokens_do_not_leak(bad, w):
    """A token with a NaN or an infinity in its value, and one whose incoming
    gradient has it, leave every row and key that does not meet them as it is."""
    wl = di.Workload("f32_leak", 63, 1, 2, 1, 61, 64, 16, w, "f32")
    inp = di.make_backward_inputs(wl)
    q, k, v, wd, dout = (to_dev(inp[n]) for n in ("q", "k", "v", "wd", "dout"))
    o0, lse0 = dar.dar_attn_prefill(q, k, v, wd, None, w, return_lse=True)
    g0 = dar.dar_attn_prefill_backward(q, k, v, wd, None, w, o0, lse0, dout)
    v1, d1 = v.clone(), dout.clone()
    v1[0, 0, 37, 5] = bad
    d1[0, 1, 21, 9] = bad
    # (a tile that holds the bad value is added in another order: fp32 rounding
    # of sums of up to 61 unit-scale terms, 61 * 2^-24 < 1e-5)
    def same(a, b):
        torch.testing.assert_close(a, b, rtol=1e-5, atol=1e-5)

    o1 = dar.dar_attn_prefill(q, k, v1, wd, None, w)
    same(o1[:, :, :37], o0[:, :, :37])
    assert not torch.isfinite(o1[:, :, 37:]).all(dim=-1).any()
    g1 = dar.dar_attn_prefill_backward(q, k, v, wd, None, w, o0, lse0, d1)
    rows = [i for i in range(61) if i != 21]
    same(g1[0][:, 0], g0[0][:, 0])
    same(g1[0][:, 1, rows], g0[0][:, 1, rows])
    same(g1[1][:, :, 22:], g0[1][:, :, 22:])
    same(g1[2][:, :, 22:], g0[2][:, :, 22:])
