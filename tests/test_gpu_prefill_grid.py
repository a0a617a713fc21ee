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


@pytest.mark.parametrize("B,H,T", [(3, 33, 512), (1, 51, 1100), (2, 24, 1000), (1, 257, 100), (1, 32, 1100)])
def test_second_half_of_the_grid_in_turned_order(B, H, T):
    """256 to 512 blocks: the workgroups from the 257th on take the remaining
    blocks shortest first, with the heads dealt to the XCDs (a multiple of eight)
    and without, even and odd block counts, one block past the line. Rows that no
    workgroup takes, or that two do, show against the same call with the batch
    and heads cut to grids of at most 256 blocks, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(T)
    q, k, v = (torch.randn(B, H, T, 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    wd = (torch.randn(H, 64, 16, generator=g, device="cuda") / 8).to(torch.bfloat16)
    nblk = (T + 127) // 128
    assert 256 < nblk * B * H <= 512
    o = torch.full_like(q, float("nan"))
    dar.dar_attn_prefill(q, k, v, wd, None, 70, o=o)
    n = 16 if H % 16 == 0 else 17
    for b in range(B):
        for h in range(0, H, n):
            s = slice(h, min(h + n, H))
            part = dar.dar_attn_prefill(*(x[b:b + 1, s].contiguous() for x in (q, k, v)),
                                        wd[s].contiguous(), None, 70)
            assert torch.equal(o[b:b + 1, s].view(torch.int16), part.view(torch.int16)), (b, h)


@pytest.mark.parametrize("H,T", [(30, 1100), (56, 1024), (57, 1000), (64, 1000), (65, 1000)])
def test_shared_latents_one_workgroup_a_unit(H, T):
    """Shared latents at d = 128, d_down = 32 hold a compute unit's LDS alone:
    one block each up to 448 blocks, pairs past that (on both sides of the line
    and of 512)."""
    d, dd, w = 128, 32, 70
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn(1, H, T, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    c = torch.randn(1, H, T, dd, generator=g, device="cuda").to(torch.bfloat16)
    uk, uv = ((torch.randn(H, dd, d, generator=g, device="cuda") / 6).to(torch.bfloat16) for _ in range(2))
    o = torch.full_like(q, float("nan"))
    dar.dar_attn_prefill_shared(q, k, v, c, uk, uv, w, o=o)
    for h in range(0, H, 13):
        s = slice(h, min(h + 13, H))
        part = dar.dar_attn_prefill_shared(*(x[:, s].contiguous() for x in (q, k, v, c)),
                                           uk[s].contiguous(), uv[s].contiguous(), w)
        assert torch.equal(o[:, s].view(torch.int16), part.view(torch.int16)), h


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,dd,w", [(64, 16, 100), (128, 32, 300), (64, 32, 0)])
def test_large_chunks_against_their_sequences(d, dd, w, paged):
    """A chunk over more than 512 blocks (pairs) and more than 8192 blocks of 32
    positions (norms of eight blocks a wavefront) against its sequences one by
    one, which take one block a workgroup and one a wavefront: the same rows,
    log-sum-exps and cache, bit for bit."""
    B, H, L, n, page = 9, 8, 4001, 1000, 64
    assert ((n + 127) // 128) * B * H > 512 and ((L + n + 31) // 32) * B * H > 8192
    assert ((n + 127) // 128) * H <= 512 and ((L + n + 31) // 32) * H <= 8192
    g = torch.Generator(device="cuda").manual_seed(d + w)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    lat, win = [randn(B, H, L, dd) for _ in range(2)], [randn(B, H, max(w, 1), d) for _ in range(2)]
    q, k, v = (randn(B, H, n, d) for _ in range(3))
    wd = (torch.randn(H, d, dd, generator=g, device="cuda") * d ** -0.5).to(torch.bfloat16)
    nb = (L + n + page - 1) // page

    def run(s):
        m = q[s].shape[0]
        if paged:
            c = dar.DarPagedCache(m, H, d, dd, w, page, nb, m * nb, torch.bfloat16)
            c.block_table.copy_(torch.arange(m * nb, dtype=torch.int32).view(m, nb))
            c.lens.fill_(L)
            for pool, x in zip((c.k_pool, c.v_pool), lat):
                pad = torch.zeros(m, H, nb * page, dd, dtype=torch.bfloat16, device="cuda")
                pad[:, :, :L] = x[s]
                pool.copy_(pad.view(m, H, nb, page, dd).transpose(1, 2).reshape(m * nb, H, page, dd))
        else:
            c = dar.DarCache(m, H, d, dd, w, L + n, torch.bfloat16)
            c.struct.len = L
            c.k_lat[:, :, :L], c.v_lat[:, :, :L] = lat[0][s], lat[1][s]
        c.k_win.copy_(win[0][s]), c.v_win.copy_(win[1][s])
        f = dar.dar_attn_prefill_chunk_paged if paged else dar.dar_attn_prefill_chunk
        o, lse = f(c, q[s].contiguous(), k[s].contiguous(), v[s].contiguous(), wd, return_lse=True)
        pool = [t.view(m, nb, H, page, dd) for t in (c.k_pool, c.v_pool)] if paged else [c.k_lat, c.v_lat]
        return [o, lse, c.k_win, c.v_win] + pool

    whole = run(slice(None))
    assert torch.isfinite(whole[0]).all()
    for b in range(B):
        for a, p in zip(whole, run(slice(b, b + 1))):
            assert torch.equal(a[b:b + 1].view(torch.int16), p.view(torch.int16)), b


def test_rotary_rows_in_one_or_two_launches():
    """Queries and keys are rotated in one launch while their heads fit its
    grid (65535): past that, in two; the same rows come out either way."""
    H, T, d, dd = 33000, 2, 64, 16
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, H, T, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    wd = (torch.randn(H, d, dd, generator=g, device="cuda") / 8).to(torch.bfloat16)
    rope = dar.Rope(16, n_pos=T)
    o = dar.dar_attn_prefill_rope(q, k, v, wd, None, 1, rope)
    n = 200
    for h in (0, 16000, H - n):
        s = slice(h, h + n)
        part = dar.dar_attn_prefill_rope(*(x[:, s].contiguous() for x in (q, k, v)), wd[s].contiguous(),
                                         None, 1, rope)
        assert torch.equal(o[:, s].view(torch.int16), part.view(torch.int16)), h
