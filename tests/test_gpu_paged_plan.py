"""The paged decode's job plan: batches of at most 64 sequences make it in one
wavefront, larger ones with the general block-wide plan. A sequence without
tokens adds no work, so a batch of n sequences (n <= 64) filled up with empty
ones past 64 takes the general plan and cuts the same parts: every real row
must come out bit for bit the same, and every empty one as NaN."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

dar = pytest.importorskip("paper_2606_18587_amd")

PAGE, BLOCKS = 32, 48


def decode(lens, extra, Hq, Hkv, d, dd, w, r, seed):
    B = len(lens) + extra
    n_pages = 4 * BLOCKS
    g = torch.Generator(device="cuda").manual_seed(seed)
    c = dar.DarPagedCache(B, Hkv, d, dd, w, PAGE, BLOCKS, n_pages, torch.bfloat16)
    n = len(lens)

    def fill(t, rows):  # the same values whatever the batch size
        t[:rows] = torch.randn(rows, *t.shape[1:], generator=g, device="cuda").to(t.dtype)

    fill(c.k_pool, n_pages)
    fill(c.v_pool, n_pages)
    fill(c.k_win, n)
    fill(c.v_win, n)
    tab = np.random.default_rng(seed).integers(0, n_pages, (n, BLOCKS)).astype(np.int32)
    c.block_table[:n] = torch.from_numpy(tab).cuda()
    c.lens[:n] = torch.tensor(lens, dtype=torch.int32)
    q = torch.zeros(B, Hq, d, dtype=torch.bfloat16, device="cuda")
    fill(q, n)
    wd = (torch.randn(Hkv, d, dd, generator=g, device="cuda") * d ** -0.5).to(torch.bfloat16)
    if r:
        o = dar.dar_attn_decode_paged_rope(c, q, wd, dar.Rope(r, n_pos=c.cap))
    else:
        o = dar.dar_attn_decode_paged(c, q, wd)
    torch.cuda.synchronize()
    return o


@pytest.mark.parametrize("n,Hq,Hkv,d,dd,w,r", [(1, 4, 4, 64, 16, 100, 0), (2, 8, 1, 64, 32, 64, 0),
                                               (7, 8, 2, 128, 32, 33, 0), (33, 4, 2, 64, 16, 0, 0),
                                               (64, 8, 8, 64, 16, 200, 0), (64, 2, 1, 128, 16, 1, 64),
                                               (20, 8, 4, 64, 16, 48, 16)])
def test_plans_agree(n, Hq, Hkv, d, dd, w, r):
    rng = np.random.default_rng(n + 100 * d)
    cap = PAGE * BLOCKS
    lens = [int(x) for x in rng.integers(1, cap + 1, n)]
    if n > 2:  # the longest, the shortest, an empty and an overflowed sequence, and ties
        lens[0], lens[1], lens[2] = cap, 1, 0
        lens[-1] = -1 - cap
    if n > 10:
        lens[5] = lens[6] = lens[7]
    a = decode(lens, 0, Hq, Hkv, d, dd, w, r, n)
    b = decode(lens, 65 - n, Hq, Hkv, d, dd, w, r, n)
    live = [i for i, x in enumerate(lens) if x > 0]
    dead = [i for i, x in enumerate(lens) if x <= 0]
    assert torch.isfinite(a[live]).all()
    assert torch.equal(a[live].view(torch.int16), b[live].view(torch.int16))
    assert torch.isnan(a[dead]).all() and torch.isnan(b[dead]).all() and torch.isnan(b[n:]).all()
