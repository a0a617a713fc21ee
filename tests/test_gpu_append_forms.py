"""The matrix-core appends request a token's four rows ahead while they have few
wavefronts (up to 1024, fewer than 32768 tokens) and one at a time past that. A
batch over the line and the same batch cut into sequences under it must leave the
same bytes in the cache: one token and many, with the ring rewritten in one
launch (n <= w) and in two, without a window, dense, paged and in paged chunks."""
import pytest
import torch

pytestmark = pytest.mark.gpu

dar = pytest.importorskip("paper_2606_18587_amd")


def bits(t):
    return t.view(torch.int16)


def randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda").to(torch.bfloat16)


@pytest.mark.parametrize("d,dd", [(64, 16), (128, 32)])
@pytest.mark.parametrize("B,Hkv,n,w,pre", [(64, 16, 1, 40, 60), (65, 16, 1, 40, 60), (8, 16, 256, 256, 300),
                                           (8, 16, 255, 256, 10), (9, 16, 300, 100, 130), (9, 16, 300, 0, 5)])
def test_dense(d, dd, B, Hkv, n, w, pre):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    k0, v0, k1, v1 = (randn(g, B, Hkv, t, d) for t in (pre, pre, n, n))
    wd = randn(g, Hkv, d, dd)

    def run(sl):
        c = dar.DarCache(k0[sl].shape[0], Hkv, d, dd, w, pre + n, torch.bfloat16)
        for t in (c.k_lat, c.v_lat, c.k_win, c.v_win):
            if t is not None:
                t.zero_()
        dar.dar_cache_append(c, k0[sl].contiguous(), v0[sl].contiguous(), wd)
        dar.dar_cache_append(c, k1[sl].contiguous(), v1[sl].contiguous(), wd)
        return [t for t in (c.k_lat, c.v_lat, c.k_win, c.v_win) if t is not None]

    whole = run(slice(None))
    for b in (0, B // 2, B - 1):
        for a, p in zip(whole, run(slice(b, b + 1))):
            assert torch.equal(bits(a[b:b + 1]), bits(p)), b


@pytest.mark.parametrize("d,dd", [(64, 16), (128, 32)])
@pytest.mark.parametrize("B,Hkv,n,w", [(128, 8, 1, 33), (129, 8, 1, 33), (8, 16, 256, 256), (9, 16, 300, 64),
                                       (9, 16, 290, 0)])
def test_paged(d, dd, B, Hkv, n, w):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    page = 32
    blocks = (80 + n + page - 1) // page
    lens = torch.randint(0, 70, (B,), generator=g, device="cuda", dtype=torch.int32)
    new = torch.randint(0, n + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    win = [randn(g, B, Hkv, w, d) for _ in range(2)]
    k1, v1 = randn(g, B, Hkv, n, d), randn(g, B, Hkv, n, d)
    wd, q = randn(g, Hkv, d, dd), randn(g, B, Hkv, n, d)

    def run(idx):
        m = len(idx)
        c = dar.DarPagedCache(m, Hkv, d, dd, w, page, blocks, m * blocks, torch.bfloat16)
        c.k_pool.zero_(), c.v_pool.zero_()
        c.block_table.copy_(torch.arange(m * blocks, dtype=torch.int32).view(m, blocks))
        c.lens.copy_(lens[idx])
        if w > 0:
            c.k_win.copy_(win[0][idx]), c.v_win.copy_(win[1][idx])
        if n == 1:
            dar.dar_cache_append_paged(c, k1[idx, :, 0].contiguous(), v1[idx, :, 0].contiguous(), wd)
        else:
            dar.dar_attn_prefill_chunk_paged(c, q[idx].contiguous(), k1[idx].contiguous(),
                                             v1[idx].contiguous(), wd, n_new=new[idx].contiguous())
        pools = [t.view(m, blocks, *t.shape[1:]) for t in (c.k_pool, c.v_pool)]
        return pools + ([c.k_win, c.v_win] if w > 0 else []) + [c.lens]

    whole = run(list(range(B)))
    for b in (0, B // 2, B - 1):
        for a, p in zip(whole, run([b])):
            assert torch.equal(a[b:b + 1].view(torch.int16), p.view(torch.int16)), b
