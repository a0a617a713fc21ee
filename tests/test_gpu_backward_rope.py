"""GPU backward of the prefill with the rotary embedding of Eq. 3
(dar_attn_prefill_rope_backward through the C ABI) against the fp64 oracle's
rotary backward on the same seeded inputs.

The GPU backward is fed the GPU rotary forward's own o and lse. Tolerance as
for the plain backward: the forward's bf16 bound 2e-2 relative to each
gradient tensor's scale,
  max |got - ref| <= tol * max(1, max |ref|)   per tensor (dq, dk, dv, dW),
and an elementwise bound |got - ref| <= B * tol * max(1, |ref|) with B from
ELEM_BOUND (the gradients are sums with cancellation: an element's error
follows the terms that built it, and the weight gradients sum over every row
of the batch).
"""
import numpy as np
import pytest
import torch

import dar_inputs as di
from oracle import oracle
from tests.dev import to_dev, to_host64, tol

pytestmark = pytest.mark.gpu

dar = pytest.importorskip("paper_2606_18587_amd")

ELEM_BOUND = {"dq": 1.4, "dk": 1.4, "dv": 1.4, "dwd": 12.0, "dwu": 12.0}


def compare(got, ref, what):
    t = tol("bf16")
    worst = {}
    for n, a, b in zip(("dq", "dk", "dv", "dwd", "dwu"), got, ref):
        if b is None:
            assert a is None, n
            continue
        assert a.shape == b.shape, (n, a.shape, b.shape)
        assert np.isfinite(a).all(), what + " " + n + " not finite"
        err = np.abs(a - b)
        ratio = err.max() / (t * max(1.0, np.abs(b).max()))
        elem = (err / (t * np.maximum(1.0, np.abs(b)))).max()
        worst[n] = ratio
        worst[n + "_elem"] = elem
        assert ratio <= 1.0, "%s %s: error %.3g of the normwise bound (max abs err %.3g)" % (
            what, n, ratio, err.max())
        assert elem <= ELEM_BOUND[n], "%s %s: elementwise error %.3g of the bound" % (what, n, elem)
    return worst


def run_gpu(inp, w, r, base, pos0):
    q, k, v = to_dev(inp["q"]), to_dev(inp["k"]), to_dev(inp["v"])
    wd, wu = to_dev(inp["wd"]), to_dev(inp["wu"])
    dout = to_dev(inp["dout"])
    T = q.shape[2]
    rope = dar.Rope(r, base, n_pos=pos0 + T)
    o, lse = dar.dar_attn_prefill_rope(q, k, v, wd, wu, w, rope, pos0=pos0, return_lse=True)
    grads = dar.dar_attn_prefill_rope_backward(q, k, v, wd, wu, w, rope, o, lse, dout, pos0=pos0)
    torch.cuda.synchronize()
    return [None if g is None else to_host64(g) for g in grads]


def full_compare(wl, r, untied=False, base=10000.0, pos0=0, seed_shift=0):
    inp = di.make_backward_inputs(wl, untied=untied, seed_shift=seed_shift)
    got = run_gpu(inp, wl.w, r, base, pos0)
    ref = oracle.backward_rope(inp["q"].f64, inp["k"].f64, inp["v"].f64, inp["wd"].f64,
                               None if inp["wu"] is None else inp["wu"].f64, wl.w, r, base,
                               inp["dout"].f64, pos0=pos0)
    worst = compare(got, ref, "%s w=%d T=%d r=%d" % (wl.name, wl.w, wl.T, r))
    print(wl.name, wl.w, wl.T, r, " ".join("%s=%.3f" % kv for kv in worst.items()))
    return worst


BF16_SMALL = di.Workload("rope_bwd_small", 50, 1, 4, 2, 300, 64, 16, 128, "bf16")


@pytest.mark.parametrize("w", [0, 1, 64, 128, 299, 300, 1000])
@pytest.mark.parametrize("untied", [False, True])
def test_d64_window_sweep(w, untied):
    full_compare(BF16_SMALL.with_(w=w), 16 if w % 2 == 0 else 64, untied=untied)


@pytest.mark.parametrize("T", [1, 2, 61, 129, 257])
def test_d64_ragged_lengths(T):
    full_compare(BF16_SMALL.with_(T=T, w=32, B=2), 32)


@pytest.mark.parametrize("w,r,untied", [(0, 128, False), (100, 32, True), (512, 64, False)])
def test_d128_gqa(w, r, untied):
    full_compare(di.Workload("rope_bwd_d128", 51, 1, 8, 2, 400, 128, 32, w, "bf16"), r,
                 untied=untied, base=500000.0)


@pytest.mark.parametrize("d,dd,w,T,r", [(64, 32, 40, 333, 64), (128, 16, 77, 290, 16),
                                        (64, 8, 33, 97, 24), (128, 48, 50, 150, 2)])
def test_other_shapes_and_rotary_dims(d, dd, w, T, r):
    """d_down 8 and 48, rotary dims that are not multiples of 16."""
    full_compare(di.Workload("rope_bwd_mixed", 52, 2, 4, 1, T, d, dd, w, "bf16"), r, untied=True)


@pytest.mark.parametrize("d,dd,w,T,r", [(64, 12, 31, 129, 2), (64, 33, 32, 128, 64),
                                        (64, 64, 1, 191, 10), (128, 65, 33, 161, 128),
                                        (128, 73, 0, 127, 34), (128, 33, 130, 131, 48)])
def test_chain_rule_column_tiles(d, dd, w, T, r):
    """d_down at the edges of the 32-column tiles up to the largest accepted,
    rotary dims with and without whole runs of eight, lengths around the
    workgroup's 128 keys (untied and tied)."""
    wl = di.Workload("rope_bwd_tiles", 53, 1, 4, 2, T, d, dd, w, "bf16")
    full_compare(wl, r, untied=True)
    full_compare(wl, r, pos0=3)


@pytest.mark.parametrize("B,Hq,Hkv,T,d,dd,w,r",
                         [(2, 2, 2, 300, 128, 64, 150, 32), (2, 8, 1, 290, 128, 64, 40, 128),
                          (2, 4, 4, 400, 128, 73, 200, 16), (2, 8, 1, 270, 128, 65, 129, 34),
                          (1, 8, 1, 300, 64, 64, 140, 64), (2, 4, 4, 390, 64, 33, 5, 16)])
def test_wide_latents_over_several_key_blocks(B, Hq, Hkv, T, d, dd, w, r):
    """Two and three column tiles up to the largest accepted d_down, with
    distant rows for several blocks of 128 keys, windows longer than one, one
    or eight query heads a KV head (untied and tied). ELEM_BOUND holds for the
    weight gradients while their largest entry stays below about 60: their
    error, the rounding of the summands, is about 0.2 of the normwise bound
    whatever the entry, so a small entry's is 0.2 max |dW| of its own (one
    sequence where eight heads and a short head size would pass that)."""
    wl = di.Workload("rope_bwd_wide", 54, B, Hq, Hkv, T, d, dd, w, "bf16")
    full_compare(wl, r, untied=True)
    full_compare(wl, r, pos0=1)


def exact_chain_inputs(rng, B, Hq, Hkv, T, d, dd, w):
    """Inputs whose distant scores are zero and whose P, dS and sums before the
    chain rule are exact, so that only the chain rule can round:
      * d splits into L = 16..d/2-1 (queries) and U = d/2..d-1 (lifted keys), and
        the latent columns into A (the keys' and values') and the rest C; W_up
        sends A into U and C into L, W_down fills A alone, keys lie in U: the
        scores are 0 and, with lse = 0, P = 1;
      * values are one element each that W_down and W_up send to the one element z
        of U, and o = 0: dS = dO[z] 2^m, a bf16 number;
      * entries are whole numbers: u / s and dvd are whole numbers below 2^24.
    w = T - 10: ten distant keys. Returns torch-free fp64 arrays."""
    h = d // 2
    nA = dd // 2
    perm = rng.permutation(h)
    z, ups = h + perm[0], h + perm[1:]
    ys, xs = ups[:5], ups[5:15]  # rows of W_down that the values and the keys use
    wd = np.zeros((Hkv, d, dd))
    wu = np.zeros((Hkv, dd, d))
    for g in range(Hkv):
        wd[g, ys, 0] = 1.0
        for n, x in enumerate(xs):
            wd[g, x, 1 + n % (nA - 1)] = rng.integers(129, 256)
        wu[g, 0, z] = 1.0
        for c in range(1, nA):
            wu[g, c, ups[rng.integers(len(ups))]] = rng.integers(1, 9)
        for c in range(nA, dd):
            wu[g, c, rng.integers(16, h)] = rng.integers(129, 256)
    q = np.zeros((B, Hq, T, d))
    q[..., 16:h] = rng.integers(-255, 256, (B, Hq, T, h - 16))
    dout = rng.integers(-255, 256, (B, Hq, T, d)) * 2.0 ** rng.integers(0, 5, (B, Hq, T, d))
    dout[..., z] = rng.integers(-3, 4, (B, Hq, T)) * 2.0 ** rng.integers(0, 6, (B, Hq, T))
    k = np.zeros((B, Hkv, T, d))
    v = np.zeros((B, Hkv, T, d))
    for t in range(T):
        k[:, :, t, xs[t % 10]] = rng.integers(129, 256, (B, Hkv))
        v[:, :, t, ys[t % 5]] = 2.0 ** rng.integers(0, 3, (B, Hkv))
    return q, k, v, wd, wu, dout


@pytest.mark.parametrize("B,Hq,Hkv,T,d,dd,r", [(1, 2, 2, 10, 64, 16, 16), (2, 8, 2, 140, 64, 64, 0),
                                               (1, 4, 4, 60, 128, 32, 16), (1, 4, 1, 30, 128, 64, 2),
                                               (2, 2, 2, 11, 128, 73, 16)])
def test_chain_rule_keeps_fp32(B, Hq, Hkv, T, d, dd, r):
    """The fp32 weight gradients against fp64 with nothing rounded before the
    chain rule. What is left is fp32: the scale (2^-24), one sum over d or a
    window of exact terms, and one over at most ten keys of each of B sequences,
    each rounding at 2^-24 of what it has summed; 2^-20 of the summed magnitudes
    is sixteen such roundings. A factor cut to 16 significant bits misses it by
    far (2^-17 of a single term)."""
    rng = np.random.default_rng(d + dd + T)
    w = T - 10
    q, k, v, wd, wu, dout = exact_chain_inputs(rng, B, Hq, Hkv, T, d, dd, w)
    up = lambda x: torch.from_numpy(x).to(torch.bfloat16).cuda()
    for x in (q, k, v, wd, wu, dout):
        assert np.array_equal(torch.from_numpy(x).to(torch.bfloat16).double().numpy(), x)
    lse = torch.zeros(B, Hq, T, device="cuda")
    got = dar.dar_attn_prefill_rope_backward(up(q), up(k), up(v), up(wd), up(wu), w,
                                             dar.Rope(r, n_pos=T), torch.zeros_like(up(q)), lse, up(dout))
    torch.cuda.synchronize()
    G, Td, s = Hq // Hkv, T - w, d ** -0.5
    dwd, dwu = np.zeros_like(wd), np.zeros_like(wu)
    awd, awu = np.zeros_like(wd), np.zeros_like(wu)
    for b in range(B):
        for g in range(Hkv):
            vd = v[b, g, :Td] @ wd[g] @ wu[g]
            far = np.arange(T)[:, None] - np.arange(Td)[None, :] >= w
            u = np.zeros((Td, d))
            dvd = np.zeros((Td, d))
            for h in range(g * G, (g + 1) * G):
                ds = np.where(far, dout[b, h] @ vd.T, 0.0)
                assert np.array_equal(torch.from_numpy(ds).to(torch.bfloat16).double().numpy(), ds)
                u += ds.T @ q[b, h]
                dvd += far.T.astype(float) @ dout[b, h]
            assert max(np.abs(u).max(), np.abs(dvd).max()) < 2 ** 24
            u *= s
            kk, vv, gk, gv = k[b, g, :Td], v[b, g, :Td], u @ wu[g].T, dvd @ wu[g].T
            ck, cv = kk @ wd[g], vv @ wd[g]
            dwd[g] += kk.T @ gk + vv.T @ gv
            dwu[g] += ck.T @ u + cv.T @ dvd
            agk, agv = np.abs(u) @ np.abs(wu[g]).T, np.abs(dvd) @ np.abs(wu[g]).T
            awd[g] += np.abs(kk).T @ agk + np.abs(vv).T @ agv
            awu[g] += np.abs(ck).T @ np.abs(u) + np.abs(cv).T @ np.abs(dvd)
    for n, a, ref, mag in (("dwd", got[3], dwd, awd), ("dwu", got[4], dwu, awu)):
        err = np.abs(to_host64(a) - ref)
        assert (mag > 0).any()
        worst = (err[mag > 0] / mag[mag > 0]).max()
        print(n, d, dd, "largest error 2^%.1f of the summed magnitudes" % np.log2(max(worst, 2.0 ** -60)))
        assert worst <= 2.0 ** -20, (n, worst)
        assert not err[mag == 0].any(), n


def test_offset_positions_and_zero_rotary_dim():
    """Rows at positions 77.. of a longer sequence, and r = 0, whose gradients
    are those of the plain backward (checked against the oracle's)."""
    wl = BF16_SMALL.with_(w=48, T=200)
    full_compare(wl, 64, pos0=77, base=500000.0)
    inp = di.make_backward_inputs(wl, untied=True, seed_shift=3)
    got = run_gpu(inp, wl.w, 0, 10000.0, 0)
    ref = oracle.backward(inp["q"].f64, inp["k"].f64, inp["v"].f64, inp["wd"].f64,
                          inp["wu"].f64, wl.w, inp["dout"].f64)
    compare(got, ref, "r=0 against the plain backward")


def test_many_short_sequences():
    """A batch of more than 65535 blocks of 32 keys, in the workspace that is
    asked for and nothing past it, against the same sequences in two halves: dq,
    dk and dv bit for bit, dW_down as their fp32 sum."""
    B, T, d, dd, w, r = 2100, 1000, 64, 16, 900, 16
    assert B * ((T + 31) // 32) > 65535
    g = torch.Generator(device="cuda").manual_seed(8)
    q, k, v, dout = (torch.randn(B, 1, T, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    wd = (torch.randn(1, d, dd, generator=g, device="cuda") / 8).to(torch.bfloat16)
    rope = dar.Rope(r, n_pos=T)

    def grads(s, ws=None):
        x = [t[s] for t in (q, k, v, dout)]
        o, lse = dar.dar_attn_prefill_rope(*x[:3], wd, None, w, rope, return_lse=True)
        return dar.dar_attn_prefill_rope_backward(*x[:3], wd, None, w, rope, o, lse, x[3], ws=ws)

    need = dar.dar_prefill_rope_backward_workspace_bytes(dar.make_shape(B, 1, 1, d, dd, w, torch.bfloat16), T)
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    whole = grads(slice(None), ws[:need])
    assert bool((ws[need:] == 0x5A).all())
    halves = [grads(slice(0, B // 2)), grads(slice(B // 2, B))]
    for n in range(3):
        for s, h in zip((slice(0, B // 2), slice(B // 2, B)), halves):
            assert torch.equal(whole[n][s].view(torch.int16), h[n].view(torch.int16))
    torch.testing.assert_close(whole[3], halves[0][3] + halves[1][3], rtol=1e-4, atol=1e-4 * float(whole[3].abs().max()))


def test_deterministic():
    wl = BF16_SMALL.with_(w=64, T=333, B=2)
    inp = di.make_backward_inputs(wl, untied=True)
    a = run_gpu(inp, wl.w, 32, 10000.0, 5)
    b = run_gpu(inp, wl.w, 32, 10000.0, 5)
    for x, y in zip(a, b):
        assert (x is None and y is None) or np.array_equal(x, y)


def test_full_size_pythia70m_one_head():
    """B8 H8 T2048 d64 d_down16 w256 with rotary dimension 16 (the Pythia
    models' rotary width) on the GPU; the oracle recomputes the gradients of
    one KV head over the whole batch (dq/dk/dv of its rows and the head's full
    dW_down)."""
    wl = di.WORKLOADS["pythia70m"]
    inp = di.make_backward_inputs(wl)
    got = run_gpu(inp, wl.w, 16, 10000.0, 0)
    g = 2
    G = wl.Hq // wl.Hkv
    hs = slice(g * G, (g + 1) * G)
    ref = oracle.backward_rope(inp["q"].f64[:, hs], inp["k"].f64[:, g:g + 1], inp["v"].f64[:, g:g + 1],
                               inp["wd"].f64[g:g + 1], None, wl.w, 16, 10000.0, inp["dout"].f64[:, hs])
    sub = [got[0][:, hs], got[1][:, g:g + 1], got[2][:, g:g + 1], got[3][g:g + 1], None]
    worst = compare(sub, ref, "pythia70m rope head %d" % g)
    print("pythia70m rope head", g, " ".join("%s=%.3f" % kv for kv in worst.items()))
