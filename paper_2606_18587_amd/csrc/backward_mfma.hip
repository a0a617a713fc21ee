// Matrix-core (MFMA) backward of the causal DAR prefill, bf16 storage, fp32
// accumulation, gfx950. The gradient formulas are those of the vector-ALU
// backward (backward.hip): one softmax over both regions (its log-sum-exp is
// the forward's), window pairs at full d, distant pairs in d_down space with
// W_up absorbed.
//
// Kernels, in launch order:
//  * bwd_prep_rows_kernel / bwd_prep_keys_kernel: q~ = q W_up^T (scaled by
//    log2(e)/sqrt(d)), dO~ = dO W_up^T, delta = dO . O and the log-sum-exp in
//    log2 units per query row; the latents c^K, c^V (Eq. 1) per key; all
//    operands bf16, each also stored in 32-token blocks transposed
//    ([T/32][d_down][32]) for the products that contract over tokens. Token
//    counts are padded to a multiple of 32 with zero rows.
//  * bwd_rows_dist_kernel: one wavefront per 32 query rows, distant keys only
//    (d_down wide), scores transposed (S^T = c^K q~^T, one query per lane
//    column, as in the forward): h^T += c^K^T dS^T and ol^T += c^V^T P^T.
//  * bwd_cols_dist_kernel: one wavefront per 32 keys, distant rows only, scores
//    in the other orientation (S = q~ c^K^T, one key per lane column) so that
//    P and dS are directly the B operands of gK^T += q~^T dS, gV^T += dO~^T P.
//  * bwd_rows_local_kernel: window keys at full d through LDS tiles,
//    dq^T += K^T dS^T (K^T read transposed from LDS); the epilogue adds the
//    lifted distant part (h W_up, h as a bf16 hi + lo pair) and the
//    workgroup's share of dW_up.
//  * bwd_cols_local_kernel: window rows, dV^T += dO^T P and dK^T += Q^T dS;
//    the epilogue adds gK W_down^T, gV W_down^T and the workgroup's share of
//    dW_down.
//  * bwd_wreduce_kernel (backward.hip): the shares summed in a fixed order.
// No kernel accumulates with atomics, so the result does not depend on
// timing. Masked pairs get a score of -inf (P = 0, dS = 0). Each row's
// exponentials use its log-sum-exp as the reference, fed as the accumulator
// input of the score product (distant) or through one FMA (window), and
// -delta is the accumulator input of dP, so dS = P * dP' needs one multiply.
#include "../../include/dar.h"
#include "dar_common.hpp"
#include "dar_kernels.hpp"
#include "mfma_common.hpp"

namespace dar {

namespace {

constexpr float kLog2eB = 1.4426950408889634f;

// 16 floats of a per-token array for the tokens acc_row(r, g) of a 32-token
// block: two runs of 8.
__device__ __forceinline__ f32x16_t load_row16(const float* p, int g, float sign) {
    const float4 a = *reinterpret_cast<const float4*>(p + 8 * g);
    const float4 b = *reinterpret_cast<const float4*>(p + 8 * g + 4);
    const float4 c = *reinterpret_cast<const float4*>(p + 16 + 8 * g);
    const float4 d = *reinterpret_cast<const float4*>(p + 16 + 8 * g + 4);
    f32x16_t r;
    r[0] = sign * a.x; r[1] = sign * a.y; r[2] = sign * a.z; r[3] = sign * a.w;
    r[4] = sign * b.x; r[5] = sign * b.y; r[6] = sign * b.z; r[7] = sign * b.w;
    r[8] = sign * c.x; r[9] = sign * c.y; r[10] = sign * c.z; r[11] = sign * c.w;
    r[12] = sign * d.x; r[13] = sign * d.y; r[14] = sign * d.z; r[15] = sign * d.w;
    return r;
}

// Store 4 consecutive fp32 accumulator registers as 4 bf16 (8 bytes).
__device__ __forceinline__ void store_bf16x4(bf16_t* p, float a, float b, float c, float d) {
    *reinterpret_cast<uint2*>(p) = make_uint2(pack2(a, b), pack2(c, d));
}

// A operand rows of a transposed latent block [32][32] (latent rows past
// d_down are zero): row R carries latent column perm_row(R), so the
// accumulator rows come out in B-operand order; tokens 16 half + 8 g + 0..7.
__device__ __forceinline__ bf16x8_t latT_operand(const bf16_t* blk, int qc, int hg, int half) {
    return load_bf16x8(blk + (size_t)perm_row(qc) * 32 + 16 * half + 8 * hg);
}

// Eight bf16 [hi, mid, lo, 0, 0, 0, 0, 0] of -x: hi + mid + lo carries about
// 24 significant bits of -x once summed in fp32.
__device__ __forceinline__ uint4 neg_split3(float x) {
    const float v = -x;
    const uint32_t h = pack2(v, 0.f) & 0xffffu;
    const float r1 = v - __uint_as_float(h << 16);
    const uint32_t m = pack2(r1, 0.f) & 0xffffu;
    const float r2 = r1 - __uint_as_float(m << 16);
    const uint32_t lo = pack2(r2, 0.f) & 0xffffu;
    return make_uint4(h | (m << 16), lo, 0u, 0u);
}

// B operand that sums the first three k slots of half `g1` (ones there, zeros
// elsewhere): with the row-constant A operand it adds -lse (g1 = 0) or
// -delta (g1 = 1) to every accumulator of the row.
__device__ __forceinline__ bf16x8_t ones3(int hg, int g1) {
    return hg == g1 ? __builtin_bit_cast(bf16x8_t, make_uint4(0x3f803f80u, 0x3f80u, 0u, 0u))
                    : zero_bf16x8();
}

// 8 fp32 values (16-byte aligned).
struct f32x8 {
    float4 a, b;
};
__device__ __forceinline__ f32x8 load_f8(const float* p) {
    return f32x8{*reinterpret_cast<const float4*>(p), *reinterpret_cast<const float4*>(p + 4)};
}
__device__ __forceinline__ void add_f8(f32x8& r, const f32x8& x) {
    r.a.x += x.a.x; r.a.y += x.a.y; r.a.z += x.a.z; r.a.w += x.a.w;
    r.b.x += x.b.x; r.b.y += x.b.y; r.b.z += x.b.z; r.b.w += x.b.w;
}

// 8 fp32 values times f, as a bf16 hi + lo pair.
__device__ __forceinline__ void split_f8(const f32x8& y, float f, bf16x8_t& hi, bf16x8_t& lo) {
    f32x16_t x;
    x[0] = y.a.x; x[1] = y.a.y; x[2] = y.a.z; x[3] = y.a.w;
    x[4] = y.b.x; x[5] = y.b.y; x[6] = y.b.z; x[7] = y.b.w;
    split8(x, 0, f, hi, lo);
}

// 8 fp32 values times f, as one bf16 operand.
__device__ __forceinline__ bf16x8_t pack_f8(const f32x8& y, float f) {
    return __builtin_bit_cast(bf16x8_t,
                              make_uint4(pack2(y.a.x * f, y.a.y * f), pack2(y.a.z * f, y.a.w * f),
                                         pack2(y.b.x * f, y.b.y * f), pack2(y.b.z * f, y.b.w * f)));
}

// Workgroup share of a weight gradient: every wavefront adds its C tiles
// (rows e = 32 t + accumulator row, column c = lane % 32 < DD) into pbuf in
// wavefront order, then the workgroup writes pbuf [D][DD] to `out`. Every
// wavefront of the workgroup must call this (it holds barriers).
template <int D, int DD, int NW>
__device__ __forceinline__ void wg_share(const f32x16_t (&acc)[D / 32], float* pbuf, int wave,
                                         int lane, int tid, float* __restrict__ out) {
    const int qc = lane & 31, hg = lane >> 5;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
        if (wave == wv && qc < DD) {
#pragma unroll
            for (int t = 0; t < D / 32; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int e = 32 * t + 8 * (r >> 2) + 4 * hg + (r & 3);
                    float* cell = pbuf + e * DD + qc;
                    *cell = (wv == 0) ? acc[t][r] : *cell + acc[t][r];
                }
        }
        __syncthreads();
    }
    for (int idx = tid; idx < D * DD; idx += NW * 64) out[idx] = pbuf[idx];
}

// wg_share for one 32-column tile (columns c0 + 0..31, those below dd stored)
// of a share of run-time width dd: pbuf holds [D][32]. The caller puts a
// barrier after it before pbuf is used again.
template <int D, int NW>
__device__ __forceinline__ void wg_share_cols(const f32x16_t (&acc)[D / 32], float* pbuf, int wave,
                                              int lane, int tid, int dd, int c0,
                                              float* __restrict__ out) {
    const int qc = lane & 31, hg = lane >> 5;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int t = 0; t < D / 32; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int e = 32 * t + 8 * (r >> 2) + 4 * hg + (r & 3);
                    float* cell = pbuf + e * 32 + qc;
                    *cell = (wv == 0) ? acc[t][r] : *cell + acc[t][r];
                }
        }
        __syncthreads();
    }
    for (int idx = tid; idx < D * 32; idx += NW * 64) {
        const int c = c0 + (idx & 31);
        if (c < dd) out[(size_t)(idx >> 5) * dd + c] = pbuf[idx];
    }
}

// Cooperative staging of a 64-row tile of two row-major [rows][D] bf16 arrays
// through registers into LDS (rows at or past `n` read as zero): fetch() for
// the next tile is issued before the current one is computed on, so its
// global latency hides behind that work.
template <int D, int NW>
struct TilePair {
    static constexpr int C8 = D / 8, PER = 64 * C8 / (NW * 64);  // 16-byte chunks per thread
    uint4 a[PER], b[PER];
    __device__ __forceinline__ void fetch(const bf16_t* ga, const bf16_t* gb, int t, int n,
                                          int tid) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = tid + u * NW * 64;
            const int row = t + idx / C8, c8 = idx % C8;
            const size_t off = (size_t)imin(row, n - 1) * D + c8 * 8;  // clamped: no branch
            a[u] = *reinterpret_cast<const uint4*>(ga + off);
            b[u] = *reinterpret_cast<const uint4*>(gb + off);
            if (row >= n) {
                a[u] = make_uint4(0, 0, 0, 0);
                b[u] = make_uint4(0, 0, 0, 0);
            }
        }
    }
    __device__ __forceinline__ void store(bf16_t* la, bf16_t* lb, int ld, int tid) const {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = tid + u * NW * 64;
            const int r = idx / C8, c8 = idx % C8;
            *reinterpret_cast<uint4*>(la + r * ld + c8 * 8) = a[u];
            *reinterpret_cast<uint4*>(lb + r * ld + c8 * 8) = b[u];
        }
    }
};

}  // namespace

// ---------------------------------------------------------------- preparation

// Per query row i (padded rows get zeros): q~s = (q W_up^T) log2(e)/sqrt(d)
// and dO~ = dO W_up^T in bf16, row-major and in transposed 32-row blocks, and
// -delta = -dO . O and -lse (the forward's, in log2 units), in fp32 and as
// bf16 hi + mid + lo row constants. One wavefront per 32 rows on the matrix
// cores: U W^T with U = W_up gives one latent row per lane column (the
// row-major store), Q U^T one token per lane column (the transposed store);
// latent rows past d_down come out zero from U's zero rows.
// Grid: (Tr / (32 NW), B * Hq).
template <int D, int DD, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_prep_rows_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
    const float* __restrict__ lse, const bf16_t* __restrict__ wd, const bf16_t* __restrict__ wu,
    bf16_t* __restrict__ qts, bf16_t* __restrict__ qtT, bf16_t* __restrict__ dts,
    bf16_t* __restrict__ dtT, bf16_t* __restrict__ rc, float* __restrict__ nd,
    float* __restrict__ nl2, int Hq, int Hkv, int T, int Tr, float qscale) {
    constexpr int KS = D / 16, DS = DD / 16, LDU = D + 8;
    __shared__ __attribute__((aligned(16))) bf16_t U[32 * LDU];  // U[c][e] = W_up[c][e]
    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bh = wg_id_y();
    const int g = (bh % Hq) / (Hq / Hkv);
    const bf16_t* wdg = wd + (size_t)g * D * DD;
    const bf16_t* wug = wu ? wu + (size_t)g * DD * D : nullptr;
    // (all of this thread's elements requested at once, indices clamped, no
    // load under a branch: one memory round trip before the barrier)
    constexpr int UPT = 32 * D / (NW * 64);
    bf16_t uv[UPT];
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int idx = tid + j * NW * 64, c = imin(idx / D, DD - 1), e = idx % D;
        uv[j] = *(wug ? wug + (size_t)c * D + e : wdg + (size_t)e * DD + c);
    }
    // the rows and the row's lse are requested now too, so that the whole
    // kernel waits for one memory round trip (rows clamped into the array and
    // zeroed past T afterwards: no load under a branch)
    const int r0 = wg_id_x() * NW * 32 + wave * 32;
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc);
    const int rb = r0 + qc, ra = r0 + prow;  // B-layout row, A-layout row
    const int rbc = imin(rb, T - 1), rac = imin(ra, T - 1);
    const bf16_t* qh = q + (size_t)bh * T * D;
    const bf16_t* dh = dout + (size_t)bh * T * D;
    const bf16_t* oh = o + (size_t)bh * T * D;
    bf16x8_t qB[KS], dB[KS], oB[KS], qA[KS], dA[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int e = s * 16 + hg * 8;
        qB[s] = load_bf16x8(qh + (size_t)rbc * D + e);
        dB[s] = load_bf16x8(dh + (size_t)rbc * D + e);
        oB[s] = load_bf16x8(oh + (size_t)rbc * D + e);
        qA[s] = load_bf16x8(qh + (size_t)rac * D + e);
        dA[s] = load_bf16x8(dh + (size_t)rac * D + e);
    }
    const float lse_r = lse[(size_t)bh * T + rbc];
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int idx = tid + j * NW * 64, c = idx / D, e = idx % D;
        U[c * LDU + e] = c < DD ? uv[j] : (bf16_t)0;
    }
    // the rows are consumed here, so they are loaded ahead of the barrier
    // rather than at their first use behind the early return
#pragma unroll
    for (int s = 0; s < KS; ++s)
        __asm__ volatile("" ::"v"(qB[s]), "v"(dB[s]), "v"(oB[s]), "v"(qA[s]), "v"(dA[s]));
    __asm__ volatile("" ::"v"(lse_r));
    __syncthreads();
    if (r0 >= Tr) return;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        if (rb >= T) { qB[s] = zero_bf16x8(); dB[s] = zero_bf16x8(); oB[s] = zero_bf16x8(); }
        if (ra >= T) { qA[s] = zero_bf16x8(); dA[s] = zero_bf16x8(); }
    }
    // latent rows of row rb: U Q^T, A rows = latent columns in perm_row order
    f32x16_t qt = splat16(0.f), dt = splat16(0.f), qn = splat16(0.f), dn = splat16(0.f);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const bf16x8_t ua = load_bf16x8(U + prow * LDU + s * 16 + hg * 8);
        const bf16x8_t ub = load_bf16x8(U + qc * LDU + s * 16 + hg * 8);
        qt = mfma(ua, qB[s], qt);
        dt = mfma(ua, dB[s], dt);
        qn = mfma(qA[s], ub, qn);
        dn = mfma(dA[s], ub, dn);
    }
    const size_t prw = (size_t)bh * Tr + rb;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        *reinterpret_cast<bf16x8_t*>(qts + prw * DD + s * 16 + hg * 8) = pack8(qt, 8 * s, qscale);
        *reinterpret_cast<bf16x8_t*>(dts + prw * DD + s * 16 + hg * 8) = pack8(dt, 8 * s);
    }
    // transposed block: lane column = latent c, registers = tokens 8 hg + r, 16 + 8 hg + r
    const size_t blk = (((size_t)bh * (Tr / 32) + r0 / 32) * 32 + qc) * 32;
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
        *reinterpret_cast<bf16x8_t*>(qtT + blk + 16 * h2 + 8 * hg) = pack8(qn, 8 * h2, qscale);
        *reinterpret_cast<bf16x8_t*>(dtT + blk + 16 * h2 + 8 * hg) = pack8(dn, 8 * h2);
    }
    float dl = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) dl = dot8(dB[s], oB[s], dl);
    dl = pair_sum(dl);
    if (hg == 0) {
        const float L2 = rb < T ? lse_r * kLog2eB : 0.f;
        nd[prw] = -dl;
        nl2[prw] = -L2;
        *reinterpret_cast<uint4*>(rc + prw * 16) = neg_split3(L2);
        *reinterpret_cast<uint4*>(rc + prw * 16 + 8) = neg_split3(dl);
    }
}

// Per key token j (padded rows get zeros): c^K = k W_down, c^V = v W_down
// (Eq. 1) in bf16, row-major and in transposed 32-token blocks, computed as
// in bwd_prep_rows_kernel with U = W_down^T. Grid: (Tr / (32 NW), B * Hkv).
template <int D, int DD, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_prep_keys_kernel(
    const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, const bf16_t* __restrict__ wd,
    bf16_t* __restrict__ ckb, bf16_t* __restrict__ ckT, bf16_t* __restrict__ cvb,
    bf16_t* __restrict__ cvT, int Hkv, int T, int Tr) {
    constexpr int KS = D / 16, DS = DD / 16, LDU = D + 8;
    __shared__ __attribute__((aligned(16))) bf16_t U[32 * LDU];  // U[c][e] = W_down[e][c]
    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bg = wg_id_y();
    const bf16_t* wdg = wd + (size_t)(bg % Hkv) * D * DD;
    // (all of this thread's elements requested at once, indices clamped, no
    // load under a branch: one memory round trip before the barrier)
    constexpr int UPT = 32 * D / (NW * 64);
    bf16_t uv[UPT];
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int idx = tid + j * NW * 64, c = imin(idx / D, DD - 1), e = idx % D;
        uv[j] = wdg[(size_t)e * DD + c];
    }
    // rows requested before the barrier, clamped and zeroed past T afterwards,
    // as in bwd_prep_rows_kernel
    const int r0 = wg_id_x() * NW * 32 + wave * 32;
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc);
    const int rb = r0 + qc, ra = r0 + prow;
    const int rbc = imin(rb, T - 1), rac = imin(ra, T - 1);
    const bf16_t* kh = k + (size_t)bg * T * D;
    const bf16_t* vh = v + (size_t)bg * T * D;
    bf16x8_t kB[KS], vB[KS], kA[KS], vA[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int e = s * 16 + hg * 8;
        kB[s] = load_bf16x8(kh + (size_t)rbc * D + e);
        vB[s] = load_bf16x8(vh + (size_t)rbc * D + e);
        kA[s] = load_bf16x8(kh + (size_t)rac * D + e);
        vA[s] = load_bf16x8(vh + (size_t)rac * D + e);
    }
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int idx = tid + j * NW * 64, c = idx / D, e = idx % D;
        U[c * LDU + e] = c < DD ? uv[j] : (bf16_t)0;
    }
#pragma unroll
    for (int s = 0; s < KS; ++s)
        __asm__ volatile("" ::"v"(kB[s]), "v"(vB[s]), "v"(kA[s]), "v"(vA[s]));
    __syncthreads();
    if (r0 >= Tr) return;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        if (rb >= T) { kB[s] = zero_bf16x8(); vB[s] = zero_bf16x8(); }
        if (ra >= T) { kA[s] = zero_bf16x8(); vA[s] = zero_bf16x8(); }
    }
    f32x16_t kt = splat16(0.f), vt = splat16(0.f), kn = splat16(0.f), vn = splat16(0.f);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const bf16x8_t ua = load_bf16x8(U + prow * LDU + s * 16 + hg * 8);
        const bf16x8_t ub = load_bf16x8(U + qc * LDU + s * 16 + hg * 8);
        kt = mfma(ua, kB[s], kt);
        vt = mfma(ua, vB[s], vt);
        kn = mfma(kA[s], ub, kn);
        vn = mfma(vA[s], ub, vn);
    }
    const size_t prw = (size_t)bg * Tr + rb;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        *reinterpret_cast<bf16x8_t*>(ckb + prw * DD + s * 16 + hg * 8) = pack8(kt, 8 * s);
        *reinterpret_cast<bf16x8_t*>(cvb + prw * DD + s * 16 + hg * 8) = pack8(vt, 8 * s);
    }
    const size_t blk = (((size_t)bg * (Tr / 32) + r0 / 32) * 32 + qc) * 32;
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
        *reinterpret_cast<bf16x8_t*>(ckT + blk + 16 * h2 + 8 * hg) = pack8(kn, 8 * h2);
        *reinterpret_cast<bf16x8_t*>(cvT + blk + 16 * h2 + 8 * hg) = pack8(vn, 8 * h2);
    }
}

// ---------------------------------------------------------------- distant tiles

// Cooperative copy of a 64-token operand tile through registers into LDS.
// The tile is up to five contiguous global segments of n_k 16-byte chunks
// (each a multiple of 64), laid out in LDS in the same order. Load u of
// wavefront `wave` moves the 64 chunks of group wave + NW u, so every load's
// segment is the same for the whole wavefront (no divergent address choice).
// seg_fetch() for the next tile is issued before the current one is computed
// on; the registers travel by value (a struct updated through a reference
// would be kept in scratch memory).
template <int NW, int NCH>
struct SegRegs {
    static_assert(NCH % 64 == 0, "tile segments are whole 64-chunk groups");
    static constexpr int NGRP = NCH / 64;
    static constexpr int PER = (NGRP + NW - 1) / NW;
    uint4 r[PER];
};

struct Segs {
    const uint4 *s0, *s1, *s2, *s3, *s4;
    int n0, n1, n2, n3;
};

template <int NW, int NCH>
__device__ __forceinline__ SegRegs<NW, NCH> seg_fetch(const Segs& g, int wave, int lane) {
    using R = SegRegs<NW, NCH>;
    R o;
#pragma unroll
    for (int u = 0; u < R::PER; ++u) {
        int grp = wave + NW * u;  // wave-uniform
        if (R::NGRP % NW != 0 && grp >= R::NGRP) grp = R::NGRP - 1;  // spare loads repeat a group
        const int c = grp * 64, b1 = g.n0, b2 = b1 + g.n1, b3 = b2 + g.n2, b4 = b3 + g.n3;
        const uint4* src = c < b1 ? g.s0 + c
                         : c < b2 ? g.s1 + (c - b1)
                         : c < b3 ? g.s2 + (c - b2)
                         : c < b4 ? g.s3 + (c - b3)
                                  : g.s4 + (c - b4);
        o.r[u] = src[lane];
    }
    return o;
}

// (lds points at the tile's first chunk, or at a later segment's)
template <int NW, int NCH>
__device__ __forceinline__ void seg_store(const SegRegs<NW, NCH> st, uint4* lds, int wave,
                                          int lane) {
    using R = SegRegs<NW, NCH>;
#pragma unroll
    for (int u = 0; u < R::PER; ++u) {
        const int grp = wave + NW * u;
        if (R::NGRP % NW == 0 || grp < R::NGRP) lds[grp * 64 + lane] = st.r[u];
    }
}

// ---------------------------------------------------------------- distant: h, ol

// One workgroup of NW wavefronts = 32 NW query rows of one (batch, query
// head); distant keys j <= i - w only. The d_down-wide key operands of each
// 64-key tile (c^K and c^V rows, their transposed blocks) are copied once into
// LDS for the workgroup, the next tile's loads in flight meanwhile. Tiles
// whose keys are distant for every row of the workgroup are computed without
// masks, both 32-key subtiles in one straight-line block so that the products
// of one overlap the exponentials of the other. Writes h = sum dS c^K and
// ol = sum P c^V (fp32) of every real row (zero without distant keys).
// Grid: ceil(T / (32 NW)) * B * Hq workgroups (xcd_block_head); row blocks
// with the most keys first.
template <int DD, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_rows_dist_kernel(
    const bf16_t* __restrict__ ckb, const bf16_t* __restrict__ ckT,
    const bf16_t* __restrict__ cvb, const bf16_t* __restrict__ cvT,
    const bf16_t* __restrict__ qts, const bf16_t* __restrict__ dts,
    const float* __restrict__ nl2, const float* __restrict__ nd, float* __restrict__ hk,
    float* __restrict__ ol, int Hq, int Hkv, int T, int Tr, int w, int BH) {
    constexpr int DS = DD / 16, BM = NW * 32;
    constexpr int NK = 8 * DD, NT = 256;       // 16-byte chunks: 64 latent rows, 2 blocks
    constexpr int NCH = 2 * NK + 2 * NT;
    __shared__ __attribute__((aligned(16))) uint4 tile[NCH];
    const bf16_t* lck = reinterpret_cast<const bf16_t*>(tile);
    const bf16_t* lcv = lck + 64 * DD;
    const bf16_t* lkt = lcv + 64 * DD;
    const bf16_t* lvt = lkt + 2 * 1024;

    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (T + BM - 1) / BM;
    int rbi, bh;
    xcd_block_head(wg_id_x(), BH, rbi, bh);
    const int rb = nblk - 1 - rbi;  // row blocks with the most keys first
    const int b = bh / Hq, h = bh % Hq;
    const int bg = b * Hkv + h / (Hq / Hkv);
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc), lrow = perm_row(qc);
    const int i0 = rb * BM, r0 = i0 + wave * 32, i = r0 + qc;
    const bool live = r0 < T;
    const int i_hi = imin(r0 + 31, T - 1);
    const int ii = imin(i, T - 1);
    const int T32 = Tr / 32;
    const size_t prw = (size_t)bh * Tr + ii;

    bf16x8_t qtop[DS], dtop[DS];
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        qtop[s] = load_bf16x8(qts + prw * DD + s * 16 + hg * 8);
        dtop[s] = load_bf16x8(dts + prw * DD + s * 16 + hg * 8);
    }
    const f32x16_t negL = splat16(nl2[prw]), negd = splat16(nd[prw]);
    f32x16_t hT = splat16(0.f), olT = splat16(0.f);

    // one 32-key subtile at offset `sub` of the LDS tile (keys js..js+31)
    auto step = [&](int sub, int js, bool masked) {
        const bf16_t* ckr = lck + (sub * 32 + prow) * DD + hg * 8;
        const bf16_t* cvr = lcv + (sub * 32 + prow) * DD + hg * 8;
        f32x16_t x = mfma(load_bf16x8(ckr), qtop[0], negL);
        f32x16_t dp = mfma(load_bf16x8(cvr), dtop[0], negd);
        if (DS == 2) {
            x = mfma(load_bf16x8(ckr + 16), qtop[DS - 1], x);
            dp = mfma(load_bf16x8(cvr + 16), dtop[DS - 1], dp);
        }
        if (masked) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (js + acc_row(r, hg) > i - w) x[r] = -INFINITY;
        }
        f32x16_t p, ds;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            p[r] = __builtin_amdgcn_exp2f(x[r]);
            ds[r] = p[r] * dp[r];
        }
        const bf16_t* kt = lkt + sub * 1024 + lrow * 32 + hg * 8;
        const bf16_t* vt = lvt + sub * 1024 + lrow * 32 + hg * 8;
        hT = mfma(load_bf16x8(kt), pack8(ds, 0), hT);
        hT = mfma(load_bf16x8(kt + 16), pack8(ds, 8), hT);
        olT = mfma(load_bf16x8(vt), pack8(p, 0), olT);
        olT = mfma(load_bf16x8(vt + 16), pack8(p, 8), olT);
    };

    const int jd_wg = imin(i0 + BM - 1, T - 1) - w;  // last distant key of the workgroup
    const int jd_end = live ? i_hi - w : -1;         // ... of this wavefront
    if (jd_wg >= 0) {
        const uint4* g_ck = reinterpret_cast<const uint4*>(ckb + (size_t)bg * Tr * DD);
        const uint4* g_cv = reinterpret_cast<const uint4*>(cvb + (size_t)bg * Tr * DD);
        const uint4* g_kt = reinterpret_cast<const uint4*>(ckT + (size_t)bg * T32 * 1024);
        const uint4* g_vt = reinterpret_cast<const uint4*>(cvT + (size_t)bg * T32 * 1024);
        auto segs = [&](int t) {
            // rows t..t+63 (DD / 8 chunks each); transposed blocks t/32, t/32 + 1 (128 each)
            const size_t tb = (size_t)(t / 32) * 128;
            // four segments: the fifth is never read
            return Segs{g_ck + (size_t)t * DD / 8, g_cv + (size_t)t * DD / 8, g_kt + tb, g_vt + tb,
                        g_vt + tb, NK, NK, NT, NT};
        };
        SegRegs<NW, NCH> st = seg_fetch<NW, NCH>(segs(0), wave, lane);
        for (int t = 0; t <= jd_wg; t += 64) {
            __syncthreads();  // the previous tile is no longer read
            seg_store<NW, NCH>(st, tile, wave, lane);
            __syncthreads();
            if (t + 64 <= jd_wg) st = seg_fetch<NW, NCH>(segs(t + 64), wave, lane);
            const bool interior = t + 63 <= r0 - w;  // every key distant for every row
            if (live && interior) {
                step(0, t, false);
                step(1, t + 32, false);
            }
            if (live && !interior && t <= jd_end) step(0, t, t + 31 > r0 - w);
            if (live && !interior && t + 32 <= jd_end) step(1, t + 32, t + 63 > r0 - w);
        }
    }
    if (!live || i >= T) return;
    float* hr = hk + ((size_t)bh * T + i) * DD;
    float* orr = ol + ((size_t)bh * T + i) * DD;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        const int c = 16 * s + 8 * hg;
        *reinterpret_cast<float4*>(hr + c) = make_float4(hT[8 * s], hT[8 * s + 1], hT[8 * s + 2], hT[8 * s + 3]);
        *reinterpret_cast<float4*>(hr + c + 4) = make_float4(hT[8 * s + 4], hT[8 * s + 5], hT[8 * s + 6], hT[8 * s + 7]);
        *reinterpret_cast<float4*>(orr + c) = make_float4(olT[8 * s], olT[8 * s + 1], olT[8 * s + 2], olT[8 * s + 3]);
        *reinterpret_cast<float4*>(orr + c + 4) = make_float4(olT[8 * s + 4], olT[8 * s + 5], olT[8 * s + 6], olT[8 * s + 7]);
    }
}

// ---------------------------------------------------------------- distant: gK, gV

// One workgroup of NW wavefronts = 32 NW keys of one (batch, KV head); the
// distant rows i >= j + w of every query head of the group. The row operands
// of each 64-row tile (q~ and dO~ rows, their transposed blocks, the row
// constants) are copied once into LDS for the workgroup, as in the query-side
// kernel. Each row's -lse and -delta enter through one more product each,
// the row-constant operand (hi + mid + lo) against ones3. Writes
// gK = sum dS q~ (q~ unscaled) and gV = sum P dO~ (fp32) of every real key
// over the (head, row tile) pairs [pt p, pt p + pt) of part p (col_parts) into
// that part's arrays, gk, gv for part 0 and array p - 1 of gkx, gvx for the
// others (a block without distant rows has no part and writes nothing). Grid: np * ceil(T / (32 NW)) * B * Hkv workgroups
// (xcd_block_head), part 0 first, within a part key block 0 (most rows) first.
template <int DD, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_cols_dist_kernel(
    const bf16_t* __restrict__ ckb, const bf16_t* __restrict__ cvb,
    const bf16_t* __restrict__ qts, const bf16_t* __restrict__ qtT,
    const bf16_t* __restrict__ dts, const bf16_t* __restrict__ dtT,
    const bf16_t* __restrict__ rc, float* __restrict__ gk, float* __restrict__ gv,
    float* __restrict__ gkx, float* __restrict__ gvx, int Hq, int Hkv, int T, int Tr, int w,
    float gscale, int BKV, int pt) {
    constexpr int DS = DD / 16, BK = NW * 32;
    static_assert(BK == 128, "bwd_col_tiles");
    constexpr int NQ = 8 * DD, NT = 256, NC = 128;  // 16-byte chunks per 64-row tile
    constexpr int NCH = 2 * NQ + 2 * NT + NC;
    __shared__ __attribute__((aligned(16))) uint4 tile[NCH];
    const bf16_t* lq = reinterpret_cast<const bf16_t*>(tile);
    const bf16_t* ld = lq + 64 * DD;
    const bf16_t* lqt = ld + 64 * DD;
    const bf16_t* ldt = lqt + 2 * 1024;
    const bf16_t* lrc = ldt + 2 * 1024;

    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int cbi, bg;
    xcd_block_head(wg_id_x(), BKV, cbi, bg);
    const int nblk = (T + BK - 1) / BK;
    const int part = cbi / nblk, cb = cbi - part * nblk;
    const int b = bg / Hkv, g = bg % Hkv;
    const int G = Hq / Hkv;
    const int ntile = bwd_col_tiles(cb, T, w);
    const int n0 = part * pt, n1 = imin(n0 + pt, G * ntile);
    if (n0 >= n1) return;  // workgroup-uniform
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc);
    const int cwg = cb * BK;
    const int c0 = cwg + wave * 32, j = c0 + qc;
    const bool live = c0 < T;
    const int jj = imin(j, T - 1);
    const int T32 = Tr / 32;

    bf16x8_t ckop[DS], cvop[DS];
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        ckop[s] = load_bf16x8(ckb + ((size_t)bg * Tr + jj) * DD + s * 16 + hg * 8);
        cvop[s] = load_bf16x8(cvb + ((size_t)bg * Tr + jj) * DD + s * 16 + hg * 8);
    }
    const bf16x8_t b_lse = ones3(hg, 0), b_del = ones3(hg, 1);
    f32x16_t gkT = splat16(0.f), gvT = splat16(0.f);

    auto step = [&](int sub, int is, bool masked) {
        const bf16_t* qr = lq + (sub * 32 + prow) * DD + hg * 8;
        const bf16_t* dr = ld + (sub * 32 + prow) * DD + hg * 8;
        const bf16x8_t cst = load_bf16x8(lrc + (sub * 32 + prow) * 16 + hg * 8);
        f32x16_t x = mfma(cst, b_lse, splat16(0.f));
        f32x16_t dp = mfma(cst, b_del, splat16(0.f));
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            x = mfma(load_bf16x8(qr + s * 16), ckop[s], x);
            dp = mfma(load_bf16x8(dr + s * 16), cvop[s], dp);
        }
        if (masked) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = is + acc_row(r, hg);
                if (i - j < w || i >= T) x[r] = -INFINITY;
            }
        }
        f32x16_t p, ds;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            p[r] = __builtin_amdgcn_exp2f(x[r]);
            ds[r] = p[r] * dp[r];
        }
        const bf16_t* qt = lqt + sub * 1024 + prow * 32 + hg * 8;
        const bf16_t* dt = ldt + sub * 1024 + prow * 32 + hg * 8;
        gkT = mfma(load_bf16x8(qt), pack8(ds, 0), gkT);
        gkT = mfma(load_bf16x8(qt + 16), pack8(ds, 8), gkT);
        gvT = mfma(load_bf16x8(dt), pack8(p, 0), gvT);
        gvT = mfma(load_bf16x8(dt + 16), pack8(p, 8), gvT);
    };

    const int t0 = (cwg + w) & ~63;  // first row tile with a distant pair in the workgroup
    // two copies per tile (the operand rows and blocks, then the row constants):
    // each keeps at most four loads per thread in registers
    constexpr int NA = NCH - NC;
    auto segs = [&](int n, bool consts) {
        const int hh = n / ntile, t = t0 + (n - hh * ntile) * 64;
        const size_t bh = (size_t)b * Hq + g * G + hh;
        const uint4* rcs = reinterpret_cast<const uint4*>(rc + (bh * Tr + t) * 16);
        if (consts) return Segs{rcs, rcs, rcs, rcs, rcs, NC, 0, 0, 0};
        return Segs{reinterpret_cast<const uint4*>(qts + (bh * Tr + t) * DD),
                    reinterpret_cast<const uint4*>(dts + (bh * Tr + t) * DD),
                    reinterpret_cast<const uint4*>(qtT + (bh * T32 + t / 32) * 1024),
                    reinterpret_cast<const uint4*>(dtT + (bh * T32 + t / 32) * 1024),
                    rcs, NQ, NQ, NT, NT};
    };
    SegRegs<NW, NA> sa = seg_fetch<NW, NA>(segs(n0, false), wave, lane);
    SegRegs<NW, NC> sc = seg_fetch<NW, NC>(segs(n0, true), wave, lane);
    for (int n = n0; n < n1; ++n) {
        const int t = t0 + (n % ntile) * 64;
        __syncthreads();  // the previous tile is no longer read
        seg_store<NW, NA>(sa, tile, wave, lane);
        seg_store<NW, NC>(sc, tile + NA, wave, lane);
        __syncthreads();
        const int nn = imin(n + 1, n1 - 1);  // the last fetch repeats
        sa = seg_fetch<NW, NA>(segs(nn, false), wave, lane);
        sc = seg_fetch<NW, NC>(segs(nn, true), wave, lane);
        const bool interior = t >= c0 + 31 + w && t + 63 < T;  // every pair distant and real
        if (live && interior) {
            step(0, t, false);
            step(1, t + 32, false);
        }
        if (live && !interior && t + 31 >= c0 + w) step(0, t, true);
        if (live && !interior && t + 63 >= c0 + w && t + 32 < T) step(1, t + 32, true);
    }
    if (!live || j >= T) return;
    const size_t xrow = (((size_t)imax(part - 1, 0) * BKV + bg) * T + j) * DD;
    float* gkr = (part == 0 ? gk : gkx) + xrow;
    float* gvr = (part == 0 ? gv : gvx) + xrow;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        const int c = 16 * s + 8 * hg;
        *reinterpret_cast<float4*>(gkr + c) =
            make_float4(gkT[8 * s] * gscale, gkT[8 * s + 1] * gscale, gkT[8 * s + 2] * gscale, gkT[8 * s + 3] * gscale);
        *reinterpret_cast<float4*>(gkr + c + 4) =
            make_float4(gkT[8 * s + 4] * gscale, gkT[8 * s + 5] * gscale, gkT[8 * s + 6] * gscale, gkT[8 * s + 7] * gscale);
        *reinterpret_cast<float4*>(gvr + c) = make_float4(gvT[8 * s], gvT[8 * s + 1], gvT[8 * s + 2], gvT[8 * s + 3]);
        *reinterpret_cast<float4*>(gvr + c + 4) = make_float4(gvT[8 * s + 4], gvT[8 * s + 5], gvT[8 * s + 6], gvT[8 * s + 7]);
    }
}

// ---------------------------------------------------------------- window: dq, dW_up

// One wavefront per 32 query rows, window keys i - w < j <= i through 64-key
// K/V tiles in LDS. Epilogue: dq = s (dq_win + h W_up) and the workgroup's
// share of dW_up^T = sum_i q_i^T (s h_i) + dO_i^T ol_i (chunk
// (b * G + h % G) * nblk + row block). Grid: ceil(T / (32 NW)) * B * Hq
// workgroups (xcd_block_head).
template <int D, int DD, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_rows_local_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ dout, const bf16_t* __restrict__ wd, const bf16_t* __restrict__ wu,
    const float* __restrict__ hk, const float* __restrict__ ol, const float* __restrict__ nl2,
    const float* __restrict__ nd, bf16_t* __restrict__ dq, float* __restrict__ wpart, int Hq,
    int Hkv, int T, int Tr, int w, float qscale, float scale, int nchunk, int BH) {
    constexpr int KS = D / 16, NT = D / 32, DS = DD / 16, BN = 64, LDK = D + 8, LDH = 40;
    constexpr int BM = NW * 32;
    __shared__ __attribute__((aligned(16))) bf16_t lds_kv[2 * BN * LDK];  // K tile, V tile
    __shared__ __attribute__((aligned(16))) bf16_t lds_h[NW * 32 * LDH];
    __shared__ __attribute__((aligned(16))) float pbuf[D * DD];
    bf16_t* lds_k = lds_kv;
    bf16_t* lds_v = lds_kv + BN * LDK;

    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (T + BM - 1) / BM;
    int rbi, bh;
    xcd_block_head(wg_id_x(), BH, rbi, bh);
    const int rb = nblk - 1 - rbi;
    const int b = bh / Hq, h = bh % Hq;
    const int G = Hq / Hkv;
    const int g = h / G;
    const int bg = b * Hkv + g;
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc);
    const int i0 = rb * BM, r0 = i0 + wave * 32, i = r0 + qc;
    const bool live = r0 < T;
    const int i_hi = imin(r0 + 31, T - 1);
    const int iwg_hi = imin(i0 + BM - 1, T - 1);
    const int ii = imin(i, T - 1);

    const bf16_t* qrow = q + ((size_t)bh * T + ii) * D;
    const bf16_t* drow = dout + ((size_t)bh * T + ii) * D;
    bf16x8_t qop[KS], doop[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        qop[s] = load_bf16x8(qrow + s * 16 + hg * 8);
        doop[s] = load_bf16x8(drow + s * 16 + hg * 8);
    }
    const size_t prw = (size_t)bh * Tr + ii;
    const float nL = nl2[prw];
    const f32x16_t negd = splat16(nd[prw]);
    f32x16_t dqT[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) dqT[t] = splat16(0.f);

    const bf16_t* kg = k + (size_t)bg * T * D;
    const bf16_t* vg = v + (size_t)bg * T * D;
    if (w > 0) {
        const int t_first = imax(0, i0 - w + 1) & ~(BN - 1);
        TilePair<D, NW> tp;
        tp.fetch(kg, vg, t_first, T, tid);
        for (int t = t_first; t <= iwg_hi; t += BN) {
            __syncthreads();  // the previous tile is no longer read
            tp.store(lds_k, lds_v, LDK, tid);
            __syncthreads();
            if (t + BN <= iwg_hi) tp.fetch(kg, vg, t + BN, T, tid);
            if (!live) continue;
#pragma unroll
            for (int sub = 0; sub < BN / 32; ++sub) {
                const int js = t + sub * 32;
                if (js > i_hi || js + 31 <= r0 - w) continue;
                f32x16_t sc = splat16(0.f), dp = negd;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    sc = mfma(load_bf16x8(lds_k + (sub * 32 + prow) * LDK + s * 16 + hg * 8), qop[s], sc);
                    dp = mfma(load_bf16x8(lds_v + (sub * 32 + prow) * LDK + s * 16 + hg * 8), doop[s], dp);
                }
                f32x16_t x;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = __builtin_fmaf(sc[r], qscale, nL);
                if (!(js > i_hi - w && js + 31 <= r0)) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int j = js + acc_row(r, hg);
                        if (j <= i - w || j > i) x[r] = -INFINITY;
                    }
                }
                f32x16_t ds;
#pragma unroll
                for (int r = 0; r < 16; ++r) ds[r] = __builtin_amdgcn_exp2f(x[r]) * dp[r];
                const bf16x8_t s0 = pack8(ds, 0), s1 = pack8(ds, 8);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    dqT[tt] = mfma(lds_tr_operand(lds_k, LDK, sub * 32, tt * 32, lane), s0, dqT[tt]);
                    dqT[tt] = mfma(lds_tr_operand(lds_k, LDK, sub * 32 + 16, tt * 32, lane), s1, dqT[tt]);
                }
            }
        }
    }
    __syncthreads();  // the K/V tiles are reused below

    // ---- dq = s (dq_win + h W_up), h from the distant kernel as hi + lo bf16
    const bool real = live && i < T;
    const float* hrow = hk + ((size_t)bh * T + ii) * DD;
    const float* orow = ol + ((size_t)bh * T + ii) * DD;
    const bool any_dist = live && i_hi - w >= 0;  // wave-uniform
    if (any_dist) {
        const bf16_t* wdg = wd + (size_t)g * D * DD;
        const bf16_t* wug = wu ? wu + (size_t)g * DD * D : nullptr;
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            bf16x8_t hhi, hlo;
            split_f8(load_f8(hrow + s * 16 + hg * 8), 1.f, hhi, hlo);
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                // A[e][c] = W_up[c][e], rows e = 32 tt + qc, c = 16 s + 8 hg + 0..7
                const int e = tt * 32 + qc, cb = s * 16 + hg * 8;
                bf16x8_t a;
                if (wug) {
                    uint16_t a8[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) a8[u] = wug[(size_t)(cb + u) * D + e];
                    a = __builtin_bit_cast(bf16x8_t, a8);
                } else {
                    a = load_bf16x8(wdg + (size_t)e * DD + cb);
                }
                dqT[tt] = mfma(a, hhi, dqT[tt]);
                dqT[tt] = mfma(a, hlo, dqT[tt]);
            }
        }
    }
    if (real) {
        bf16_t* dqr = dq + ((size_t)bh * T + i) * D;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int a = 0; a < 4; ++a)
                store_bf16x4(dqr + tt * 32 + 8 * a + 4 * hg, dqT[tt][4 * a] * scale,
                             dqT[tt][4 * a + 1] * scale, dqT[tt][4 * a + 2] * scale,
                             dqT[tt][4 * a + 3] * scale);
    }

    // ---- share of dW_up^T [e][c] = sum_i q_i[e] s h_i[c] + dO_i[e] ol_i[c]
    f32x16_t pw[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) pw[t] = splat16(0.f);
    if (any_dist) {
        bf16_t* xs = lds_kv + wave * 32 * LDK;  // this wavefront's 32 rows of q, then dO
        bf16_t* ys = lds_h + wave * 32 * LDH;   // its 32 rows of s h, then ol (bf16, zero padded)
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
                *reinterpret_cast<bf16x8_t*>(xs + qc * LDK + s * 16 + hg * 8) = pass ? doop[s] : qop[s];
            const float f = real ? (pass ? 1.f : scale) : 0.f;  // rows past T add nothing
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int c = s * 16 + hg * 8;
                *reinterpret_cast<bf16x8_t*>(ys + qc * LDH + c) =
                    s < DS ? pack_f8(load_f8((pass ? orow : hrow) + c), f) : zero_bf16x8();
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const bf16x8_t bop = lds_tr_operand(ys, LDH, hf * 16, 0, lane);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt)
                    pw[tt] = mfma(lds_tr_operand(xs, LDK, hf * 16, tt * 32, lane), bop, pw[tt]);
            }
        }
    }
    const int chunk = (b * G + h % G) * nblk + rb;
    wg_share<D, DD, NW>(pw, pbuf, wave, lane, tid,
                        wpart + (((size_t)Hkv + g) * nchunk + chunk) * D * DD);
}

// ---------------------------------------------------------------- window: dk, dv, dW_down

// One wavefront per 32 keys, window rows j <= i < j + w of every query head
// of the group through 64-row Q / dO tiles in LDS. Epilogue: the distant part
// gK W_down^T, gV W_down^T (hi + lo bf16), and the workgroup's share of
// dW_down = sum_j k_j^T s gK_j + v_j^T gV_j (chunk b * nkb + key block).
// Grid: ceil(T / (32 NW)) * B * Hkv workgroups (xcd_block_head).
template <int D, int DD, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_cols_local_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ dout, const bf16_t* __restrict__ wd,
    const float* __restrict__ gk, const float* __restrict__ gv, const float* __restrict__ gkx,
    const float* __restrict__ gvx, const float* __restrict__ nl2, const float* __restrict__ nd,
    bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, float* __restrict__ wpart, int Hq, int Hkv, int T, int Tr, int w, float qscale, float scale,
    int nchunk, int BKV, int pt) {
    constexpr int KS = D / 16, NT = D / 32, DS = DD / 16, BN = 64, LDK = D + 8, LDH = 40;
    constexpr int BK = NW * 32;
    __shared__ __attribute__((aligned(16))) bf16_t lds_qd[2 * BN * LDK];  // Q tile, dO tile
    __shared__ __attribute__((aligned(16))) float lds_lse[BN];  // -lse (log2 units)
    __shared__ __attribute__((aligned(16))) float lds_del[BN];  // -delta
    __shared__ __attribute__((aligned(16))) bf16_t lds_g[NW * 32 * LDH];
    __shared__ __attribute__((aligned(16))) float pbuf[D * DD];
    bf16_t* lds_q = lds_qd;
    bf16_t* lds_do = lds_qd + BN * LDK;

    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int cb, bg;
    xcd_block_head(wg_id_x(), BKV, cb, bg);
    const int nkb = (T + BK - 1) / BK;
    const int b = bg / Hkv, g = bg % Hkv;
    const int G = Hq / Hkv;
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc);
    const int cwg_lo = cb * BK;
    const int c0 = cwg_lo + wave * 32, j = c0 + qc;
    const bool live = c0 < T;
    const int j_hi = imin(c0 + 31, T - 1);
    const int cwg_hi = imin(cwg_lo + BK - 1, T - 1);
    const int jj = imin(j, T - 1);

    bf16x8_t kop[KS], vop[KS];
    const bf16_t* krow = k + ((size_t)bg * T + jj) * D;
    const bf16_t* vrow = v + ((size_t)bg * T + jj) * D;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        kop[s] = load_bf16x8(krow + s * 16 + hg * 8);
        vop[s] = load_bf16x8(vrow + s * 16 + hg * 8);
    }
    f32x16_t dkT[NT], dvT[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) { dkT[t] = splat16(0.f); dvT[t] = splat16(0.f); }
    const int loc_hi = w > 0 ? imin(T - 1, cwg_hi + w - 1) : -1;  // last row with a window pair

    // (head, 64-row tile) pairs in order, the next one fetched during the
    // current one's work
    const int ntile = loc_hi >= cwg_lo ? (loc_hi - cwg_lo) / BN + 1 : 0;
    TilePair<D, NW> tp;
    float sv = 0.f;  // -lse (threads 0..63) or -delta (64..127) of one tile row
    auto fetch = [&](int n) {
        const int hh = n / ntile, t = cwg_lo + (n - hh * ntile) * BN;
        const size_t bh = (size_t)b * Hq + g * G + hh;
        tp.fetch(q + bh * T * D, dout + bh * T * D, t, T, tid);
        if (tid < 2 * BN) {
            const int r = tid & (BN - 1);
            const float* src = (tid < BN ? nl2 : nd) + bh * Tr;
            sv = t + r < Tr ? src[imin(t + r, Tr - 1)] : 0.f;
        }
    };
    if (ntile > 0) fetch(0);
    for (int n = 0; n < G * ntile; ++n) {
        const int t = cwg_lo + (n % ntile) * BN;
        {
            __syncthreads();  // the previous tile is no longer read
            tp.store(lds_q, lds_do, LDK, tid);
            if (tid < BN) lds_lse[tid] = sv;
            else if (tid < 2 * BN) lds_del[tid - BN] = sv;
            __syncthreads();
            if (n + 1 < G * ntile) fetch(n + 1);
            if (!live) continue;
#pragma unroll
            for (int sub = 0; sub < BN / 32; ++sub) {
                const int is = t + sub * 32;
                if (is + 31 < c0 || is > j_hi + w - 1) continue;
                f32x16_t sc = splat16(0.f);
                f32x16_t dp = load_row16(lds_del + sub * 32, hg, 1.f);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    sc = mfma(load_bf16x8(lds_q + (sub * 32 + prow) * LDK + s * 16 + hg * 8), kop[s], sc);
                    dp = mfma(load_bf16x8(lds_do + (sub * 32 + prow) * LDK + s * 16 + hg * 8), vop[s], dp);
                }
                const f32x16_t ln = load_row16(lds_lse + sub * 32, hg, 1.f);
                f32x16_t x;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = __builtin_fmaf(sc[r], qscale, ln[r]);
                if (!(is >= c0 + 31 && is + 31 - c0 < w && is + 31 < T)) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int i = is + acc_row(r, hg);
                        if (i < j || i - j >= w || i >= T) x[r] = -INFINITY;
                    }
                }
                f32x16_t p, ds;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    p[r] = __builtin_amdgcn_exp2f(x[r]);
                    ds[r] = p[r] * dp[r];
                }
                const bf16x8_t p0 = pack8(p, 0), p1 = pack8(p, 8);
                const bf16x8_t s0 = pack8(ds, 0), s1 = pack8(ds, 8);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    dvT[tt] = mfma(lds_tr_operand(lds_do, LDK, sub * 32, tt * 32, lane), p0, dvT[tt]);
                    dvT[tt] = mfma(lds_tr_operand(lds_do, LDK, sub * 32 + 16, tt * 32, lane), p1, dvT[tt]);
                    dkT[tt] = mfma(lds_tr_operand(lds_q, LDK, sub * 32, tt * 32, lane), s0, dkT[tt]);
                    dkT[tt] = mfma(lds_tr_operand(lds_q, LDK, sub * 32 + 16, tt * 32, lane), s1, dkT[tt]);
                }
            }
        }
    }
    __syncthreads();  // the Q/dO tiles are reused below

    // ---- dk = s dk_win + (s gK) W_down^T, dv = dv_win + gV W_down^T
    const bool real = live && j < T;
    const bf16_t* wdg = wd + (size_t)g * D * DD;
    const float* gkr = gk + ((size_t)bg * T + jj) * DD;
    const float* gvr = gv + ((size_t)bg * T + jj) * DD;
    const bool any_dist = live && c0 + w < T;  // wave-uniform
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int r = 0; r < 16; ++r) dkT[tt][r] *= scale;
    f32x8 ksum[DS], vsum[DS];  // the distant kernel's parts
    if (any_dist) {
        const int np = (G * bwd_col_tiles(cb, T, w) + pt - 1) / pt;
        const size_t stride = (size_t)BKV * T * DD;
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            ksum[s] = load_f8(gkr + s * 16 + hg * 8);
            vsum[s] = load_f8(gvr + s * 16 + hg * 8);
        }
        for (int pt_i = 1; pt_i < np; ++pt_i) {  // in part order, one round trip each
            f32x8 kx[DS], vx[DS];
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                const size_t at = (pt_i - 1) * stride + ((size_t)bg * T + jj) * DD + s * 16 + hg * 8;
                kx[s] = load_f8(gkx + at);
                vx[s] = load_f8(gvx + at);
            }
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                add_f8(ksum[s], kx[s]);
                add_f8(vsum[s], vx[s]);
            }
        }
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            bf16x8_t khi, klo, vhi, vlo;
            split_f8(ksum[s], scale, khi, klo);
            split_f8(vsum[s], 1.f, vhi, vlo);
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                const bf16x8_t a = load_bf16x8(wdg + (size_t)(tt * 32 + qc) * DD + s * 16 + hg * 8);
                dkT[tt] = mfma(a, khi, dkT[tt]);
                dkT[tt] = mfma(a, klo, dkT[tt]);
                dvT[tt] = mfma(a, vhi, dvT[tt]);
                dvT[tt] = mfma(a, vlo, dvT[tt]);
            }
        }
    }
    if (real) {
        bf16_t* dkr = dk + ((size_t)bg * T + j) * D;
        bf16_t* dvr = dv + ((size_t)bg * T + j) * D;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                store_bf16x4(dkr + tt * 32 + 8 * a + 4 * hg, dkT[tt][4 * a], dkT[tt][4 * a + 1],
                             dkT[tt][4 * a + 2], dkT[tt][4 * a + 3]);
                store_bf16x4(dvr + tt * 32 + 8 * a + 4 * hg, dvT[tt][4 * a], dvT[tt][4 * a + 1],
                             dvT[tt][4 * a + 2], dvT[tt][4 * a + 3]);
            }
    }

    // ---- share of dW_down [e][c] = sum_j k_j[e] s gK_j[c] + v_j[e] gV_j[c]
    f32x16_t pw[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) pw[t] = splat16(0.f);
    if (any_dist) {
        bf16_t* xs = lds_qd + wave * 32 * LDK;  // this wavefront's 32 keys, then values
        bf16_t* ys = lds_g + wave * 32 * LDH;   // s gK, then gV (bf16, zero padded)
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
                *reinterpret_cast<bf16x8_t*>(xs + qc * LDK + s * 16 + hg * 8) = pass ? vop[s] : kop[s];
            const float f = real ? (pass ? 1.f : scale) : 0.f;  // keys past T add nothing
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int c = s * 16 + hg * 8;
                *reinterpret_cast<bf16x8_t*>(ys + qc * LDH + c) =
                    s < DS ? pack_f8(pass ? vsum[imin(s, DS - 1)] : ksum[imin(s, DS - 1)], f)
                           : zero_bf16x8();
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const bf16x8_t bop = lds_tr_operand(ys, LDH, hf * 16, 0, lane);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt)
                    pw[tt] = mfma(lds_tr_operand(xs, LDK, hf * 16, tt * 32, lane), bop, pw[tt]);
            }
        }
    }
    wg_share<D, DD, NW>(pw, pbuf, wave, lane, tid,
                        wpart + ((size_t)g * nchunk + b * nkb + cb) * D * DD);
}

// ---------------------------------------------------------------- host

bool bwd_mfma_supported(int d, int dd, bool bf16) {
    return bf16 && (d == 64 || d == 128) && (dd == 16 || dd == 32);
}

// Parts of the key-side distant kernel: pt (head, row tile) pairs each, at most
// np of a key block. With several query heads per KV head its blocks are few
// and long, and its causal blocks differ in length by the whole sequence: the
// first one is the time (B2 Hq16 Hkv4 T4001 d128 d_down32 w512: 256 blocks,
// 267 us). A block's pairs are cut into parts of about one of kSlots equal
// shares of the whole work, at least 8 tiles each (a part costs about two
// tiles to start and finish), each with its own fp32 sums, which the window
// kernel adds in part order: the training step there 717 -> 552 us (with
// 512 shares: 561). 1 + Hq / Hkv parts fit the workspace. With a block
// for every resident workgroup already (four on each of 256 compute units)
// the parts only add their sums (B8 H8 T2048 d64 w256, 1024 blocks: 246.2
// against 245.3 us), so there is one. The query side has a block per query
// head and gains nothing from the same cut (83 against 81 us there, 38.3
// against 36.8 us at B8 H8 T2048 d64 w256).
struct ColParts {
    int pt, np;
};
static ColParts col_parts(int B, int Hq, int Hkv, int T, int w) {
    constexpr long long kSlots = 1280;
    const int nblk = (T + 127) / 128, G = Hq / Hkv;
    const long long most = (long long)bwd_col_tiles(0, T, w) * G;
    if (most == 0 || (long long)nblk * B * Hkv >= 4 * 256) return {(int)(most > 1 ? most : 1), 1};
    long long cols = 0;
    for (int i = 0; i < nblk; ++i) cols += (long long)bwd_col_tiles(i, T, w) * G;
    long long pt = (cols * B * Hkv + kSlots - 1) / kSlots;
    const long long fit = (most + G) / (1 + G);  // so that 1 + G parts are enough
    pt = pt > fit ? pt : fit;
    pt = pt > 8 ? pt : 8;
    return {(int)pt, (int)((most + pt - 1) / pt)};
}

template <int D, int DD>
static hipError_t launch_bwd_mfma_t(const bf16_t* q, const bf16_t* k, const bf16_t* v,
                                    const bf16_t* o, const float* lse, const bf16_t* dout,
                                    const bf16_t* wd, const bf16_t* wu, bf16_t* dq, bf16_t* dk,
                                    bf16_t* dv, float* dwd, float* dwu, char* ws, const BwdWs& L,
                                    int B, int Hq, int Hkv, int T, int w, hipStream_t st) {
    constexpr int NW = 4;
    const int Tr = round_up(T, 64);
    const size_t nrow = (size_t)B * Hq * Tr * DD, ntok = (size_t)B * Hkv * Tr * DD;  // bf16
    float* nl2 = (float*)(ws + L.lse_off);
    float* nd = (float*)(ws + L.delta_off);
    bf16_t* rc = (bf16_t*)(ws + L.rc_off);
    bf16_t* qts = (bf16_t*)(ws + L.qt_off);
    bf16_t* qtT = qts + nrow;
    bf16_t* dts = (bf16_t*)(ws + L.dot_off);
    bf16_t* dtT = dts + nrow;
    bf16_t* ckb = (bf16_t*)(ws + L.ck_off);
    bf16_t* ckT = ckb + ntok;
    bf16_t* cvb = (bf16_t*)(ws + L.cv_off);
    bf16_t* cvT = cvb + ntok;
    float* hk = (float*)(ws + L.hk_off);
    float* ol = (float*)(ws + L.ol_off);
    float* gk = (float*)(ws + L.gk_off);
    float* gv = (float*)(ws + L.gv_off);
    float* part = (float*)(ws + L.wpart_off);
    const float scale = 1.f / sqrtf((float)D);
    const float qscale = scale * kLog2eB;
    const int nblk = (T + NW * 32 - 1) / (NW * 32);

    const int nprep = (Tr + NW * 32 - 1) / (NW * 32);
    hipLaunchKernelGGL((bwd_prep_rows_kernel<D, DD, NW>), dim3(nprep, B * Hq), dim3(NW * 64), 0,
                       st, q, o, dout, lse, wd, wu, qts, qtT, dts, dtT, rc, nd, nl2, Hq, Hkv, T, Tr,
                       qscale);
    hipLaunchKernelGGL((bwd_prep_keys_kernel<D, DD, NW>), dim3(nprep, B * Hkv), dim3(NW * 64), 0,
                       st, k, v, wd, ckb, ckT, cvb, cvT, Hkv, T, Tr);
    const ColParts cp = col_parts(B, Hq, Hkv, T, w);
    auto cols_dist = [&] {
        hipLaunchKernelGGL((bwd_cols_dist_kernel<DD, NW>), dim3(cp.np * nblk * B * Hkv), dim3(NW * 64), 0,
                           st, (const bf16_t*)ckb, (const bf16_t*)cvb, (const bf16_t*)qts,
                           (const bf16_t*)qtT, (const bf16_t*)dts, (const bf16_t*)dtT,
                           (const bf16_t*)rc, gk, gv, hk, ol, Hq, Hkv, T, Tr, w, 1.f / qscale, B * Hkv,
                           cp.pt);
    };
    auto cols_local = [&] {
        hipLaunchKernelGGL((bwd_cols_local_kernel<D, DD, NW>), dim3(nblk * B * Hkv), dim3(NW * 64), 0,
                           st, q, k, v, dout, wd, (const float*)gk, (const float*)gv, (const float*)hk,
                           (const float*)ol, (const float*)nl2, (const float*)nd, dk, dv, part, Hq, Hkv,
                           T, Tr, w, qscale, scale, L.nchunk, B * Hkv, cp.pt);
    };
    auto rows_dist = [&] {
        hipLaunchKernelGGL((bwd_rows_dist_kernel<DD, NW>), dim3(nblk * B * Hq), dim3(NW * 64), 0, st,
                           (const bf16_t*)ckb, (const bf16_t*)ckT, (const bf16_t*)cvb,
                           (const bf16_t*)cvT, (const bf16_t*)qts, (const bf16_t*)dts,
                           (const float*)nl2, (const float*)nd, hk, ol, Hq, Hkv, T, Tr, w, B * Hq);
    };
    auto rows_local = [&] {
        hipLaunchKernelGGL((bwd_rows_local_kernel<D, DD, NW>), dim3(nblk * B * Hq), dim3(NW * 64), 0,
                           st, q, k, v, dout, wd, wu, (const float*)hk, (const float*)ol,
                           (const float*)nl2, (const float*)nd, dq, part, Hq, Hkv, T, Tr, w,
                           qscale, scale, L.nchunk, B * Hq);
    };
    if (cp.np > 1) {
        // the key side first: until the row side runs, hk and ol hold its parts
        cols_dist();
        cols_local();
        rows_dist();
        rows_local();
    } else {
        // (both distant kernels read the latents, both window kernels q and
        // dO: in the order above B8 H8 T2048 d64 w256 takes 0.9 % longer)
        rows_dist();
        cols_dist();
        rows_local();
        cols_local();
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_bwd_wreduce(part, dwd, dwu, Hkv, D, DD, L, st);
}

hipError_t launch_bwd_mfma(const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* o,
                           const float* lse, const bf16_t* dout, const bf16_t* wd,
                           const bf16_t* wu, bf16_t* dq, bf16_t* dk, bf16_t* dv, float* dwd,
                           float* dwu, char* ws, const BwdWs& L, int B, int Hq, int Hkv, int T,
                           int d, int dd, int w, hipStream_t st) {
#define DAR_BWD_CASE(D_, DD_)                                                                   \
    if (d == D_ && dd == DD_)                                                                   \
        return launch_bwd_mfma_t<D_, DD_>(q, k, v, o, lse, dout, wd, wu, dq, dk, dv, dwd, dwu,  \
                                          ws, L, B, Hq, Hkv, T, w, st);
    DAR_BWD_CASE(64, 16)
    DAR_BWD_CASE(64, 32)
    DAR_BWD_CASE(128, 16)
    DAR_BWD_CASE(128, 32)
#undef DAR_BWD_CASE
    return hipErrorInvalidValue;
}


// ================================================================ rotary embedding
//
// Backward of dar_attn_prefill_rope (Eq. 3 with the rotation; Section 2.3
// trains through it). The forward attends at full d: rotated queries qr,
// rotated window keys kr with values v, lifted-then-rotated distant keys kd
// with lifted values vd (the rotary pre-pass writes them; kd, vd hold
// positions 0..Td-1, Td = T - w). The softmax is recomputed against the
// forward's log-sum-exp:
//   bwd_rope_rowprep_kernel  -lse (log2 units) and -delta = -dO . O per row
//   bwd_rope_rows_kernel     dqr = s sum_j dS_ij key_ij over both regions, then
//                            dq = R^T dqr
//   bwd_rope_keys_kernel     per key, s sum_i dS_ij qr_i and sum_i P_ij dO_i over
//                            the rows that see it at distance (dkd, dvd) and in
//                            the window (dkr, dvw); the rotation taken back and
//                            the chain rule through the lift x' = (x W_down) W_up
//                            for keys and values, with the weight-gradient shares
//   bwd_wreduce_kernel       the shares summed in a fixed order
// with s = 1/sqrt(d). The main loops are the window kernels' loops with the
// key range and mask of either region; the key, row and latent gradients stay
// in registers from the sums to the bf16 stores (written out in fp32 and read
// back by separate rotation and chain-rule kernels they cost 135 MB and
// 220 us at B4 H16 T2048 d64 d_down16 w128).

namespace {

// -lse (log2 units) and -delta per row, zero for the padding rows. One
// thread per row (16-byte loads along the row).
template <int D>
__global__ __launch_bounds__(256) void bwd_rope_rowprep_kernel(const bf16_t* __restrict__ o,
                                                               const bf16_t* __restrict__ dout,
                                                               const float* __restrict__ lse,
                                                               float* __restrict__ nl2,
                                                               float* __restrict__ nd, int T,
                                                               int Tr) {
    const int bh = wg_id_y();
    const int i = wg_id_x() * 256 + lane_id_x();
    if (i >= Tr) return;
    float acc = 0.f;
    if (i < T) {
        const size_t row = ((size_t)bh * T + i) * D;
#pragma unroll
        for (int e = 0; e < D; e += 8) {
            const uint4 a = *reinterpret_cast<const uint4*>(o + row + e);
            const uint4 b = *reinterpret_cast<const uint4*>(dout + row + e);
            const uint32_t ua[4] = {a.x, a.y, a.z, a.w}, ub[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc = __builtin_fmaf(__uint_as_float(ua[q] << 16), __uint_as_float(ub[q] << 16), acc);
                acc = __builtin_fmaf(__uint_as_float(ua[q] & 0xffff0000u), __uint_as_float(ub[q] & 0xffff0000u), acc);
            }
        }
    }
    nd[(size_t)bh * Tr + i] = i < T ? -acc : 0.f;
    nl2[(size_t)bh * Tr + i] = i < T ? -lse[(size_t)bh * T + i] * kLog2eB : 0.f;
}

// Dynamic LDS: the rows kernel's two tiles, or its wavefronts' fp32 rows; the
// keys kernel's part below the weights (a wavefront's fp32 rows, or its bf16
// tile with a latent tile's three parts; the tiles and row constants fit in the
// same).
__host__ __device__ constexpr int rope_rows_lds_bytes(int D, int NW) {
    return 2 * 64 * (D + 8) * 2 > NW * 32 * (D + 4) * 4 ? 2 * 64 * (D + 8) * 2 : NW * 32 * (D + 4) * 4;
}
__host__ __device__ constexpr int rope_keys_scratch_bytes(int D, int NW) {
    return NW * (32 * (D + 4) * 4 > 32 * (D + 8) * 2 + 3 * 32 * 40 * 2 ? 32 * (D + 4) * 4
                                                                       : 32 * (D + 8) * 2 + 3 * 32 * 40 * 2);
}
static_assert(rope_keys_scratch_bytes(64, 4) >= 2 * 64 * 72 * 2 + 2 * 64 * 4 &&
                  rope_keys_scratch_bytes(128, 4) >= 2 * 64 * 136 * 2 + 2 * 64 * 4 &&
                  rope_keys_scratch_bytes(64, 4) >= 64 * 32 * 4 &&
                  rope_keys_scratch_bytes(128, 4) >= 128 * 32 * 4,
              "the row tiles and the share's sum fit in the scratch");

// f x, then the rotation taken back (R_p^T: the pairs (m, m + r/2) turned by
// -p base^(-2m/r); FWD: applied, R_p), for a wavefront's 32 tokens: accumulators in acc_row order
// (register 8 h + u of tile tt holds element 32 tt + 16 h + 8 hg + u of token
// qc). The pair's other element may sit in any register of either half, so
// the rows go through the wavefront's LDS (F, 32 rows of D + 4 floats). tabp:
// the angle row of this lane's token (r / 2 cos, then sin). Rotary dimensions
// that are multiples of 16 turn whole runs of eight with vector loads.
template <int D, bool FWD>
__device__ __forceinline__ void rotate_tile(f32x16_t (&x)[D / 32], float f, float* F, int r,
                                              const float* __restrict__ tabp, int qc, int hg) {
    constexpr int NT = D / 32, LDF = D + 4;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int q = 0; q < 16; ++q) x[tt][q] *= f;
    if (r == 0) return;  // uniform
    float* row = F + qc * LDF;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int q = 0; q < 8; q += 4)
                *reinterpret_cast<float4*>(row + 32 * tt + 16 * h2 + 8 * hg + q) =
                    make_float4(x[tt][8 * h2 + q], x[tt][8 * h2 + q + 1], x[tt][8 * h2 + q + 2],
                                x[tt][8 * h2 + q + 3]);
    wave_lds_order();
    const int h = r >> 1;
    const bool runs = (r & 15) == 0;  // uniform
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            const int e0 = 32 * tt + 16 * h2 + 8 * hg;
            if (32 * tt + 16 * h2 >= r) continue;  // uniform: both halves past the rotated part
            if (runs) {
                if (e0 < r) {
                    const bool first = e0 < h;  // of its pair
                    const int m = first ? e0 : e0 - h, o = first ? e0 + h : e0 - h;
#pragma unroll
                    for (int q = 0; q < 8; q += 4) {
                        const float4 c = *reinterpret_cast<const float4*>(tabp + m + q);
                        const float4 s = *reinterpret_cast<const float4*>(tabp + h + m + q);
                        const float4 y = *reinterpret_cast<const float4*>(row + o + q);
                        const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {s.x, s.y, s.z, s.w};
                        const float yy[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                        for (int z = 0; z < 4; ++z)
                            x[tt][8 * h2 + q + z] =
                                __builtin_fmaf(x[tt][8 * h2 + q + z], cc[z],
                                               first != FWD ? yy[z] * ss[z] : -yy[z] * ss[z]);
                    }
                }
            } else {
#pragma unroll
                for (int z = 0; z < 8; ++z) {
                    const int e = e0 + z;
                    if (e < r) {
                        const bool first = e < h;
                        const int m = first ? e : e - h;
                        const float y = row[first ? e + h : e - h], s = tabp[h + m];
                        x[tt][8 * h2 + z] =
                            __builtin_fmaf(x[tt][8 * h2 + z], tabp[m], first != FWD ? y * s : -y * s);
                    }
                }
            }
        }
    wave_lds_order();
}

// One wavefront per 32 query rows: dqr^T += K^T dS^T over the window keys
// (kr, v: i - w < j <= i) and the distant keys (kd, vd: j <= i - w), 64-key
// tiles staged through LDS for the workgroup. Writes dq = R^T (s dqr) of every
// real row. Grid: ceil(T / (32 NW)) * B * Hq workgroups (xcd_block_head).
template <int D, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_rope_rows_kernel(
    const bf16_t* __restrict__ qr, const bf16_t* __restrict__ kr, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ kd, const bf16_t* __restrict__ vd, const bf16_t* __restrict__ dout,
    const float* __restrict__ nl2, const float* __restrict__ nd, const float* __restrict__ tab,
    bf16_t* __restrict__ dq, int Hq, int Hkv, int T, int Tr, int w, int r, int pos0, float qscale,
    float scale, int BH) {
    constexpr int KS = D / 16, NT = D / 32, BN = 64, LDK = D + 8;
    constexpr int BM = NW * 32;
    // K tile and V tile, later each wavefront's fp32 rows for the rotation
    extern __shared__ __align__(16) char sm[];
    bf16_t* lds_k = reinterpret_cast<bf16_t*>(sm);
    bf16_t* lds_v = lds_k + BN * LDK;

    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (T + BM - 1) / BM;
    int rbi, bh;
    xcd_block_head(wg_id_x(), BH, rbi, bh);
    const int rb = nblk - 1 - rbi;
    const int b = bh / Hq, h = bh % Hq;
    const int G = Hq / Hkv;
    const int g = h / G;
    const int bg = b * Hkv + g;
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc);
    const int i0 = rb * BM, r0 = i0 + wave * 32, i = r0 + qc;
    const bool live = r0 < T;
    const int i_hi = imin(r0 + 31, T - 1);
    const int iwg_hi = imin(i0 + BM - 1, T - 1);
    const int ii = imin(i, T - 1);
    const int Td = imax(T - w, 0);

    const bf16_t* qrow = qr + ((size_t)bh * T + ii) * D;
    const bf16_t* drow = dout + ((size_t)bh * T + ii) * D;
    bf16x8_t qop[KS], doop[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        qop[s] = load_bf16x8(qrow + s * 16 + hg * 8);
        doop[s] = load_bf16x8(drow + s * 16 + hg * 8);
    }
    const size_t prw = (size_t)bh * Tr + ii;
    const float nL = nl2[prw];
    const f32x16_t negd = splat16(nd[prw]);
    f32x16_t dqT[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) dqT[t] = splat16(0.f);

    // keys [t_first, t_last] of one region (workgroup-uniform bounds: every
    // thread reaches the barriers)
    auto region = [&](const bf16_t* kg, const bf16_t* vg, int nkeys, int t_first, int t_last,
                      bool dist) {
        TilePair<D, NW> tp;
        tp.fetch(kg, vg, t_first, nkeys, tid);
        for (int t = t_first; t <= t_last; t += BN) {
            __syncthreads();  // the previous tile is no longer read
            tp.store(lds_k, lds_v, LDK, tid);
            __syncthreads();
            if (t + BN <= t_last) tp.fetch(kg, vg, t + BN, nkeys, tid);
            if (!live) continue;
#pragma unroll
            for (int sub = 0; sub < BN / 32; ++sub) {
                const int js = t + sub * 32;
                if (dist ? js > i_hi - w : (js > i_hi || js + 31 <= r0 - w)) continue;
                f32x16_t sc = splat16(0.f), dp = negd;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    sc = mfma(load_bf16x8(lds_k + (sub * 32 + prow) * LDK + s * 16 + hg * 8), qop[s], sc);
                    dp = mfma(load_bf16x8(lds_v + (sub * 32 + prow) * LDK + s * 16 + hg * 8), doop[s], dp);
                }
                f32x16_t x;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = __builtin_fmaf(sc[r], qscale, nL);
                const bool full = dist ? js + 31 <= r0 - w : (js > i_hi - w && js + 31 <= r0);
                if (!full) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int j = js + acc_row(r, hg);
                        if (dist ? j > i - w : (j <= i - w || j > i)) x[r] = -INFINITY;
                    }
                }
                f32x16_t ds;
#pragma unroll
                for (int r = 0; r < 16; ++r) ds[r] = __builtin_amdgcn_exp2f(x[r]) * dp[r];
                const bf16x8_t s0 = pack8(ds, 0), s1 = pack8(ds, 8);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    dqT[tt] = mfma(lds_tr_operand_perm(lds_k, LDK, sub * 32, tt * 32, lane), s0, dqT[tt]);
                    dqT[tt] = mfma(lds_tr_operand_perm(lds_k, LDK, sub * 32 + 16, tt * 32, lane), s1, dqT[tt]);
                }
            }
        }
    };
    if (w > 0) region(kr + (size_t)bg * T * D, v + (size_t)bg * T * D, T, imax(0, i0 - w + 1) & ~(BN - 1),
                      iwg_hi, false);
    if (iwg_hi - w >= 0) region(kd + (size_t)bg * Td * D, vd + (size_t)bg * Td * D, Td, 0, iwg_hi - w, true);

    __syncthreads();  // the tiles are no longer read
    rotate_tile<D, false>(dqT, scale, reinterpret_cast<float*>(sm) + wave * 32 * (D + 4), r,
                     tab + (size_t)(pos0 + ii) * r, qc, hg);
    if (live && i < T) {
        bf16_t* out = dq + ((size_t)bh * T + i) * D + 8 * hg;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2)
                *reinterpret_cast<bf16x8_t*>(out + tt * 32 + h2 * 16) = pack8(dqT[tt], 8 * h2);
    }
}

// One workgroup of NW wavefronts = 32 NW keys of one (batch, KV head), the
// rows of every query head of the group that see them, through 64-row Q / dO
// tiles in LDS: dk^T += Q^T dS, dv^T += dO^T P. First the rows at distance
// (i >= j + w) against the lifted keys (kd, vd), then the window's rows
// (j <= i < j + w) against (kr, v), each key's sums in one lane column. With
// u = R^T s dkd between the two:
//   gK = u W_up^T,  gV = dvd W_up^T,  cK = k W_down,  cV = v W_down
//   dW_down += k^T gK + v^T gV,  dW_up^T += u^T cK + dvd^T cV  (shares)
//   dk = R^T s dkr + gK W_down^T,  dv = dvw + gV W_down^T
// on the matrix cores; u, dvd, gK, gV, cK, cV are fp32 sums and enter as bf16
// triples hi + mid + lo, so that a product with a bf16 factor carries the 24
// bits of fp32 (three products) and one of two fp32 factors as well (six). The
// chain rule adds about 130 products per wavefront to the 16 of each of its
// 32-row subtiles at d = 64: forward and backward at B4 H16 T2048 d64 d_down16
// w128 take 348 us (550 with the chain rule on the vector ALUs; 338 with hi +
// lo pairs, 75 products, whose weight gradients carried 16 bits: 2^-16.5 of the
// summed magnitudes off where the triples are 2^-22). The window's sums start from gK W_down^T and gV W_down^T
// instead of keeping gK and gV in registers through the window's loop. d_down
// <= 32 DT columns, zero padded. Writes the share of chunk b * nkb + key block.
// Grid: ceil(T / (32 NW)) * B * Hkv workgroups
// (xcd_block_head), key block 0 (most rows) first.
template <int D, int DT, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_rope_keys_kernel(
    const bf16_t* __restrict__ qr, const bf16_t* __restrict__ kr, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ kd, const bf16_t* __restrict__ vd, const bf16_t* __restrict__ dout,
    const float* __restrict__ nl2, const float* __restrict__ nd, const bf16_t* __restrict__ k,
    const bf16_t* __restrict__ wd, const bf16_t* __restrict__ wu, const float* __restrict__ tab,
    bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, float* __restrict__ wpart, int Hq, int Hkv,
    int T, int Tr, int dd, int w, int r, int pos0, float qscale, float scale, int nchunk, int BKV) {
    constexpr int KS = D / 16, NT = D / 32, BN = 64, LDK = D + 8, LDH = 40;
    constexpr int BK = NW * 32;
    extern __shared__ __align__(16) char sm[];
    // Q tile, dO tile, -lse and -delta of their rows; between and after the
    // regions the wavefronts' scratch (fp32 rows for the rotation, or a bf16
    // tile and a latent tile's three parts) and the weight shares' sum
    bf16_t* lds_q = reinterpret_cast<bf16_t*>(sm);
    bf16_t* lds_do = lds_q + BN * LDK;
    float* lds_lse = reinterpret_cast<float*>(lds_do + BN * LDK);
    float* lds_del = lds_lse + BN;
    bf16_t* wds = reinterpret_cast<bf16_t*>(sm + rope_keys_scratch_bytes(D, NW));  // W_down^T [c][e]
    bf16_t* wus = wu ? wds + 32 * DT * LDK : wds;                                  // W_up [c][e]

    const int tid = lane_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int cb, bg;
    xcd_block_head(wg_id_x(), BKV, cb, bg);
    const int b = bg / Hkv, g = bg % Hkv;
    const int G = Hq / Hkv;
    const int qc = lane & 31, hg = lane >> 5, prow = perm_row(qc);
    const int cwg_lo = cb * BK;
    const int c0 = cwg_lo + wave * 32, j = c0 + qc;
    const bool live = c0 < T;
    const int jj = imin(j, T - 1);
    const int Td = imax(T - w, 0);

    {
        const bf16_t* wdg = wd + (size_t)g * D * dd;
        const bf16_t* wug = wu ? wu + (size_t)g * dd * D : nullptr;
        for (int idx = tid; idx < 32 * DT * D; idx += NW * 64) {
            const int c = idx / D, e = idx % D, cc = imin(c, dd - 1);
            const bf16_t x = wdg[(size_t)e * dd + cc];
            wds[c * LDK + e] = c < dd ? x : (bf16_t)0;
            if (wug) {
                const bf16_t y = wug[(size_t)cc * D + e];
                wus[c * LDK + e] = c < dd ? y : (bf16_t)0;
            }
        }
    }

    f32x16_t dkT[NT], dvT[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) { dkT[t] = splat16(0.f); dvT[t] = splat16(0.f); }
    // the sums over one region's rows, added to dkT, dvT (workgroup-uniform
    // bounds: every thread reaches the barriers)
    auto region = [&](const bf16_t* kx, const bf16_t* vx, int nkeys, bool dist) {
        const int j_hi = imin(c0 + 31, nkeys - 1);
        const int cwg_hi = imin(cwg_lo + BK - 1, nkeys - 1);
        bf16x8_t kop[KS], vop[KS];
        const bf16_t* krow = kx + ((size_t)bg * nkeys + imin(j, nkeys - 1)) * D;
        const bf16_t* vrow = vx + ((size_t)bg * nkeys + imin(j, nkeys - 1)) * D;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            kop[s] = load_bf16x8(krow + s * 16 + hg * 8);
            vop[s] = load_bf16x8(vrow + s * 16 + hg * 8);
        }
        // the workgroup's rows: window [cwg_lo, cwg_hi + w - 1], at distance [cwg_lo + w, T - 1]
        const int row_lo = dist ? cwg_lo + w : cwg_lo;
        const int row_hi = dist ? T - 1 : imin(T - 1, cwg_hi + w - 1);
        const int ntile = row_hi >= row_lo ? (row_hi - row_lo) / BN + 1 : 0;
        TilePair<D, NW> tp;
        float sv = 0.f;  // -lse (threads 0..63) or -delta (64..127) of one tile row
        auto fetch = [&](int n) {
            const int hh = n / ntile, t = row_lo + (n - hh * ntile) * BN;
            const size_t bh = (size_t)b * Hq + g * G + hh;
            tp.fetch(qr + bh * T * D, dout + bh * T * D, t, T, tid);
            if (tid < 2 * BN) {
                const int rr = tid & (BN - 1);
                const float* src = (tid < BN ? nl2 : nd) + bh * Tr;
                sv = t + rr < Tr ? src[imin(t + rr, Tr - 1)] : 0.f;
            }
        };
        if (ntile > 0) fetch(0);
        for (int n = 0; n < G * ntile; ++n) {
            const int t = row_lo + (n % ntile) * BN;
            __syncthreads();  // the previous tile is no longer read
            tp.store(lds_q, lds_do, LDK, tid);
            if (tid < BN) lds_lse[tid] = sv;
            else if (tid < 2 * BN) lds_del[tid - BN] = sv;
            __syncthreads();
            if (n + 1 < G * ntile) fetch(n + 1);
            if (!live) continue;
#pragma unroll
            for (int sub = 0; sub < BN / 32; ++sub) {
                const int is = t + sub * 32;
                if (dist ? is + 31 < c0 + w : (is + 31 < c0 || is > j_hi + w - 1)) continue;
                f32x16_t sc = splat16(0.f);
                f32x16_t dp = load_row16(lds_del + sub * 32, hg, 1.f);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    sc = mfma(load_bf16x8(lds_q + (sub * 32 + prow) * LDK + s * 16 + hg * 8), kop[s], sc);
                    dp = mfma(load_bf16x8(lds_do + (sub * 32 + prow) * LDK + s * 16 + hg * 8), vop[s], dp);
                }
                const f32x16_t ln = load_row16(lds_lse + sub * 32, hg, 1.f);
                f32x16_t x;
#pragma unroll
                for (int q = 0; q < 16; ++q) x[q] = __builtin_fmaf(sc[q], qscale, ln[q]);
                const bool full = dist ? (is >= j_hi + w && is + 31 < T)
                                       : (is >= c0 + 31 && is + 31 - c0 < w && is + 31 < T);
                if (!full) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const int i = is + acc_row(q, hg);
                        if (dist ? (i - j < w || i >= T) : (i < j || i - j >= w || i >= T))
                            x[q] = -INFINITY;
                    }
                }
                f32x16_t p, ds;
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    p[q] = __builtin_amdgcn_exp2f(x[q]);
                    ds[q] = p[q] * dp[q];
                }
                const bf16x8_t p0 = pack8(p, 0), p1 = pack8(p, 8);
                const bf16x8_t s0 = pack8(ds, 0), s1 = pack8(ds, 8);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    dvT[tt] = mfma(lds_tr_operand_perm(lds_do, LDK, sub * 32, tt * 32, lane), p0, dvT[tt]);
                    dvT[tt] = mfma(lds_tr_operand_perm(lds_do, LDK, sub * 32 + 16, tt * 32, lane), p1, dvT[tt]);
                    dkT[tt] = mfma(lds_tr_operand_perm(lds_q, LDK, sub * 32, tt * 32, lane), s0, dkT[tt]);
                    dkT[tt] = mfma(lds_tr_operand_perm(lds_q, LDK, sub * 32 + 16, tt * 32, lane), s1, dkT[tt]);
                }
            }
        }
        __syncthreads();  // the tiles are no longer read (and the weights are staged)
    };

    float* F = reinterpret_cast<float*>(sm + wave * (rope_keys_scratch_bytes(D, NW) / NW));
    bf16_t* xs = reinterpret_cast<bf16_t*>(F);  // [32][LDK]: 32 tokens at full d
    bf16_t* ys = xs + 32 * LDK;                 // [3][32][LDH]: a 32-column latent tile, hi, mid, lo
    const float* tabp = tab + (size_t)(pos0 + jj) * r;
    const bool any_dist = live && c0 + w < T;  // wave-uniform
    const int nkb = (T + BK - 1) / BK;
    const size_t n_out = (size_t)D * dd;
    const int chunk = b * nkb + cb;

    if (Td > cwg_lo) region(kd, vd, Td, true);  // (workgroup-uniform) some key is distant for some row
    else __syncthreads();                       // the weights are staged
    rotate_tile<D, false>(dkT, scale, F, r, tabp, qc, hg);  // u
    // u and dvd stay in fp32 and are split where they enter a product
    f32x16_t u[NT], dvd[NT];
    // gK W_down^T and gV W_down^T; the window's sums are added on top, the
    // first (rotated forward, over s) in the rotated keys' frame
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        u[t] = dkT[t];
        dvd[t] = dvT[t];
        dkT[t] = splat16(0.f);
        dvT[t] = splat16(0.f);
    }
    const size_t own = ((size_t)bg * T + jj) * D + hg * 8;
    // acc[e][c] += sum_j X[j][e] Y[j][c] with the parts hi .. of Y down to part
    // `last` (smallest first); x(s): step s of this lane's token
    auto share = [&](f32x16_t (&acc)[NT], auto x, int last) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
            *reinterpret_cast<bf16x8_t*>(xs + qc * LDK + s * 16 + hg * 8) = x(s);
        wave_lds_order();
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            bf16x8_t y[3];
#pragma unroll
            for (int p = 0; p <= last; ++p) y[p] = lds_tr_operand(ys + p * 32 * LDH, LDH, hf * 16, 0, lane);
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                const bf16x8_t a = lds_tr_operand(xs, LDK, hf * 16, tt * 32, lane);
#pragma unroll
                for (int p = last; p >= 0; --p) acc[tt] = mfma(a, y[p], acc[tt]);
            }
        }
        wave_lds_order();
    };
    // one of the two sides (keys: u, k, dkT; values: dvd, v, dvT) of 32 columns,
    // so that no instance spills a register: with the sides and the column tiles
    // side by side d = 128, d_down > 32 took all 512 and scratch besides, and a
    // tuple spilled partly to accumulation registers and partly to scratch may
    // come back incomplete (tests/test_kernel_resources.py).
    // up 0: gX = x W_up^T, dW_down += row^T gX, g += gX W_down^T;
    // up 1: cX = row W_down, dW_up^T += x^T cX
    auto side = [&](int up, int ct, const f32x16_t (&x)[NT], const bf16_t* rows, f32x16_t (&g)[NT],
                    f32x16_t (&pw)[NT]) {
        f32x16_t y = splat16(0.f);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8_t a = load_bf16x8((up ? wds : wus) + (32 * ct + prow) * LDK + s * 16 + hg * 8);
            if (up) {
                y = mfma(a, load_bf16x8(rows + own + s * 16), y);
            } else {
                bf16x8_t xp[3];
                split8x3(x[s >> 1], 8 * (s & 1), xp);
#pragma unroll
                for (int p = 2; p >= 0; --p) y = mfma(a, xp[p], y);
            }
        }
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            bf16x8_t yp[3];
            split8x3(y, 8 * h2, yp);
#pragma unroll
            for (int p = 0; p < 3; ++p)
                *reinterpret_cast<bf16x8_t*>(ys + (p * 32 + qc) * LDH + 16 * h2 + 8 * hg) = yp[p];
            if (up == 0) {
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    const bf16x8_t a = lds_tr_operand_perm(wds, LDK, 32 * ct + 16 * h2, 32 * tt, lane);
#pragma unroll
                    for (int p = 2; p >= 0; --p) g[tt] = mfma(a, yp[p], g[tt]);
                }
            }
        }
        if (up) {
            // every product of the two factors' parts that reaches 2^-24: lo hi,
            // mid (mid, hi), hi (lo, mid, hi)
#pragma unroll
            for (int p = 2; p >= 0; --p)
                share(pw, [&](int s) {
                    bf16x8_t xp[3];
                    split8x3(x[s >> 1], 8 * (s & 1), xp);
                    return xp[p];
                }, 2 - p);
        } else {
            share(pw, [&](int s) { return load_bf16x8(rows + own + s * 16); }, 2);
        }
    };
#pragma nounroll
    for (int ct = 0; ct < DT; ++ct)
#pragma unroll
        for (int up = 0; up < 2; ++up) {
            f32x16_t pw[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) pw[t] = splat16(0.f);
            if (any_dist) {
                wave_lds_order();
                side(up, ct, u, k, dkT, pw);
                side(up, ct, dvd, v, dvT, pw);
            }
            // the wavefronts' shares added in order (pbuf is the scratch)
            __syncthreads();
            wg_share_cols<D, NW>(pw, reinterpret_cast<float*>(sm), wave, lane, tid, dd, 32 * ct,
                                 wpart + ((size_t)(up ? Hkv + g : g) * nchunk + chunk) * n_out);
            __syncthreads();
        }

    if (w > 0) {
        rotate_tile<D, true>(dkT, 1.f / scale, F, r, tabp, qc, hg);
        __syncthreads();  // the scratch becomes the tiles
        region(kr, v, T, false);
        rotate_tile<D, false>(dkT, scale, F, r, tabp, qc, hg);
    }
    if (live && j < T) {
        bf16_t* dkr = dk + ((size_t)bg * T + j) * D + 8 * hg;
        bf16_t* dvr = dv + ((size_t)bg * T + j) * D + 8 * hg;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                *reinterpret_cast<bf16x8_t*>(dkr + tt * 32 + h2 * 16) = pack8(dkT[tt], 8 * h2);
                *reinterpret_cast<bf16x8_t*>(dvr + tt * 32 + h2 * 16) = pack8(dvT[tt], 8 * h2);
            }
    }
}

// Above 64 KB a kernel's dynamic LDS has to be asked for.
hipError_t allow_lds(const void* fn, int bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

}  // namespace

// d_down up to d, and at d = 128 up to 73, the interface's limit (three column
// tiles would hold 96 in 120 KB of LDS)
bool bwd_rope_mfma_supported(int d, int dd, bool bf16) {
    return bf16 && ((d == 64 && dd <= 64) || (d == 128 && dd <= 73));
}

template <int D, int DT, int NW>
static hipError_t launch_rope_keys_t(const RopeBwdArgs& a, hipStream_t st) {
    const int nkb = (a.T + NW * 32 - 1) / (NW * 32);
    const float scale = 1.f / sqrtf((float)D);
    const int lds = rope_keys_scratch_bytes(D, NW) + (a.wu ? 2 : 1) * 32 * DT * (D + 8) * 2;
    const hipError_t e = allow_lds((const void*)bwd_rope_keys_kernel<D, DT, NW>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bwd_rope_keys_kernel<D, DT, NW>), dim3(nkb * a.B * a.Hkv), dim3(NW * 64), lds,
                       st, a.qr, a.kr, a.v, a.kd, a.vd, a.dout, (const float*)a.nl2,
                       (const float*)a.nd, a.k, a.wd, a.wu, a.tab, a.dk, a.dv, a.wpart, a.Hq, a.Hkv,
                       a.T, round_up(a.T, 64), a.dd, a.w, a.r, a.pos0, scale * kLog2eB, scale,
                       a.L.nchunk, a.B * a.Hkv);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_bwd_rope_t(const RopeBwdArgs& a, hipStream_t st) {
    constexpr int NW = 4;
    const int B = a.B, Hq = a.Hq, Hkv = a.Hkv, T = a.T, w = a.w, dd = a.dd, r = a.r;
    const int Tr = round_up(T, 64);
    const float scale = 1.f / sqrtf((float)D);
    const float qscale = scale * kLog2eB;
    const int nblk = (T + NW * 32 - 1) / (NW * 32);
    hipLaunchKernelGGL(bwd_rope_rowprep_kernel<D>, dim3((Tr + 255) / 256, B * Hq), dim3(256), 0, st, a.o, a.dout,
                       a.lse, a.nl2, a.nd, T, Tr);
    const int rlds = rope_rows_lds_bytes(D, NW);
    hipError_t e = allow_lds((const void*)bwd_rope_rows_kernel<D, NW>, rlds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bwd_rope_rows_kernel<D, NW>), dim3(nblk * B * Hq), dim3(NW * 64), rlds, st,
                       a.qr, a.kr, a.v, a.kd, a.vd, a.dout, (const float*)a.nl2, (const float*)a.nd,
                       a.tab, a.dq, Hq, Hkv, T, Tr, w, r, a.pos0, qscale, scale, B * Hq);
    if (dd <= 32) e = launch_rope_keys_t<D, 1, NW>(a, st);
    else if (dd <= 64) e = launch_rope_keys_t<D, 2, NW>(a, st);
    else if constexpr (D == 128) e = launch_rope_keys_t<D, 3, NW>(a, st);
    else e = hipErrorInvalidValue;
    if (e != hipSuccess) return e;
    return launch_bwd_wreduce(a.wpart, a.dwd, a.dwu, Hkv, D, dd, a.L, st);
}

hipError_t launch_bwd_rope_mfma(const RopeBwdArgs& a, int d, hipStream_t st) {
    if (d == 64) return launch_bwd_rope_t<64>(a, st);
    if (d == 128) return launch_bwd_rope_t<128>(a, st);
    return hipErrorInvalidValue;
}

}  // namespace dar
