// fp32 prefill and backward on the fp32 matrix cores (v_mfma_f32_16x16x4_f32:
// fp32 operands, products and sums) for heads up to
// 128 wide, gfx950.
//
// One wavefront per 16 query rows (or 16 keys) and no LDS: the instruction's
// layouts, lane l = 16 qd + c16,
//   A (16 x 4): A[c16][k = qd]   B (4 x 16): B[k = qd][c16]
//   C (16 x 16): register r holds C[4 qd + r][c16]
// let every product take its operands as they come. Which four k a step
// covers is free as long as A and B agree:
//  * a product over d takes k = qd D/4 + s at step s: a lane reads D/4
//    consecutive elements of its row;
//  * a product over the 16 rows of an accumulator tile (keys of S^T for P V,
//    latent columns for the lift, ...) takes k = 4 qd + r at step r, so the
//    accumulator registers are the B operand without any movement, and the A
//    operand is read 16 elements of a row at a time, consecutive over lanes.
// Rows are padded with zeros to D (64 or 128) and latents to DD in registers.
//
// What bounds it: at the sizes fp32 is used for (gradient checks, short
// fine-tunes) the chip is mostly idle and the longest row's chain of loads,
// products and exponentials is the time; 16-row wavefronts keep that chain
// short and give T / 16 wavefronts a head. Forward and backward at B1 H8 T331
// d64 d_down16 w64 took 605 us with one wavefront per row on the vector ALUs
// (every lane reading its own key row element by element), 130 us here.
//
// A masked pair (after the row, outside the region) has weight exactly zero,
// but a product multiplies it all the same: a subtile with masked pairs whose
// operand holds an infinity or a NaN is added pair by pair (add_product), so
// that a token never reaches a row that does not see it.
#include "dar_common.hpp"
#include "dar_kernels.hpp"

namespace dar {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;

__device__ __forceinline__ f32x4_t mma(float a, float b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4_t zero4() { return f32x4_t{0.f, 0.f, 0.f, 0.f}; }

// Sum / maximum over the four lanes of a column.
__device__ __forceinline__ float col_sum(float x) {
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float col_max(float x) {
    x = fmaxf(x, __shfl_xor(x, 16, 64));
    return fmaxf(x, __shfl_xor(x, 32, 64));
}

// Element e of a row of n, zero past it. (Here and below the address is
// clamped and the value selected: loads under a condition each keep a lane
// mask, and the scalar registers for those ran out.)
__device__ __forceinline__ float load1(const float* row, int e, int n) {
    const float x = row[imin(e, n - 1)];
    return e < n ? x : 0.f;
}

// Four elements e..e+3 of a row of n (zeros past it); whole: n is the padded
// width (uniform), rows are then 16-byte aligned.
__device__ __forceinline__ float4 load4(const float* row, int e, int n, bool whole) {
    if (whole) return *reinterpret_cast<const float4*>(row + e);
    return make_float4(load1(row, e, n), load1(row, e + 1, n), load1(row, e + 2, n),
                       load1(row, e + 3, n));
}

// W[c][e] of a lift: wu [dd][d], or wd [d][dd] transposed; zero outside.
__device__ __forceinline__ float weight(const float* wd, const float* wu, int c, int e, int d,
                                        int dd) {
    const int cc = imin(c, dd - 1), ee = imin(e, d - 1);
    const float x = *(wu ? wu + (size_t)cc * d + ee : wd + (size_t)ee * dd + cc);
    return c < dd && e < d ? x : 0.f;
}

// This lane's D/4 elements of a row of d, times f.
template <int D>
__device__ __forceinline__ void load_row(const float* row, int qd, int d, float f,
                                         float (&x)[D / 4]) {
    const bool whole = d == D;
#pragma unroll
    for (int s = 0; s < D / 4; s += 4) {
        const float4 v = load4(row, qd * (D / 4) + s, d, whole);
        x[s] = v.x * f; x[s + 1] = v.y * f; x[s + 2] = v.z * f; x[s + 3] = v.w * f;
    }
}

// A operands of one 16-row step over rows `row(r)` (r = 0..3, this lane's k):
// a[r][t] = X[row][16 t + c16], X rows of n elements.
template <int NT, class F>
__device__ __forceinline__ void load_cols(float (&a)[4][NT], F row, int c16, int n) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float* p = row(r);
#pragma unroll
        for (int t = 0; t < NT; ++t) a[r][t] = load1(p, 16 * t + c16, n);
    }
}

// The bits of x, opaque: the sources are compiled with NaN taken as absent, so
// a comparison that only a NaN decides would be dropped.
__device__ __forceinline__ uint32_t bits_of(float x) {
    uint32_t u = __float_as_uint(x);
    __asm__ volatile("" : "+v"(u));
    return u;
}

// acc[t] += sum_r A(r, t) p[r]: 16 rows of A against the weights p. edge: some
// pair is masked (p = 0 there) and must not meet an infinity or a NaN.
template <int NT>
__device__ __forceinline__ void add_product(f32x4_t (&acc)[NT], const float (&a)[4][NT],
                                            const float (&p)[4], bool edge, int qd, int c16) {
    if (edge) {
        bool odd = false;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                odd |= (bits_of(a[r][t]) & 0x7f800000u) == 0x7f800000u;
        if (__builtin_amdgcn_ballot_w64(odd)) {
            // register u of a lane is row 16 t + 4 qd + u of the product
            for (int kq = 0; kq < 4; ++kq)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float pk = __shfl(p[r], 16 * kq + c16, 64);
                    const uint32_t keep = (bits_of(pk) << 1) != 0u ? 0xffffffffu : 0u;
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float x = __shfl(a[r][t], 16 * kq + 4 * qd + u, 64);
                            acc[t][u] = __builtin_fmaf(__uint_as_float(bits_of(x) & keep), pk,
                                                       acc[t][u]);
                        }
                }
            return;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = mma(a[r][t], p[r], acc[t]);
}

// y^T[c][token] = sum_e U[c][e] x[token][e] (U = W_up, or W_down^T): x the
// lane's row elements, register r of tile ct is column 16 ct + 4 qd + r.
template <int D, int DD>
__device__ __forceinline__ void project(const float* wd, const float* wu, int d, int dd, int qd,
                                        int c16, const float (&x)[D / 4], f32x4_t (&y)[DD / 16]) {
#pragma unroll
    for (int ct = 0; ct < DD / 16; ++ct) {
        y[ct] = zero4();
#pragma unroll
        for (int s = 0; s < D / 4; ++s)
            y[ct] = mma(weight(wd, wu, 16 * ct + c16, qd * (D / 4) + s, d, dd), x[s], y[ct]);
    }
}

// acc^T[e][token] += sum_c W[c][e] y^T[c][token], W = wu [dd][d] or, transposed,
// wd [d][dd].
template <int D, int DD>
__device__ __forceinline__ void lift(const float* wd, const float* wu, int d, int dd, int qd,
                                     int c16, const f32x4_t (&y)[DD / 16], f32x4_t (&acc)[D / 16]) {
#pragma unroll
    for (int ct = 0; ct < DD / 16; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < D / 16; ++t)
                acc[t] = mma(weight(wd, wu, 16 * ct + 4 * qd + r, 16 * t + c16, d, dd), y[ct][r], acc[t]);
}

// Row of n from accumulator tiles (register r of tile t: element 16 t + 4 qd + r).
template <int NT>
__device__ __forceinline__ void store_row(float* out, const f32x4_t (&x)[NT], int qd, int n,
                                          float f) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int e = 16 * t + 4 * qd;
        if (n == 16 * NT) {
            *reinterpret_cast<float4*>(out + e) =
                make_float4(x[t][0] * f, x[t][1] * f, x[t][2] * f, x[t][3] * f);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (e + r < n) out[e + r] = x[t][r] * f;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------- prefill

// One wavefront per 16 query rows of one (batch, query head), 32 keys a step:
// the distant keys in d_down space against q~ = q W_up^T, the window's keys at
// full d, one running maximum and sum (Eq. 4), the latent part lifted once at
// the end. Arguments as prefill_valu_kernel. Grid: (ceil(n_rows / 16), B Hq),
// longest rows first.
template <int D, int DD>
__global__ __launch_bounds__(64) void prefill_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ wd, const float* __restrict__ wu, const float* __restrict__ cK,
    const float* __restrict__ cVt, float* __restrict__ o, float* __restrict__ lse, int Hq, int Hkv,
    int q0, int n_rows, int kv0, int Tkv, int d, int dd, int w, int Tp, float qscale,
    const float* __restrict__ wv, const int* __restrict__ seq_lens) {
    constexpr int NT = D / 16, CT = DD / 16;
    const int lane = lane_id_x(), qd = lane >> 4, c16 = lane & 15;
    const int row0 = ((n_rows + 15) / 16 - 1 - wg_id_x()) * 16;
    const int bh = wg_id_y();
    const int b = bh / Hq, h = bh - (bh / Hq) * Hq;
    const int g = h / (Hq / Hkv);
    const int bg = b * Hkv + g;
    const int total = q0 + n_rows;
    const int end = seq_lens ? imin(total, imax(seq_lens[b], 0)) : total;  // rows at or past it: none
    const int i_lo = q0 + row0;
    if (i_lo >= end) return;
    const int i_hi = imin(i_lo + 15, end - 1);
    const int i = i_lo + c16, ii = imin(i, i_hi);
    const float* wdg = wd + (size_t)g * d * dd;
    const float* wug = wu ? wu + (size_t)g * dd * d : nullptr;
    const float* wvg = wv ? wv + (size_t)g * dd * d : wug;  // value lift

    float qv[D / 4];
    load_row<D>(q + ((size_t)bh * n_rows + (ii - q0)) * d, qd, d, qscale, qv);
    float m = -INFINITY, l = 0.f;
    f32x4_t ow[NT], ol[CT];
#pragma unroll
    for (int t = 0; t < NT; ++t) ow[t] = zero4();
#pragma unroll
    for (int t = 0; t < CT; ++t) ol[t] = zero4();

    // the weights of one step's scores x[8], the maximum moved if needed
    auto weights = [&](const float (&x)[8], float (&p0)[4], float (&p1)[4]) {
        float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                         fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
        const float mn = fmaxf(m, col_max(mx));
        if (__builtin_amdgcn_ballot_w64(mn > m)) {
            const float corr = m == -INFINITY ? 0.f : exp2f(m - mn);
            l *= corr;
#pragma unroll
            for (int t = 0; t < NT; ++t) ow[t] *= corr;
#pragma unroll
            for (int t = 0; t < CT; ++t) ol[t] *= corr;
            m = mn;
        }
        const float ref = m == -INFINITY ? 0.f : m;  // no key of the row yet: every x is -inf
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p0[r] = exp2f(x[r] - ref);
            p1[r] = exp2f(x[4 + r] - ref);
            s += p0[r] + p1[r];
        }
        l += col_sum(s);
    };

    const int jd = i_hi - w;  // last distant key of any row here
    if (jd >= 0) {
        f32x4_t qt[CT];
        project<D, DD>(wdg, wug, d, dd, qd, c16, qv, qt);
        const float* ck = cK + (size_t)bg * Tp * dd;
        const float* cv = cVt + (size_t)bg * Tp * dd;
        const bool whole = dd == DD;
        for (int j0 = 0; j0 <= jd; j0 += 32) {
            float4 kk[2][CT], vv[2][CT];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float* kr = ck + (size_t)imin(j0 + 16 * s + c16, jd) * dd;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    kk[s][ct] = load4(kr, 16 * ct + 4 * qd, dd, whole);
                    // (32-token blocks [dd][32]: this lane's four keys of one column)
                    const int c = imin(16 * ct + c16, dd - 1);
                    vv[s][ct] = *reinterpret_cast<const float4*>(
                        cv + (size_t)j0 * dd + (size_t)c * 32 + 16 * s + 4 * qd);
                }
            }
            const bool edge = j0 + 31 > i_lo - w;  // some pair is not distant
            float x[8];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                f32x4_t sc = zero4();
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    sc = mma(kk[s][ct].x, qt[ct][0], sc);
                    sc = mma(kk[s][ct].y, qt[ct][1], sc);
                    sc = mma(kk[s][ct].z, qt[ct][2], sc);
                    sc = mma(kk[s][ct].w, qt[ct][3], sc);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    x[4 * s + r] = edge && j0 + 16 * s + 4 * qd + r > i - w ? -INFINITY : sc[r];
            }
            float p[2][4];
            weights(x, p[0], p[1]);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float a[4][CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const bool in = 16 * ct + c16 < dd;
                    a[0][ct] = in ? vv[s][ct].x : 0.f;
                    a[1][ct] = in ? vv[s][ct].y : 0.f;
                    a[2][ct] = in ? vv[s][ct].z : 0.f;
                    a[3][ct] = in ? vv[s][ct].w : 0.f;
                }
                add_product<CT>(ol, a, p[s], edge, qd, c16);
            }
        }
    }

    const float* kg = k + (size_t)bg * Tkv * d;  // row of position j: j - kv0
    const float* vg = v + (size_t)bg * Tkv * d;
    if (w > 0) {
        for (int j0 = imax(0, i_lo - w + 1); j0 <= i_hi; j0 += 32) {
            const bool edge = j0 + 31 > i_lo || j0 <= i_hi - w;
            float x[8], a[2][4][NT];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float kx[D / 4];
                load_row<D>(kg + (size_t)(imin(j0 + 16 * s + c16, i_hi) - kv0) * d, qd, d, 1.f, kx);
                load_cols<NT>(
                    a[s],
                    [&](int r) { return vg + (size_t)(imin(j0 + 16 * s + 4 * qd + r, i_hi) - kv0) * d; },
                    c16, d);
                f32x4_t sc = zero4();
#pragma unroll
                for (int e = 0; e < D / 4; ++e) sc = mma(kx[e], qv[e], sc);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = j0 + 16 * s + 4 * qd + r;
                    x[4 * s + r] = edge && (j > i || j <= i - w || j > i_hi) ? -INFINITY : sc[r];
                }
            }
            float p[2][4];
            weights(x, p[0], p[1]);
#pragma unroll
            for (int s = 0; s < 2; ++s) add_product<NT>(ow, a[s], p[s], edge, qd, c16);
        }
    }

    if (jd >= 0) lift<D, DD>(wdg, wvg, d, dd, qd, c16, ol, ow);
    if (i >= end) return;
    const size_t row = (size_t)bh * n_rows + (i - q0);
    if (lse && qd == 0) lse[row] = (m + log2f(l)) * kLn2F;
    store_row<NT>(o + row * d, ow, qd, d, 1.f / l);
}

// ---------------------------------------------------------------- backward

// c^K, c^V (Eq. 1) row-major [T][dd]. One wavefront per 16 tokens; grid
// (ceil(T / 16), B Hkv).
template <int D, int DD>
__global__ __launch_bounds__(64) void bwd_f32_latent_kernel(
    const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ wd,
    float* __restrict__ ck, float* __restrict__ cv, int Hkv, int T, int d, int dd) {
    const int lane = lane_id_x(), qd = lane >> 4, c16 = lane & 15;
    const int bg = wg_id_y();
    const int j = wg_id_x() * 16 + c16;
    const size_t tok = (size_t)bg * T + imin(j, T - 1);
    const float* wdg = wd + (size_t)(bg % Hkv) * d * dd;
    float x[D / 4], y[D / 4];
    load_row<D>(k + tok * d, qd, d, 1.f, x);
    load_row<D>(v + tok * d, qd, d, 1.f, y);
    f32x4_t cx[DD / 16], cy[DD / 16];
    project<D, DD>(wdg, nullptr, d, dd, qd, c16, x, cx);
    project<D, DD>(wdg, nullptr, d, dd, qd, c16, y, cy);
    if (j >= T) return;
    store_row<DD / 16>(ck + tok * dd, cx, qd, dd, 1.f);
    store_row<DD / 16>(cv + tok * dd, cy, qd, dd, 1.f);
}

// One wavefront per 16 query rows of one (batch, query head): q~, dO~ and
// delta (kept, and written for the key side), then P from the forward's
// log-sum-exp, dS = P (dP - delta) and dq^T += K^T dS^T (window),
// h^T += c^K^T dS^T, ol^T += c^V^T P^T (distant); dq = s (dq + h W_up).
// Grid: (ceil(T / 16), B Hq), longest rows first.
template <int D, int DD>
__global__ __launch_bounds__(64) void bwd_f32_rows_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ o, const float* __restrict__ dout, const float* __restrict__ wd,
    const float* __restrict__ wu, const float* __restrict__ ck, const float* __restrict__ cv,
    const float* __restrict__ lse, float* __restrict__ qt_out, float* __restrict__ dot_out,
    float* __restrict__ delta, float* __restrict__ hk, float* __restrict__ ol_out,
    float* __restrict__ dq, int Hq, int Hkv, int T, int d, int dd, int w, float scale) {
    constexpr int NT = D / 16, CT = DD / 16;
    const int lane = lane_id_x(), qd = lane >> 4, c16 = lane & 15;
    const int bh = wg_id_y();
    const int b = bh / Hq, h = bh % Hq, g = h / (Hq / Hkv);
    const int bg = b * Hkv + g;
    const int i_lo = ((T + 15) / 16 - 1 - wg_id_x()) * 16;
    const int i_hi = imin(i_lo + 15, T - 1);
    const int i = i_lo + c16, ii = imin(i, i_hi);
    const size_t row = (size_t)bh * T + ii;
    const float* wdg = wd + (size_t)g * d * dd;
    const float* wug = wu ? wu + (size_t)g * dd * d : nullptr;
    const float qscale = scale * kLog2eF;

    float qv[D / 4], dv[D / 4];
    load_row<D>(q + row * d, qd, d, 1.f, qv);
    load_row<D>(dout + row * d, qd, d, 1.f, dv);
    float dl = 0.f;
    {
        float ov[D / 4];
        load_row<D>(o + row * d, qd, d, 1.f, ov);
#pragma unroll
        for (int s = 0; s < D / 4; ++s) dl = __builtin_fmaf(dv[s], ov[s], dl);
        dl = col_sum(dl);
    }
    const float L2 = lse[row] * kLog2eF;
    f32x4_t qt[CT], dt[CT];
    project<D, DD>(wdg, wug, d, dd, qd, c16, qv, qt);
    project<D, DD>(wdg, wug, d, dd, qd, c16, dv, dt);
    if (i < T) {
        store_row<CT>(qt_out + row * dd, qt, qd, dd, 1.f);
        store_row<CT>(dot_out + row * dd, dt, qd, dd, 1.f);
        if (qd == 0) delta[row] = dl;
    }
    f32x4_t dqa[NT], ha[CT], oa[CT];
#pragma unroll
    for (int t = 0; t < NT; ++t) dqa[t] = zero4();
#pragma unroll
    for (int t = 0; t < CT; ++t) ha[t] = oa[t] = zero4();

    const int jd = i_hi - w;
    const bool whole = dd == DD;
    const float* ckg = ck + (size_t)bg * T * dd;
    const float* cvg = cv + (size_t)bg * T * dd;
#pragma unroll 2
    for (int j0 = 0; j0 <= jd; j0 += 16) {
        const float* kr = ckg + (size_t)imin(j0 + c16, jd) * dd;
        const float* vr = cvg + (size_t)imin(j0 + c16, jd) * dd;
        float4 kk[CT], vv[CT];
        float ka[4][CT], va[4][CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            kk[ct] = load4(kr, 16 * ct + 4 * qd, dd, whole);
            vv[ct] = load4(vr, 16 * ct + 4 * qd, dd, whole);
        }
        load_cols<CT>(ka, [&](int r) { return ckg + (size_t)imin(j0 + 4 * qd + r, jd) * dd; }, c16, dd);
        load_cols<CT>(va, [&](int r) { return cvg + (size_t)imin(j0 + 4 * qd + r, jd) * dd; }, c16, dd);
        f32x4_t sc = zero4(), dp = zero4();
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            sc = mma(kk[ct].x, qt[ct][0], sc); dp = mma(vv[ct].x, dt[ct][0], dp);
            sc = mma(kk[ct].y, qt[ct][1], sc); dp = mma(vv[ct].y, dt[ct][1], dp);
            sc = mma(kk[ct].z, qt[ct][2], sc); dp = mma(vv[ct].z, dt[ct][2], dp);
            sc = mma(kk[ct].w, qt[ct][3], sc); dp = mma(vv[ct].w, dt[ct][3], dp);
        }
        const bool edge = j0 + 15 > i_lo - w;
        float p[4], ds[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool out = edge && j0 + 4 * qd + r > i - w;
            p[r] = out ? 0.f : exp2f(__builtin_fmaf(sc[r], qscale, -L2));
            ds[r] = out ? 0.f : p[r] * (dp[r] - dl);
        }
        add_product<CT>(ha, ka, ds, edge, qd, c16);
        add_product<CT>(oa, va, p, edge, qd, c16);
    }
    if (w > 0) {
        const float* kg = k + (size_t)bg * T * d;
        const float* vg = v + (size_t)bg * T * d;
        for (int j0 = imax(0, i_lo - w + 1); j0 <= i_hi; j0 += 16) {
            const size_t jr = (size_t)imin(j0 + c16, i_hi) * d;
            float kx[D / 4], vx[D / 4], ka[4][NT];
            load_row<D>(kg + jr, qd, d, 1.f, kx);
            load_row<D>(vg + jr, qd, d, 1.f, vx);
            load_cols<NT>(ka, [&](int r) { return kg + (size_t)imin(j0 + 4 * qd + r, i_hi) * d; }, c16, d);
            f32x4_t sc = zero4(), dp = zero4();
#pragma unroll
            for (int e = 0; e < D / 4; ++e) {
                sc = mma(kx[e], qv[e], sc);
                dp = mma(vx[e], dv[e], dp);
            }
            const bool edge = j0 + 15 > i_lo || j0 <= i_hi - w;
            float ds[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = j0 + 4 * qd + r;
                const bool out = edge && (j > i || j <= i - w || j > i_hi);
                ds[r] = out ? 0.f : exp2f(__builtin_fmaf(sc[r], qscale, -L2)) * (dp[r] - dl);
            }
            add_product<NT>(dqa, ka, ds, edge, qd, c16);
        }
    }
    if (jd >= 0) lift<D, DD>(wdg, wug, d, dd, qd, c16, ha, dqa);
    if (i >= T) return;
    store_row<CT>(hk + row * dd, ha, qd, dd, 1.f);
    store_row<CT>(ol_out + row * dd, oa, qd, dd, 1.f);
    store_row<NT>(dq + row * d, dqa, qd, d, scale);
}

// One wavefront per 16 keys of one (batch, KV head), the rows of every query
// head of the group that see them, S = Q K^T so that P and dS are the B
// operands of dV^T += dO^T P, dK^T += Q^T dS (window rows), gV^T += dO~^T P,
// gK^T += q~^T dS (distant rows); dk = s (dk + gK W_down^T), dv = dv + gV
// W_down^T. Grid: (ceil(T / 16), B Hkv), first keys (most rows) first.
template <int D, int DD>
__global__ __launch_bounds__(64) void bwd_f32_cols_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ dout, const float* __restrict__ wd, const float* __restrict__ ck,
    const float* __restrict__ cv, const float* __restrict__ qt, const float* __restrict__ dot,
    const float* __restrict__ delta, const float* __restrict__ lse, float* __restrict__ gk,
    float* __restrict__ gv, float* __restrict__ dk, float* __restrict__ dv, int Hq, int Hkv, int T,
    int d, int dd, int w, float scale) {
    constexpr int NT = D / 16, CT = DD / 16;
    const int lane = lane_id_x(), qd = lane >> 4, c16 = lane & 15;
    const int bg = wg_id_y();
    const int b = bg / Hkv, g = bg % Hkv, G = Hq / Hkv;
    const int j_lo = wg_id_x() * 16, j = j_lo + c16;
    const int j_hi = imin(j_lo + 15, T - 1);
    const size_t tok = (size_t)bg * T + imin(j, T - 1);
    const float qscale = scale * kLog2eF;
    f32x4_t dka[NT], dva[NT], gka[CT], gva[CT];
#pragma unroll
    for (int t = 0; t < NT; ++t) dka[t] = dva[t] = zero4();
#pragma unroll
    for (int t = 0; t < CT; ++t) gka[t] = gva[t] = zero4();
    float kx[D / 4], vx[D / 4];
    load_row<D>(k + tok * d, qd, d, 1.f, kx);
    load_row<D>(v + tok * d, qd, d, 1.f, vx);
    const bool whole = dd == DD;
    float4 ckx[CT], cvx[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        ckx[ct] = load4(ck + tok * dd, 16 * ct + 4 * qd, dd, whole);
        cvx[ct] = load4(cv + tok * dd, 16 * ct + 4 * qd, dd, whole);
    }
    for (int hh = 0; hh < G; ++hh) {
        const size_t r0 = ((size_t)b * Hq + g * G + hh) * T;
        const float* qh = q + r0 * d;
        const float* dh = dout + r0 * d;
        // P and dS of the rows i0 + 4 qd + r against this lane's key
        auto weights = [&](const f32x4_t& sc, const f32x4_t& dp, int i0, bool edge, bool far,
                           float (&p)[4], float (&ds)[4]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + 4 * qd + r;
                const size_t ic = r0 + imin(i, T - 1);
                const float L2 = lse[ic] * kLog2eF, dl = delta[ic];
                const bool out = edge && (i >= T || (far ? i - j < w : (i < j || i - j >= w)));
                p[r] = out ? 0.f : exp2f(__builtin_fmaf(sc[r], qscale, -L2));
                ds[r] = out ? 0.f : p[r] * (dp[r] - dl);
            }
        };
        if (w > 0) {
            const int last = imin(T - 1, j_hi + imin(w, T) - 1);
            for (int i0 = j_lo; i0 <= last; i0 += 16) {
                const size_t ir = (size_t)imin(i0 + c16, T - 1) * d;
                float qx[D / 4], dx[D / 4], qa[4][NT], da[4][NT];
                load_row<D>(qh + ir, qd, d, 1.f, qx);
                load_row<D>(dh + ir, qd, d, 1.f, dx);
                load_cols<NT>(qa, [&](int r) { return qh + (size_t)imin(i0 + 4 * qd + r, T - 1) * d; }, c16, d);
                load_cols<NT>(da, [&](int r) { return dh + (size_t)imin(i0 + 4 * qd + r, T - 1) * d; }, c16, d);
                f32x4_t sc = zero4(), dp = zero4();
#pragma unroll
                for (int e = 0; e < D / 4; ++e) {
                    sc = mma(qx[e], kx[e], sc);
                    dp = mma(dx[e], vx[e], dp);
                }
                const bool edge = i0 < j_hi || i0 + 15 - j_lo >= w || i0 + 15 >= T;
                float p[4], ds[4];
                weights(sc, dp, i0, edge, false, p, ds);
                add_product<NT>(dka, qa, ds, edge, qd, c16);
                add_product<NT>(dva, da, p, edge, qd, c16);
            }
        }
        const float* qth = qt + r0 * dd;
        const float* dth = dot + r0 * dd;
        if (j_lo < T - w)  // (w may exceed T)
#pragma unroll 2
            for (int i0 = j_lo + w; i0 < T; i0 += 16) {
                const size_t ir = (size_t)imin(i0 + c16, T - 1) * dd;
                float4 qx[CT], dx[CT];
                float qa[4][CT], da[4][CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    qx[ct] = load4(qth + ir, 16 * ct + 4 * qd, dd, whole);
                    dx[ct] = load4(dth + ir, 16 * ct + 4 * qd, dd, whole);
                }
                load_cols<CT>(qa, [&](int r) { return qth + (size_t)imin(i0 + 4 * qd + r, T - 1) * dd; }, c16, dd);
                load_cols<CT>(da, [&](int r) { return dth + (size_t)imin(i0 + 4 * qd + r, T - 1) * dd; }, c16, dd);
                f32x4_t sc = zero4(), dp = zero4();
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    sc = mma(qx[ct].x, ckx[ct].x, sc); dp = mma(dx[ct].x, cvx[ct].x, dp);
                    sc = mma(qx[ct].y, ckx[ct].y, sc); dp = mma(dx[ct].y, cvx[ct].y, dp);
                    sc = mma(qx[ct].z, ckx[ct].z, sc); dp = mma(dx[ct].z, cvx[ct].z, dp);
                    sc = mma(qx[ct].w, ckx[ct].w, sc); dp = mma(dx[ct].w, cvx[ct].w, dp);
                }
                const bool edge = i0 < j_hi + w || i0 + 15 >= T;
                float p[4], ds[4];
                weights(sc, dp, i0, edge, true, p, ds);
                add_product<CT>(gka, qa, ds, edge, qd, c16);
                add_product<CT>(gva, da, p, edge, qd, c16);
            }
    }
    if (j_lo < T - w) {  // dk^T[e] += W_down[e][c] gK^T[c]: the lift with W_down^T
        const float* wdg = wd + (size_t)g * d * dd;
        lift<D, DD>(wdg, nullptr, d, dd, qd, c16, gka, dka);
        lift<D, DD>(wdg, nullptr, d, dd, qd, c16, gva, dva);
    }
    if (j >= T) return;
    store_row<CT>(gk + tok * dd, gka, qd, dd, 1.f);
    store_row<CT>(gv + tok * dd, gva, qd, dd, 1.f);
    store_row<NT>(dk + tok * d, dka, qd, d, scale);
    store_row<NT>(dv + tok * d, dva, qd, d, 1.f);
}

// Weight-gradient share of one chunk of rows, stored [e][c], as
// bwd_wpart_kernel: z = 0 sum k_e (s gK_c) + v_e gV_c over the tokens of KV
// head g, z = 1 sum q_e (s h_c) + dO_e ol_c over its group's query rows; the
// rows are the products' k, four at a step. One workgroup per (chunk, KV head,
// z, 16 columns), its eight wavefronts an eighth of the rows each (a chunk is
// 256 rows or more: with one wavefront a chunk, 64 dependent steps), added in
// order in LDS. Grid (nchunk, Hkv, 2 * DD / 16).
constexpr int kPartWaves = 8;
template <int D, int DD>
__global__ __launch_bounds__(64 * kPartWaves) void bwd_f32_wpart_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ dout, const float* __restrict__ gk, const float* __restrict__ gv,
    const float* __restrict__ hk, const float* __restrict__ ol, float* __restrict__ part, int B,
    int Hq, int Hkv, int T, int d, int dd, int nchunk_d, int nchunk_u, int nchunk, float scale) {
    constexpr int NT = D / 16;
    __shared__ f32x4_t sum[NT][64];
    const int tid = lane_id_x(), lane = tid & 63, qd = lane >> 4, c16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = wg_id_x(), g = wg_id_y();
    const int z = wg_id_z() & 1, ct = wg_id_z() >> 1;
    const int nch = z == 0 ? nchunk_d : nchunk_u;
    if (chunk >= nch || 16 * ct >= dd) return;  // workgroup-uniform
    const int H = z == 0 ? Hkv : Hq, n = z == 0 ? 1 : Hq / Hkv;  // heads of an array, of the group
    const float *x1 = z == 0 ? k : q, *x2 = z == 0 ? v : dout;
    const float *y1 = z == 0 ? gk : hk, *y2 = z == 0 ? gv : ol;
    const long long rows = (long long)B * n * T;
    const long long per = (rows + nch - 1) / nch;
    const long long end = (chunk + 1) * per < rows ? (chunk + 1) * per : rows;
    const long long wper = (per + 4 * kPartWaves - 1) / (4 * kPartWaves) * 4;
    const long long r0 = (long long)chunk * per + wave * wper;
    const long long r1 = r0 + wper < end ? r0 + wper : end;
    const int c = 16 * ct + c16;
    f32x4_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = zero4();
    // this lane's row: token i of sequence-and-head bh = b * n + head of the group
    int bh = (int)(r0 / T), i = (int)(r0 - (long long)bh * T) + qd;
#pragma unroll 2
    for (long long r = r0; r < r1; r += 4) {
        while (i >= T) {
            i -= T;
            ++bh;
        }
        const bool in = r + qd < r1;
        const size_t row = in ? ((size_t)(bh / n) * H + g * n + bh % n) * T + i : 0;
        i += 4;
        const int dd_r = in ? dd : 0, d_r = in ? d : 0;  // a row past the chunk reads as zeros
        const float b1 = y1[row * dd + imin(c, dd - 1)] * scale, b2 = y2[row * dd + imin(c, dd - 1)];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int e = 16 * t + c16;
            const float a1 = x1[row * d + imin(e, d - 1)], a2 = x2[row * d + imin(e, d - 1)];
            acc[t] = mma(e < d_r ? a1 : 0.f, c < dd_r ? b1 : 0.f, acc[t]);
            acc[t] = mma(e < d_r ? a2 : 0.f, c < dd_r ? b2 : 0.f, acc[t]);
        }
    }
    for (int wv = 0; wv < kPartWaves; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int t = 0; t < NT; ++t) sum[t][lane] = wv == 0 ? acc[t] : sum[t][lane] + acc[t];
        }
        __syncthreads();
    }
    float* out = part + (((size_t)z * Hkv + g) * nchunk + chunk) * (size_t)d * dd;
    if (wave != 0 || c >= dd) return;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = 16 * t + 4 * qd + r;
            if (e < d) out[(size_t)e * dd + c] = sum[t][lane][r];
        }
}

// ---------------------------------------------------------------- host

// The register budget: d up to 64 with any d_down, up to 128 with d_down up to
// 32 (the key side then holds 256 accumulators and operands of its own); the
// rest takes the vector-ALU kernels.
bool f32_mfma_supported(int d, int dd) { return d <= 64 ? dd <= d : d <= 128 && dd <= 32; }

// the instance for (d, dd): rows padded to 64 or 128, latents to 16, 32 or 64
#define DAR_F32_DISPATCH(CALL)                   \
    do {                                         \
        if (d <= 64) {                           \
            if (dd <= 16) { CALL(64, 16); }      \
            else if (dd <= 32) { CALL(64, 32); } \
            else { CALL(64, 64); }               \
        } else {                                 \
            CALL(128, 32);                       \
        }                                        \
    } while (0)

hipError_t launch_prefill_f32(const float* q, const float* k, const float* v, const float* wd,
                              const float* wu, const float* cK, const float* cVt, float* o,
                              float* lse, int B, int Hq, int Hkv, const PrefillGeo& geo, int d,
                              int dd, int w, hipStream_t st, const float* wv) {
    const int Tp = prefill_tp(geo.total(), w);
    const float qscale = kLog2eF / sqrtf((float)d);
    const dim3 grid((geo.n_rows + 15) / 16, B * Hq);
#define DAR_F32_CALL(D_, DD_)                                                                       \
    hipLaunchKernelGGL((prefill_f32_kernel<D_, DD_>), grid, dim3(64), 0, st, q, k, v, wd, wu, cK,  \
                       cVt, o, lse, Hq, Hkv, geo.q0, geo.n_rows, geo.kv0, geo.Tkv, d, dd, w, Tp,   \
                       qscale, wv, geo.seq_lens)
    DAR_F32_DISPATCH(DAR_F32_CALL);
#undef DAR_F32_CALL
    return hipGetLastError();
}

hipError_t launch_bwd_f32(const float* q, const float* k, const float* v, const float* o,
                          const float* lse, const float* dout, const float* wd, const float* wu,
                          float* dq, float* dk, float* dv, float* dwd, float* dwu, char* ws,
                          const BwdWs& L, int B, int Hq, int Hkv, int T, int d, int dd, int w,
                          hipStream_t st) {
    float* delta = (float*)(ws + L.delta_off);
    float* qt = (float*)(ws + L.qt_off);
    float* dot = (float*)(ws + L.dot_off);
    float* hk = (float*)(ws + L.hk_off);
    float* ol = (float*)(ws + L.ol_off);
    float* ck = (float*)(ws + L.ck_off);
    float* cv = (float*)(ws + L.cv_off);
    float* gk = (float*)(ws + L.gk_off);
    float* gv = (float*)(ws + L.gv_off);
    float* part = (float*)(ws + L.wpart_off);
    const float scale = 1.f / sqrtf((float)d);
    const int nb = (T + 15) / 16;
#define DAR_F32_CALL(D_, DD_)                                                                        \
    hipLaunchKernelGGL((bwd_f32_latent_kernel<D_, DD_>), dim3(nb, B * Hkv), dim3(64), 0, st, k, v,  \
                       wd, ck, cv, Hkv, T, d, dd);                                                  \
    hipLaunchKernelGGL((bwd_f32_rows_kernel<D_, DD_>), dim3(nb, B * Hq), dim3(64), 0, st, q, k, v,  \
                       o, dout, wd, wu, (const float*)ck, (const float*)cv, lse, qt, dot, delta,    \
                       hk, ol, dq, Hq, Hkv, T, d, dd, w, scale);                                    \
    hipLaunchKernelGGL((bwd_f32_cols_kernel<D_, DD_>), dim3(nb, B * Hkv), dim3(64), 0, st, q, k, v, \
                       dout, wd, (const float*)ck, (const float*)cv, (const float*)qt,              \
                       (const float*)dot, (const float*)delta, lse, gk, gv, dk, dv, Hq, Hkv, T, d,  \
                       dd, w, scale);                                                               \
    hipLaunchKernelGGL((bwd_f32_wpart_kernel<D_, DD_>), dim3(L.nchunk, Hkv, 2 * (DD_ / 16)),        \
                       dim3(64 * kPartWaves), 0, st, q, k, v, dout, (const float*)gk, (const float*)gv,          \
                       (const float*)hk, (const float*)ol, part, B, Hq, Hkv, T, d, dd, L.nchunk_d,  \
                       L.nchunk_u, L.nchunk, scale)
    DAR_F32_DISPATCH(DAR_F32_CALL);
#undef DAR_F32_CALL
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_bwd_wreduce(part, dwd, dwu, Hkv, d, dd, L, st);
}

}  // namespace dar
