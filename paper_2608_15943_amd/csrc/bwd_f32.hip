// Attention of fp32 models over whole sequences (the small configurations), forward and
// backward: plain fp32 on the vector ALUs, the same data flow as the bf16 path.  With
// S = Q K^T / sqrt(d) (masked), P = softmax(S), O = P V (Sec. 2.2, Eq. 2): dV = P^T dO,
// dP = dO V^T, dS = P * (dP - D), D = rowsum(dO * O), dQ = dS K / sqrt(d),
// dK = dS^T Q / sqrt(d); dQ and dK are rotated back through RoPE (orthogonal per position); a
// consumer's dK, dV add into its producer's fp32 sums (Eq. 3).
//
// A workgroup owns 16 queries of one head (forward, dQ) or 16 keys of one KV head (dK, dV);
// its four waves take every fourth tile of the other axis (attn_f32.h).  Measured on the
// four-layer stack (128 tokens, 4 heads of 64), per layer, against one thread per row with
// rows read from global memory: dK/dV 1150 -> 19 us, dQ and the row statistics 719 -> 21 us;
// the forward 22 -> 14 us against one wave per (token, head).  Unrolling the row loops or
// masking by selects instead of branches made all three slower (14 -> 17, 21 -> 26, 19 -> 27
// us): a kernel this short also pays for the instructions it fetches.  Short sequences take
// the forward by rows (attn_seq_f32).
//
// A key or query outside the causal mask is never multiplied into a sum, so a value that is
// not finite reaches only the rows that see it.
#include <math.h>

#include "attn_f32.h"
#include "kernels.h"

namespace kvp {
namespace {

// Running softmax of the lane's row over a tile's scaled scores (-inf where hidden): returns
// the factor of what was summed before.
__device__ __forceinline__ float softmax_step(float (&s)[4], float& m, float& l) {
    const float mt = quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
    const float mn = fmaxf(m, mt);
    // A row that has seen no key yet (rows past the end) keeps its empty sum.
    const float a = mn == -INFINITY ? 1.f : expf(m - mn);
    float t = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        // By the score, not by the maximum, which passes over NaN: a NaN score stays one.
        s[e] = s[e] == -INFINITY ? 0.f : expf(s[e] - mn);
        t += s[e];
    }
    l = l * a + quad_sum(t);
    m = mn;
    return a;
}

template <int D>
__global__ __launch_bounds__(256) void attn_tile_f32_kernel(const float* __restrict__ q, const float* __restrict__ kc,
                                                            const float* __restrict__ vc, float* __restrict__ o, int B,
                                                            int S, int a, int g, int cap) {
    constexpr int P = F32Tile<D>::P, N4 = D / 16;
    __shared__ F32Tile<D> qs, ks[4], vs[4];
    __shared__ float ps[4][FT][FT + 1], ml[4][2][FT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane >> 2, c = lane & 3;
    const int nqt = (S + FT - 1) / FT;
    const int qt = nqt - 1 - blockIdx.x / (B * a), bh = blockIdx.x % (B * a);   // longest rows first
    const int b = bh / a, h = bh - b * a, kvh = h / (a / g);
    const int q0 = qt * FT;
    const float scale = 1.0f / sqrtf((float)D);
    const float* kb = kc + ((size_t)b * g + kvh) * cap * D;
    const float* vb = vc + ((size_t)b * g + kvh) * D * cap;
    {
        RowLoad<D, 256> x;
        x.load(q + ((size_t)(b * S + q0) * a + h) * D, (size_t)a * D, min(S - q0, FT), tid);
        x.store(qs, tid);
    }
    __syncthreads();
    f32x4 acc[N4];
#pragma unroll
    for (int i = 0; i < N4; ++i) acc[i] = f32x4{};
    float m = -INFINITY, l = 0.f;
    RowLoad<D, 64> kl;
    ColLoad<D, 64> vl;
    auto fetch = [&](int t) {
        kl.load(kb + (size_t)t * FT * D, D, min(S - t * FT, FT), lane);
        vl.load(vb + t * FT, cap, min(S - t * FT, FT), lane);
    };
    if (wave <= qt) fetch(wave);
    for (int t = wave; t <= qt; t += 4) {
        wave_sync();
        kl.store(ks[wave], lane);
        vl.store(vs[wave], lane);
        if (t + 4 <= qt) fetch(t + 4);
        wave_sync();
        float s[4];
        dot_tile<D>(qs, ks[wave], r, c, s);
        const int lim = min(q0 + r, S - 1) - t * FT;      // last visible key of the row in the tile
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = 4 * c + e <= lim ? s[e] * scale : -INFINITY;
        const float f = softmax_step(s, m, l);
#pragma unroll
        for (int i = 0; i < N4; ++i) acc[i] *= f;
#pragma unroll
        for (int e = 0; e < 4; ++e) ps[wave][r][4 * c + e] = s[e];
        wave_sync();
        for (int j = 0; j < FT; ++j)
            if (j <= lim) add_row<D>(acc, vs[wave], j, c, ps[wave][r][j]);
    }
    // Merge the waves: weights exp(m_w - M), in wave order.
    wave_sync();
#pragma unroll
    for (int i = 0; i < N4; ++i) *(f32x4*)&ks[wave].v[r * P + 16 * i + 4 * c] = acc[i];
    if (c == 0) {
        ml[wave][0][r] = m;
        ml[wave][1][r] = l;
    }
    __syncthreads();
    for (int id = tid; id < FT * D; id += 256) {
        const int row = id / D, d = id % D;
        if (q0 + row >= S) continue;
        const float M = fmaxf(fmaxf(ml[0][0][row], ml[1][0][row]), fmaxf(ml[2][0][row], ml[3][0][row]));
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float wt = expf(ml[w][0][row] - M);
            num = fmaf(wt, ks[w].v[row * P + d], num);
            den = fmaf(wt, ml[w][1][row], den);
        }
        o[((size_t)(b * S + q0 + row) * a + h) * D + d] = num / den;
    }
}

// Rotates the pair (x1, x2) = (dim i, dim i + D/2) back by the position's angle.
__device__ __forceinline__ void rope_back(float2 cs, float& x1, float& x2) {
    const float y1 = x1 * cs.x + x2 * cs.y, y2 = x2 * cs.x - x1 * cs.y;
    x1 = y1;
    x2 = y2;
}

// dQ, and on the way the row statistics that dK, dV need: the log-sum-exp of the scaled
// scores (a first sweep over the keys) and D.
template <int D>
__global__ __launch_bounds__(256) void dq_f32_kernel(AttnBwdF32 A) {
    constexpr int P = F32Tile<D>::P, N4 = D / 16, HALF = D / 2;
    __shared__ F32Tile<D> qs, ds, ks[4], vs[4];
    __shared__ float ps[4][FT][FT + 1], ml[4][2][FT], lse_s[FT], dsum_s[FT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane >> 2, c = lane & 3;
    const int S = A.S, a = A.a, nqt = (S + FT - 1) / FT;
    const int qt = nqt - 1 - blockIdx.x / (A.B * a), bh = blockIdx.x % (A.B * a);
    const int b = bh / a, h = bh - b * a, kvh = h / (a / A.g);
    const int q0 = qt * FT, nq = min(S - q0, FT);
    const float scale = 1.0f / sqrtf((float)D);
    const float* kb = A.kc + ((size_t)b * A.g + kvh) * A.cap * D;
    const float* vb = A.vc + ((size_t)b * A.g + kvh) * D * A.cap;
    const size_t row0 = ((size_t)(b * S + q0) * a + h) * D;
    {
        RowLoad<D, 256> x, y;
        x.load(A.q + row0, (size_t)a * D, nq, tid);
        y.load(A.dO + row0, (size_t)a * D, nq, tid);
        x.store(qs, tid);
        y.store(ds, tid);
    }
    __syncthreads();
    {
        const int row = tid >> 4, sub = tid & 15;
        float t = 0.f;
        if (row < nq)
            for (int d = sub; d < D; d += 16) t = fmaf(ds.v[row * P + d], A.O[row0 + (size_t)row * a * D + d], t);
#pragma unroll
        for (int k = 8; k >= 1; k >>= 1) t += __shfl_xor(t, k);
        if (sub == 0) dsum_s[row] = t;
    }
    const int lim0 = min(q0 + r, S - 1);
    auto visible = [&](int t) { return lim0 - t * FT; };   // last visible key of the row in tile t
    float m = -INFINITY, l = 0.f;
    RowLoad<D, 64> kl;
    ColLoad<D, 64> vl;
    auto fetch_k = [&](int t) { kl.load(kb + (size_t)t * FT * D, D, min(S - t * FT, FT), lane); };
    auto fetch_v = [&](int t) { vl.load(vb + t * FT, A.cap, min(S - t * FT, FT), lane); };
    if (wave <= qt) fetch_k(wave);
    for (int t = wave; t <= qt; t += 4) {
        wave_sync();
        kl.store(ks[wave], lane);
        if (t + 4 <= qt) fetch_k(t + 4);
        wave_sync();
        float s[4];
        dot_tile<D>(qs, ks[wave], r, c, s);
        const int lim = visible(t);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = 4 * c + e <= lim ? s[e] * scale : -INFINITY;
        softmax_step(s, m, l);
    }
    if (wave <= qt) {
        fetch_k(wave);
        fetch_v(wave);
    }
    if (c == 0) {
        ml[wave][0][r] = m;
        ml[wave][1][r] = l;
    }
    __syncthreads();
    if (tid < FT) {
        const float M = fmaxf(fmaxf(ml[0][0][tid], ml[1][0][tid]), fmaxf(ml[2][0][tid], ml[3][0][tid]));
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) den = fmaf(expf(ml[w][0][tid] - M), ml[w][1][tid], den);
        const float lse = M + logf(den);
        lse_s[tid] = lse;
        if (tid < nq) {
            const size_t i = (size_t)(b * S + q0 + tid) * a + h;
            A.lse[i] = lse;
            A.dsum[i] = dsum_s[tid];
        }
    }
    __syncthreads();
    const float lse = lse_s[r], dd = dsum_s[r];
    f32x4 acc[N4];
#pragma unroll
    for (int i = 0; i < N4; ++i) acc[i] = f32x4{};
    for (int t = wave; t <= qt; t += 4) {
        wave_sync();
        kl.store(ks[wave], lane);
        vl.store(vs[wave], lane);
        if (t + 4 <= qt) {
            fetch_k(t + 4);
            fetch_v(t + 4);
        }
        wave_sync();
        float s[4], dp[4];
        dot_tile<D>(qs, ks[wave], r, c, s);
        dot_tile<D>(ds, vs[wave], r, c, dp);
        const int lim = visible(t);
#pragma unroll
        for (int e = 0; e < 4; ++e) ps[wave][r][4 * c + e] = expf(s[e] * scale - lse) * (dp[e] - dd);
        wave_sync();
        for (int j = 0; j < FT; ++j)
            if (j <= lim) add_row<D>(acc, ks[wave], j, c, ps[wave][r][j]);
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < N4; ++i) *(f32x4*)&ks[wave].v[r * P + 16 * i + 4 * c] = acc[i];
    __syncthreads();
    for (int id = tid; id < FT * HALF; id += 256) {
        const int row = id / HALF, i = id % HALF;
        if (row >= nq) continue;
        float x1 = 0.f, x2 = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            x1 += ks[w].v[row * P + i];
            x2 += ks[w].v[row * P + i + HALF];
        }
        x1 *= scale;
        x2 *= scale;
        rope_back(A.rope[(size_t)(q0 + row) * HALF + i], x1, x2);
        float* dst = A.out_q + (size_t)(b * S + q0 + row) * A.ldo + h * D;
        dst[i] = x1;
        dst[i + HALF] = x2;
    }
}

// dK, dV of 16 keys: the sum over the r query heads and the query tiles at or after them.
template <int D>
__global__ __launch_bounds__(256) void dkv_f32_kernel(AttnBwdF32 A) {
    constexpr int P = F32Tile<D>::P, N4 = D / 16, HALF = D / 2;
    __shared__ F32Tile<D> ks, vs, qs[4], ds[4];
    __shared__ float ps[4][FT][FT + 1], dss[4][FT][FT + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane >> 2, c = lane & 3;
    const int S = A.S, a = A.a, g = A.g, rep = a / g, nqt = (S + FT - 1) / FT;
    const int kt = blockIdx.x / (A.B * g), bk = blockIdx.x % (A.B * g);   // most query tiles first
    const int b = bk / g, kvh = bk - b * g;
    const int k0 = kt * FT, nk = min(S - k0, FT);
    const float scale = 1.0f / sqrtf((float)D);
    {
        RowLoad<D, 256> x;
        ColLoad<D, 256> y;
        x.load(A.kc + (((size_t)b * g + kvh) * A.cap + k0) * D, D, nk, tid);
        y.load(A.vc + ((size_t)b * g + kvh) * D * A.cap + k0, A.cap, nk, tid);
        x.store(ks, tid);
        y.store(vs, tid);
    }
    __syncthreads();
    f32x4 dk[N4], dv[N4];
#pragma unroll
    for (int i = 0; i < N4; ++i) dk[i] = dv[i] = f32x4{};
    const int per = nqt - kt, n = rep * per;      // query tiles per head, all
    RowLoad<D, 64> ql, dl;
    float lse_n = 0.f, dd_n = 0.f;                // of the lane's row, next tile
    auto fetch = [&](int it) {
        const int h = kvh * rep + it / per, q0 = (kt + it % per) * FT, nq = min(S - q0, FT);
        const size_t row0 = ((size_t)(b * S + q0) * a + h) * D;
        ql.load(A.q + row0, (size_t)a * D, nq, lane);
        dl.load(A.dO + row0, (size_t)a * D, nq, lane);
        const size_t i = (size_t)(b * S + q0 + min(r, nq - 1)) * a + h;
        lse_n = A.lse[i];
        dd_n = A.dsum[i];
    };
    if (wave < n) fetch(wave);
    for (int it = wave; it < n; it += 4) {
        const int q0 = (kt + it % per) * FT, nq = min(S - q0, FT);
        const float lse = lse_n, dd = dd_n;
        wave_sync();
        ql.store(qs[wave], lane);
        dl.store(ds[wave], lane);
        if (it + 4 < n) fetch(it + 4);
        wave_sync();
        float s[4], dp[4];
        dot_tile<D>(qs[wave], ks, r, c, s);
        dot_tile<D>(ds[wave], vs, r, c, dp);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p = expf(s[e] * scale - lse);
            ps[wave][r][4 * c + e] = p;
            dss[wave][r][4 * c + e] = p * (dp[e] - dd);
        }
        wave_sync();
        // The lane's key is k0 + r: queries q0 + j >= it, below S.
        for (int j = 0; j < nq; ++j)
            if (q0 + j >= k0 + r) {
                add_row<D>(dv, ds[wave], j, c, ps[wave][j][r]);
                add_row<D>(dk, qs[wave], j, c, dss[wave][j][r]);
            }
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < N4; ++i) {
        *(f32x4*)&qs[wave].v[r * P + 16 * i + 4 * c] = dk[i];
        *(f32x4*)&ds[wave].v[r * P + 16 * i + 4 * c] = dv[i];
    }
    __syncthreads();
    for (int id = tid; id < FT * HALF; id += 256) {
        const int row = id / HALF, i = id % HALF, key = k0 + row;
        if (row >= nk) continue;
        float yk[2] = {0.f, 0.f}, yv[2] = {0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                yk[z] += qs[w].v[row * P + i + z * HALF];
                yv[z] += ds[w].v[row * P + i + z * HALF];
            }
        yk[0] *= scale;
        yk[1] *= scale;
        rope_back(A.rope[(size_t)key * HALF + i], yk[0], yk[1]);
        const size_t ai = (((size_t)b * g + kvh) * S + key) * D;
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const int d = i + z * HALF;
            if (A.acc_in_k) {
                yk[z] += A.acc_in_k[ai + d];
                yv[z] += A.acc_in_v[ai + d];
            }
            if (A.acc_out_k) {
                A.acc_out_k[ai + d] = yk[z];
                A.acc_out_v[ai + d] = yv[z];
            }
            if (A.out_kv) {
                float* out = A.out_kv + (size_t)(b * S + key) * A.ldo + kvh * D;
                out[A.col_k + d] = yk[z];
                out[A.col_v + d] = yv[z];
            }
        }
    }
}

}  // namespace

hipError_t attn_seq_f32(const float* q, const float* kc, const float* vc, float* o, int B, int S, int a, int g, int d,
                        int cap, hipStream_t st) {
    // Short sequences: one wave per (token, head), as in decode, where the device has a SIMD for
    // each and the longest has few keys.  Prefill of four (8 heads, 8 and more sequences: two)
    // layers on tiles over that by rows: one head of 128, 4 x 5 tokens 96 us / 72 us = 1.34, 4 x
    // 32 1.17, 4 x 48 1.02; 8 heads of 128, 8 x 16 (1024 waves) 1.17, 16 x 16 0.98, 8 x 24 1.00,
    // 4 x 48 0.86; 4 heads of 64, 8 x 32 1.07, 16 x 24 0.97; 4 heads of 16, 1 x 16 1.02, 1 x 24
    // 0.98; 8 heads of 32, 8 x 16 1.05, 8 x 24 0.97.
    if (S <= (d >= 64 ? 32 : 16) && (int64_t)B * S * a <= 1024)
        return attn_rows_f32(q, kc, vc, o, B, S, a, g, d, cap, st);
    const dim3 grid((S + FT - 1) / FT * B * a), block(256);
    switch (d) {
        case 16: hipLaunchKernelGGL(attn_tile_f32_kernel<16>, grid, block, 0, st, q, kc, vc, o, B, S, a, g, cap); break;
        case 32: hipLaunchKernelGGL(attn_tile_f32_kernel<32>, grid, block, 0, st, q, kc, vc, o, B, S, a, g, cap); break;
        case 64: hipLaunchKernelGGL(attn_tile_f32_kernel<64>, grid, block, 0, st, q, kc, vc, o, B, S, a, g, cap); break;
        case 128: hipLaunchKernelGGL(attn_tile_f32_kernel<128>, grid, block, 0, st, q, kc, vc, o, B, S, a, g, cap); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t attn_bwd_f32(const AttnBwdF32& p, hipStream_t st) {
    const int nt = (p.S + FT - 1) / FT;
    const dim3 gq(nt * p.B * p.a), gk(nt * p.B * p.g), block(256);
#define KVP_BWD_F32(DD)                                                  \
    hipLaunchKernelGGL(dq_f32_kernel<DD>, gq, block, 0, st, p);          \
    hipLaunchKernelGGL(dkv_f32_kernel<DD>, gk, block, 0, st, p)
    switch (p.d) {
        case 16: KVP_BWD_F32(16); break;
        case 32: KVP_BWD_F32(32); break;
        case 64: KVP_BWD_F32(64); break;
        case 128: KVP_BWD_F32(128); break;
        default: return hipErrorInvalidValue;
    }
#undef KVP_BWD_F32
    return hipGetLastError();
}

}  // namespace kvp
