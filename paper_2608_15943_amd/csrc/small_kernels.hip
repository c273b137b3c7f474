// Smaller kernels of the path:
//   rope_table    -- cos/sin of pos * theta_i in double, stored as fp32 pairs.
//   rope_scatter  -- RoPE on fp32 projections, then Q to its buffer and K, V
//                    (transposed) into the producer's slot; used by decode
//                    (position len_b of each sequence) and by fp32 models.
//   gemm_f32 (_nn, _tn), attn_f32, attn_rows_f32 -- the full-precision path for fp32 models
//                    (vector ALU, no reduced-precision matrix modes).
#include <math.h>

#include "attn_f32.h"
#include "kernels.h"

namespace kvp {
namespace {

// ---------------------------------------------------------------------------
// RoPE
// ---------------------------------------------------------------------------

__global__ void rope_table_kernel(float2* t, int S, int half, int d, double base) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= S * half) return;
    const int pos = idx / half, i = idx - pos * half;
    const double theta = pow(base, -2.0 * i / d);
    double s, c;
    sincos((double)pos * theta, &s, &c);
    t[idx] = make_float2((float)c, (float)s);
}

template <typename T>
__device__ __forceinline__ void put(T* p, size_t i, float v);
template <>
__device__ __forceinline__ void put<float>(float* p, size_t i, float v) { p[i] = v; }
template <>
__device__ __forceinline__ void put<uint16_t>(uint16_t* p, size_t i, float v) { p[i] = f2bf(v); }

template <typename T>
__global__ __launch_bounds__(256) void rope_scatter_kernel(const float* __restrict__ proj, int nsplit,
                                                           size_t split_stride, int S,
                                                           const int32_t* __restrict__ lens, int a,
                                                           int g, int d, int cap, double base,
                                                           int producer, T* q, T* kc, T* vc) {
    __shared__ float2 cs[64];                 // (cos, sin) of this row's position, d / 2 <= 64
    const int r = blockIdx.x;
    int b, pos;
    if (lens) {
        b = r;
        pos = max(0, min(lens[r], cap - 1));   // never outside the slot
    } else {
        b = r / S;
        pos = r - b * S;
    }
    const int half = d / 2, nq = a * d, nkv = g * d;
    const int ncols = nq + (producer ? 2 * nkv : 0);
    const float* pr = proj + (size_t)r * ncols;
    // Sum of the K slices of the projection (one slice unless the GEMM split K).
    auto val = [&](int c) {
        float v = pr[c];
        for (int s = 1; s < nsplit; ++s) v += pr[(size_t)s * split_stride + c];
        return v;
    };
    for (int i = threadIdx.x; i < half; i += blockDim.x) {
        const double theta = pow(base, -2.0 * i / d);
        double sd, cd;
        sincos((double)pos * theta, &sd, &cd);
        cs[i] = make_float2((float)cd, (float)sd);
    }
    __syncthreads();
    const int heads = a + (producer ? g : 0);
    for (int j = threadIdx.x; j < heads * half; j += blockDim.x) {
        const int h = j / half, i = j - h * half;
        const float c = cs[i].x, s = cs[i].y;
        const float x1 = val(h * d + i), x2 = val(h * d + i + half);
        const float o1 = x1 * c - x2 * s, o2 = x2 * c + x1 * s;
        if (h < a) {
            put(q, (size_t)r * nq + h * d + i, o1);
            put(q, (size_t)r * nq + h * d + i + half, o2);
        } else {
            const size_t kb = (((size_t)b * g + (h - a)) * cap + pos) * d;
            put(kc, kb + i, o1);
            put(kc, kb + i + half, o2);
        }
    }
    if (producer) {
        for (int j = threadIdx.x; j < nkv; j += blockDim.x) {
            const int h = j / d, c = j - h * d;
            put(vc, (((size_t)b * g + h) * d + c) * cap + pos, val(nq + nkv + j));
        }
    }
}

// ---------------------------------------------------------------------------
// fp32 path
// ---------------------------------------------------------------------------

// fp32 products C[m][n] (+ res) = sum_k A(m, k) B(k, n).  AK / BK_: the operand is contiguous
// along k (else along m / n).  B may be stacked from three blocks (along n when contiguous
// along k, else along k) and C from three row blocks.  Row strides, and the extents along
// the contiguous axes, are multiples of 4 (widths of fp32 models are multiples of 16).
struct F32Dst {
    float* p[3];
    int rows[3];
};
__device__ __forceinline__ const float* f32_block(const WRows& B, int r, int& row) {   // stacked row r
    if (r < B.rows[0]) { row = r; return (const float*)B.p[0]; }
    r -= B.rows[0];
    if (r < B.rows[1]) { row = r; return (const float*)B.p[1]; }
    row = r - B.rows[1];
    return (const float*)B.p[2];
}
__device__ __forceinline__ float* f32_dst_row(const F32Dst& dst, int m, size_t ldc, size_t& off) {
    int i = 0;
    if (m >= dst.rows[0]) {
        m -= dst.rows[0];
        i = 1;
        if (m >= dst.rows[1]) {
            m -= dst.rows[1];
            i = 2;
        }
    }
    off = (size_t)m * ldc;
    return i == 0 ? dst.p[0] : i == 1 ? dst.p[1] : dst.p[2];
}

// Products with few tiles: latency, not arithmetic.  Each of the four waves multiplies a
// quarter of K for the whole 32 x 32 tile (4 x 4 elements a lane, K steps of 32 through its
// own LDS, no barrier between steps, the next step's values already requested), and the four
// partial tiles are added in wave order.  At 128 tokens x width 256, against the four waves
// sharing the tile and walking all of K together: 12.8 -> 6.4 us a product (the backward's
// products, one wave per 64 elements: 30.7 -> 4.6 to 6.6 us).
// KN: values of k a wave multiplies per step, 32, or 16 for K <= 64, so that all four waves
// have some (a bound taken from K in place of a constant made every product 2 to 4 % longer).
template <bool AK, bool BK_, int KN>
__global__ __launch_bounds__(256) void gemm_f32_split_kernel(const float* __restrict__ A, size_t lda, WRows B,
                                                             size_t ldb, int M, int N, int K, F32Dst dst, size_t ldc,
                                                             const float* res) {
    constexpr int TM = 32, KS = 32, LD = 36;   // LDS rows: 32 values, padded to spread 8 rows over the banks
    __shared__ float sh[4][2][32 * LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tx = lane & 7, ty = lane >> 3;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
    const int kw = (K + 4 * KN - 1) / (4 * KN) * KN, kb = wave * kw, ke = min(kb + kw, K);
    float* as = sh[wave][0];
    float* bs = sh[wave][1];
    f32x4 av[4], bv[4];
    // 32 x 32 values of an operand: row i of the tile (k-contiguous: m or n; else k), 4 values.
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = ty + 8 * i, c = 4 * tx;
            av[i] = f32x4{};
            bv[i] = f32x4{};
            if (AK ? (m0 + r < M && k0 + c < ke) : (k0 + r < ke && m0 + c < M))
                av[i] = *(const f32x4*)(AK ? A + (size_t)(m0 + r) * lda + k0 + c : A + (size_t)(k0 + r) * lda + m0 + c);
            if (BK_ ? (n0 + r < N && k0 + c < ke) : (k0 + r < ke && n0 + c < N)) {
                int row;
                const float* p = f32_block(B, BK_ ? n0 + r : k0 + r, row);
                bv[i] = *(const f32x4*)(p + (size_t)row * ldb + (BK_ ? k0 : n0) + c);
            }
        }
    };
    float acc[4][4] = {};
    if (kb < ke) load(kb);
    for (int k0 = kb; k0 < ke; k0 += KS) {
        wave_sync();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            *(f32x4*)&as[(ty + 8 * i) * LD + 4 * tx] = av[i];
            *(f32x4*)&bs[(ty + 8 * i) * LD + 4 * tx] = bv[i];
        }
        if (k0 + KS < ke) load(k0 + KS);
        wave_sync();
        // Rows ty + 8 i (k-contiguous) or 4 ty + i of the tile; columns likewise.
#pragma unroll 2
        for (int kk = 0; kk < KN; kk += 4) {
            f32x4 a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = *(const f32x4*)(AK ? &as[(ty + 8 * i) * LD + kk] : &as[(kk + i) * LD + 4 * ty]);
                b[i] = *(const f32x4*)(BK_ ? &bs[(tx + 8 * i) * LD + kk] : &bs[(kk + i) * LD + 4 * tx]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] = fmaf(AK ? a[i][k] : a[k][i], BK_ ? b[j][k] : b[k][j], acc[i][j]);
        }
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            as[(AK ? ty + 8 * i : 4 * ty + i) * LD + (BK_ ? tx + 8 * j : 4 * tx + j)] = acc[i][j];
    __syncthreads();
    const int r = tid >> 3, c = 4 * (tid & 7), m = m0 + r, n = n0 + c;
    if (m >= M || n >= N) return;
    f32x4 v = *(const f32x4*)&sh[0][0][r * LD + c];
#pragma unroll
    for (int w = 1; w < 4; ++w) v += *(const f32x4*)&sh[w][0][r * LD + c];
    size_t off;
    float* p = f32_dst_row(dst, m, ldc, off);
    off += n;
    if (res) v += *(const f32x4*)(res + off);
    *(f32x4*)(p + off) = v;
}

// Larger products: 64 x 64 tile, 4 x 4 elements per thread, k in order (one fmaf chain per
// element), 32-wide K steps through LDS with the next step's values already requested.
template <bool AK, bool BK_>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, size_t lda, WRows B, size_t ldb,
                                                       int M, int N, int K, F32Dst dst, size_t ldc,
                                                       const float* res) {
    constexpr int T = 4, TM = 16 * T, KS = 32, PER = TM * KS / 256;
    __shared__ float As[KS][TM + 4], Bs[KS][TM + 4];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
    float av[PER], bv[PER];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int id = tid + 256 * i;
            {
                const int kk = AK ? id % KS : id / TM, mm = AK ? id / KS : id % TM;
                const int m = m0 + mm, k = k0 + kk;
                av[i] = (m < M && k < K) ? (AK ? A[(size_t)m * lda + k] : A[(size_t)k * lda + m]) : 0.f;
            }
            {
                const int kk = BK_ ? id % KS : id / TM, nn = BK_ ? id / KS : id % TM;
                const int n = n0 + nn, k = k0 + kk;
                bv[i] = 0.f;
                if (n < N && k < K) {
                    int row;
                    const float* p = f32_block(B, BK_ ? n : k, row);
                    bv[i] = p[(size_t)row * ldb + (BK_ ? k : n)];
                }
            }
        }
    };
    float acc[T][T] = {};
    load(0);
    for (int k0 = 0; k0 < K; k0 += KS) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int id = tid + 256 * i;
            As[AK ? id % KS : id / TM][AK ? id / KS : id % TM] = av[i];
            Bs[BK_ ? id % KS : id / TM][BK_ ? id / KS : id % TM] = bv[i];
        }
        __syncthreads();
        if (k0 + KS < K) load(k0 + KS);
#pragma unroll 8
        for (int kk = 0; kk < KS; ++kk) {
            float a[T], b[T];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                a[i] = As[kk][ty * T + i];
                b[i] = Bs[kk][tx * T + i];
            }
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int m = m0 + ty * T + i;
        if (m >= M) continue;
        size_t row;
        float* c = f32_dst_row(dst, m, ldc, row);
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int n = n0 + tx * T + j;
            if (n >= N) continue;
            const size_t off = row + n;
            c[off] = res ? res[off] + acc[i][j] : acc[i][j];
        }
    }
}

template <bool AK, bool BK_>
hipError_t launch_f32(const float* a, size_t lda, const WRows& b, size_t ldb, int M, int N, int K, const F32Dst& dst,
                      size_t ldc, const float* res, hipStream_t st) {
    if (M < 1 || N < 1) return hipSuccess;
    // 64 x 64 tiles once they fill the 256 CUs.
    if ((int64_t)((M + 63) / 64) * ((N + 63) / 64) >= 256)
        hipLaunchKernelGGL((gemm_f32_kernel<AK, BK_>), dim3((N + 63) / 64, (M + 63) / 64), dim3(256), 0, st, a, lda, b,
                           ldb, M, N, K, dst, ldc, res);
    else if (K > 64)
        hipLaunchKernelGGL((gemm_f32_split_kernel<AK, BK_, 32>), dim3((N + 31) / 32, (M + 31) / 32), dim3(256), 0, st, a,
                           lda, b, ldb, M, N, K, dst, ldc, res);
    else
        hipLaunchKernelGGL((gemm_f32_split_kernel<AK, BK_, 16>), dim3((N + 31) / 32, (M + 31) / 32), dim3(256), 0, st, a,
                           lda, b, ldb, M, N, K, dst, ldc, res);
    return hipGetLastError();
}

// One wave per (row, query head): the keys [0, pos] go through in chunks of 64, lane j
// scoring key t0 + j (a D-long dot product from its K row); the chunk's maximum and sum are
// wave reductions (online softmax in fp32), and lane j accumulates output dimensions j and
// j + 64 over the chunk's keys, each key's weight broadcast from its lane.
template <int D>
__device__ __forceinline__ void attn_row_f32(const float* __restrict__ q, const float* __restrict__ kc,
                                             const float* __restrict__ vc, float* __restrict__ o, int r, int h, int b,
                                             int pos, int a, int g, int cap, int lane) {
    constexpr int DPL = (D + 63) / 64;   // output dimensions per lane
    const int kvh = h / (a / g);
    const float scale = 1.0f / sqrtf((float)D);
    float qv[D];
#pragma unroll
    for (int i = 0; i < D; ++i) qv[i] = q[((size_t)r * a + h) * D + i];
    const float* kb = kc + ((size_t)b * g + kvh) * cap * D;
    const float* vb = vc + ((size_t)b * g + kvh) * D * cap;
    float acc[DPL];
#pragma unroll
    for (int k = 0; k < DPL; ++k) acc[k] = 0.f;
    float m = -INFINITY, l = 0.f;
    for (int t0 = 0; t0 <= pos; t0 += 64) {
        const int t = t0 + lane;
        float sc = -INFINITY;
        if (t <= pos) {
            float d = 0.f;
#pragma unroll
            for (int i = 0; i < D; ++i) d = fmaf(qv[i], kb[(size_t)t * D + i], d);
            sc = d * scale;
        }
        const float m_new = fmaxf(m, wave_max(sc));      // finite: key t0 is always visible
        const float alpha = expf(m - m_new);
        const float p = t <= pos ? expf(sc - m_new) : 0.f;
        l = l * alpha + wave_sum(p);
#pragma unroll
        for (int k = 0; k < DPL; ++k) acc[k] *= alpha;
        const int nk = min(64, pos + 1 - t0);
        for (int j = 0; j < nk; ++j) {
            const float pj = __shfl(p, j);
#pragma unroll
            for (int k = 0; k < DPL; ++k) {
                const int d = lane + 64 * k;
                if (d < D) acc[k] = fmaf(pj, vb[(size_t)d * cap + t0 + j], acc[k]);
            }
        }
        m = m_new;
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int k = 0; k < DPL; ++k) {
        const int d = lane + 64 * k;
        if (d < D) o[((size_t)r * a + h) * D + d] = acc[k] * inv;
    }
}

// Row r: sequence r at position lens[r].
template <int D>
__global__ __launch_bounds__(256) void attn_f32_kernel(const float* __restrict__ q,
                                                       const float* __restrict__ kc,
                                                       const float* __restrict__ vc,
                                                       const int32_t* __restrict__ lens,
                                                       float* __restrict__ o, int rows, int a, int g,
                                                       int cap) {
    const int wid = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63;
    if (wid >= rows * a) return;         // wave-uniform
    const int r = wid / a, h = wid - r * a;
    attn_row_f32<D>(q, kc, vc, o, r, h, r, max(0, min(lens[r], cap - 1)), a, g, cap, lane);
}

// Row r: sequence r / S at position r % S.
template <int D>
__global__ __launch_bounds__(256) void attn_rows_f32_kernel(const float* __restrict__ q, const float* __restrict__ kc,
                                                            const float* __restrict__ vc, float* __restrict__ o,
                                                            int rows, int S, int a, int g, int cap) {
    const int wid = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63;
    if (wid >= rows * a) return;         // wave-uniform
    const int r = wid / a, h = wid - r * a, b = r / S;
    attn_row_f32<D>(q, kc, vc, o, r, h, b, r - b * S, a, g, cap, lane);
}

}  // namespace

hipError_t rope_table(float2* table, int S, int d, double base, hipStream_t st) {
    const int n = S * (d / 2);
    hipLaunchKernelGGL(rope_table_kernel, dim3((n + 255) / 256), dim3(256), 0, st, table, S, d / 2, d,
                       base);
    return hipGetLastError();
}

hipError_t rope_scatter(const float* proj, int nsplit, size_t split_stride, int rows, int S,
                        const int32_t* lens, int a, int g, int d, int cap, double base, bool producer,
                        bool bf16, void* q, void* kc, void* vc, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    if (d > 128 || nsplit < 1) return hipErrorInvalidValue;
    if (bf16)
        hipLaunchKernelGGL(rope_scatter_kernel<uint16_t>, dim3(rows), dim3(256), 0, st, proj, nsplit,
                           split_stride, S, lens, a, g, d, cap, base, producer ? 1 : 0, (uint16_t*)q,
                           (uint16_t*)kc, (uint16_t*)vc);
    else
        hipLaunchKernelGGL(rope_scatter_kernel<float>, dim3(rows), dim3(256), 0, st, proj, nsplit,
                           split_stride, S, lens, a, g, d, cap, base, producer ? 1 : 0, (float*)q,
                           (float*)kc, (float*)vc);
    return hipGetLastError();
}

hipError_t gemm_f32(const float* a, const WRows& w, int M, int N, int K, float* out,
                    const float* x_res, hipStream_t st) {
    return launch_f32<true, true>(a, K, w, K, M, N, K, F32Dst{{out, out, out}, {M, 0, 0}}, N, x_res, st);
}

hipError_t gemm_f32_nn(const float* a, size_t lda, const WRows& b, size_t ldb, const float* res, float* c, size_t ldc,
                       int M, int N, int K, hipStream_t st) {
    return launch_f32<true, false>(a, lda, b, ldb, M, N, K, F32Dst{{c, c, c}, {M, 0, 0}}, ldc, res, st);
}

hipError_t gemm_f32_tn(const float* a, size_t lda, const float* b, size_t ldb, float* const c[3], const int rows[3],
                       int M, int N, int K, hipStream_t st) {
    return launch_f32<false, false>(a, lda, WRows{{b, b, b}, {K, 0, 0}}, ldb, M, N, K,
                                    F32Dst{{c[0], c[1], c[2]}, {rows[0], rows[1], rows[2]}}, N, nullptr, st);
}

hipError_t attn_f32(const float* q, const float* kc, const float* vc, const int32_t* lens, float* o,
                    int rows, int a, int g, int d, int cap, hipStream_t st) {
    const int n = rows * a;                  // one wave each, four waves per block
    dim3 grid((n + 3) / 4), block(256);
    switch (d) {
        case 16: hipLaunchKernelGGL(attn_f32_kernel<16>, grid, block, 0, st, q, kc, vc, lens, o, rows, a, g, cap); break;
        case 32: hipLaunchKernelGGL(attn_f32_kernel<32>, grid, block, 0, st, q, kc, vc, lens, o, rows, a, g, cap); break;
        case 64: hipLaunchKernelGGL(attn_f32_kernel<64>, grid, block, 0, st, q, kc, vc, lens, o, rows, a, g, cap); break;
        case 128: hipLaunchKernelGGL(attn_f32_kernel<128>, grid, block, 0, st, q, kc, vc, lens, o, rows, a, g, cap); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t attn_rows_f32(const float* q, const float* kc, const float* vc, float* o, int B, int S, int a, int g, int d,
                         int cap, hipStream_t st) {
    const int rows = B * S;
    const dim3 grid((rows * a + 3) / 4), block(256);
    switch (d) {
        case 16: hipLaunchKernelGGL(attn_rows_f32_kernel<16>, grid, block, 0, st, q, kc, vc, o, rows, S, a, g, cap); break;
        case 32: hipLaunchKernelGGL(attn_rows_f32_kernel<32>, grid, block, 0, st, q, kc, vc, o, rows, S, a, g, cap); break;
        case 64: hipLaunchKernelGGL(attn_rows_f32_kernel<64>, grid, block, 0, st, q, kc, vc, o, rows, S, a, g, cap); break;
        case 128: hipLaunchKernelGGL(attn_rows_f32_kernel<128>, grid, block, 0, st, q, kc, vc, o, rows, S, a, g, cap); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace kvp
