// Epilogues of the bf16 GEMMs (gemm_bf16.hip).  A workgroup's fp32 accumulators go through
// LDS: a pass stages ROWS rows of the tile's BN columns (st_block()), then all NT threads copy
// the pass out with coalesced 16-byte global accesses (flush()), applying the fused work.
// The global inputs of a pass (cos/sin rows, residual) are requested by prefetch(): before
// the staging in gemm_small, so that their latency runs under the LDS writes and the
// barrier; after it in the 8-wave kernels, in the registers that the staging has freed.
//
// Staged layout: row m is BN floats; its 16-byte chunk c sits at position
// c ^ ((m / 8) % 16) ^ (8 if m & 4).  An accumulator lane pair (l, l + 32) writes 128
// contiguous bytes of rows m and m + 4, the row flush reads chunks along one row and the
// transposed V flush reads one column of 16 groups of 8 rows: all three spread over the 64
// banks.
#pragma once

#include "common.h"
#include "kernels.h"

namespace kvp {
namespace {

template <int BN>
__device__ __forceinline__ int st_off(int m, int n) {
    return m * (BN * 4) + (((n >> 2) ^ ((m >> 3) & 15) ^ ((m & 4) << 1)) << 4) + ((n & 3) << 2);
}
template <int BN>
__device__ __forceinline__ u32x4 st_chunk(const char* st, int m, int c) {
    return *(const u32x4*)(st + st_off<BN>(m, 4 * c));
}
// One 32 x 32 accumulator block at rows m.., columns n.. of the pass.
template <int BN>
__device__ __forceinline__ void st_block(char* st, const f32x16& acc, int m, int n, int lane) {
    const int l32 = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int i = 0; i < 16; ++i) *(float*)(st + st_off<BN>(m + 8 * (i >> 2) + 4 * hi + (i & 3), n + l32)) = acc[i];
}

// Q, K (rotated) and V (transposed) of the projection GEMM.  A tile column block of 128 is
// one head, so the rotate-half partner of column c is column c + 64 of the same pass.  The
// 64-column tile takes rotary pairs 32 sub .. 32 sub + 31 of one head: columns
// 32 sub + i and 64 + 32 sub + i (kPairedCols tells the GEMM to load its W rows so).
struct QkvEpi {
    static constexpr bool kPairedCols = true;
    template <int ROWS, int BN, int NT>
    struct Pre {
        u32x4 cs[ROWS * BN / 16 / NT][4];
    };
    QkvOut o;
    __device__ __forceinline__ void set_split(int) {}
    // Element offsets of K row s and of V^T element (dimension n, position s) of
    // sequence b, KV head `head`: in the contiguous slot or in s's page.
    __device__ __forceinline__ size_t k_row(int b, int head, int s) const {
        if (o.pages.pt)
            return (((size_t)head * o.pages.n + page_at(o.pages, b, s / kPage)) * kPage + s % kPage) * 128;
        return (((size_t)b * o.g + head) * o.cap + s) * 128;
    }
    __device__ __forceinline__ size_t v_at(int b, int head, int n, int s) const {
        if (o.pages.pt)
            return (((size_t)head * o.pages.n + page_at(o.pages, b, s / kPage)) * 128 + n) * kPage + s % kPage;
        return (((size_t)b * o.g + head) * 128 + n) * o.cap + s;
    }
    // Region of the 128 columns at nw: 0 = Q, 1 = K, 2 = V, -1 = past N.
    __device__ __forceinline__ int region(int nw, int N, int* head) const {
        if (nw >= N) return -1;
        if (nw < o.n_q) { *head = nw >> 7; return 0; }
        if (nw < o.n_q + o.n_kv) { *head = (nw - o.n_q) >> 7; return 1; }
        *head = (nw - o.n_q - o.n_kv) >> 7;
        return 2;
    }
    // Items of a head block: (row, 8 rotation pairs), tid + NT t of them.
    template <int ROWS, int BN, int NT>
    __device__ __forceinline__ void prefetch(int m0, int n0, int tid, int M, int N, Pre<ROWS, BN, NT>& pre) const {
        constexpr int HALF = BN == 64 ? 32 : 64, G8 = HALF / 8, HB = BN / (2 * HALF), T = ROWS * G8 / NT;
        const int sub = BN == 64 ? (n0 & 64) / 2 : 0;
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
            int head;
            const int reg = region((n0 & ~127) + 128 * hb, N, &head);
            if (reg != 0 && reg != 1) continue;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int id = tid + NT * t;
                const int m = min(m0 + id / G8, M - 1);
                const u32x4* tab = (const u32x4*)(o.rope + (size_t)(m % o.S) * 64 + sub + 8 * (id % G8));
#pragma unroll
                for (int q = 0; q < 4; ++q) pre.cs[hb * T + t][q] = tab[q];
            }
        }
    }
    template <int ROWS, int BN, int NT>
    __device__ __forceinline__ void flush(int m0, int n0, int tid, int M, int N, const char* st,
                                          const Pre<ROWS, BN, NT>& pre) const {
        constexpr int HALF = BN == 64 ? 32 : 64, G8 = HALF / 8, HB = BN / (2 * HALF), T = ROWS * G8 / NT;
        const int sub = BN == 64 ? (n0 & 64) / 2 : 0;
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
            int head;
            const int reg = region((n0 & ~127) + 128 * hb, N, &head);
            if (reg < 0) continue;
            const int c0 = 2 * HALF * hb;     // the head block's first staged column
            if (reg == 2) {
                // V^T: item (column n, 8 rows from d0 + 8 k), consecutive lanes along k.  d0 moves
                // the runs to positions that are multiples of 8, aligned in the slot and inside
                // one page; the d0 rows before the first run follow one value a lane, and a run
                // that leaves the pass, the sequence or M goes out value by value.  (Eight
                // 2-byte stores, or misaligned 16-byte ones, for every run made the epilogue of
                // 2 x 777 tokens 14 us longer.)
                constexpr int KC = ROWS / 8, TV = KC * 2 * HALF / NT;
                const int s0 = m0 % o.S, d0 = (8 - s0 % 8) % 8;
                auto dim_of = [&](int n) { return BN == 64 ? sub + (n & 31) + 2 * (n & 32) : n; };
                auto put = [&](int m, int n, float x) {
                    const int b = m / o.S;
                    o.vc[v_at(b, head, dim_of(n), m - b * o.S)] = f2bf(x);
                };
#pragma unroll
                for (int t = 0; t < TV; ++t) {
                    const int id = tid + NT * t;
                    const int r = 8 * (id % KC) + d0, n = id / KC;
                    const int m = m0 + r;
                    if (m >= M) continue;
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        x[e] = *(const float*)(st + st_off<BN>(min(r + e, ROWS - 1), c0 + n));
                    const int b = m / o.S, s = m - b * o.S;
                    if (s % 8 == 0 && s + 8 <= o.S && r + 8 <= ROWS && m + 8 <= M) {
                        *(u32x4*)(o.vc + v_at(b, head, dim_of(n), s)) =
                            u32x4{pack2bf(x[0], x[1]), pack2bf(x[2], x[3]), pack2bf(x[4], x[5]), pack2bf(x[6], x[7])};
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (r + e < ROWS && m + e < M) put(m + e, n, x[e]);
                    }
                }
                if (d0)
                    for (int id = tid; id < 8 * 2 * HALF; id += NT) {
                        const int e = id % 8, n = id / 8;
                        if (e < d0 && m0 + e < M) put(m0 + e, n, *(const float*)(st + st_off<BN>(e, c0 + n)));
                    }
                continue;
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int id = tid + NT * t, k = id % G8, row = id / G8;
                const int m = m0 + row;
                if (m >= M) continue;
                const int c = c0 / 4 + 2 * k;
                const u32x4 a0 = st_chunk<BN>(st, row, c), a1 = st_chunk<BN>(st, row, c + 1);
                const u32x4 b0 = st_chunk<BN>(st, row, c + HALF / 4), b1 = st_chunk<BN>(st, row, c + HALF / 4 + 1);
                float x1[8], x2[8], cc[8], sn[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x1[e] = __uint_as_float(a0[e]);
                    x1[e + 4] = __uint_as_float(a1[e]);
                    x2[e] = __uint_as_float(b0[e]);
                    x2[e + 4] = __uint_as_float(b1[e]);
                }
                const auto& cs = pre.cs[hb * T + t];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    cc[e] = __uint_as_float(cs[e >> 1][2 * (e & 1)]);
                    sn[e] = __uint_as_float(cs[e >> 1][2 * (e & 1) + 1]);
                }
                u32x4 lo, up;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    lo[e] = pack2bf(x1[2 * e] * cc[2 * e] - x2[2 * e] * sn[2 * e],
                                    x1[2 * e + 1] * cc[2 * e + 1] - x2[2 * e + 1] * sn[2 * e + 1]);
                    up[e] = pack2bf(x2[2 * e] * cc[2 * e] + x1[2 * e] * sn[2 * e],
                                    x2[2 * e + 1] * cc[2 * e + 1] + x1[2 * e + 1] * sn[2 * e + 1]);
                }
                uint16_t* dst;
                if (reg == 0) {
                    dst = o.q + (size_t)m * o.n_q + head * 128;
                } else {
                    const int b = m / o.S;
                    dst = o.kc + k_row(b, head, m - b * o.S);
                }
                *(u32x4*)(dst + sub + 8 * k) = lo;
                *(u32x4*)(dst + sub + 8 * k + 64) = up;
            }
        }
    }
};

// Residual update y = x + acc.  x is the bf16 layer input (XF32 = false) or the fp32
// residual stream (XF32 = true, updated in place through yf); y is written in bf16,
// yf (optional) in fp32.
template <bool XF32>
struct ResidEpi {
    static constexpr bool kPairedCols = false;
    // Items of the pass: (row, 8 columns), tid + NT t of them.
    template <int ROWS, int BN, int NT>
    struct Pre {
        u32x4 xv[ROWS * BN / 8 / NT][XF32 ? 2 : 1];
    };
    const void* x;
    uint16_t* y;
    float* yf;
    __device__ __forceinline__ void set_split(int) {}
    template <int ROWS, int BN, int NT>
    __device__ __forceinline__ void prefetch(int m0, int n0, int tid, int M, int N, Pre<ROWS, BN, NT>& pre) const {
        constexpr int C8 = BN / 8;
#pragma unroll
        for (int t = 0; t < ROWS * C8 / NT; ++t) {
            const int id = tid + NT * t;
            const size_t off = (size_t)min(m0 + id / C8, M - 1) * N + min(n0 + 8 * (id % C8), N - 8);
            if (XF32) {
                pre.xv[t][0] = *(const u32x4*)((const float*)x + off);
                pre.xv[t][XF32 ? 1 : 0] = *(const u32x4*)((const float*)x + off + 4);
            } else {
                pre.xv[t][0] = *(const u32x4*)((const uint16_t*)x + off);
            }
        }
    }
    template <int ROWS, int BN, int NT>
    __device__ __forceinline__ void flush(int m0, int n0, int tid, int M, int N, const char* st,
                                          const Pre<ROWS, BN, NT>& pre) const {
        constexpr int C8 = BN / 8;
#pragma unroll
        for (int t = 0; t < ROWS * C8 / NT; ++t) {
            const int id = tid + NT * t, row = id / C8, c8 = id % C8;
            const int m = m0 + row, n = n0 + 8 * c8;
            if (m >= M || n >= N) continue;
            const u32x4 p0 = st_chunk<BN>(st, row, 2 * c8), p1 = st_chunk<BN>(st, row, 2 * c8 + 1);
            float r[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a0 = __uint_as_float(p0[e]), a1 = __uint_as_float(p1[e]);
                float x0, x1;
                if (XF32) {
                    x0 = __uint_as_float(pre.xv[t][0][e]);
                    x1 = __uint_as_float(pre.xv[t][XF32 ? 1 : 0][e]);
                } else {
                    const uint32_t w0 = pre.xv[t][0][e >> 1], w1 = pre.xv[t][0][2 + (e >> 1)];
                    x0 = __uint_as_float((e & 1) ? (w0 & 0xFFFF0000u) : (w0 << 16));
                    x1 = __uint_as_float((e & 1) ? (w1 & 0xFFFF0000u) : (w1 << 16));
                }
                r[e] = x0 + a0;
                r[4 + e] = x1 + a1;
            }
            const size_t off = (size_t)m * N + n;
            u32x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = pack2bf(r[2 * e], r[2 * e + 1]);
            *(u32x4*)(y + off) = out;
            if (yf) {
                *(u32x4*)(yf + off) = u32x4{__float_as_uint(r[0]), __float_as_uint(r[1]),
                                            __float_as_uint(r[2]), __float_as_uint(r[3])};
                *(u32x4*)(yf + off + 4) = u32x4{__float_as_uint(r[4]), __float_as_uint(r[5]),
                                                __float_as_uint(r[6]), __float_as_uint(r[7])};
            }
        }
    }
};

// Plain store of C (no fused work): bf16 [M][N], or fp32: rows [0, rows0) of C to dst0, the
// next rows1 to dst1, the rest to dst2, or (split K) plane `split` of dst0.
template <bool BF16>
struct OutEpi {
    static constexpr bool kPairedCols = false;
    template <int ROWS, int BN, int NT>
    struct Pre {};
    void* dst0;
    float* dst1;
    float* dst2;
    int rows0, rows1;
    size_t plane;
    int split;
    __device__ __forceinline__ void set_split(int s) { split = s; }
    template <int ROWS, int BN, int NT>
    __device__ __forceinline__ void prefetch(int, int, int, int, int, Pre<ROWS, BN, NT>&) const {}
    template <int ROWS, int BN, int NT>
    __device__ __forceinline__ void flush(int m0, int n0, int tid, int M, int N, const char* st,
                                          const Pre<ROWS, BN, NT>&) const {
        constexpr int C8 = BN / 8;
#pragma unroll
        for (int t = 0; t < ROWS * C8 / NT; ++t) {
            const int id = tid + NT * t, row = id / C8, c8 = id % C8;
            int m = m0 + row;
            const int n = n0 + 8 * c8;
            if (m >= M || n >= N) continue;
            const u32x4 p0 = st_chunk<BN>(st, row, 2 * c8), p1 = st_chunk<BN>(st, row, 2 * c8 + 1);
            if constexpr (BF16) {
                u32x4 o;
                o[0] = pack2bf(__uint_as_float(p0[0]), __uint_as_float(p0[1]));
                o[1] = pack2bf(__uint_as_float(p0[2]), __uint_as_float(p0[3]));
                o[2] = pack2bf(__uint_as_float(p1[0]), __uint_as_float(p1[1]));
                o[3] = pack2bf(__uint_as_float(p1[2]), __uint_as_float(p1[3]));
                *(u32x4*)((uint16_t*)dst0 + (size_t)m * N + n) = o;
            } else {
                float* dst = (float*)dst0;
                if (m >= rows0) {
                    m -= rows0;
                    dst = dst1;
                    if (m >= rows1) {
                        m -= rows1;
                        dst = dst2;
                    }
                }
                dst += split * plane + (size_t)m * N + n;
                *(u32x4*)dst = p0;
                *(u32x4*)(dst + 4) = p1;
            }
        }
    }
};

}  // namespace
}  // namespace kvp
