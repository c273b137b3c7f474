// Single-token decode attention over a long KV cache (Sec. 2.2: each new token
// attends to every cached position; a consumer reads its producer's cache,
// Eq. 3), split along the cache ("split-K") and merged by a second kernel.
//
// Schedule: the work of one layer is the list of 64-position tiles of every
// (sequence b, KV head) pair, in (b, head, tile) order.  The grid has one wave per
// SIMD of the device, all resident at once, and wave w streams a contiguous
// range of that list: every wave reads the same number of tiles, or one more (the
// T mod W of the waves), whatever the mix of lengths, and a range may run
// from the end of one pair into the next without a pipeline bubble.  (With ranges of
// ceil(T / W) tiles the last waves had none: 8 sequences of 4100 positions are 4.004
// tiles a wave, 5 for four fifths of the waves, 26.7 us.)  Some short lists
// run on fewer waves (Split).  Each piece
// of a range that lies in one pair ends in a partial result (running max m, sum
// l, unnormalised O); the piece of wave w in pair P goes to slot w + P, which is
// unique because w and P never both decrease along the list.
//
// Per tile: S^T[16 pos x 16 heads] blocks via v_mfma_f32_16x16x32_bf16 with
// A = K rows and B = Q^T (the r query heads of the KV head, padded to 16), then
// O^T[128 x 16] += V^T P^T.  The MFMA row -> position assignment is permuted so
// that after the score MFMAs each lane holds 8 consecutive positions of its
// head, which is exactly the k-slice the PV MFMA needs and a 16-byte run of the
// V^T row: K and V^T are read as 64-byte row segments straight from HBM into
// registers (no LDS: every byte is used once) and P never leaves registers.  The
// next tile's loads (and the next pair's queries) are issued before the current
// tile is consumed.

#include <math.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace kvp {
namespace {

constexpr int D = 128, TILE = 64, PSTRIDE = D + 4;  // O[128], m, l, pad
constexpr int kCombineThreads = 256;
constexpr float kLazy = 8.0f;

struct DTile {
    u32x4 k[4][4];   // [block tb][k step ks]
    u32x4 v[8][2];   // [d block db][pv step s]
};

// Tiles of every sequence (lanes < B) and their inclusive prefix over sequences.
struct SeqTiles {
    int len, n, pre;
};

__device__ __forceinline__ SeqTiles seq_tiles(const int32_t* lens, int B, int cap, int lane) {
    SeqTiles t;
    t.len = lane < B ? max(0, min(lens[lane], cap - 1)) + 1 : 0;
    t.n = (t.len + TILE - 1) / TILE;
    t.pre = t.n;
    for (int off = 1; off < B; off <<= 1) {
        const int v = __shfl_up(t.pre, off);
        if (lane >= off) t.pre += v;
    }
    return t;
}

// The list's split over W waves: wave w starts at tile floor(w T / W)
// (T < 2^31: 64 sequences of at most 2^17 tiles and at most 256 KV heads).  Waves with one
// tile more than others are spread over the grid: starts at one power-of-two stride (64
// sequences of 32K: 256 tiles) meet in the same memory channels, 0.7 % slower.
// Where it takes at most 3/4 of the waves to give none more than ceil(T / waves) = 2 or 3 tiles,
// no more run: the longest range is the same, and 768 waves of a short range finish sooner than
// 1024.  Decode steps, us, all waves / as few as it takes, 8/4 heads, 24 layers: T / waves 1.25
// 979 / 937, 1.5 980 / 943, 1.75 (896 waves) 995 / 1005, 2.25 1086 / 1044, 2.5 1094 / 1115, 2.75
// 1104 / 1134, on pages 1117 / 1164; 32/8, 6 layers: 1.5 288 / 279, 1.75 291 / 295, 2.25 315 / 305,
// 2.5 317 / 324.  The attention alone at 3.06 (784 waves) 23.7 / 24.1, 4.06 27.9 / 28.2, 6.06
// 35.9 / 36.9.
struct Split {
    uint32_t T, W, q, rem;
    static __device__ __forceinline__ uint32_t waves_of(uint32_t T, uint32_t waves) {
        // Constant divisors: a division by a value of the list's took each kernel 0.1 us.
        if (T <= waves) return T;
        if (T <= waves + waves / 2) return (T + 1) / 2;
        if (T > 2 * waves && T <= 2 * waves + waves / 4) return (T + 2) / 3;
        return waves;
    }
    __device__ __forceinline__ Split(uint32_t T_, uint32_t waves) : T(T_), W(waves_of(T_, waves)), q(T_ / W), rem(T_ % W) {}
    __device__ __forceinline__ uint32_t start(uint32_t w) const { return w * q + w * rem / W; }   // w <= W <= 4096
    // The wave that holds tile x: ceil((x + 1) W / T) - 1.  The quotient is exact in double (an
    // integer below 2^43 over one below 2^31).
    __device__ __forceinline__ uint32_t wave_of(uint32_t x) const {
        return (uint32_t)(((double)(x + 1) * (double)W - 1.0) / (double)T);
    }
};

// One wave per workgroup, one workgroup per SIMD (the grid is sized to the device).
// PAGED: every 64-position tile is one page, looked up once per tile.
template <bool PAGED>
__global__ __launch_bounds__(64, 1) void decode_attn_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Kc, const uint16_t* __restrict__ Vc,
    const int32_t* __restrict__ lens, float* __restrict__ part, int B, int a, int g, int cap,
    float scale_log2, Pages pages) {
    const int lane = threadIdx.x;
    const int W = gridDim.x, w = blockIdx.x;
    const int r = a / g;
    const SeqTiles st = seq_tiles(lens, B, cap, lane);
    const uint32_t T = (uint32_t)g * __shfl(st.pre, B - 1);
    const Split sp(T, W);
    if (w >= (int)sp.W) return;
    uint32_t x = sp.start(w);
    const uint32_t x_end = sp.start(w + 1);

    // Locate tile x: sequence b is the number of sequences that end at or before x.
    int b = __popcll(__ballot(lane < B && (uint32_t)g * st.pre <= x));
    int n = __shfl(st.n, b), len = __shfl(st.len, b);
    const uint32_t into = x - (uint32_t)g * (__shfl(st.pre, b) - n);
    int kvh = (int)(into / n), t = (int)(into % n);

    const int col = lane & 15, grp = lane >> 4;    // MFMA column (head) and lane group

    // Q^T fragments: lane (col, grp) holds head kvh*r + col, dims 32 ks + 8 grp + 0..7.
    auto load_q = [&](int qb, int qh, bf16x8* qf) {
        const bool real = col < r;
        const uint16_t* qrow = Q + (size_t)qb * a * D + (size_t)(qh * r + (real ? col : 0)) * D + 8 * grp;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            u32x4 v = *(const u32x4*)(qrow + 32 * ks);
            if (!real) v = u32x4{0, 0, 0, 0};
            qf[ks] = as_bf16x8(v);
        }
    };

    // Position held by MFMA row rho (= lane & 15 for the A operand) of score block tb
    // of a tile: block 2s + e covers positions 32 s + 8 (rho / 4) + 4 e + rho % 4.
    // Tiles start at multiples of 64 and cap % 64 == 0, so every load stays in the slot
    // (or, paged, in the tile's page).  Paged: the wave keeps 64 consecutive entries of a
    // table row in a register (lane i: entry 64 c + i of row pb) and reads the tile's entry
    // with readlane, so a dependent table load is paid once per 64 tiles, not per tile.
    int pb = -1, pc = -1, pgv = 0;
    auto load = [&](int lb, int lh, int t0, DTile& tl) {
        const uint16_t* kbase;
        const uint16_t* vbase;
        int vld;
        if constexpr (PAGED) {
            const int j = t0 / TILE;
            if (lb != pb || (j >> 6) != pc) {
                pb = lb;
                pc = j >> 6;
                const int e = 64 * pc + lane;
                pgv = e < pages.stride ? pages.pt[(size_t)lb * pages.stride + e] : 0;
            }
            const int pg = min(max(__builtin_amdgcn_readlane(pgv, j & 63), 0), pages.n - 1);
            kbase = Kc + ((size_t)lh * pages.n + pg) * TILE * D - (size_t)t0 * D;
            vbase = Vc + ((size_t)lh * pages.n + pg) * D * TILE - t0;
            vld = TILE;
        } else {
            kbase = Kc + ((size_t)lb * g + lh) * cap * D;
            vbase = Vc + ((size_t)lb * g + lh) * D * cap;
            vld = cap;
        }
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            const int s = tb >> 1, e = tb & 1;
            const int pos = t0 + 32 * s + 8 * (col >> 2) + 4 * e + (col & 3);
            const uint16_t* kr = kbase + (size_t)pos * D + 8 * grp;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) tl.k[tb][ks] = *(const u32x4*)(kr + 32 * ks);
        }
#pragma unroll
        for (int db = 0; db < 8; ++db) {
            const uint16_t* vr = vbase + (size_t)(16 * db + col) * vld + t0 + 8 * grp;
#pragma unroll
            for (int s = 0; s < 2; ++s) tl.v[db][s] = *(const u32x4*)(vr + 32 * s);
        }
    };

    bf16x8 qf[4], qn[4];
    load_q(b, kvh, qf);
    f32x4 o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = f32x4{};
    float m_run = kNoScore, l_run = 0.f;

    DTile cur, nxt;
    load(b, kvh, TILE * t, cur);
    for (; x < x_end; ++x) {
        // Next tile of the range, possibly in the next pair.
        const bool more = x + 1 < x_end;
        int nb = b, nh = kvh, nt = t + 1, nn = n, nl = len;
        bool pair_ends = !more;
        if (more) {
            if (nt == n) {
                nt = 0;
                pair_ends = true;
                if (++nh == g) {
                    nh = 0;
                    ++nb;
                    nn = __shfl(st.n, nb);
                    nl = __shfl(st.len, nb);
                }
                load_q(nb, nh, qn);
            }
            load(nb, nh, TILE * nt, nxt);
        }

        // ---- scores --------------------------------------------------------------
        const int t0 = TILE * t;
        f32x4 sc[4];
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            sc[tb] = f32x4{};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) sc[tb] = mfma16x16x32(as_bf16x8(cur.k[tb][ks]), qf[ks], sc[tb]);
        }
        // Lane (col, grp) now holds head col at positions t0 + 32 s + 8 grp + 4 e + i.
        const bool edge = t0 + TILE > len;
        float mx = -INFINITY;
#pragma unroll
        for (int tb = 0; tb < 4; ++tb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (edge) {
                    const int pos = t0 + 32 * (tb >> 1) + 8 * grp + 4 * (tb & 1) + i;
                    if (pos >= len) sc[tb][i] = -INFINITY;
                }
                mx = fmaxf(mx, sc[tb][i]);
            }
        mx = pair32_max(pair16_max(mx));
        const float mt = mx * scale_log2;
        if (__any(mt > m_run + kLazy)) {
            const float m_new = fmaxf(m_run, mt);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < 8; ++db) o[db] *= alpha;
        }
        bf16x8 pb[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float p[8];
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    p[4 * e + i] = __builtin_amdgcn_exp2f(fmaf(sc[2 * s + e][i], scale_log2, -m_run));
                    l_run += p[4 * e + i];
                }
            u32x4 wv;
            wv[0] = pack2bf(p[0], p[1]);
            wv[1] = pack2bf(p[2], p[3]);
            wv[2] = pack2bf(p[4], p[5]);
            wv[3] = pack2bf(p[6], p[7]);
            pb[s] = as_bf16x8(wv);
        }
        // ---- O^T += V^T P^T; positions >= len carry P = 0 but their V must be finite:
        // zero them (the cache beyond len_b may hold anything).
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int p0 = t0 + 32 * s + 8 * grp;
#pragma unroll
            for (int db = 0; db < 8; ++db) {
                u32x4 v = cur.v[db][s];
                if (edge) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int pa = p0 + 2 * e;
                        const uint32_t m = (pa < len ? 0x0000FFFFu : 0u) | (pa + 1 < len ? 0xFFFF0000u : 0u);
                        v[e] &= m;
                    }
                }
                o[db] = mfma16x16x32(as_bf16x8(v), pb[s], o[db]);
            }
        }

        if (pair_ends) {
            // ---- partial result of this wave's piece of pair (b, kvh) -----------------
            const float lt = pair32_sum(pair16_sum(l_run));
            if (col < r) {
                float* pr = part + (((size_t)w + (size_t)b * g + kvh) * r + col) * PSTRIDE;
                // O^T block db: lane holds dims 16 db + 4 grp + 0..3 of head col.
#pragma unroll
                for (int db = 0; db < 8; ++db) *(f32x4*)(pr + 16 * db + 4 * grp) = o[db];
                if (grp == 0) {
                    pr[D] = m_run;
                    pr[D + 1] = lt;
                }
            }
            if (more) {
#pragma unroll
                for (int i = 0; i < 8; ++i) o[i] = f32x4{};
                m_run = kNoScore;
                l_run = 0.f;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) qf[ks] = qn[ks];
            }
        }
        b = nb;
        kvh = nh;
        t = nt;
        n = nn;
        len = nl;
        if (more) cur = nxt;
    }
}

// Merge the pieces of one (sequence, query head): the waves that covered its pair are
// w_first..w_last (recomputed from the lengths exactly as the attention kernel splits
// the tile list).  Wave v of the workgroup takes pieces v, v + 4, ...: lane i holds the
// maximum and sum of its i-th, every lane two of the 128 dimensions, so nothing is shared
// before the four waves' results meet in LDS.  The kernel is a few dependent load latencies
// and the fetch of its own code; weights in LDS for the whole workgroup, with three barriers,
// or the values requested early by unrolled code were 0.8 us longer at one sequence of 977
// positions (4.4 and 5.2 us).  The values of 8 and then of 4 pieces are requested at once: one
// piece after the other took (step of two layers, 16/1 heads, one sequence of 120 000: 1024
// pieces) 204 us, this 81; 64/8 heads, 8000: 162 and 152; batches of 4 alone 97 and 152, of 16
// 72 and 155 (their remainder goes one by one).
// MANY: with the batches.  Without them, for up to 8 tiles a sequence (at most two pieces a wave),
// the kernel is half as long and takes 26 registers for 50.  Same bits.
template <bool MANY>
__global__ __launch_bounds__(kCombineThreads) void decode_combine_kernel(
    const float* __restrict__ part, const int32_t* __restrict__ lens, uint16_t* __restrict__ O, int B,
    int a, int g, int cap, int W) {
    constexpr int NW = kCombineThreads / 64;
    __shared__ float num_s[NW][D], m_s[NW], den_s[NW];
    const int bh = blockIdx.x, b = bh / a, j = bh % a, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int r = a / g, kvh = j / r, jr = j % r;
    const SeqTiles st = seq_tiles(lens, B, cap, lane);
    const Split sp((uint32_t)g * __shfl(st.pre, B - 1), W);
    const int n = __shfl(st.n, b);
    const uint32_t g0 = (uint32_t)g * (__shfl(st.pre, b) - n) + (uint32_t)kvh * n;
    const int w_first = __builtin_amdgcn_readfirstlane((int)sp.wave_of(g0));
    const int ns = __builtin_amdgcn_readfirstlane((int)sp.wave_of(g0 + n - 1)) - w_first + 1;
    const size_t step = (size_t)NW * r * PSTRIDE;     // from one of the wave's pieces to the next
    const float* pr = part + (((size_t)w_first + (size_t)b * g + kvh + wave) * r + jr) * PSTRIDE;
    const int mine = (ns - wave + NW - 1) / NW;
    float M = -INFINITY, den = 0.f;
    f32x2 num = {0.f, 0.f};
    for (int s0 = 0; s0 < mine; s0 += 64, pr += 64 * step) {
        const int c = min(mine - s0, 64);
        float m = -INFINITY, l = 0.f;
        if (lane < c) {
            m = pr[lane * step + D];
            l = pr[lane * step + D + 1];
        }
        const float Mn = fmaxf(M, wave_max(m)), f = exp2f(M - Mn);
        const float wt = exp2f(m - Mn);
        den = den * f + wave_sum(wt * l);
        num *= f;
        M = Mn;
        auto add = [&](auto n_t, int s) __attribute__((always_inline)) {
            constexpr int n = decltype(n_t)::value;
            f32x2 x[n];
#pragma unroll
            for (int i = 0; i < n; ++i) x[i] = *(const f32x2*)(pr + (s + i) * step + 2 * lane);
#pragma unroll
            for (int i = 0; i < n; ++i) {
                const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wt), s + i));
                num[0] += w * x[i][0];
                num[1] += w * x[i][1];
            }
        };
        int s = 0;
        if constexpr (MANY) {
            for (; s + 8 <= c; s += 8) add(std::integral_constant<int, 8>{}, s);
            for (; s + 4 <= c; s += 4) add(std::integral_constant<int, 4>{}, s);
        }
        for (; s < c; ++s) add(std::integral_constant<int, 1>{}, s);
    }
    *(f32x2*)&num_s[wave][2 * lane] = num;
    if (lane == 0) {
        m_s[wave] = M;
        den_s[wave] = den;
    }
    __syncthreads();
    if (t >= D) return;
    float Mx = m_s[0];
#pragma unroll
    for (int v = 1; v < NW; ++v) Mx = fmaxf(Mx, m_s[v]);
    float nsum = 0.f, dsum = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        const float f = exp2f(m_s[v] - Mx);
        nsum += f * num_s[v][t];
        dsum += f * den_s[v];
    }
    O[(size_t)bh * D + t] = f2bf(nsum / dsum);
}

}  // namespace

hipError_t decode_attn_bf16(const uint16_t* q, const uint16_t* kc, const uint16_t* vc,
                            const int32_t* lens, float* part, int B, int a, int g, int cap, int waves,
                            const Pages& pages, hipStream_t st) {
    if (B < 1 || B > 64 || waves < 1 || waves > kMaxDecodeSplits) return hipErrorInvalidValue;
    const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));
    if (pages.pt) {
        if (pages.n < 1 || pages.stride < 1 || cap != TILE * pages.stride) return hipErrorInvalidValue;
        hipLaunchKernelGGL(decode_attn_kernel<true>, dim3(waves), dim3(64), 0, st, q, kc, vc, lens, part, B, a,
                           g, cap, scale_log2, pages);
    } else {
        hipLaunchKernelGGL(decode_attn_kernel<false>, dim3(waves), dim3(64), 0, st, q, kc, vc, lens, part, B,
                           a, g, cap, scale_log2, pages);
    }
    return hipGetLastError();
}

hipError_t decode_combine_bf16(const float* part, const int32_t* lens, uint16_t* o, int B, int a, int g,
                               int cap, int waves, int max_len, hipStream_t st) {
    if (B < 1 || B > 64 || waves < 1 || waves > kMaxDecodeSplits) return hipErrorInvalidValue;
    if (max_len >= 8 * TILE)
        hipLaunchKernelGGL(decode_combine_kernel<true>, dim3(B * a), dim3(kCombineThreads), 0, st, part, lens, o, B, a,
                           g, cap, waves);
    else
        hipLaunchKernelGGL(decode_combine_kernel<false>, dim3(B * a), dim3(kCombineThreads), 0, st, part, lens, o, B, a,
                           g, cap, waves);
    return hipGetLastError();
}

}  // namespace kvp
