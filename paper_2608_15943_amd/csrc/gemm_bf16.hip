// GEMMs of the prefill and the backward on bf16 matrix cores (gfx950).
//
// C[M][N] = A[M][K] * W[N][K]^T with both operands K-contiguous ([out, in]
// weights), fp32 accumulation in v_mfma_f32_32x32x16_bf16, K summed in order in steps of
// 16 whatever the tile (every tile size gives the same bits), and fused epilogues
// (gemm_epi.h): RoPE + Q / K / V^T writes (Sec. 2.2, Eq. 1; a consumer runs it with
// N = a * d_h, Q only), the residual update X_{l+1} = X_l + O W_O^T, or a plain store.
//
// gemm_big: 256 x 256 x 64 per workgroup of 8 waves, two per SIMD (waves w and w + 4), which
// take turns: in every slot one group of four waves runs 16 matrix instructions from
// registers while the other reads its next fragments from LDS and requests later tiles; a
// barrier ends the slot and the groups change places.  One wave per SIMD (four waves of
// 128 x 128) had nothing to run while it waited for its fragments and for the tile behind
// the barrier.  Operands go from global memory straight into LDS, two stages of 64 KB; each
// part of a stage is requested again as soon as its fragments are in registers, so a load
// has two pairs of slots (a whole K step of the workgroup) before its wait, which leaves the
// newer loads in flight.
//
// gemm_half (128 x 256, the same turns) and gemm_small (128 x 128, 64 x 64 per workgroup of 4
// waves): products whose 256 x 256 tiles would leave CUs without work.
//
// LDS rows are 128 B (64 k) with the 16-byte chunk index XOR-swizzled by ((row >> 1) & 7),
// which spreads the fragment reads over all 64 banks.  Tiles are ordered so that each XCD
// works on a contiguous group of M-panels (its own L2 keeps the A and W panels hot).
#include "common.h"
#include "gemm_epi.h"
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace kvp {
namespace {

constexpr int BM = 256, BN = 256, BK = 64, GROUP_M = 8;

// Word 3 of a raw buffer resource: a valid (32-bit) data format.
constexpr int kRsrcWord3 = 0x00020000;

typedef __attribute__((address_space(3))) void lvoid_t;

// LDS position of 16-byte chunk c of tile row r (rows are 128 B): spreads 16 consecutive
// rows of one chunk column over all 64 banks.
__device__ __forceinline__ int swz(int r, int c) { return c ^ ((r >> 1) & 7); }

// Buffer resource of `rows` rows of K values at p: reads past them return zeros.  Made
// scalar word by word (a resource in vector registers costs a loop around every load).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const uint16_t* p, int rows, int K) {
    const uint64_t a = (uint64_t)p;
    const uint64_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)a) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32;
    return __builtin_amdgcn_make_buffer_rsrc((void*)u, 0, __builtin_amdgcn_readfirstlane(max(rows, 0) * K * 2),
                                             kRsrcWord3);
}

// First row of the 128-row weight block at stacked row n (n % 128 == 0, block sizes are
// multiples of 128).
__device__ __forceinline__ const uint16_t* w_block(const WRows& w, int n, int K) {
    if (n < w.rows[0]) return (const uint16_t*)w.p[0] + (size_t)n * K;
    n -= w.rows[0];
    if (n < w.rows[1]) return (const uint16_t*)w.p[1] + (size_t)n * K;
    n -= w.rows[1];
    return (const uint16_t*)w.p[2] + (size_t)n * K;
}

// Tile of workgroup `lid` (row tile, column tile): groups of gm row tiles, rows fastest.
__device__ __forceinline__ void tile_of(int lid, int ntm, int ntn, int gm, int& tm, int& tn) {
    const int group = lid / (gm * ntn), first = group * gm;
    const int gsz = min(ntm - first, gm);
    const int in_g = lid - group * gm * ntn;
    tm = first + in_g % gsz;
    tn = in_g / gsz;
}

// Fragment reads: four 16-wide k steps of one or two 32-row blocks per operand, addresses
// per k step plus a constant for the block.  The reads and their wait are one asm block: the
// compiler, which cannot tell the LDS stages apart, would wait for every load into LDS
// before a plain read.
typedef u32x4 Frag[4];   // [k step]
// A rows +0 and +32, B rows +0 and +128.
__device__ __forceinline__ void read_a2b2_half(Frag (&fa)[2], Frag (&fb)[2], const uint32_t (&a)[4],
                                            const uint32_t (&b)[4]) {
    asm volatile("ds_read_b128 %0, %16\n\tds_read_b128 %4, %16 offset:4096\n\t"
                 "ds_read_b128 %8, %20\n\tds_read_b128 %12, %20 offset:16384\n\t"
                 "ds_read_b128 %1, %17\n\tds_read_b128 %5, %17 offset:4096\n\t"
                 "ds_read_b128 %9, %21\n\tds_read_b128 %13, %21 offset:16384\n\t"
                 "ds_read_b128 %2, %18\n\tds_read_b128 %6, %18 offset:4096\n\t"
                 "ds_read_b128 %10, %22\n\tds_read_b128 %14, %22 offset:16384\n\t"
                 "ds_read_b128 %3, %19\n\tds_read_b128 %7, %19 offset:4096\n\t"
                 "ds_read_b128 %11, %23\n\tds_read_b128 %15, %23 offset:16384\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(fa[0][0]), "=&v"(fa[0][1]), "=&v"(fa[0][2]), "=&v"(fa[0][3]), "=&v"(fa[1][0]),
                   "=&v"(fa[1][1]), "=&v"(fa[1][2]), "=&v"(fa[1][3]), "=&v"(fb[0][0]), "=&v"(fb[0][1]),
                   "=&v"(fb[0][2]), "=&v"(fb[0][3]), "=&v"(fb[1][0]), "=&v"(fb[1][1]), "=&v"(fb[1][2]),
                   "=&v"(fb[1][3])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3])
                 : "memory");
}
// A and B rows +0 and +32.
__device__ __forceinline__ void read_a2b2(Frag (&fa)[2], Frag (&fb)[2], const uint32_t (&a)[4],
                                            const uint32_t (&b)[4]) {
    asm volatile("ds_read_b128 %0, %16\n\tds_read_b128 %4, %16 offset:4096\n\t"
                 "ds_read_b128 %8, %20\n\tds_read_b128 %12, %20 offset:4096\n\t"
                 "ds_read_b128 %1, %17\n\tds_read_b128 %5, %17 offset:4096\n\t"
                 "ds_read_b128 %9, %21\n\tds_read_b128 %13, %21 offset:4096\n\t"
                 "ds_read_b128 %2, %18\n\tds_read_b128 %6, %18 offset:4096\n\t"
                 "ds_read_b128 %10, %22\n\tds_read_b128 %14, %22 offset:4096\n\t"
                 "ds_read_b128 %3, %19\n\tds_read_b128 %7, %19 offset:4096\n\t"
                 "ds_read_b128 %11, %23\n\tds_read_b128 %15, %23 offset:4096\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(fa[0][0]), "=&v"(fa[0][1]), "=&v"(fa[0][2]), "=&v"(fa[0][3]), "=&v"(fa[1][0]),
                   "=&v"(fa[1][1]), "=&v"(fa[1][2]), "=&v"(fa[1][3]), "=&v"(fb[0][0]), "=&v"(fb[0][1]),
                   "=&v"(fb[0][2]), "=&v"(fb[0][3]), "=&v"(fb[1][0]), "=&v"(fb[1][1]), "=&v"(fb[1][2]),
                   "=&v"(fb[1][3])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3])
                 : "memory");
}
// A rows +128 and +160.
__device__ __forceinline__ void read_a2_upper(Frag (&fa)[2], const uint32_t (&a)[4]) {
    asm volatile("ds_read_b128 %0, %8 offset:16384\n\tds_read_b128 %4, %8 offset:20480\n\t"
                 "ds_read_b128 %1, %9 offset:16384\n\tds_read_b128 %5, %9 offset:20480\n\t"
                 "ds_read_b128 %2, %10 offset:16384\n\tds_read_b128 %6, %10 offset:20480\n\t"
                 "ds_read_b128 %3, %11 offset:16384\n\tds_read_b128 %7, %11 offset:20480\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(fa[0][0]), "=&v"(fa[0][1]), "=&v"(fa[0][2]), "=&v"(fa[0][3]), "=&v"(fa[1][0]),
                   "=&v"(fa[1][1]), "=&v"(fa[1][2]), "=&v"(fa[1][3])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
                 : "memory");
}
// One block of A and one of B.
__device__ __forceinline__ void read_a1b1(Frag& fa, Frag& fb, const uint32_t (&a)[4], const uint32_t (&b)[4]) {
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %4, %12\n\t"
                 "ds_read_b128 %1, %9\n\tds_read_b128 %5, %13\n\t"
                 "ds_read_b128 %2, %10\n\tds_read_b128 %6, %14\n\t"
                 "ds_read_b128 %3, %11\n\tds_read_b128 %7, %15\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(fa[0]), "=&v"(fa[1]), "=&v"(fa[2]), "=&v"(fa[3]), "=&v"(fb[0]), "=&v"(fb[1]), "=&v"(fb[2]),
                   "=&v"(fb[3])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3])
                 : "memory");
}

// 64 lanes x 16 bytes at r + voff + soff (bytes) to 1 KB of LDS at dst.
__device__ __forceinline__ void load_1k(__amdgpu_buffer_rsrc_t r, u32x4* dst, uint32_t voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lvoid_t*)dst, 16, voff, soff, 0, 0);
}

template <int N>
__device__ __forceinline__ void vm_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}
__device__ __forceinline__ void slot_end() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

constexpr int kBigNT = 512;

// Slots.  A K tile is two phases: phase a multiplies tile rows 0..127 (each wave 64 of them)
// by all columns, phase b rows 128..255; a phase is a read slot and a product slot, and the
// second wave group runs one slot behind the first.  Tile parts A0, A1 (rows 0..127,
// 128..255) and B0, B1 (columns likewise) of tile kt + 2 are requested into stage kt % 2 once
// both groups have read tile kt's (A0, B0, B1: in phase b of tile kt; A1: in phase a of tile
// kt + 1), 16 KB each, two loads per wave.  Every read slot ends with a wait for the parts
// the next phase reads; the 8 newer loads stay in flight, also at the end, where tiles past
// the last one are requested beyond their resource.
template <class Epi>
__global__ __launch_bounds__(kBigNT, 2) void gemm_big(const uint16_t* __restrict__ A, WRows W, int M, int N, int K,
                                                     int splits, Epi epi) {
    __shared__ u32x4 lds[8192];   // A [stage][half][128 rows][8 chunks], then B likewise
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int l32 = lane & 31, hi = lane >> 5;

    const int ntm = (M + BM - 1) / BM, ntn = (N + BN - 1) / BN;
    // With split K, workgroup slot `split` of every tile takes the 64-wide K tiles
    // [split * n / splits, (split + 1) * n / splits) of n; consecutive ids share a slice.
    const int lid0 = xcd_remap(blockIdx.x, gridDim.x);
    const int split = __builtin_amdgcn_readfirstlane(lid0 / (ntm * ntn));
    int tm, tn;
    tile_of(lid0 - split * (ntm * ntn), ntm, ntn, GROUP_M, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int kt0 = __builtin_amdgcn_readfirstlane(split * (K / BK) / splits);
    const int nk = __builtin_amdgcn_readfirstlane((split + 1) * (K / BK) / splits) - kt0, kofs = kt0 * BK;
    epi.set_split(split);

    // Resources of the four half tiles; a half past M has no rows, one past N repeats the first.
    const __amdgpu_buffer_rsrc_t ra[2] = {row_rsrc(A + (size_t)m0 * K, min(M - m0, 128), K),
                                          row_rsrc(A + (size_t)(m0 + (m0 + 128 < M ? 128 : 0)) * K, min(M - m0 - 128, 128), K)};
    const __amdgpu_buffer_rsrc_t rb[2] = {row_rsrc(w_block(W, n0, K), 128, K),
                                          row_rsrc(w_block(W, n0 + 128 < N ? n0 + 128 : n0, K), 128, K)};
    // Wave w requests rows 16 w .. 16 w + 15 of a half in two 1 KB instructions (8 rows each);
    // lane l covers row l / 8 and fetches the global chunk that belongs at position l % 8.
    uint32_t goff[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = 16 * wave + 8 * j + (lane >> 3);
        goff[j] = (uint32_t)(row * K + kofs + 8 * swz(row, lane & 7)) * 2u;
    }
    // A tile past the last one is requested at offsets past the resource: nothing is fetched,
    // and the wait counts stay the same to the end.
    auto issue = [&](const __amdgpu_buffer_rsrc_t& r, int part, int half, int kt) __attribute__((always_inline)) {
        u32x4* dst = &lds[part * 4096 + ((kt & 1) * 2 + half) * 1024 + wave * 128];
        const uint32_t past = kt < nk ? 0u : 0x80000000u;
        const int ko = kt < nk ? kt * BK * 2 : 0;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            load_1k(r, dst + 64 * j, goff[j] | past, ko);
    };

    // LDS byte addresses of the lane's fragments (k step ks) in half 0 of stage 0.
    uint32_t aa[4], ab[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const uint32_t c = (uint32_t)(((2 * ks + hi) ^ ((l32 >> 1) & 7)) * 16);
        aa[ks] = (uint32_t)(uintptr_t)&lds[(64 * wm + l32) * 8] + c;
        ab[ks] = (uint32_t)(uintptr_t)&lds[4096 + (32 * wn + l32) * 8] + c;
    }
    f32x16 acc[2][2][2];   // [row half][column half][32-row block]
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i >> 2][(i >> 1) & 1][i & 1] = f32x16{};
    Frag fa[2], fb[2];
    // The products stay in their slot: nothing else orders them against the barriers.
    auto products = [&](f32x16 (&c)[2][2]) __attribute__((always_inline)) {
        asm volatile("" : "+v"(c[0][0]), "+v"(c[0][1]), "+v"(c[1][0]), "+v"(c[1][1]));
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
                    c[j][mb] = mfma32x32x16(as_bf16x8(fa[mb][ks]), as_bf16x8(fb[j][ks]), c[j][mb]);
        __builtin_amdgcn_s_setprio(0);
        asm volatile("" : "+v"(c[0][0]), "+v"(c[0][1]), "+v"(c[1][0]), "+v"(c[1][1]));
    };
    issue(ra[0], 0, 0, 0);
    issue(rb[0], 1, 0, 0);
    issue(rb[1], 1, 1, 0);
    issue(ra[1], 0, 1, 0);
    issue(ra[0], 0, 0, 1);
    issue(rb[0], 1, 0, 1);
    issue(rb[1], 1, 1, 1);
    vm_wait<8>();
    slot_end();
    if (wm == 1) slot_end();   // the second group runs one slot behind
    for (int kt = 0; kt < nk; ++kt) {
        // phase a
        issue(ra[1], 0, 1, kt + 1);
        read_a2b2_half(fa, fb, aa, ab);
        vm_wait<8>();
        slot_end();
        products(acc[0]);
        slot_end();
        // phase b
        issue(ra[0], 0, 0, kt + 2);
        issue(rb[0], 1, 0, kt + 2);
        issue(rb[1], 1, 1, kt + 2);
        read_a2_upper(fa, aa);
        vm_wait<8>();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            aa[ks] ^= 32768u;
            ab[ks] ^= 32768u;
        }
        slot_end();
        products(acc[1]);
        slot_end();
    }
    if (wm == 0) slot_end();
    vm_wait<0>();
    // Pass i: rows 128 i .. + 127 of the tile.
    char* st = (char*)&lds[0];
    auto pass = [&](auto i_t) __attribute__((always_inline)) {
        constexpr int i = decltype(i_t)::value;
        __syncthreads();   // the LDS is free: last fragment reads / previous flush are done
        typename Epi::template Pre<128, BN, kBigNT> pre;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) st_block<BN>(st, acc[i][j][mb], 64 * wm + 32 * mb, 128 * j + 32 * wn, lane);
        // Requested in the registers that the staging has freed.
        __builtin_amdgcn_sched_barrier(0);
        epi.template prefetch<128, BN, kBigNT>(m0 + 128 * i, n0, tid, M, N, pre);
        __syncthreads();
        epi.template flush<128, BN, kBigNT>(m0 + 128 * i, n0, tid, M, N, st, pre);
    };
    pass(std::integral_constant<int, 0>{});
    pass(std::integral_constant<int, 1>{});
}

// 128 x 256 tile, the first of gemm_big's two phases alone: 64 x 64 per wave, 16 products a
// slot.  A K tile is one read slot and one product slot per group; three stages of 48 KB, tile
// kt + 3 requested in the read slot of tile kt + 1 (both groups have read tile kt by then) and
// waited for in that of tile kt + 2.
template <class Epi>
__global__ __launch_bounds__(kBigNT, 2) void gemm_half(const uint16_t* __restrict__ A, WRows W, int M, int N, int K,
                                                      int splits, Epi epi) {
    constexpr int kStage = 384 * 8;            // [A 128 rows, B 256 rows][8 chunks]
    __shared__ u32x4 lds[3 * kStage];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int l32 = lane & 31, hi = lane >> 5;

    const int ntm = (M + 127) / 128, ntn = (N + BN - 1) / BN;
    const int lid0 = xcd_remap(blockIdx.x, gridDim.x);
    const int split = __builtin_amdgcn_readfirstlane(lid0 / (ntm * ntn));
    int tm, tn;
    tile_of(lid0 - split * (ntm * ntn), ntm, ntn, 2 * GROUP_M, tm, tn);
    const int m0 = tm * 128, n0 = tn * BN;
    const int kt0 = __builtin_amdgcn_readfirstlane(split * (K / BK) / splits);
    const int nk = __builtin_amdgcn_readfirstlane((split + 1) * (K / BK) / splits) - kt0, kofs = kt0 * BK;
    epi.set_split(split);

    const __amdgpu_buffer_rsrc_t ra = row_rsrc(A + (size_t)m0 * K, min(M - m0, 128), K);
    const __amdgpu_buffer_rsrc_t rb[2] = {row_rsrc(w_block(W, n0, K), 128, K),
                                          row_rsrc(w_block(W, n0 + 128 < N ? n0 + 128 : n0, K), 128, K)};
    uint32_t goff[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = 16 * wave + 8 * j + (lane >> 3);
        goff[j] = (uint32_t)(row * K + kofs + 8 * swz(row, lane & 7)) * 2u;
    }
    auto issue = [&](int kt, int stg) __attribute__((always_inline)) {
        u32x4* dst = &lds[stg * kStage + wave * 128];
        const uint32_t past = kt < nk ? 0u : 0x80000000u;
        const int ko = kt < nk ? kt * BK * 2 : 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            load_1k(ra, dst + 64 * j, goff[j] | past, ko);
            load_1k(rb[0], dst + 1024 + 64 * j, goff[j] | past, ko);
            load_1k(rb[1], dst + 2048 + 64 * j, goff[j] | past, ko);
        }
    };
    f32x16 c[2][2];   // [column half][32-row block]
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i >> 1][i & 1] = f32x16{};
    Frag fa[2], fb[2];

    issue(0, 0);
    issue(1, 1);
    issue(2, 2);
    vm_wait<12>();
    slot_end();
    if (wm == 1) slot_end();   // the second group runs one slot behind
    int stg = 0;
    for (int kt = 0; kt < nk; ++kt) {
        if (kt > 0) issue(kt + 2, stg == 0 ? 2 : stg - 1);
        uint32_t aa[4], ab[4];
        const uint32_t base = (uint32_t)(uintptr_t)&lds[0] + stg * (kStage * 16);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const uint32_t ch = (uint32_t)(((2 * ks + hi) ^ ((l32 >> 1) & 7)) * 16);
            aa[ks] = base + (64 * wm + l32) * 128 + ch;
            ab[ks] = base + 16384 + (32 * wn + l32) * 128 + ch;
        }
        read_a2b2_half(fa, fb, aa, ab);
        vm_wait<6>();
        slot_end();
        asm volatile("" : "+v"(c[0][0]), "+v"(c[0][1]), "+v"(c[1][0]), "+v"(c[1][1]));
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
                    c[j][mb] = mfma32x32x16(as_bf16x8(fa[mb][ks]), as_bf16x8(fb[j][ks]), c[j][mb]);
        __builtin_amdgcn_s_setprio(0);
        asm volatile("" : "+v"(c[0][0]), "+v"(c[0][1]), "+v"(c[1][0]), "+v"(c[1][1]));
        slot_end();
        stg = stg == 2 ? 0 : stg + 1;
    }
    if (wm == 0) slot_end();
    vm_wait<0>();
    char* st = (char*)&lds[0];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) st_block<BN>(st, c[j][mb], 64 * wm + 32 * mb, 128 * j + 32 * wn, lane);
    __builtin_amdgcn_sched_barrier(0);
    typename Epi::template Pre<128, BN, kBigNT> pre;
    epi.template prefetch<128, BN, kBigNT>(m0, n0, tid, M, N, pre);
    __syncthreads();
    epi.template flush<128, BN, kBigNT>(m0, n0, tid, M, N, st, pre);
}

// BM_ x BN_ tile of 4 waves (2 x 2), STAGES K tiles in LDS: tile kt + STAGES - 1 is requested
// once tile kt - 1 is read, and a wave waits only for tile kt's loads, so STAGES - 1 tiles of
// latency are covered; another workgroup of the CU (PER_CU = 2) runs under the rest.  Stages
// and K per stage measured: 128 x 128 tiles, one round of 256 (1024 tokens at width 4096,
// output): 2 stages 63 us, 3 stages 46.5, 4 stages 47; 64 x 64 (200 tokens, width 4096): 4
// stages 33 us, 5 stages 33, 8 stages 41 (one workgroup per CU), 128 of K per stage 34 to 40.
template <class Epi, int BM_, int BN_, int STAGES, int GM, int PER_CU>
__global__ __launch_bounds__(256, PER_CU) void gemm_small(const uint16_t* __restrict__ A, WRows W, int M, int N, int K,
                                                    int splits, Epi epi) {
    constexpr int ROWS = BM_ + BN_, LPT = ROWS / 32;   // LDS rows of a stage, loads per wave and tile
    constexpr int MB = BM_ / 64, NB = BN_ / 64;
    static_assert((MB == 2 && NB == 2) || (MB == 1 && NB == 1), "fragment reads are written for these tiles");
    __shared__ u32x4 lds[STAGES * ROWS * 8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, hi = lane >> 5;

    const int ntm = (M + BM_ - 1) / BM_, ntn = (N + BN_ - 1) / BN_;
    const int lid0 = xcd_remap(blockIdx.x, gridDim.x);
    const int split = __builtin_amdgcn_readfirstlane(lid0 / (ntm * ntn));
    int tm, tn;
    tile_of(lid0 - split * (ntm * ntn), ntm, ntn, GM, tm, tn);
    const int m0 = tm * BM_, n0 = tn * BN_;
    const int kt0 = __builtin_amdgcn_readfirstlane(split * (K / BK) / splits);
    const int nk = __builtin_amdgcn_readfirstlane((split + 1) * (K / BK) / splits) - kt0, kofs = kt0 * BK;
    epi.set_split(split);

    const __amdgpu_buffer_rsrc_t ra = row_rsrc(A + (size_t)m0 * K, min(M - m0, BM_), K);
    const __amdgpu_buffer_rsrc_t rb = row_rsrc(w_block(W, n0 & ~127, K), 128, K);
    // LDS rows 8 u .. 8 u + 7 (u = wave * LPT + j): A's rows, then B's.
    uint32_t goff[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int r = 8 * (wave * LPT + j) + (lane >> 3);
        int row = r;
        if (r >= BM_) {
            row = r - BM_;
            if (BN_ == 64) row = Epi::kPairedCols ? (n0 & 64) / 2 + (row & 31) + 2 * (row & 32) : (n0 & 64) + row;
        }
        goff[j] = (uint32_t)(row * K + kofs + 8 * swz(r, lane & 7)) * 2u;
    }
    auto issue = [&](int kt, int stg) __attribute__((always_inline)) {
        u32x4* dst = &lds[(stg * ROWS + 8 * wave * LPT) * 8];
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            if (8 * (wave * LPT + j) < BM_)
                load_1k(ra, dst + 64 * j, goff[j], kt * BK * 2);
            else
                load_1k(rb, dst + 64 * j, goff[j], kt * BK * 2);
        }
    };
    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x16{};

    // Tiles past the last one are requested again as the last: the wait counts stay the same
    // and their stages are never read.
#pragma unroll
    for (int t = 0; t < STAGES - 1; ++t) issue(min(t, nk - 1), t);
    int stg = 0;
    for (int kt = 0; kt < nk; ++kt) {
        vm_wait<LPT * (STAGES - 2)>();
        slot_end();   // tile kt has landed for every wave, and every wave has read tile kt - 1
        issue(min(kt + STAGES - 1, nk - 1), stg == 0 ? STAGES - 1 : stg - 1);
        uint32_t aa[4], ab[4];
        const uint32_t base = (uint32_t)(uintptr_t)&lds[0] + stg * (ROWS * 128);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const uint32_t c = (uint32_t)(((2 * ks + hi) ^ ((l32 >> 1) & 7)) * 16);
            aa[ks] = base + (wm * (BM_ / 2) + l32) * 128 + c;
            ab[ks] = base + (BM_ + wn * (BN_ / 2) + l32) * 128 + c;
        }
        if constexpr (MB == 2) {
            Frag fa[2], fb[2];
            read_a2b2(fa, fb, aa, ab);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = mfma32x32x16(as_bf16x8(fa[i][ks]), as_bf16x8(fb[j][ks]), acc[i][j]);
        } else {
            Frag fa, fb;
            read_a1b1(fa, fb, aa, ab);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) acc[0][0] = mfma32x32x16(as_bf16x8(fa[ks]), as_bf16x8(fb[ks]), acc[0][0]);
        }
        stg = stg + 1 == STAGES ? 0 : stg + 1;
    }
    vm_wait<0>();
    __syncthreads();   // no load into LDS is in flight and every fragment is read
    static_assert(BM_ * BN_ * 4 <= STAGES * ROWS * 128, "the tile is staged in one pass");
    char* st = (char*)&lds[0];
    typename Epi::template Pre<BM_, BN_, 256> pre;
    epi.template prefetch<BM_, BN_, 256>(m0, n0, tid, M, N, pre);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) st_block<BN_>(st, acc[i][j], wm * (BM_ / 2) + 32 * i, wn * (BN_ / 2) + 32 * j, lane);
    __syncthreads();
    epi.template flush<BM_, BN_, 256>(m0, n0, tid, M, N, st, pre);
}

// Estimated time (us) of a product on each tile, k = K / 1024, t = number of tiles: fitted to
// the layer projections at widths 2048, 4096 and 8192 and 64 to 16384 tokens with weights read
// from HBM.  The 256 x 256, 128 x 256 and 128 x 128 tiles have a CU to themselves: a round
// takes longer with every CU busy than with few (the matrix cores' clock falls, the epilogues
// share the HBM).  The 64 x 64 tiles run two workgroups per CU.  Measured (us; big / half /
// 128 / 64): 200 tokens at width 4096, Q|K|V 79 / 56 / 44 / 33; 1024 tokens at 2048, output
// 42 / 33 / 26 / 21; 1024 tokens at 4096, Q|K|V 84 / 62 / 88 / 97; 3000 tokens at 2048, output
// 43 / 34 / 47 / 49, Q|K|V 56 / 67 / 72 / 91; 8192 tokens at 8192, output 757 / 963 / - / -.
enum Tile { kBig, kHalf, kMid, kLow };
struct Pick {
    Tile tile;
    float us;
};
int64_t tiles(int M, int N, int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn); }
Pick pick_tile(int M, int N, int K, int splits) {
    const float k = (float)K / (float)splits / 1024.f;
    auto rounds = [&](int64_t t, float full, float least, float load) {
        return (float)(t / 256) * full + (t % 256 ? least + (float)(t % 256) / 256.f * load : 0.f);
    };
    Pick p{kBig, rounds(tiles(M, N, 256, 256) * splits, 17.5f + 21.7f * k, 13.f + 13.5f * k, 4.5f + 8.2f * k)};
    const float half = rounds(tiles(M, N, 128, 256) * splits, 10.5f + 13.4f * k, 3.f + 13.3f * k, 7.f);
    if (half < p.us) p = {kHalf, half};
    const float mid = rounds(tiles(M, N, 128, 128) * splits, 10.f + 9.5f * k, 5.5f + 9.5f * k, 2.5f);
    if (mid < p.us) p = {kMid, mid};
    const float low = std::max(2.f + 5.5f * k, (float)(tiles(M, N, 64, 64) * splits) / 512.f * (3.f + 7.5f * k));
    if (low < p.us) p = {kLow, low};
    return p;
}

template <class Epi>
hipError_t launch(const uint16_t* A, const WRows& W, int M, int N, int K, const Epi& epi,
                  hipStream_t st, int splits = 1) {
    if (M < 1 || N % 128 || K % BK || splits < 1 || splits > K / BK)
        return hipErrorInvalidValue;
    switch (pick_tile(M, N, K, splits).tile) {
        case kBig:
            hipLaunchKernelGGL(gemm_big<Epi>, dim3(tiles(M, N, 256, 256) * splits), dim3(kBigNT), 0, st, A, W, M, N, K,
                               splits, epi);
            break;
        case kHalf:
            hipLaunchKernelGGL(gemm_half<Epi>, dim3(tiles(M, N, 128, 256) * splits), dim3(kBigNT), 0, st, A, W, M, N, K,
                               splits, epi);
            break;
        case kMid:
            hipLaunchKernelGGL((gemm_small<Epi, 128, 128, 3, 8, 1>), dim3(tiles(M, N, 128, 128) * splits), dim3(256), 0,
                               st, A, W, M, N, K, splits, epi);
            break;
        case kLow:
            hipLaunchKernelGGL((gemm_small<Epi, 64, 64, 4, 16, 2>), dim3(tiles(M, N, 64, 64) * splits), dim3(256), 0, st,
                               A, W, M, N, K, splits, epi);
            break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t gemm_qkv_bf16(const uint16_t* x, const WRows& w, int M, int N, int K, const QkvOut& o,
                         hipStream_t st) {
    return launch(x, w, M, N, K, QkvEpi{o}, st);
}

hipError_t gemm_resid_bf16(const uint16_t* a, const uint16_t* w, const void* x_res, bool x_f32,
                           uint16_t* y, float* yf, int M, int N, int K, hipStream_t st) {
    WRows W{{w, nullptr, nullptr}, {N, 0, 0}};
    if (x_f32) return launch(a, W, M, N, K, ResidEpi<true>{x_res, y, yf}, st);
    return launch(a, W, M, N, K, ResidEpi<false>{x_res, y, yf}, st);
}

hipError_t gemm_out_bf16(const uint16_t* a, const uint16_t* w, int M, int N, int K, uint16_t* c,
                         hipStream_t st) {
    WRows W{{w, nullptr, nullptr}, {N, 0, 0}};
    return launch(a, W, M, N, K, OutEpi<true>{c, nullptr, nullptr, M, 0, 0, 0}, st);
}

hipError_t gemm_out_f32(const uint16_t* a, const uint16_t* w, int M, int N, int K, int splits, float* part, float* dst0,
                        int rows0, float* dst1, int rows1, float* dst2, hipStream_t st) {
    WRows W{{w, nullptr, nullptr}, {N, 0, 0}};
    if (splits == 1) return launch(a, W, M, N, K, OutEpi<false>{dst0, dst1, dst2, rows0, rows1, 0, 0}, st);
    return launch(a, W, M, N, K, OutEpi<false>{part, nullptr, nullptr, M, 0, (size_t)M * N, 0}, st, splits);
}

// Splitting K adds workgroups and shortens their chain, and pays for the fp32 planes: written,
// read again and summed by a kernel of its own (about 5 us and 4.5 TB/s).
int gemm_out_splits(int M, int N, int K, size_t part_floats) {
    int best = 1;
    float t = pick_tile(M, N, K, 1).us;
    for (int s = 2; s <= 8 && s <= K / BK && (size_t)s * M * N <= part_floats; s *= 2) {
        const float u = pick_tile(M, N, K, s).us + 5.f + (float)(s + 1) * (float)M * (float)N * 4.f / 4.5e6f;
        if (u < t) {
            t = u;
            best = s;
        }
    }
    return best;
}

}  // namespace kvp
