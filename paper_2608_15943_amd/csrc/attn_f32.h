// Tiles of the fp32 attention kernels (forward and backward): 16 queries x 16 keys per
// wave.  Lane (r = lane / 4, c = lane % 4) holds the entries (row r, columns 4 c .. 4 c + 3)
// of a score tile and, of a 16-row accumulator, row r at dims 16 i + 4 c .. + 3.  Staged rows
// are D + 4 floats, so that 16 rows at one dim spread over the LDS banks.
//
// The small full-precision models are bound by latency and by the length of one wave's chain
// of tiles, not by arithmetic: the four waves of a workgroup take every fourth tile and their
// results are added in wave order, and the next tile's rows are requested before the current
// tile is multiplied.
#pragma once

#include "common.h"

namespace kvp {
namespace {

constexpr int FT = 16;   // tile edge

template <int D>
struct F32Tile {
    static constexpr int P = D + 4;
    float v[FT * P];
};

// LDS written and read by one wave: in order in hardware, kept in order for the compiler.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 16 rows of D floats (row stride ld) by NT threads, through registers; rows >= n are zeros.
template <int D, int NT>
struct RowLoad {
    static constexpr int PER = FT * D / 4 / NT > 0 ? FT * D / 4 / NT : 1;
    f32x4 x[PER];
    __device__ __forceinline__ void load(const float* src, size_t ld, int n, int tid) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int id = tid + NT * i, row = id / (D / 4), c = id % (D / 4);
            x[i] = f32x4{};
            if (row < n) x[i] = *(const f32x4*)(src + (size_t)row * ld + 4 * c);   // n <= 16
        }
    }
    __device__ __forceinline__ void store(F32Tile<D>& t, int tid) const {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int id = tid + NT * i, row = id / (D / 4), c = id % (D / 4);
            if (row < FT) *(f32x4*)&t.v[row * F32Tile<D>::P + 4 * c] = x[i];
        }
    }
};

// Positions 0 .. n - 1 (n <= 16) of a transposed slot [D][cap] at src, stored position-major.
template <int D, int NT>
struct ColLoad {
    static constexpr int PER = FT * D / NT;
    float x[PER];
    __device__ __forceinline__ void load(const float* src, size_t cap, int n, int tid) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int id = tid + NT * i, key = id % FT, d = id / FT;
            x[i] = key < n ? src[(size_t)d * cap + key] : 0.f;
        }
    }
    __device__ __forceinline__ void store(F32Tile<D>& t, int tid) const {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int id = tid + NT * i;
            t.v[(id % FT) * F32Tile<D>::P + id / FT] = x[i];
        }
    }
};

// s[e] = sum_d a[r][d] b[4 c + e][d], d in order.
template <int D>
__device__ __forceinline__ void dot_tile(const F32Tile<D>& a, const F32Tile<D>& b, int r, int c, float (&s)[4]) {
    constexpr int P = F32Tile<D>::P;
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = 0.f;
#pragma unroll 2
    for (int d = 0; d < D; d += 4) {
        const f32x4 x = *(const f32x4*)&a.v[r * P + d];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const f32x4 y = *(const f32x4*)&b.v[(4 * c + e) * P + d];
#pragma unroll
            for (int i = 0; i < 4; ++i) s[e] = fmaf(x[i], y[i], s[e]);
        }
    }
}

// acc[i] += w * row `row` of t at dims 16 i + 4 c.
template <int D>
__device__ __forceinline__ void add_row(f32x4 (&acc)[D / 16], const F32Tile<D>& t, int row, int c, float w) {
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
        const f32x4 y = *(const f32x4*)&t.v[row * F32Tile<D>::P + 16 * i + 4 * c];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][e] = fmaf(w, y[e], acc[i][e]);
    }
}
__device__ __forceinline__ float quad_max(float v) {
    v = fmaxf(v, __shfl_xor(v, 1));
    return fmaxf(v, __shfl_xor(v, 2));
}
__device__ __forceinline__ float quad_sum(float v) {
    v += __shfl_xor(v, 1);
    return v + __shfl_xor(v, 2);
}

}  // namespace
}  // namespace kvp
