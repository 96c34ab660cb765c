// What the kernels of split fp32 products share (kernels_gemm_split.hip, kernels_gemm_half.hip): loads from a uniform base and a
// lane's byte offset, and the way of a tile of 32 x 32 blocks to memory.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

template <typename T>
__device__ __forceinline__ T load_at(const void* base, uint32_t byte_offset) {
    return *reinterpret_cast<const T*>(static_cast<const char*>(base) + byte_offset);
}
// Four floats from any address of a float (the device loads 16 bytes from there just as well).
__device__ __forceinline__ float4 load4_at(const void* base, uint32_t byte_offset) {
    typedef float any4 __attribute__((ext_vector_type(4), aligned(4)));
    const any4 v = *reinterpret_cast<const any4*>(static_cast<const char*>(base) + byte_offset);
    return make_float4(v[0], v[1], v[2], v[3]);
}

// Stores a wavefront's blocks: accumulator register v of a lane is element (8 * (v / 4) + 4 * (lane / 32) + v % 4, lane % 32) of block
// (i, j), whose first element is (row0 + 32 i, col0 + 32 j) of C (m x n, rows `pitch` apart). inside: the workgroup's tile lies wholly
// inside C (all but the last row and column of tiles). It is then stored through one scalar
// base per output row plus one 32-bit lane offset, so that the address arithmetic
// runs on the scalar unit and the vector unit only sees the loads, adds and stores; the edge tiles take the
// path with per-element tests and clamped addresses. When C is added to, the old values of a block are fetched
// by loads that are all issued before the first one is used, not one round trip per element.
template <int TMB, int TNB>
__device__ __forceinline__ void store_tile(const float __attribute__((ext_vector_type(16))) (&acc)[TMB][TNB], float* base, int64_t pitch, int32_t m, int32_t n,
                                           int32_t row0, int32_t col0, bool inside, int lane, bool add_old, bool relu) {
    const int lrow = lane & 31, lk = lane >> 5;
    if (inside) {
        float* const tile = base + int64_t(row0) * pitch + col0;                        // scalar
        const uint32_t lane_off = uint32_t(4 * lk) * uint32_t(pitch) + uint32_t(lrow);  // a tile spans < 2^32 elements
#pragma unroll
        for (int i = 0; i < TMB; ++i) {
#pragma unroll
            for (int j = 0; j < TNB; ++j) {
                float old[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) old[v] = 0.f;
                if (add_old) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        old[v] = (tile + int64_t(i * 32 + 8 * (v >> 2) + (v & 3)) * pitch + j * 32)[lane_off];
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float x = acc[i][j][v] + old[v];
                    if (relu) x = fmaxf(x, 0.f);
                    (tile + int64_t(i * 32 + 8 * (v >> 2) + (v & 3)) * pitch + j * 32)[lane_off] = x;
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TMB; ++i) {
#pragma unroll
        for (int j = 0; j < TNB; ++j) {
            float* ptr[16];
            bool ok[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int32_t row = row0 + i * 32 + 4 * lk + 8 * (v >> 2) + (v & 3), col = col0 + lrow + j * 32;
                ok[v] = row < m && col < n;
                ptr[v] = base + int64_t(min(row, m - 1)) * pitch + min(col, n - 1);
            }
            float old[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) old[v] = 0.f;
            if (add_old) {
#pragma unroll
                for (int v = 0; v < 16; ++v) old[v] = *ptr[v];
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float x = acc[i][j][v] + old[v];
                if (relu) x = fmaxf(x, 0.f);
                if (ok[v]) *ptr[v] = x;
            }
        }
    }
}
