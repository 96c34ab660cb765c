// The copies of the weights that the matrix kernels read: device side (kernels_gemm_split.hip, kernels_spmm.hip).
#pragma once

#include "elem.h"
#include "gemm_tile.h"
#include "half_terms.h"
#include "varco_internal.h"

// Weight copies (see PrepJob). Copies in terms: element (term p, row r, column c) sits at
//   (((r / bn) * (pitch / kPrepStage) + c / kPrepStage) * terms + p) * bn * kPrepStage + (r % bn) * kPrepStage + c % kPrepStage,
// bn = rows of a B tile (64 for at most 64 rows, else 128). Behind two fp16 terms (rows_padded * pitch * 2 elements) follow the
// scale exponents of the rows as 32-bit integers; there a workgroup takes 32 rows, looks for the largest value of each and splits them.
// All copies of a step are made by one launch, on small graphs by the one of the first aggregation: a copy is a few
// thousand elements, far less than a launch costs.
constexpr int kPrepThreads = 256;
constexpr int kPrepStage = 32;          // reduction steps of a stage
template <int CAP>
struct PrepJobs {
    PrepJob job[CAP];
    int32_t n;
};
// (not transposed) Eight lanes to a row, each with every eighth group of 8 columns: whole lines per load, and the largest value of
// a row is found among the eight.
__device__ __forceinline__ void prep_halves(const PrepJob& jb, int32_t block, int32_t thread) {
    constexpr int HELD = 4;                                          // groups kept in registers between the two passes (256 columns)
    const int32_t r = block * 32 + (thread >> 3), g0 = thread & 7, groups = jb.pitch / 8, bn = jb.rows <= 64 ? 64 : 128;
    const float* const row = jb.h + int64_t(min(r, jb.rows - 1)) * jb.ld;
    auto read = [&](int32_t g, float (&x)[8]) {
        const int32_t left = r < jb.rows ? jb.cols - g * 8 : 0;
        if (left >= 8) {
            const float4 u = load4_at(row, uint32_t(g) * 32u), v = load4_at(row, uint32_t(g) * 32u + 16u);
            x[0] = u.x, x[1] = u.y, x[2] = u.z, x[3] = u.w, x[4] = v.x, x[5] = v.y, x[6] = v.z, x[7] = v.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = i < left ? row[g * 8 + i] : 0.f;
        }
    };
    float held[HELD][8], m = 0.f;
#pragma unroll
    for (int q = 0; q < HELD; ++q) {
        if (g0 + 8 * q < groups) read(g0 + 8 * q, held[q]);
    }
#pragma unroll
    for (int q = 0; q < HELD; ++q)
        if (g0 + 8 * q < groups) {
#pragma unroll
            for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(held[q][i]));
        }
    for (int32_t g = g0 + 8 * HELD; g < groups; g += 8) {
        float x[8];
        read(g, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(x[i]));
    }
#pragma unroll
    for (int d = 4; d; d >>= 1) m = fmaxf(m, __shfl_xor(m, d));
    const int e = scale_exponent(m, kHalfTop);
    const float s = power_of_two(e);
    uint16_t* const out = static_cast<uint16_t*>(jb.out);
    auto write = [&](int32_t g, const float (&x)[8]) {
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) split_pair(x[2 * i] * s, x[2 * i + 1] * s, hi[i], lo[i]);
        const int64_t at = (int64_t(r / bn) * (jb.pitch / kPrepStage) + g * 8 / kPrepStage) * 2;
        uint16_t* const dst = out + at * bn * kPrepStage + (r % bn) * kPrepStage + g * 8 % kPrepStage;
        *reinterpret_cast<uint4*>(dst) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        *reinterpret_cast<uint4*>(dst + bn * kPrepStage) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    };
#pragma unroll
    for (int q = 0; q < HELD; ++q)
        if (g0 + 8 * q < groups) write(g0 + 8 * q, held[q]);
    for (int32_t g = g0 + 8 * HELD; g < groups; g += 8) {
        float x[8];
        read(g, x);
        write(g, x);
    }
    if (g0 == 0) reinterpret_cast<int32_t*>(out + int64_t(jb.rows_padded) * jb.pitch * 2)[r] = e;
}
// What thread `thread` of kPrepThreads does in workgroup `at_block` of all copies (lanes of a wavefront are consecutive threads).
template <int CAP>
__device__ __forceinline__ void prep_weights(const PrepJobs<CAP>& jobs, int32_t at_block, int32_t thread) {
    int32_t at = 0;
    while (at + 1 < jobs.n && at_block >= jobs.job[at + 1].first_block) ++at;
    const PrepJob& jb = jobs.job[at];
    const int32_t block = at_block - jb.first_block;
    if (jb.terms == kHalfTerms) {
        prep_halves(jb, block, thread);
        return;
    }
    const int64_t idx = int64_t(block) * kPrepThreads + thread;
    if (idx >= int64_t(jb.rows_padded) * jb.pitch) return;
    const int32_t r = int32_t(idx / jb.pitch), c = int32_t(idx % jb.pitch);
    float x = 0.f;
    if (r < jb.rows && c < jb.cols) x = jb.transpose ? jb.h[int64_t(c) * jb.ld + r] : jb.h[int64_t(r) * jb.ld + c];
    uint16_t* const out = static_cast<uint16_t*>(jb.out);
    if (jb.terms == 1) {
        out[idx] = float_to_bf16(x);
        return;
    }
    const bool exact = jb.terms == kExactTerms;
    const int32_t bn = jb.rows <= 64 ? 64 : 128, terms = exact ? 3 : jb.terms;
    const int64_t first = (int64_t(r / bn) * (jb.pitch / kPrepStage) + c / kPrepStage) * terms;
    const int32_t inside = (r % bn) * kPrepStage + c % kPrepStage;
    if (exact) {
        // Cut, not rounded: every term has the sign of the value, and none but that of a zero is zero (where one or two terms would do, the last of them is
        // halved), so that an infinite element of a row, or of the weights, gives the infinity or NaN that it gives in one product. The terms add up to
        // values of 2^-109 and more; below, bits under 2^-133 (the smallest bf16 number, which stands in for a zero term too) are lost: 2^-131 in all.
        auto cut = [](float v) { return __uint_as_float(__float_as_uint(v) & 0xFFFF0000u); };
        const uint32_t sign = __float_as_uint(x) & 0x80000000u;
        const bool number = isfinite(x), some = x != 0.f;
        float t[3] = {x != x ? __uint_as_float(0x7FC00000u) : cut(x)};                         // (a NaN whose upper bits say infinity)
        const float rest = number ? x - t[0] : 0.f;
        t[1] = cut(rest), t[2] = cut(rest - t[1]);
        if (number && t[1] == 0.f) t[1] = t[0] = 0.5f * t[0];
        if (number && t[2] == 0.f) t[2] = t[1] = 0.5f * t[1];
        for (int p = 0; p < 3; ++p) {
            uint32_t u = __float_as_uint(t[p]) >> 16;
            if (some && (u & 0x7FFFu) == 0u) u = sign >> 16 | 1u;
            out[(first + p) * bn * kPrepStage + inside] = uint16_t(u);
        }
        return;
    }
    for (int p = 0; p < terms; ++p) {
        const uint16_t t = float_to_bf16(x);
        out[(first + p) * bn * kPrepStage + inside] = t;
        x -= __uint_as_float(uint32_t(t) << 16);
    }
}
