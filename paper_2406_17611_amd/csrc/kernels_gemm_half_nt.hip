// Input gradients of eq. (2) for fp32-stored activations whose reduction takes 65 to 512 steps (hidden layers), dM = dZ H^T and with two taps
// dZ H0^T, from the two scaled fp16 terms of kernels_gemm_half.hip (same products; a row of dZ has one scale, that of its largest value, which
// is known before the first product, so that no sum ever follows a smaller one).
//
// The weights stay in registers: a wavefront holds 32 columns of them (16 beyond 256 steps), both terms, 128 registers, for all the rows
// that its workgroup walks over. Blocks of 32 rows (64 up to 128 steps) come in whole rows, 16 lanes to one, one block ahead in registers; they
// are masked, scaled and split once for the eight wavefronts and lie in LDS as the matrix unit reads them, [stage][term][16 rows][eight steps][row],
// rows swapped by their place so that neither writes nor reads meet in a bank; two buffers, one barrier per block. One half of the
// wavefronts splits the next block while the other multiplies, and the other way round: every SIMD holds one of either half.
// v_mfma_f32_16x16x32_f16 rather than 32x32x16: its result is ready after half the time, and one wavefront alone keeps the matrix unit busy. The
// weights are the first operand: a lane then holds four consecutive columns of a row and stores them together.
// Bound by the memory (a read of dZ and of what masks it, a write per tap): 4.3 to 5.4 TB/s of them (matrix units 42 % busy, vector ALUs 39 %). 128 x 128 tiles that each split their rows again and fetch
// weights by stage / this, us, masked:
//   2,449,029 rows 256 -> 256 two taps 3,530 / 2,340, one 2,050 / 1,400     169,343 rows 256 -> 256 one tap 142 / 104, 128 -> 128 50 / 48
//   410,003 rows 256 -> 256 two taps 607 / 468, 512 -> 256 two taps 1,161 / 912     50,021 rows 136 -> 200 two taps 64 / 41
//   1,000,000 rows 96 -> 64 two taps 274 / 236; at 64 steps and below the tiles are level or ahead (30,000 rows 17 -> 64 8.5 / 9.6, 2,449,029 rows
//   47 -> 256 two taps 1,490 / 1,560)
// The last rows and columns are stored four columns at a time like the others: element by element, the remainder alone took a launch of few blocks 2 to 4 us
// (3,000 rows 72 -> 256 12.2 / 8.2, two taps 13.6 / 8.7, 6,000 rows 96 -> 256 11.6 / 8.6, 45,000 rows 256 -> 200 29.3 / 27.4).
// (Measured and not kept: rows in registers and weights through LDS, 6,100 us for the first; 32x32x16 instructions, whose two sums wait for each other, 3,190;
// both halves in step, 2,590.)
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "gemm_tile.h"
#include "half_terms.h"
#include "varco_internal.h"

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kUnits = 256;          // compute units: one workgroup is resident on each
constexpr int kRows = 32;            // rows of a block
constexpr int kStage = 32;           // reduction steps of a stage of the weights' split copy
constexpr int kShortest = 64;        // reductions up to this many steps are left to kernels_gemm_half.hip (figures above)

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float any4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t words4 __attribute__((ext_vector_type(4)));

struct InputGrad {
    const float *a, *gate;
    int64_t lda;
    int32_t m, n, k;
    const uint16_t* b[2];            // split copies of the weights
    int32_t tile_rows;               // rows of a tile of theirs
    int64_t pitch, exps;             // their padded reduction length; place of the scale exponents (elements)
    float* c[2];
    int64_t ldc;
    int32_t accumulate;
    int32_t units, all_units;        // columns of a wavefront: so many in one product, and in all
    int32_t groups, stride;          // groups of eight wavefronts; workgroups of a group
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_at(const float* p, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, 0x00027000);
}

// Blocks of 32 rows that a workgroup takes at a time (as many values whatever the reduction's length), and tiles of 16 columns that a
// wavefront holds the weights of (128 registers), for a reduction of `stages` stages of 32 steps.
constexpr int row_blocks(int stages) { return stages <= 4 ? 2 : 1; }
constexpr int column_tiles(int stages) { return stages <= 8 ? 2 : 1; }

template <int KT, bool GATE>
__global__ __launch_bounds__(kThreads, 2) void input_grad_kernel(InputGrad g) {
    constexpr int J = (KT + 1) / 2, RB = row_blocks(KT), ROWS = kRows * RB, RT = 2 * RB;      // loads of a row's lane, tiles of 16 rows
    constexpr int CT = column_tiles(KT), CW = 16 * CT;                          // tiles of 16 columns of a wavefront
    constexpr int kBlock = KT * 2 * RT * 512;                                   // fp16 elements: [stage][term][row tile][eight steps][row]
    __shared__ __attribute__((aligned(16))) uint16_t smem[2][kBlock];
    __shared__ __attribute__((aligned(16))) int32_t exps[2][ROWS];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3, group = within % g.groups;
    const int32_t first = (within / g.groups) * 8 + xcd, n_blocks = (g.m + ROWS - 1) / ROWS;
    if (first >= n_blocks || first >= g.stride) return;         // whole workgroup

    // this wavefront's columns of the weights
    const int32_t unit0 = group * kWaves + wave;
    const bool mine = unit0 < g.all_units;
    const int32_t unit = min(unit0, g.all_units - 1), p = unit >= g.units ? 1 : 0, n0 = (unit - p * g.units) * CW;
    halfx8 w0[KT][CT], w1[KT][CT];
    int4 eb[CT];
    {
        const int32_t plane = g.tile_rows * kStage;             // elements of a stage's term
        const uint16_t* const at = g.b[p] + int64_t(n0 / g.tile_rows) * (g.pitch / kStage) * 2 * plane + (n0 % g.tile_rows + l16) * kStage + lg * 8;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                w0[t][ct] = w1[t][ct] = halfx8{};
                if (KT > 8 && t * kStage >= g.pitch) continue;      // (an odd number of stages)
                w0[t][ct] = __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4*>(at + 2 * t * plane + ct * 16 * kStage));
                w1[t][ct] = __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4*>(at + (2 * t + 1) * plane + ct * 16 * kStage));
            }
            eb[ct] = *reinterpret_cast<const int4*>(reinterpret_cast<const int32_t*>(g.b[p] + g.exps) + n0 + ct * 16 + 4 * lg);
        }
    }

    // rows of A: a group of 16 lanes holds a row, every lane four values of every 64
    float4 x[RB][J], y[GATE ? RB : 1][GATE ? J : 1];
    const int32_t row_bytes = int32_t(g.lda) * 4, k_last = 64 * (J - 1) + 4 * l16;
    const uint32_t off = uint32_t(lg) * uint32_t(row_bytes) + 16u * uint32_t(l16), off_last = k_last < g.k ? off + 256u * (J - 1) : 0x7FFFFFF0u;
    auto fetch = [&](int32_t block) __attribute__((always_inline)) {          // (rows that do not exist: no bytes, zeros)
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int32_t row = block * ROWS + (wave * RB + i) * 4, rows = min(4, g.m - row);
            const int32_t bytes = rows > 0 ? (rows - 1) * row_bytes + g.k * 4 : 0;
            const auto from = row_at(g.a + int64_t(row) * g.lda, bytes), mask = row_at(GATE ? g.gate + int64_t(row) * g.lda : g.a, bytes);
#pragma unroll
            for (int j = 0; j < J; ++j) {
                x[i][j] = __builtin_bit_cast(float4, words4(__builtin_amdgcn_raw_buffer_load_b128(from, j + 1 < J ? off : off_last, j + 1 < J ? 256 * j : 0, 0)));
                if constexpr (GATE) y[i][j] = __builtin_bit_cast(float4, words4(__builtin_amdgcn_raw_buffer_load_b128(mask, j + 1 < J ? off : off_last, j + 1 < J ? 256 * j : 0, 0)));
            }
        }
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            float m = 0.f;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                float4& v = x[i][j];
                if constexpr (GATE) {
                    v.x = y[i][j].x > 0.f ? v.x : 0.f, v.y = y[i][j].y > 0.f ? v.y : 0.f;
                    v.z = y[i][j].z > 0.f ? v.z : 0.f, v.w = y[i][j].w > 0.f ? v.w : 0.f;
                }
                if (j + 1 == J && (g.k & 3)) {                  // past the row's end: the next row's values
                    const int left = g.k - k_last;
                    v.y = left > 1 ? v.y : 0.f, v.z = left > 2 ? v.z : 0.f, v.w = left > 3 ? v.w : 0.f;
                }
                m = fmaxf(fmaxf(fmaxf(m, fabsf(v.x)), fmaxf(fabsf(v.y), fabsf(v.z))), fabsf(v.w));
            }
            const int e = scale_exponent(largest_of_lanes<16>(m), kHalfTop), row = (wave * RB + i) * 4 + lg;
            const float sc = power_of_two(e);
            if (l16 == 0) exps[buf][row] = e;
            uint16_t* const at = &smem[buf][((l16 >> 3) * 2 * RT + (row >> 4)) * 512 + ((l16 >> 1 & 3) * 16 + ((row & 15) ^ (l16 & 14))) * 8 + (l16 & 1) * 4];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const float4 v = x[i][j];
                uint32_t h[2], l[2];
                split_pair(v.x * sc, v.y * sc, h[0], l[0]);
                split_pair(v.z * sc, v.w * sc, h[1], l[1]);
                if (KT % 2 == 0 || j + 1 < J || l16 < 8) {
                    *reinterpret_cast<uint2*>(at + j * 4 * RT * 512) = make_uint2(h[0], h[1]);
                    *reinterpret_cast<uint2*>(at + (j * 4 + 1) * RT * 512) = make_uint2(l[0], l[1]);
                }
            }
        }
    };
    fetch(first);
    stash(0);
    fetch(first + g.stride);
    __syncthreads();

    const bool early = wave >= kWaves / 2;
    int buf = 0;
    for (int32_t block = first; block < n_blocks; block += g.stride, buf ^= 1) {
        auto next = [&]() __attribute__((always_inline)) {
            stash(buf ^ 1);
            fetch(block + 2 * g.stride);
        };
        if (early) next();
        floatx4 acc[RT][CT], low[RT][CT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = low[rt][ct] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (mine) {
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const uint16_t* const at = &smem[buf][t * 2 * RT * 512 + (lg * 16 + (l16 ^ (2 * lg + 8 * (t & 1)))) * 8];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const halfx8 a0 = __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4*>(at + rt * 512));
                    const halfx8 a1 = __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4*>(at + (RT + rt) * 512));
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w0[t][ct], a0, acc[rt][ct], 0, 0, 0);
                        low[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[t][ct], a0, low[rt][ct], 0, 0, 0);
                    }
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) low[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w0[t][ct], a1, low[rt][ct], 0, 0, 0);
                }
            }
        }
        if (!early) next();
        if (mine) {
            float* const c = g.c[p] + int64_t(block) * ROWS * g.ldc + n0;
            const bool inside = (block + 1) * ROWS <= g.m && n0 + CW <= g.n;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int row = rt * 16 + l16, ea = exps[buf][row];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const int e[4] = {eb[ct].x, eb[ct].y, eb[ct].z, eb[ct].w};
                    floatx4 o;
#pragma unroll
                    for (int v = 0; v < 4; ++v) o[v] = __builtin_ldexpf(acc[rt][ct][v] + low[rt][ct][v] * (1.f / kHalfLow), -(ea + e[v]));
                    const int col = ct * 16 + 4 * lg;
                    float* const dst = c + int64_t(row) * g.ldc + col;
                    if (!inside && block * ROWS + row >= g.m) continue;
                    if (inside || n0 + col + 4 <= g.n) {
                        if (g.accumulate) o += *reinterpret_cast<const any4*>(dst);
                        *reinterpret_cast<any4*>(dst) = o;
                    } else {
#pragma unroll
                        for (int v = 0; v < 3; ++v)
                            if (n0 + col + v < g.n) dst[v] = g.accumulate ? dst[v] + o[v] : o[v];
                    }
                }
            }
        }
        __syncthreads();
    }
}

// How the columns of both products are dealt: wavefronts' shares, groups of eight of them, and workgroups of a group.
struct Groups {
    int32_t units, all_units, groups, stride;
};
Groups groups_of(const GemmArgs& ga, int stages) {
    const int32_t cw = 16 * column_tiles(stages), units = (ga.n + cw - 1) / cw, all = units * (ga.c_dual ? 2 : 1), groups = (all + kWaves - 1) / kWaves;
    return {units, all, groups, std::max(8, kUnits / groups / 8 * 8)};
}

template <class F>
void with_flag(bool b, F&& f) {
    if (b)
        f(std::true_type{});
    else
        f(std::false_type{});
}

}  // namespace

bool varco_gemm_half_nt_usable(const GemmArgs& ga) {
    if (ga.a.transposed || ga.k <= kShortest || ga.k > 16 * kStage || !varco_gemm_half_usable(ga)) return false;
    // The tiles of kernels_gemm_half.hip are ahead where wavefronts here have no columns to multiply and the launch is a chain of blocks: `rounds` of them,
    // while `tiles` workgroups, 512 of which are resident, do their share at once. Same accuracy. Time of the tiles / of the rows, us:
    const int stages = (ga.k + kStage - 1) / kStage, taps = ga.c_dual ? 2 : 1, n_tile = ga.n <= 64 ? 64 : 128;
    const Groups at = groups_of(ga, stages);
    const int32_t rows = kRows * row_blocks(stages), rounds = ((ga.m + rows - 1) / rows + at.stride - 1) / at.stride;
    const int64_t tiles = (int64_t(ga.m) + 127) / 128 * ((ga.n + n_tile - 1) / n_tile) * taps;
    if (ga.n <= 64) {
        // up to 128 steps: 24,000 rows 80 -> 16 6.6 / 9.5, 80 -> 64 7.0 / 9.6, two taps 80 -> 16 8.3 / 10.0, 56,000 rows 96 -> 16 11.0 / 14.9. More tiles than are
        // resident: one tap 220,000 rows 96 -> 16 30.6 / 40.9, 65,536 rows 128 -> 48 16.3 / 19.0, but 110,000 rows 120 -> 32, whose rows begin inside
        // lines, 29.3 / 24.4, two taps 96 -> 32 24.6 / 23.0, and beyond four rounds of tiles 600,000 rows 80 -> 32 101 / 88. Rows that are not whole
        // 32 bytes cost the tiles more: 24,000 rows 100 -> 32 8.8 / 9.8, but 2,000 rows 8.4 / 7.2.
        const bool wave_after_wave = taps == 1 && (ga.k % kStage == 0 || ga.k <= 80);
        if (stages <= 4 && tiles <= (wave_after_wave ? 2048 : 512) && (ga.k % 8 == 0 || rounds > 1)) return false;
        // more steps: 30,000 rows 224 -> 32 12.9 / 14.8, 192 -> 16 11.6 / 12.8; 20,000 rows (three rounds) 240 -> 32 14.0 / 12.9; 40,000 rows, more
        // tiles than compute units, 22.0 / 18.1
        if (taps == 1 && rounds > 3 && tiles <= 256) return false;
    } else if (stages <= 4 && tiles <= 512 && rounds > 1 && ga.n % 128 == 0 && at.all_units > kWaves && at.all_units % kWaves) {
        return false;                  // a last group with idle wavefronts, whole tiles: 10,000 rows 96 -> 384 9.8 / 13.0, 20,000 rows 13.3 / 17.0; one round: 8,000 rows 128 -> 384 12.0 / 10.2
    }
    return true;
}

hipError_t varco_launch_gemm_half_nt(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag) {
    auto f32 = [](const void* p) { return static_cast<const float*>(p); };
    InputGrad g{};
    g.m = ga.m, g.n = ga.n, g.k = ga.k;
    g.a = f32(ga.a.ptr), g.gate = f32(ga.a.gate), g.lda = ga.a.ld;
    g.b[0] = static_cast<const uint16_t*>(ga.b_prep), g.b[1] = static_cast<const uint16_t*>(ga.b_dual_prep);
    g.tile_rows = ga.n <= 64 ? 64 : 128;
    g.pitch = ga.b_prep_ld, g.exps = 2 * ga.b_prep_plane;
    g.c[0] = static_cast<float*>(ga.c), g.c[1] = static_cast<float*>(ga.c_dual), g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0;
    tag.begin(stream);
    auto go = [&](auto kt) {
        constexpr int KT = decltype(kt)::value, ROWS = kRows * row_blocks(KT);
        const Groups at = groups_of(ga, KT);
        g.units = at.units, g.all_units = at.all_units, g.groups = at.groups, g.stride = at.stride;
        const dim3 grid{unsigned((std::min(g.stride, (ga.m + ROWS - 1) / ROWS) + 7) / 8 * 8 * g.groups)};
        with_flag(ga.a.gate != nullptr, [&](auto gt) {
            hipLaunchKernelGGL((input_grad_kernel<KT, decltype(gt)::value>), grid, dim3(kThreads), 0, stream, g);
        });
    };
    using std::integral_constant;
    switch ((ga.k + kStage - 1) / kStage) {
        case 3: go(integral_constant<int, 3>{}); break;
        case 4: go(integral_constant<int, 4>{}); break;
        case 5: go(integral_constant<int, 5>{}); break;
        case 6: go(integral_constant<int, 6>{}); break;
        case 7: go(integral_constant<int, 7>{}); break;
        case 8: go(integral_constant<int, 8>{}); break;
        case 9:
        case 10: go(integral_constant<int, 10>{}); break;
        case 11:
        case 12: go(integral_constant<int, 12>{}); break;
        case 13:
        case 14: go(integral_constant<int, 14>{}); break;
        default: go(integral_constant<int, 16>{});
    }
    tag.end(stream);
    return hipGetLastError();
}
