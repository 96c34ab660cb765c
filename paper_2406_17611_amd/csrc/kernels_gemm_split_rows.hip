// The dense transform of eq. (2) for fp32-stored activations whose reduction takes 65 to 256 steps (both taps together), act(M H + X H0), from three
// bf16 terms of either operand and six products (kernels_gemm_split.hip: the expansion and what it keeps). The same instructions on the same
// values in the same order as the tiles there, so the same bits: a ReLU whose argument is within rounding of zero decides alike in either. (Summed
// from the smallest product on 16 x 16 x 32 instructions, which round half as often, errors against fp64 are 0.73 to 0.96 of these and 169,343
// rows 256 -> 256 take 117 us; but one gate of a hub that decides otherwise moves the gradients of 50,021 nodes by 1.6e-3 as a whole.)
//
// The weights stay in registers: a wavefront holds 32 columns of them, all terms, of both taps, 24 registers per stage of 32 steps, for all the
// rows that its workgroup walks over. Blocks of 32 rows come in whole rows, 16 lanes to one, from any 4-byte address, one block (of one tap) ahead in
// registers; they are split once for the eight wavefronts and lie in LDS as the matrix unit reads them, [stage][term][16 rows][eight steps][row],
// rows swapped by their place so that neither writes nor reads meet in a bank; two buffers, one barrier per block and tap. One half of the
// wavefronts splits the next block while the other multiplies, and the other way round: every SIMD holds one of either half (all splitting and
// multiplying at once: 900,000 rows 256 -> 256 657 us). The weights are the first operand: a lane then holds four consecutive columns of a row and
// stores them together. Bound by the matrix units' chain of dependent products and, 225 steps and more, by fragments read just before their use,
// for which no registers are left to have more in flight (2,449,029 rows 100 -> 256 two taps: matrix units 59 % busy, vector ALUs 22 %).
// 128 x 128 tiles that each split their rows again and fetch weights by stage / this, us:
//   169,343 rows 256 -> 256 146 / 135     900,000 rows 256 -> 256 653 / 592, 800,000 rows 160 -> 512 787 / 750     300,007 rows 200 -> 200 218 / 170
//   50,021 rows 128 -> 136 two taps 50 / 43     300,007 rows 100 -> 256 two taps 218 / 186     3,001 rows 256 -> 256 20 / 17, 128 -> 256 two taps 20 / 16
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "gemm_tile.h"
#include "varco_internal.h"

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kUnits = 256;          // compute units: one workgroup is resident on each
constexpr int kRows = 32;            // rows of a block
constexpr int kStage = 32;           // reduction steps of a stage
constexpr int kTerms = 3;
constexpr int kColumns = 32;         // columns of a wavefront
constexpr int kMostStages = 8;       // of all taps: 192 registers of weights
constexpr int kTileRows = 128;       // rows of a tile of the expanded weights

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float any4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t words4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct Transform {
    const float* a[2];               // rows of the taps
    int64_t lda;
    int32_t m, n, k;
    const uint16_t* b[2];            // expanded copies of the weights
    int64_t pitch;                   // their padded reduction length
    float* c;
    int64_t ldc;
    int32_t accumulate, relu;
    int32_t units;                   // wavefronts' columns
    int32_t groups, stride;          // groups of eight wavefronts; workgroups of a group
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_at(const float* p, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, 0x00027000);
}

// Two fp32 values: w[p] holds term p of both.
__device__ __forceinline__ void expand2(float x0, float x1, uint32_t (&w)[kTerms]) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int p = 0; p < kTerms; ++p) {
        w[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{x0, x1}), bf16x2));
        if (p + 1 < kTerms) x0 -= __uint_as_float(w[p] << 16), x1 -= __uint_as_float(w[p] & 0xFFFF0000u);
    }
}

// KT: stages of a tap.
template <int KT, int TAPS>
__global__ __launch_bounds__(kThreads, 2) void transform_kernel(Transform g) {
    static_assert(KT * TAPS <= kMostStages, "the weights are 24 registers per stage");
    constexpr int J = (KT + 1) / 2, RT = kRows / 16;
    constexpr int kBlock = KT * kTerms * RT * 512;
    __shared__ __attribute__((aligned(16))) uint16_t smem[2][kBlock];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4, l32 = lane & 31, lk = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3, group = within % g.groups;
    const int32_t first = (within / g.groups) * 8 + xcd, n_blocks = (g.m + kRows - 1) / kRows;
    if (first >= n_blocks || first >= g.stride) return;         // whole workgroup

    const int32_t unit = group * kWaves + wave, n0 = min(unit, g.units - 1) * kColumns;
    const bool mine = unit < g.units;
    bf16x8 w[TAPS][KT][kTerms][2];       // [..][half of a stage]
    {
        const int32_t plane = kTileRows * kStage;
        const int64_t at = int64_t(n0 / kTileRows) * (g.pitch / kStage) * kTerms * plane + (n0 % kTileRows + l32) * kStage + lk * 8;
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap)
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int p = 0; p < kTerms; ++p)
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        w[tap][t][p][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(g.b[tap] + at + (kTerms * t + p) * plane + s * 16));
    }

    float4 x[J];
    const int32_t row_bytes = int32_t(g.lda) * 4, k_last = 64 * (J - 1) + 4 * l16;
    const uint32_t off = uint32_t(lg) * uint32_t(row_bytes) + 16u * uint32_t(l16), off_last = k_last < g.k ? off + 256u * (J - 1) : 0x7FFFFFF0u;
    auto fetch = [&](const float* a, int32_t block) __attribute__((always_inline)) {
        const int32_t row = block * kRows + wave * 4, rows = min(4, g.m - row);
        const auto from = rows_at(a + int64_t(row) * g.lda, rows > 0 ? (rows - 1) * row_bytes + g.k * 4 : 0);
#pragma unroll
        for (int j = 0; j < J; ++j)
            x[j] = __builtin_bit_cast(float4, words4(__builtin_amdgcn_raw_buffer_load_b128(from, j + 1 < J ? off : off_last, j + 1 < J ? 256 * j : 0, 0)));
    };
    const int row = wave * 4 + lg;
    const int to = ((l16 >> 3) * kTerms * RT + (row >> 4)) * 512 + ((l16 >> 1 & 3) * 16 + ((row & 15) ^ (l16 & 14))) * 8 + (l16 & 1) * 4;
    auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const float4 v = x[j];
            uint32_t lo[kTerms], hi[kTerms];
            expand2(v.x, v.y, lo);
            expand2(v.z, v.w, hi);
            if (KT % 2 == 0 || j + 1 < J || l16 < 8)
#pragma unroll
                for (int p = 0; p < kTerms; ++p) *reinterpret_cast<uint2*>(&smem[buf][to + (j * 2 * kTerms + p) * RT * 512]) = make_uint2(lo[p], hi[p]);
        }
    };
    fetch(g.a[0], first);
    stash(0);
    fetch(g.a[TAPS - 1], TAPS == 2 ? first : first + g.stride);
    __syncthreads();

    const bool early = wave >= kWaves / 2, half_last = g.k <= (KT - 1) * kStage + 16;        // half a stage of padding is left out
    const int32_t place = (lg & 1) * 512;
    int buf = 0;
    for (int32_t block = first; block < n_blocks; block += g.stride) {
        floatx16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap) {
            auto next = [&]() __attribute__((always_inline)) {
                stash(buf ^ 1);
                fetch(g.a[tap], block + (TAPS == 2 ? 1 : 2) * g.stride);          // what follows the values just split
            };
            if (early) next();
            if (mine) {
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        if (t + 1 == KT && s == 1 && half_last) break;
                        const int eight = 2 * s + lk;
                        const uint16_t* const at = &smem[buf][t * kTerms * RT * 512 + place + (eight * 16 + (l16 ^ (2 * eight + 8 * (t & 1)))) * 8];
                        bf16x8 f[kTerms];
#pragma unroll
                        for (int p = 0; p < kTerms; ++p) f[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(at + p * RT * 512));
                        auto multiply = [&](int pa, int pw) __attribute__((always_inline)) {
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[tap][t][pw][s], f[pa], acc, 0, 0, 0);
                        };
                        multiply(0, 0), multiply(0, 1), multiply(1, 0), multiply(1, 1), multiply(0, 2), multiply(2, 0);
                    }
            }
            if (!early) next();
            buf ^= 1;
            if (tap + 1 < TAPS) __syncthreads();
        }
        if (mine) {                  // a lane holds a row's columns 8 c + 4 lk .. + 3
            float* const c = g.c + (int64_t(block) * kRows + l32) * g.ldc + n0 + 4 * lk;
            const bool inside = (block + 1) * kRows <= g.m && n0 + kColumns <= g.n;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 o = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
                float* const dst = c + 8 * q;
                if (inside) {
                    o += g.accumulate ? floatx4(*reinterpret_cast<const any4*>(dst)) : floatx4{0.f, 0.f, 0.f, 0.f};       // (-0 becomes 0)
                    if (g.relu) o = floatx4{fmaxf(o[0], 0.f), fmaxf(o[1], 0.f), fmaxf(o[2], 0.f), fmaxf(o[3], 0.f)};
                    *reinterpret_cast<any4*>(dst) = o;
                } else if (block * kRows + l32 < g.m) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (n0 + 8 * q + 4 * lk + v < g.n) {
                            const float s = o[v] + (g.accumulate ? dst[v] : 0.f);
                            dst[v] = g.relu ? fmaxf(s, 0.f) : s;
                        }
                }
            }
        }
        __syncthreads();
    }
}

bool aligned_to(const void* p, uintptr_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

// Columns that each row is charged for when the device is full: the idle wavefronts of a group, and the compute units that no group has.
int32_t charged_columns(int32_t n) {
    const int32_t groups = ((n + kColumns - 1) / kColumns + kWaves - 1) / kWaves;
    return kUnits * kWaves * kColumns / std::max(8, kUnits / groups / 8 * 8);
}

}  // namespace

bool varco_gemm_split_rows_usable(const GemmArgs& ga) {
    auto copy_ok = [&](const void* p, int64_t ld, int64_t plane) {
        return p && aligned_to(p, 16) && ld == (int64_t(ga.k) + kStage - 1) / kStage * kStage && plane == (int64_t(ga.n) + 127) / 128 * 128 * ld;
    };
    if (ga.f32_terms != kTerms || ga.m <= 0 || ga.n <= 0 || ga.k <= 64) return false;
    if (ga.a.dtype != VARCO_F32 || ga.c_dtype != VARCO_F32 || ga.a.transposed || ga.a.gate || ga.b.gate || ga.c_dual || ga.split_k > 1 || ga.b_halves)
        return false;
    if (!copy_ok(ga.b_prep, ga.b_prep_ld, ga.b_prep_plane) || !aligned_to(ga.a.ptr, 4) || ga.a.ld > (int64_t(1) << 26)) return false;
    if (ga.k2 > 0 && (ga.k2 != ga.k || !copy_ok(ga.b2_prep, ga.b2_prep_ld, ga.b2_prep_plane) || !aligned_to(ga.a2.ptr, 4) || ga.a2.ld != ga.a.ld ||
                      ga.a2.gate || ga.a2.dtype != VARCO_F32 || ga.a2.transposed))
        return false;
    // Whole 16-byte pieces as the tiles take them; weights that fit.
    const int32_t stages = (ga.k + kStage - 1) / kStage * (ga.k2 > 0 ? 2 : 1);
    if (ga.k % 4 != 0 || stages > kMostStages) return false;
    // The tiles of kernels_gemm_split.hip are level or ahead (us, there / here):
    if (ga.n <= 64) return false;                       // idle wavefronts here: 2,449,029 rows 256 -> 47 two taps 1,094 / 1,290
    const int32_t n_blocks = (ga.m + kRows - 1) / kRows, groups = (ga.n + kColumns * kWaves - 1) / (kColumns * kWaves);
    if (int64_t(n_blocks) * groups <= kUnits) return true;           // a block for every workgroup: 3,001 rows 256 -> 256 20 / 17
    const int64_t tiles = (int64_t(ga.m) + 127) / 128 * ((int64_t(ga.n) + 127) / 128);
    if (tiles <= 2 * kUnits) return false;              // few blocks in turn: 10,007 rows 256 -> 256 21 / 23, 31,000 rows 256 -> 128 23 / 28
    if (stages <= 4) return false;                      // few products a block: 169,343 rows 128 -> 256 77 / 81
    return charged_columns(ga.n) <= (ga.n + 127) / 128 * 128;      // 169,343 rows 100 -> 320 two taps 174 / 185
}

hipError_t varco_launch_gemm_split_rows(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag) {
    Transform g{};
    g.a[0] = static_cast<const float*>(ga.a.ptr), g.a[1] = static_cast<const float*>(ga.a2.ptr);
    g.lda = ga.a.ld;
    g.m = ga.m, g.n = ga.n, g.k = ga.k;
    g.b[0] = static_cast<const uint16_t*>(ga.b_prep), g.b[1] = static_cast<const uint16_t*>(ga.b2_prep);
    g.pitch = ga.b_prep_ld;
    g.c = static_cast<float*>(ga.c), g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0, g.relu = ga.relu ? 1 : 0;
    const int32_t n_blocks = (ga.m + kRows - 1) / kRows;
    g.units = (ga.n + kColumns - 1) / kColumns;
    g.groups = (g.units + kWaves - 1) / kWaves;
    g.stride = std::max(8, kUnits / g.groups / 8 * 8);
    const dim3 grid{unsigned((std::min(g.stride, n_blocks) + 7) / 8 * 8 * g.groups)};
    tag.begin(stream);
    using std::integral_constant;
    auto go = [&](auto kt) {
        constexpr int KT = decltype(kt)::value;
        if constexpr (2 * KT <= kMostStages)
            if (ga.k2 > 0) {
                hipLaunchKernelGGL((transform_kernel<KT, 2>), grid, dim3(kThreads), 0, stream, g);
                return;
            }
        hipLaunchKernelGGL((transform_kernel<KT, 1>), grid, dim3(kThreads), 0, stream, g);
    };
    switch ((ga.k + kStage - 1) / kStage) {
        case 3: go(integral_constant<int, 3>{}); break;
        case 4: go(integral_constant<int, 4>{}); break;
        case 5: go(integral_constant<int, 5>{}); break;
        case 6: go(integral_constant<int, 6>{}); break;
        case 7: go(integral_constant<int, 7>{}); break;
        default: go(integral_constant<int, 8>{});
    }
    tag.end(stream);
    return hipGetLastError();
}
