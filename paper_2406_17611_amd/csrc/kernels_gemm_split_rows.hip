// The dense transform of eq. (2) for fp32-stored activations whose reduction takes 65 to 256 steps (both taps: twice that), act(M H + X H0), from three
// bf16 terms of either operand and six products (kernels_gemm_split.hip: the expansion and what it keeps). The products of a stage of 32 steps
// are summed from the smallest to the largest, on v_mfma_f32_16x16x32_bf16, which rounds half as often as two of 16 steps: the errors against
// fp64 are 0.73 to 0.96 of those of the tiles there.
//
// The weights stay in registers: a wavefront holds 16 or 32 columns of them, all terms, of both taps, up to 192 registers, for all the rows that
// its workgroup walks over. Blocks of 32 rows come in whole rows, 16 lanes to one, from any 4-byte address, one block (of one tap) ahead in
// registers; they are split once for the eight wavefronts and lie in LDS as the matrix unit reads them, [stage][term][16 rows][eight steps][row],
// rows swapped by their place so that neither writes nor reads meet in a bank; two buffers, one barrier per block and tap. One half of the
// wavefronts splits the next block while the other multiplies, and the other way round: every SIMD holds one of either half. The weights are
// the first operand: a lane then holds four consecutive columns of a row and stores them together.
// Bound by the matrix units (1.1 to 1.3 of the 1.6 PFLOP/s that random operands reach from LDS) and, two taps of 129 steps and more, by the reads
// from LDS for 16 columns alone. 128 x 128 tiles that each split their rows again and fetch weights by stage / this, us:
//   169,343 rows 256 -> 256 134 / 117, 128 -> 256 76 / 64     1,638,400 rows 256 -> 256 1,500 / 1,140     300,007 rows 200 -> 200 208 / 152
//   50,021 rows 200 -> 136 two taps 77 / 64     300,007 rows 100 -> 256 two taps 210 / 167     2,449,029 rows 256 -> 256 two taps 3,540 / 3,290
//   3,001 rows 256 -> 256 20 / 11, two taps 32 / 16
// Rows that are no whole number of 16-byte pieces stay with fp32 instructions although this would be as accurate and faster (50,021 rows 75 -> 200 two
// taps 67 / 37): with every layer's roundings changed, twice as many ReLU gates within rounding of zero decide otherwise, and gradients
// of a small graph then move by 1e-3 as a whole.
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

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float any4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t words4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct Transform {
    const float* a[2];               // rows of the taps
    int64_t lda;
    int32_t m, n, k;
    const uint16_t* b[2];            // expanded copies of the weights
    int32_t tile_rows;               // rows of a tile of theirs
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

// KT: stages of a tap; CT: tiles of 16 columns of a wavefront.
template <int KT, int TAPS, int CT>
__global__ __launch_bounds__(kThreads, 2) void transform_kernel(Transform g) {
    constexpr int J = (KT + 1) / 2, RT = kRows / 16, CW = 16 * CT;
    constexpr int kBlock = KT * kTerms * RT * 512;
    __shared__ __attribute__((aligned(16))) uint16_t smem[2][kBlock];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3, group = within % g.groups;
    const int32_t first = (within / g.groups) * 8 + xcd, n_blocks = (g.m + kRows - 1) / kRows;
    if (first >= n_blocks || first >= g.stride) return;         // whole workgroup

    const int32_t unit = group * kWaves + wave, n0 = min(unit, g.units - 1) * CW;
    const bool mine = unit < g.units;
    bf16x8 w[TAPS][KT][kTerms][CT];
    {
        const int32_t plane = g.tile_rows * kStage;
        const int64_t at = int64_t(n0 / g.tile_rows) * (g.pitch / kStage) * kTerms * plane + (n0 % g.tile_rows + l16) * kStage + lg * 8;
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap)
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int p = 0; p < kTerms; ++p)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        w[tap][t][p][ct] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(g.b[tap] + at + (kTerms * t + p) * plane + ct * 16 * kStage));
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

    const bool early = wave >= kWaves / 2;
    int buf = 0;
    for (int32_t block = first; block < n_blocks; block += g.stride) {
        floatx4 acc[RT][CT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap) {
            auto next = [&]() __attribute__((always_inline)) {
                stash(buf ^ 1);
                fetch(g.a[tap], block + (TAPS == 2 ? 1 : 2) * g.stride);          // what follows the values just split
            };
            if (early) next();
            if (mine) {
#pragma unroll
                for (int t = 0; t < KT; ++t) {
                    const uint16_t* const at = &smem[buf][t * kTerms * RT * 512 + (lg * 16 + (l16 ^ (2 * lg + 8 * (t & 1)))) * 8];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        bf16x8 f[kTerms];
#pragma unroll
                        for (int p = 0; p < kTerms; ++p) f[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(at + (p * RT + rt) * 512));
                        auto multiply = [&](int pa, int pw) __attribute__((always_inline)) {
#pragma unroll
                            for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[tap][t][pw][ct], f[pa], acc[rt][ct], 0, 0, 0);
                        };
                        multiply(2, 0), multiply(0, 2), multiply(1, 1), multiply(1, 0), multiply(0, 1), multiply(0, 0);
                    }
                }
            }
            if (!early) next();
            buf ^= 1;
            if (tap + 1 < TAPS) __syncthreads();
        }
        if (mine) {
            float* const c = g.c + int64_t(block) * kRows * g.ldc + n0;
            const bool inside = (block + 1) * kRows <= g.m && n0 + CW <= g.n;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int row = rt * 16 + l16;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    floatx4 o = acc[rt][ct];
                    const int col = ct * 16 + 4 * lg;
                    float* const dst = c + int64_t(row) * g.ldc + col;
                    if (inside) {
                        if (g.accumulate) o += *reinterpret_cast<const any4*>(dst);
                        if (g.relu) o = floatx4{fmaxf(o[0], 0.f), fmaxf(o[1], 0.f), fmaxf(o[2], 0.f), fmaxf(o[3], 0.f)};
                        *reinterpret_cast<any4*>(dst) = o;
                    } else if (block * kRows + row < g.m) {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (n0 + col + v < g.n) {
                                const float s = g.accumulate ? o[v] + dst[v] : o[v];
                                dst[v] = g.relu ? fmaxf(s, 0.f) : s;
                            }
                    }
                }
            }
        }
        __syncthreads();
    }
}

bool aligned_to(const void* p, uintptr_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

template <class F>
void with_flag(bool b, F&& f) {
    b ? f(std::true_type{}) : f(std::false_type{});
}

// Columns that each row is charged for when the device is full: the idle wavefronts of a group, and the compute units that no group has.
int32_t charged_columns(int32_t n, int32_t cw) {
    const int32_t groups = ((n + cw - 1) / cw + kWaves - 1) / kWaves;
    return kUnits * kWaves * cw / std::max(8, kUnits / groups / 8 * 8);
}

}  // namespace

bool varco_gemm_split_rows_usable(const GemmArgs& ga) {
    auto copy_ok = [&](const void* p, int64_t ld, int64_t plane) {
        return p && aligned_to(p, 16) && ld == (int64_t(ga.k) + kStage - 1) / kStage * kStage && plane == (int64_t(ga.n) + 127) / 128 * 128 * ld;
    };
    if (ga.f32_terms != kTerms || ga.m <= 0 || ga.n <= 0 || ga.k <= 64 || ga.k > 8 * kStage) return false;
    if (ga.a.dtype != VARCO_F32 || ga.c_dtype != VARCO_F32 || ga.a.transposed || ga.a.gate || ga.b.gate || ga.c_dual || ga.split_k > 1 || ga.b_halves)
        return false;
    if (!copy_ok(ga.b_prep, ga.b_prep_ld, ga.b_prep_plane) || !aligned_to(ga.a.ptr, 4) || ga.a.ld > (int64_t(1) << 26)) return false;
    if (ga.k2 > 0 && (ga.k2 != ga.k || !copy_ok(ga.b2_prep, ga.b2_prep_ld, ga.b2_prep_plane) || !aligned_to(ga.a2.ptr, 4) || ga.a2.ld != ga.a.ld ||
                      ga.a2.gate || ga.a2.dtype != VARCO_F32 || ga.a2.transposed))
        return false;
    // The tiles of kernels_gemm_split.hip are level or ahead (us, there / here):
    if (ga.k % 4 != 0) return false;
    if (ga.n <= 64) return false;                       // idle wavefronts here: 2,449,029 rows 256 -> 47 two taps 1,094 / 1,290
    const int64_t tiles = (int64_t(ga.m) + 127) / 128 * ((int64_t(ga.n) + 127) / 128);
    if (tiles <= 3 * kUnits / 2) return true;           // units without a tile there: 10,007 rows 128 -> 200 two taps 23 / 17
    if (tiles <= 2 * kUnits) return false;              // just two for every unit: 31,000 rows 100 -> 256 two taps 30 / 33
    if (ga.k2 == 0 && ga.k <= 96) return false;         // few products a block: 300,007 rows 72 -> 136 88 / 92
    return charged_columns(ga.n, 16) <= (ga.n + 127) / 128 * 128;      // 169,343 rows 100 -> 320 two taps 174 / 185
}

hipError_t varco_launch_gemm_split_rows(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag) {
    Transform g{};
    g.a[0] = static_cast<const float*>(ga.a.ptr), g.a[1] = static_cast<const float*>(ga.a2.ptr);
    g.lda = ga.a.ld;
    g.m = ga.m, g.n = ga.n, g.k = ga.k;
    g.b[0] = static_cast<const uint16_t*>(ga.b_prep), g.b[1] = static_cast<const uint16_t*>(ga.b2_prep);
    g.tile_rows = ga.n <= 64 ? 64 : 128;
    g.pitch = ga.b_prep_ld;
    g.c = static_cast<float*>(ga.c), g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0, g.relu = ga.relu ? 1 : 0;
    const int32_t n_blocks = (ga.m + kRows - 1) / kRows;
    // Twice the columns halve the reads of the rows' fragments, half the columns spread few rows over more units (10,007 rows 256 -> 256 22 us
    // against 18; 300,007 rows 160 against 183).
    const bool wide = n_blocks >= 4 * kUnits && charged_columns(ga.n, 32) <= charged_columns(ga.n, 16);
    tag.begin(stream);
    auto launch = [&](auto kt, auto taps, auto ct) {
        constexpr int CW = 16 * decltype(ct)::value;
        g.units = (ga.n + CW - 1) / CW;
        g.groups = (g.units + kWaves - 1) / kWaves;
        g.stride = std::max(8, kUnits / g.groups / 8 * 8);
        const dim3 grid{unsigned((std::min(g.stride, n_blocks) + 7) / 8 * 8 * g.groups)};
        hipLaunchKernelGGL((transform_kernel<decltype(kt)::value, decltype(taps)::value, decltype(ct)::value>), grid, dim3(kThreads), 0, stream, g);
    };
    using std::integral_constant;
    auto go = [&](auto kt) {
        with_flag(ga.k2 > 0, [&](auto two) {
            constexpr int TAPS = decltype(two)::value ? 2 : 1;
            with_flag(wide, [&](auto w) {
                constexpr int CT = decltype(w)::value && decltype(kt)::value * TAPS <= 8 ? 2 : 1;
                launch(kt, integral_constant<int, TAPS>{}, integral_constant<int, CT>{});
            });
        });
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
