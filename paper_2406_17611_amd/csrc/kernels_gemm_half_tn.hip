// Weight gradients of eq. (2) for fp32-stored activations, dH = M^T dZ: one reduction over the nodes, on the fp16 matrix units, from the
// two scaled fp16 terms of kernels_gemm_half.hip (same products, same order of the sums, same scales per column).
//
// Both operands have the reduction index (nodes) as the slow one. A lane loads four columns of four or eight consecutive nodes with 16-byte
// loads and splits the values of two consecutive nodes of a column together, which is the word the matrix unit wants: LDS holds operands
// as it reads them, [32 columns][16 nodes][term] of 1 KB, lane after lane, with the lanes of a column's four pieces swapped so that
// neither the writes nor the reads meet in a bank. The taps' rows count as columns of one operand (each tap's padded to 64), so that both
// taps of a layer of up to 64 inputs fill a tile of 128.
//
// Bound by what the L2s deliver to the compute units: the same pattern of loads with nothing else in the kernel takes 2.1 of 3.0 ms (256 x 256,
// both taps, 2,449,029 nodes; 20 GB out of the L2s, 12 GB into them; matrix units 31 % busy, vector ALUs 31 %). Hence the tile: 256 x 128 by 512 threads, one workgroup per compute unit,
// loads 8 KB per node where four 128 x 128 tiles of two workgroups per unit load 12, and splits a value once per 128 or 256 columns of the
// other operand. 128 columns of A where 256 would be padding. One barrier per stage of 32 nodes: the next stage is split into a second LDS buffer
// while other wavefronts still multiply. The maximum of a column is only looked at when a value leaves the range that its scale leaves (one
// test per stage and wavefront). 128 x 128 tiles / this, us, masked unless noted:
//   256 x 256 both taps   2,449,029 nodes 3,650 / 3,020      100 x 256 both taps 2,160 / 1,690    256 x 256 2,210 / 1,730
//   256 x 47 both taps, no mask           1,310 / 1,240
//   256 x 256               169,343 nodes   147 / 124        128 x 256              91 / 93      256 x 40, no mask 50 / 45
//   200 x 136 both taps      50,021 nodes    89 / 68         75 x 200 both taps     50 / 41
//   64 x 128 both taps       60,013 nodes    38 / 23         32 x 64 both taps, 16,000 nodes 12.8 / 8.9   16 x 32, 2,000 nodes 11.1 / 8.8
// (Measured and not kept: a column per lane and 4-byte loads, which needs no exchange between lanes, 4,710 us for the first; stages of 16 nodes; two
// or three stages in registers; wavefronts that split first while others multiply first; priorities; loads that touch a later stage's lines.)
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "gemm_tile.h"
#include "half_terms.h"
#include "varco_internal.h"

namespace {

constexpr int BK = 32;           // nodes per stage
constexpr int kThreads = 512;
constexpr int kFirst = 8;        // exponent that the largest value of a first stage is brought to, which leaves
constexpr int kRoom = 6;         // later ones this many binades
constexpr int kFragment = 512;   // fp16 elements of a 32-column, 16-node operand of the matrix unit (1 KB)

typedef float floatx16 __attribute__((ext_vector_type(16)));

struct WeightGrad {
    const float* a[2];           // nodes x m: the taps' rows
    const float *b, *gate;       // nodes x n: errors, and what masks them
    int64_t lda, ldb;
    int32_t m, n, nodes;
    float *c[2], *partial;
    int64_t ldc;
    int32_t accumulate;
    int32_t split, stages_per_split;
    int32_t units_per_tap, units;      // units of 64 columns of A
    int32_t tiles_n, inner;            // tiles along B, and in all
    int32_t first;                     // workgroup of a launch of several (a multiple of eight)
};
struct WeightGrads {
    WeightGrad job[kMaxWeightJobs];
    int32_t n;
};
enum Gate { kOpen, kMasked, kEither };      // B as it is, masked, or as the job says

// Descriptor of `bytes` bytes from p on; what lies behind reads as zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_at(const float* p, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, 0x00027000);
}
__device__ __forceinline__ float4 load_row4(__amdgpu_buffer_rsrc_t r, uint32_t off, int32_t row) {
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(float4, words4(__builtin_amdgcn_raw_buffer_load_b128(r, off, row, 0)));
}

template <int TMB, int TNB>
__device__ __forceinline__ void multiply(const halfx8 (&fa)[TMB], const halfx8 (&fb)[TNB], floatx16 (&acc)[TMB][TNB]) {
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fb[j], acc[i][j], 0, 0, 0);
}

__device__ __forceinline__ float& part(float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// Place of a column's piece (eight nodes, number p of its stage) among the 32 of half a fragment: what is written, or read, at once lies in
// different banks.
__device__ __forceinline__ int slot(int col, int p) { return col ^ p; }

// UM, UN: units of 64 columns of the two operands in a tile.
template <int UM, int UN, Gate GATE>
__device__ __forceinline__ void weight_grad(const WeightGrad& g, uint32_t block) {
    constexpr int BM = 64 * UM, BN = 64 * UN, COLS = BM + BN;
    constexpr int WM = 4, WN = 2, TMB = BM / 32 / WM, TNB = BN / 32 / WN;
    constexpr int kStage = COLS / 32 * 4 * kFragment;                  // fp16 elements: [32 columns][16 nodes][term]
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * kStage];
    __shared__ __attribute__((aligned(16))) int2 scales[2][COLS];      // per stage parity and column: exponent, factor the sums so far take
    __shared__ int32_t smaller_at[2];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int32_t xcd = block & 7, within = block >> 3;
    const int32_t in = within % g.inner, z = (within / g.inner) * 8 + xcd;
    if (z >= g.split) return;                  // whole workgroup leaves together: no barrier is skipped
    const int32_t all = (g.nodes + BK - 1) / BK;
    const int32_t t_begin = z * g.stages_per_split, t_end = min(all, t_begin + g.stages_per_split);
    if (t_begin >= t_end) return;
    const int32_t u0 = in / g.tiles_n * UM, n0 = in % g.tiles_n * BN;
    const float sign = (z & 1) ? -1.f : 1.f;
    const int lrow = lane & 31, lk = lane >> 5;
    const int wm = wave / WN * TMB, wn = wave % WN * TNB;              // first blocks of 32 of this wavefront

    floatx16 acc[TMB][TNB], low[TMB][TNB];
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;
    if (tid < 2) smaller_at[tid] = -1;

    auto compute = [&](int32_t t) __attribute__((always_inline)) {
        const uint16_t* const st = smem + (t & 1) * kStage;
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            const uint16_t* const at = st + (lk * 32 + slot(lrow, 2 * s + lk)) * 8;
            auto fragment = [&](int block, int term) {
                return __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4*>(at + ((block * 2 + s) * 2 + term) * kFragment));
            };
            halfx8 a0[TMB], b0[TNB], b1[TNB], a1[TMB];
#pragma unroll
            for (int i = 0; i < TMB; ++i) a0[i] = fragment(wm + i, 0);
#pragma unroll
            for (int j = 0; j < TNB; ++j) b0[j] = fragment(BM / 32 + wn + j, 0);
#pragma unroll
            for (int j = 0; j < TNB; ++j) b1[j] = fragment(BM / 32 + wn + j, 1);
            multiply<TMB, TNB>(a0, b0, acc);
            multiply<TMB, TNB>(a0, b1, low);
#pragma unroll
            for (int i = 0; i < TMB; ++i) a1[i] = fragment(wm + i, 1);
            multiply<TMB, TNB>(a1, b0, low);
        }
    };
    auto follow = [&](int32_t t) __attribute__((always_inline)) {
        if (__builtin_amdgcn_readfirstlane(smaller_at[t & 1]) != t) return;
        const int2* const sc = scales[t & 1];
#pragma unroll
        for (int j = 0; j < TNB; ++j) {
            const float f = __uint_as_float(uint32_t(sc[BM + (wn + j) * 32 + lrow].y));
#pragma unroll
            for (int i = 0; i < TMB; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float fa = __uint_as_float(uint32_t(sc[(wm + i) * 32 + 8 * (v >> 2) + 4 * lk + (v & 3)].y));
                    acc[i][j][v] = acc[i][j][v] * fa * f, low[i][j][v] = low[i][j][v] * fa * f;
                }
        }
    };

    // NK: nodes per lane (8: a wavefront serves 64 columns, 4: 32).
    auto run = [&](auto is_a, auto nk, auto idle) __attribute__((always_inline)) {
        constexpr bool A = decltype(is_a)::value, IDLE = decltype(idle)::value, G = GATE != kOpen && !A;
        constexpr int NK = decltype(nk)::value, NG = BK / NK;          // node groups
        constexpr int WC = 4 * 64 / NG;                                // columns of this wavefront
        const int w = A ? wave : wave - 4;
        const int q = lane % NG, cg = lane / NG;                       // node group, group of four columns
        const int col = w * WC + 4 * cg;                               // of the operand's tile
        const int32_t unit = A ? u0 + w * WC / 64 : 0, tap = A && unit >= g.units_per_tap ? 1 : 0;
        const int32_t extent = A ? g.m : g.n;
        const int32_t first = A ? (unit - tap * g.units_per_tap) * 64 + w * WC % 64 : n0 + w * WC;      // first column of this wavefront
        const float* const src = A ? g.a[tap] : g.b;
        const int64_t ld = A ? g.lda : g.ldb;
        const bool live = !IDLE && first < extent && (!A || unit < g.units);
        const bool masked = GATE == kMasked || g.gate;
        const int32_t row_bytes = int32_t(ld) * 4;
        const uint32_t off = uint32_t(q * NK) * uint32_t(row_bytes) + (first + 4 * cg < extent ? 16u * cg : 0u);
        float4 rx[NK], ry[G ? NK : 1];
        auto fetch = [&](int32_t t) __attribute__((always_inline)) {         // (past the slab: no bytes, zeros)
            if (IDLE) return;
            const int32_t k0 = t * BK, rows = min(BK, g.nodes - k0), bytes = live && t < t_end ? (rows - 1) * row_bytes + (extent - first) * 4 : 0;
            const auto from = rows_at(src + int64_t(k0) * ld + first, bytes);
            const auto mask = rows_at(G && masked ? g.gate + int64_t(k0) * ld + first : src, bytes);
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                rx[kk] = load_row4(from, off, kk * row_bytes);
                if constexpr (G) ry[kk] = load_row4(mask, off, kk * row_bytes);
            }
        };
        int e[4] = {126, 126, 126, 126};
        const float sg = A ? 1.f : sign;
        auto stash = [&](int32_t t) __attribute__((always_inline)) {
            if (IDLE) return;
            float m[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NK; ++kk)
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
                    float& x = part(rx[kk], ii);
                    if constexpr (G) x = part(ry[kk], ii) > 0.f || !masked ? x : 0.f;
                    m[ii] = fmaxf(m[ii], fabsf(x));
                }
            float sc[4], f[4] = {1.f, 1.f, 1.f, 1.f};
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) sc[ii] = power_of_two(e[ii]);
            if (__any(fmaxf(fmaxf(m[0] * sc[0], m[1] * sc[1]), fmaxf(m[2] * sc[2], m[3] * sc[3])) >= float(2 << (kFirst + kRoom)))) {
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
                    const int now = scale_exponent(largest_of_lanes<NG>(m[ii]), kFirst), old = e[ii];
                    if (now < old - kRoom) e[ii] = now;
                    sc[ii] = power_of_two(e[ii]), f[ii] = power_of_two(max(e[ii] - old, -126));
                }
                smaller_at[t & 1] = t;
            }
            if (q == 0) {
                int4* const at = reinterpret_cast<int4*>(&scales[t & 1][(A ? 0 : BM) + col]);
                at[0] = make_int4(e[0], __float_as_int(f[0]), e[1], __float_as_int(f[1])), at[1] = make_int4(e[2], __float_as_int(f[2]), e[3], __float_as_int(f[3]));
            }
            constexpr int P = 8 / NK;                                  // lanes that share a 16-byte piece
            const int p = q / P;                                       // eight nodes: half of an operand's column
            uint16_t* const dst = smem + (t & 1) * kStage + ((A ? 0 : BM) + col) / 32 * 4 * kFragment + (p >> 1) * 2 * kFragment + (p & 1) * 256 + (q % P) * NK;
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) {
                uint32_t hi[NK / 2], lo[NK / 2];
                const float s = sg * sc[ii];
#pragma unroll
                for (int h = 0; h < NK / 2; ++h) split_pair(part(rx[2 * h], ii) * s, part(rx[2 * h + 1], ii) * s, hi[h], lo[h]);
                uint16_t* const at = dst + slot((col & 31) + ii, p) * 8;
                if constexpr (NK == 8) {
                    *reinterpret_cast<uint4*>(at) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                    *reinterpret_cast<uint4*>(at + kFragment) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                } else {
                    *reinterpret_cast<uint2*>(at) = make_uint2(hi[0], hi[1]);
                    *reinterpret_cast<uint2*>(at + kFragment) = make_uint2(lo[0], lo[1]);
                }
            }
        };
        fetch(t_begin);
        __syncthreads();                       // smaller_at is set
        stash(t_begin);
        fetch(t_begin + 1);
        __syncthreads();
        for (int32_t t = t_begin; t < t_end; ++t) {
            follow(t);
            compute(t);
            if (t + 1 < t_end) {
                stash(t + 1);
                fetch(t + 2);
                __syncthreads();
            }
        }
    };
    using std::integral_constant;
    constexpr int NA = UM == 4 ? 8 : 4;
    if (wave < 4)
        run(std::true_type{}, integral_constant<int, NA>{}, std::false_type{});
    else if (UN == 2 || wave < 6)
        run(std::false_type{}, integral_constant<int, 4>{}, std::false_type{});
    else
        run(std::false_type{}, integral_constant<int, 4>{}, std::true_type{});

    const int2* const sc = scales[(t_end - 1) & 1];
    const bool to_partial = g.split > 1;
#pragma unroll
    for (int i = 0; i < TMB; ++i) {
        int ea[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) ea[v] = sc[(wm + i) * 32 + 8 * (v >> 2) + 4 * lk + (v & 3)].x;
#pragma unroll
        for (int j = 0; j < TNB; ++j) {
            const int eb = sc[BM + (wn + j) * 32 + lrow].x;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = __builtin_ldexpf(sign * (acc[i][j][v] + low[i][j][v] * (1.f / kHalfLow)), -(ea[v] + eb));
        }
        const int32_t unit = u0 + (wm + i) / 2, tap = unit >= g.units_per_tap ? 1 : 0, row0 = (unit - tap * g.units_per_tap) * 64 + (wm + i) % 2 * 32;
        if (unit >= g.units || row0 >= g.m) continue;
        float* const base = to_partial ? g.partial + (int64_t(tap) * g.split + z) * g.m * g.n : g.c[tap];
        store_tile<1, TNB>(reinterpret_cast<const floatx16(&)[1][TNB]>(acc[i]), base, to_partial ? int64_t(g.n) : g.ldc, g.m, g.n, row0, n0 + wn * 32,
                           row0 + 32 <= g.m && n0 + BN <= g.n, lane, !to_partial && g.accumulate, false);
    }
}

template <int UM, int UN, Gate GATE>
__global__ __launch_bounds__(kThreads, 2) void weight_grad_kernel(WeightGrad g) {
    weight_grad<UM, UN, GATE>(g, blockIdx.x);
}

// Products of several layers: each workgroup belongs to one of them.
template <int UN>
__global__ __launch_bounds__(kThreads, 2) void weight_grads_kernel(WeightGrads all) {
    int i = 0;
    while (i + 1 < all.n && int32_t(blockIdx.x) >= all.job[i + 1].first) ++i;
    weight_grad<2, UN, kEither>(all.job[i], blockIdx.x - all.job[i].first);
}

// The product `ga` in tiles of 64 UM x 64 UN, its reduction in about `split` slabs; workgroups in all.
int64_t make_job(const GemmArgs& ga, int um, int un, int64_t split_wanted, WeightGrad& g) {
    const int32_t products = ga.c_dual ? 2 : 1;
    auto f32 = [](const void* p) { return static_cast<const float*>(p); };
    g.a[0] = f32(ga.a.ptr), g.a[1] = ga.c_dual ? f32(ga.a_dual) : g.a[0];
    g.b = f32(ga.b.ptr), g.gate = f32(ga.b.gate);
    g.lda = ga.a.ld, g.ldb = ga.b.ld;
    g.m = ga.m, g.n = ga.n, g.nodes = ga.k;
    g.c[0] = static_cast<float*>(ga.c), g.c[1] = static_cast<float*>(ga.c_dual), g.partial = ga.partial;
    g.ldc = ga.ldc, g.accumulate = ga.accumulate ? 1 : 0;
    g.units_per_tap = (ga.m + 63) / 64, g.units = products * g.units_per_tap;
    g.tiles_n = (ga.n + 64 * un - 1) / (64 * un);
    g.inner = (g.units + um - 1) / um * g.tiles_n;
    const int32_t stages = (ga.k + BK - 1) / BK;
    const int32_t split = int32_t(std::max<int64_t>(1, std::min<int64_t>(split_wanted, stages)));
    g.stages_per_split = std::max(1, (stages + split - 1) / split);
    g.split = std::max(1, (stages + g.stages_per_split - 1) / g.stages_per_split);
    return int64_t((g.split + 7) / 8 * 8) * g.inner;
}

}  // namespace

int64_t varco_gemm_half_tn_tiles(const GemmArgs& ga) {
    const int32_t units = (ga.c_dual ? 2 : 1) * ((ga.m + 63) / 64);
    return int64_t((units + 1) / 2) * ((ga.n + 127) / 128);
}

hipError_t varco_launch_gemm_half_tn_jobs(const GemmArgs* ga, int32_t n, hipStream_t stream, const LaunchTag& tag, int32_t* split_used) {
    if (n < 1 || n > kMaxWeightJobs) return hipErrorInvalidValue;
    bool narrow = true;
    for (int32_t i = 0; i < n; ++i) narrow = narrow && ga[i].n <= 64;
    WeightGrads all{};
    all.n = n;
    int64_t blocks = 0;
    for (int32_t i = 0; i < n; ++i) {
        all.job[i].first = int32_t(blocks);
        blocks += make_job(ga[i], 2, narrow ? 1 : 2, ga[i].split_k, all.job[i]);
        if (blocks > 0x7FFFFFFF / kThreads || (all.job[i].split > 1 && !ga[i].partial)) return hipErrorInvalidValue;
        split_used[i] = all.job[i].split;
    }
    const dim3 grid{unsigned(blocks)};
    tag.begin(stream);
    if (narrow)
        hipLaunchKernelGGL(weight_grads_kernel<1>, grid, dim3(kThreads), 0, stream, all);
    else
        hipLaunchKernelGGL(weight_grads_kernel<2>, grid, dim3(kThreads), 0, stream, all);
    tag.end(stream);
    return hipGetLastError();
}

// Tiles of 256 columns of A unless tiles of 128 cover them with fewer; 64 columns of B where that is all there are. (The tile changes no sum.)
// Tiles of 128 x 64 where slabs are up to three stages long and all of them start at once, two to a compute unit (in place of tiles of 128 columns: one): such a launch waits
// for its first loads, and a smaller tile has fewer of them and less to write. Other tiles / these, with the sums of the slabs, us: 2,000 rows 200 x 100 15.6 / 11.3,
// 256 x 16 11.5 / 9.4, 128 x 100 11.8 / 10.3, 256 x 256 (504 of them) 19.9 / 18.5, both taps 100 x 100 16.3 / 11.8, 10,007 rows 200 x 100 21.6 / 17.9, 100 x 100 15.2 / 13.3.
// More, or longer: 2,000 rows 512 x 200 +3 %, 16 x 512 +4 %, 10,007 rows 200 x 200 +9 %, 100 x 256 +3 %, 500,000 rows 200 x 64 134 / 151.
hipError_t varco_launch_gemm_half_tn(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag, int32_t* split_used) {
    const int32_t units = (ga.c_dual ? 2 : 1) * ((ga.m + 63) / 64);
    const bool fewer_wide = (units + 3) / 4 * 4 <= (units + 1) / 2 * 2;
    WeightGrad g{};
    int64_t blocks = make_job(ga, 2, 1, ga.split_k, g);
    const bool few = g.stages_per_split <= 3 && int64_t(g.split) * g.inner <= (fewer_wide ? 512 : 256), wide = fewer_wide && !few;
    const int un = few || ga.n <= 64 ? 1 : 2;
    if (wide || un == 2) blocks = make_job(ga, wide ? 4 : 2, un, ga.split_k, g);
    if (g.split > 1 && !ga.partial) return hipErrorInvalidValue;
    if (blocks > 0x7FFFFFFF / kThreads) return hipErrorInvalidValue;
    *split_used = g.split;
    const dim3 grid{unsigned(blocks)};
    tag.begin(stream);
    using std::integral_constant;
    auto go = [&](auto m, auto n, auto gt) {
        hipLaunchKernelGGL((weight_grad_kernel<decltype(m)::value, decltype(n)::value, decltype(gt)::value>), grid, dim3(kThreads), 0, stream, g);
    };
    auto with_gate = [&](auto m, auto n) {
        if (ga.b.gate)
            go(m, n, integral_constant<Gate, kMasked>{});
        else
            go(m, n, integral_constant<Gate, kOpen>{});
    };
    auto with_n = [&](auto m) {
        if (un == 1)
            with_gate(m, integral_constant<int, 1>{});
        else
            with_gate(m, integral_constant<int, 2>{});
    };
    if (wide)
        with_n(integral_constant<int, 4>{});
    else
        with_n(integral_constant<int, 2>{});
    tag.end(stream);
    return hipGetLastError();
}
