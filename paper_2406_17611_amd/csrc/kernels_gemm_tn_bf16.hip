// Weight gradients of bf16-stored activations: C[m x n] = sum over rows r of A[r, i] B[r, j] (both operands row-major with the
// reduction index slow), optionally with a ReLU mask on B, in fp32 on the matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Both operands go to LDS as they lie in memory, rows of one reduction index, with 16-byte loads and writes, and are
// transposed when they are read: ds_read_b64_tr_b16 hands lane i of a group of 16 the i-th column of a 4 x 16 block. (Transposing
// 8 x 4 blocks in registers instead takes eight 8-byte loads, 32 word operations and as many selects per block and thread, and
// a stage of 32 rows then moves as many bytes through the vector memory unit, 64 bytes per cycle, as a 256 x 128 tile can
// multiply in that time; a 256 x 256 tile takes 3/4 of the bytes per product.)
// Row pitch in LDS: 64 bytes more than a multiple of 256, so that the four rows that a group of lanes reads start in four
// different quarters of the banks.
// Bound by reading A, B and the mask once (the tiles of one slab of rows run on one XCD and share them through its L2).
// 169,343 rows, 512 x 512, masked: transposed in registers 270 us, 163 with stages of 32 rows, 142 with 64; 2,449,029 rows in 64
// slabs: 1.93 ms with 32 x 32 x 16 blocks, 1.81 with 16 x 16 x 32 (710 TFLOP/s).
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "varco_internal.h"

namespace {

constexpr int kThreads = 512;

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

// Rows per stage: 32, and 64 for the 256 x 256 tile, whose single workgroup per compute unit has nothing else in flight while
// it waits for a stage.
constexpr int stage_rows(int bm, int bn) { return bm == 256 && bn == 256 ? 64 : 32; }

struct TnDev {
    int32_t m, n, k;
    const uint16_t* a;
    const uint16_t* b;
    const uint16_t* gate;
    const uint16_t* a_dual;
    int64_t lda, ldb;
    float* c;
    float* c_dual;
    int64_t ldc;
    int32_t accumulate;
    int32_t split_k, stages_per_split;
    float* partial;
    int32_t tiles_n, tiles, inner;
};

__device__ __forceinline__ uint32_t gate_pair(uint32_t v, uint32_t g) {
    const uint32_t lo = __uint_as_float(g << 16) > 0.f ? 0x0000FFFFu : 0u;
    const uint32_t hi = __uint_as_float(g & 0xFFFF0000u) > 0.f ? 0xFFFF0000u : 0u;
    return v & (lo | hi);
}

// One operand's share of a stage: W columns x BK rows in chunks of 8 elements, dealt to the threads row by row. Rows may have
// any alignment and any length from 8 on: a chunk that crosses the last column is loaded from before it and moved up (ANY:
// the lengths are no multiples of 8; 5 % of the 256 x 256 kernel's time).
template <int W, bool ANY, bool GATE, int BK>
struct Slab {
    static constexpr int PER_ROW = W / 8, TOTAL = PER_ROW * BK, N = (TOTAL + kThreads - 1) / kThreads, ROWS = kThreads / PER_ROW;
    static constexpr int PITCH = W * 2 + 64;               // bytes
    static_assert(kThreads % PER_ROW == 0, "a thread keeps its columns");
    uint4 v[N], g[GATE ? N : 1];
    uint32_t row;                                          // of this thread's first chunk
    int32_t col;
    bool crosses;
    int by;                                                // columns that the crossing chunk of a row is loaded early (same in all lanes)
    __device__ __forceinline__ void start(int32_t i0, int32_t extent) {
        row = threadIdx.x / PER_ROW;
        const int32_t c = i0 + int32_t(threadIdx.x % PER_ROW) * 8;
        crosses = c < extent && c + 8 > extent;
        by = extent & 7 ? 8 - (extent & 7) : 0;
        col = min(c, extent - 8);                          // (columns past the matrix: repeated ones, never stored)
    }
    // rows k0 .. k0 + BK - 1; those from kmax on are zero
    __device__ __forceinline__ void load(const uint16_t* p, const uint16_t* gate, int64_t ld, int32_t k0, int32_t kmax) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            if (TOTAL < kThreads && threadIdx.x >= TOTAL) break;
            const int64_t off = int64_t(min(k0 + int32_t(row) + h * ROWS, kmax - 1)) * ld + col;
            v[h] = load8_any(reinterpret_cast<const char*>(p + off));
            if constexpr (GATE) g[h] = load8_any(reinterpret_cast<const char*>(gate + off));
        }
    }
    __device__ __forceinline__ void store(char* s, int32_t k0, int32_t kmax) const {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            if (TOTAL < kThreads && threadIdx.x >= TOTAL) break;
            uint4 x = v[h];
            if constexpr (GATE) x = make_uint4(gate_pair(x.x, g[h].x), gate_pair(x.y, g[h].y), gate_pair(x.z, g[h].z), gate_pair(x.w, g[h].w));
            if (ANY && by) {
                const uint4 y = moved_up8(x, by);
                if (crosses) x = y;
            }
            if (k0 + int32_t(row) + h * ROWS >= kmax) x = make_uint4(0u, 0u, 0u, 0u);
            *reinterpret_cast<uint4*>(s + (row + h * ROWS) * PITCH + (threadIdx.x % PER_ROW) * 16) = x;
        }
    }
};

// B read element by element (64 columns at most, never masked): fewer than 8 columns.
template <int BK>
struct ElementSlab {
    static constexpr int N = 64 * BK / kThreads, PITCH = 64 * 2 + 64;
    uint16_t v[N];
    int32_t row[N], col[N];
    __device__ __forceinline__ void start(int32_t, int32_t extent) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int32_t e = int32_t(threadIdx.x) + h * kThreads;
            row[h] = e / extent, col[h] = e - row[h] * extent;         // row >= BK: not this thread's
        }
    }
    __device__ __forceinline__ void load(const uint16_t* p, const uint16_t*, int64_t ld, int32_t k0, int32_t kmax) {
#pragma unroll
        for (int h = 0; h < N; ++h) v[h] = p[int64_t(min(k0 + row[h], kmax - 1)) * ld + col[h]];
    }
    __device__ __forceinline__ void store(char* s, int32_t k0, int32_t kmax) const {
#pragma unroll
        for (int h = 0; h < N; ++h)
            if (row[h] < BK) *reinterpret_cast<uint16_t*>(s + row[h] * PITCH + col[h] * 2) = k0 + row[h] < kmax ? v[h] : uint16_t(0);
    }
};
template <int W, bool FEW, bool ANY, bool GATE, int BK>
using SlabOf = std::conditional_t<FEW, ElementSlab<BK>, Slab<W, ANY, GATE, BK>>;

// Fragment of 16 columns x 32 rows whose first column's element of row 0 (this lane's share of the block) is at LDS byte `at`.
template <int PITCH>
__device__ __forceinline__ bf16x8 fragment(uint32_t at) {
    using P = __attribute__((address_space(3))) shortx4*;
    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)(uintptr_t)at);
    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)(uintptr_t)(at + 4 * PITCH));
    typedef short shortx8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
}

template <int WM, int WN, int TMB, int TNB, bool FEW, bool ANY, bool GATE>
__global__ __launch_bounds__(kThreads, TMB * TNB > 4 ? 2 : 4) void gemm_tn_bf16_kernel(TnDev g) {
    static_assert(WM * WN * 64 == kThreads, "");
    constexpr int BM = 32 * TMB * WM, BN = 32 * TNB * WN, BK = stage_rows(BM, BN);
    using SA = SlabOf<BM, false, ANY, false, BK>;
    using SB = SlabOf<BN, FEW, ANY, GATE, BK>;
    extern __shared__ __attribute__((aligned(16))) char lds[];          // two buffers of BK rows of A, then of B
    constexpr int kA = BK * SA::PITCH, kB = BK * SB::PITCH;

    // slabs of rows are dealt to the 8 XCDs; all tiles of a slab go to one
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3;
    const int32_t in = within % g.inner, z = (within / g.inner) * 8 + xcd;
    if (z >= g.split_k) return;            // whole workgroup leaves together: no barrier is skipped
    const bool second = in >= g.tiles;
    const int32_t tile = second ? in - g.tiles : in;
    const int32_t m0 = tile / g.tiles_n * BM, n0 = tile % g.tiles_n * BN;
    const uint16_t* const a = second ? g.a_dual : g.a;
    const int32_t stages = (g.k + BK - 1) / BK;
    const int32_t s0 = z * g.stages_per_split, s1 = min(stages, s0 + g.stages_per_split);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave / WN) * (32 * TMB), wn = (wave % WN) * (32 * TNB);
    constexpr int NA = 2 * TMB, NB = 2 * TNB;                           // blocks of 16 x 16 per wavefront
    floatx4 acc[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = floatx4(0.f);

    // this lane's share of a 4 x 16 block: row (lane / 4) % 4, columns 4 (lane % 4) ..; group g of 16 lanes: rows 8 g of the
    // fragment
    const uint32_t row = 8 * (lane >> 4) + ((lane >> 2) & 3), sub = 8 * (lane & 3);
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lds));
    const uint32_t at_a = base + row * SA::PITCH + sub + wm * 2, at_b = base + 2 * kA + row * SB::PITCH + sub + wn * 2;

    SA sa;
    SB sb;
    sa.start(m0, g.m);
    sb.start(n0, g.n);
    if (s0 < s1) {
        sa.load(a, nullptr, g.lda, s0 * BK, g.k);
        sb.load(g.b, g.gate, g.ldb, s0 * BK, g.k);
        sa.store(lds, s0 * BK, g.k);
        sb.store(lds + 2 * kA, s0 * BK, g.k);
    }
    __syncthreads();
    for (int32_t s = s0; s < s1; ++s) {
        const uint32_t buf = uint32_t(s - s0) & 1u;
        const bool more = s + 1 < s1;
        if (more) {
            sa.load(a, nullptr, g.lda, (s + 1) * BK, g.k);
            sb.load(g.b, g.gate, g.ldb, (s + 1) * BK, g.k);
        }
#pragma unroll
        for (int h = 0; h < BK / 32; ++h) {
            bf16x8 fb[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[j] = fragment<SB::PITCH>(at_b + buf * kB + h * 32 * SB::PITCH + j * 32);
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const bf16x8 fa = fragment<SA::PITCH>(at_a + buf * kA + h * 32 * SA::PITCH + i * 32);
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[j], acc[i][j], 0, 0, 0);
            }
        }
        if (more) {
            sa.store(lds + (buf ^ 1u) * kA, (s + 1) * BK, g.k);
            sb.store(lds + 2 * kA + (buf ^ 1u) * kB, (s + 1) * BK, g.k);
        }
        __syncthreads();
    }

    // accumulator register v of a lane is element (4 * (lane / 16) + v, lane % 16)
    float* const out = g.split_k > 1 ? g.partial + (int64_t(second ? g.split_k : 0) + z) * g.m * g.n : second ? g.c_dual : g.c;
    const int64_t ldo = g.split_k > 1 ? g.n : g.ldc;
    const bool add_old = g.split_k <= 1 && g.accumulate;
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int32_t r = m0 + wm + i * 16 + 4 * (lane >> 4) + v, c = n0 + wn + j * 16 + (lane & 15);
                if (r < g.m && c < g.n) {
                    float* const p = out + int64_t(r) * ldo + c;
                    *p = add_old ? *p + acc[i][j][v] : acc[i][j][v];
                }
            }
}

bool aligned_to(const void* p, uintptr_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

}  // namespace

bool varco_gemm_tn_bf16_usable(const GemmArgs& g) {
    if (g.m <= 0 || g.n <= 0 || g.k <= 0 || !g.a.transposed || g.b.transposed || g.k2 > 0 || g.a.gate || g.relu) return false;
    if (g.a.dtype != VARCO_BF16 || g.b.dtype != VARCO_BF16 || g.c_dtype != VARCO_F32 || (g.c_dual && !g.a_dual)) return false;
    if (!aligned_to(g.a.ptr, 2) || !aligned_to(g.a_dual, 2) || !aligned_to(g.b.ptr, 2) || !aligned_to(g.b.gate, 2)) return false;
    return g.m >= 8 && (g.n >= 8 || !g.b.gate);
}

// Tile for a product of m x n: 256 rows, or 128 where 256 would be half empty; 256, 128 or 64 columns likewise.
void varco_gemm_tn_bf16_tile(int32_t m, int32_t n, int32_t* bm, int32_t* bn, int32_t* per_cu) {
    *bm = m <= 128 ? 128 : 256;
    *bn = n <= 64 ? 64 : n <= 128 ? 128 : 256;
    *per_cu = *bm == 256 && *bn == 256 ? 1 : 2;      // resident workgroups
}

hipError_t varco_launch_gemm_tn_bf16(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag, int32_t* split_used) {
    int32_t bm, bn, per_cu;
    varco_gemm_tn_bf16_tile(ga.m, ga.n, &bm, &bn, &per_cu);
    auto u16 = [](const void* p) { return static_cast<const uint16_t*>(p); };
    TnDev g;
    g.m = ga.m, g.n = ga.n, g.k = ga.k;
    g.a = u16(ga.a.ptr), g.b = u16(ga.b.ptr), g.gate = u16(ga.b.gate);
    g.a_dual = ga.c_dual ? u16(ga.a_dual) : nullptr;
    g.lda = ga.a.ld, g.ldb = ga.b.ld;
    g.c = static_cast<float*>(ga.c), g.c_dual = static_cast<float*>(ga.c_dual), g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0;
    const int32_t rows = stage_rows(bm, bn), stages = (ga.k + rows - 1) / rows;
    int32_t split = std::max(1, std::min(ga.split_k, stages));
    g.stages_per_split = (stages + split - 1) / split;
    split = (stages + g.stages_per_split - 1) / g.stages_per_split;
    g.split_k = split;
    g.partial = ga.partial;
    if (split > 1 && !ga.partial) return hipErrorInvalidValue;
    g.tiles_n = (ga.n + bn - 1) / bn;
    g.tiles = (ga.m + bm - 1) / bm * g.tiles_n;
    g.inner = g.tiles * (ga.c_dual ? 2 : 1);
    const int64_t blocks = int64_t((split + 7) / 8 * 8) * g.inner;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    *split_used = split;

    hipError_t err = hipSuccess;
    auto launch = [&](auto wm, auto wn, auto tmb, auto tnb, auto few, auto any, auto gated) {
        constexpr int WM = decltype(wm)::value, WN = decltype(wn)::value, TMB = decltype(tmb)::value, TNB = decltype(tnb)::value;
        constexpr bool F = decltype(few)::value, A = decltype(any)::value, G = decltype(gated)::value;
        constexpr int BK = stage_rows(32 * TMB * WM, 32 * TNB * WN);
        const size_t bytes = size_t(2 * BK) * (SlabOf<32 * TMB * WM, false, A, false, BK>::PITCH + SlabOf<32 * TNB * WN, F, A, G, BK>::PITCH);
        const auto kernel = gemm_tn_bf16_kernel<WM, WN, TMB, TNB, F, A, G>;
        if (bytes > 64 * 1024) {
            err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
            if (err != hipSuccess) return;
        }
        tag.begin(stream);
        hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(kThreads), bytes, stream, g);
        tag.end(stream);
    };
    auto with_gate = [&](auto wm, auto wn, auto tmb, auto tnb) {
        using Yes = std::true_type;
        using No = std::false_type;
        const bool any = ga.m % 8 || ga.n % 8;
        if (ga.n < 8) {
            if constexpr (decltype(tnb)::value * decltype(wn)::value == 2) launch(wm, wn, tmb, tnb, Yes{}, Yes{}, No{});
        } else if (g.gate) {
            any ? launch(wm, wn, tmb, tnb, No{}, Yes{}, Yes{}) : launch(wm, wn, tmb, tnb, No{}, No{}, Yes{});
        } else {
            any ? launch(wm, wn, tmb, tnb, No{}, Yes{}, No{}) : launch(wm, wn, tmb, tnb, No{}, No{}, No{});
        }
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    if (bm == 256 && bn == 256)
        with_gate(I2{}, I4{}, I4{}, I2{});
    else if (bm == 256 && bn == 128)
        with_gate(I4{}, I2{}, I2{}, I2{});
    else if (bm == 256)
        with_gate(I4{}, I2{}, I2{}, I1{});
    else if (bn == 256)
        with_gate(I2{}, I4{}, I2{}, I2{});
    else if (bn == 128)
        with_gate(I2{}, I4{}, I2{}, I1{});
    else
        with_gate(I4{}, I2{}, I1{}, I1{});
    return err != hipSuccess ? err : hipGetLastError();
}
