// Input gradients of the dense feature transform of eq. (2) for fp32-stored activations, dM = dZ H^T, on the fp16 matrix units: what all gradients of that
// storage type have in common, and the kernel for reductions of 17 to 64 and of more than 512 steps (65 to 512: kernels_gemm_half_nt.hip). Operands are scaled by
// powers of two and every value is written as two fp16 terms,
//     x s = h0 + h1 / 2048,   h0 = fp16(x s), h1 = fp16(2048 (x s - h0))
// (the difference is exact in fp32; two 11-bit significands cover 23 of the 24 bits of x, the last one is lost for a quarter of
// all values). Of the four cross products
//     a b = a0 b0 + (a0 b1 + a1 b0) / 2048 + a1 b1 / 2^22
// the first is summed in one fp32 accumulator and the two in the middle in another; the last, below fp32's own rounding, is left out
// except in short sums. Both sums meet in the epilogue, where the scales are taken back out. Three fp16 instructions
// (v_mfma_f32_32x32x16_f16) instead of the six that three bf16 terms take (kernels_gemm_split.hip).
// Two accumulators because the matrix unit drops what falls below the last place of the sum it adds to: the small products in a sum
// of their own leave the large one a single rounding per 16 products. Relative error against fp64, normal operands, three bf16 terms /
// this: K = 16 8.2e-8 / 7.7e-8 (with a1 b1), 48 1.2e-7 / 9.6e-8, 96 1.6e-7 / 1.1e-7, 256 2.5e-7 / 1.3e-7, 512 3.5e-7 / 1.7e-7, 16,384
// 2.1e-6 / 8.3e-7; alike with rectified values and with values over 12 or 20 binades. What the rounding of the accumulators leaves is
// below zero on average, so every second slab of a weight gradient (kernels_gemm_half_tn.hip, the same terms) multiplies -B (its scale is
// negative) and changes sign in the epilogue.
// Scales: the largest value of a row of the weights' copy is brought to [2^14, 2^15) when it is made. Rows of A
// (in weight gradients the columns of both operands) are scaled as they arrive, by what brings the largest value of the first stage to
// [2^8, 2^9); a later stage that exceeds that more than 64-fold takes a smaller scale, and the sums so far follow it (a power of two:
// exact). Values down to 2^-22 of the largest that they are summed with keep all bits of both terms, below that the error is 2^-44 of that
// one. An infinity or NaN makes NaN of every output it meets. (One scale for 64 columns of a weight gradient, a single maximum per
// wavefront, lost the gradients of columns far smaller than their neighbours - features of different units: 2^-31 of the largest, relative
// error 1.7e-4.)
//
// A workgroup of four wavefronts computes a 128 x 128 tile of C (128 x 64 for outputs at most 64 columns wide), a
// wavefront 64 x 64 (32 x 64); two workgroups are resident per compute unit. A stage of 32
// reduction steps is fetched into registers one step ahead, then split and written to LDS as two planes of
// fp16 rows (one output index per row, reduction index contiguous, 80-byte pitch). A is split here; B is the library's own split copy of the
// weights (varco_launch_prep_weights), zero-padded to whole tiles and copied as is. The ReLU mask of the backward pass is applied before
// the split.
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "gemm_tile.h"
#include "half_terms.h"
#include "varco_internal.h"

namespace {

constexpr int BK = 32;
constexpr int kThreads = 256;
constexpr int kPitch = BK + 8;   // fp16 elements per LDS row (80 bytes)
constexpr int kShortSum = 32;    // up to this many products per sum the fourth product is formed as well
constexpr int kFirst = 8;        // exponent that the largest value of a first stage is brought to, which leaves
constexpr int kRoom = 6;         // later ones this many binades
constexpr int kPrepRows = 128;   // split weight copies are padded to this many rows (the widest B tile) and to BK columns

typedef float floatx16 __attribute__((ext_vector_type(16)));
struct HalfOperand {
    const void* ptr;      // fp32 matrix, or the split copy of a weight matrix
    const float* gate;
    int64_t ld;
};

struct HalfGemm {
    int32_t m, n, k;
    HalfOperand a, b;
    float* c;
    int64_t ldc;
    int32_t accumulate;
    int32_t tiles_m, tiles_n;
    int32_t inner;                   // tiles along the fast direction of the workgroup order
    const void* dual;                // second split B, or null
    float* c_dual;
    int64_t exps;                    // place of the scale exponents in a split copy (elements)
};

typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float largest4(float m, const float4& x) {
    return fmaxf(fmaxf(fmaxf(m, fabsf(x.x)), fmaxf(fabsf(x.y), fabsf(x.z))), fabsf(x.w));
}
__device__ __forceinline__ float4 gate4(float4 x, float4 y) {
    x.x = y.x > 0.f ? x.x : 0.f, x.y = y.y > 0.f ? x.y : 0.f;
    x.z = y.z > 0.f ? x.z : 0.f, x.w = y.w > 0.f ? x.w : 0.f;
    return x;
}

// Consecutive groups of lanes write consecutive tile rows; with an 80-byte pitch rows r and r + 1 overlap in
// four LDS banks while rows r and r + 4 tile all of them, so the q-th row group of a wavefront goes to row
// (q with its low three bits rotated): 0 4 1 5 2 6 3 7.
__device__ __forceinline__ int tile_row(int q) { return (q & ~7) | ((q & 1) << 2) | ((q >> 1) & 3); }

// A group of four that crosses the end of its row is loaded from four elements before the end and moved up by `by` (1 to 3)
// elements; what follows the end is zero.
__device__ __forceinline__ float4 moved_up(float4 x, int by) {
    if (by == 1) return make_float4(x.y, x.z, x.w, 0.f);
    if (by == 2) return make_float4(x.z, x.w, 0.f, 0.f);
    return make_float4(x.w, 0.f, 0.f, 0.f);
}

// ---- fp32 operand with the reduction index contiguous: chunks of CH floats ----
// Addresses are a per-tile base (uniform) plus a 32-bit offset per chunk that does not change along the
// reduction. Rows beyond the matrix are clamped to its last row (their results are never stored); chunks
// beyond the reduction length re-read values of the same row, and meet zeros in B. Chunks of four may be of any
// alignment; one that crosses the end of its row, or lies beyond it, is loaded from four values before the end (the reduction has at
// least four), and the crossing one is moved up. Such a start may lie up to three values before the stage's first one, so that
// offsets count from four values before the tile's base: they are unsigned.
template <int ROWS, int CH, bool GATE>
struct RowRegs {
    static constexpr int PER_ROW = BK / CH;
    static constexpr int N = ROWS * PER_ROW / kThreads;
    float4 v[N][CH / 4];
    float4 g[GATE ? N : 1][CH / 4];
    int e[N];            // scale exponents of the chunks' rows
};

template <int ROWS, int CH>
struct RowPlan {
    static constexpr int PER_ROW = BK / CH;
    static constexpr int N = ROWS * PER_ROW / kThreads;
    uint32_t off[N];     // bytes from four values before the tile base
    __device__ __forceinline__ void init(int tid, int32_t i0, int32_t extent, int64_t ld) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int c = tid + h * kThreads;
            const int32_t r = min(tile_row(c / PER_ROW), extent - 1 - i0);
            off[h] = uint32_t(r * ld + (c % PER_ROW) * CH + 4) * 4u;
        }
    }
};

template <int ROWS, int CH, bool GATE>
__device__ __forceinline__ void load_rows(int tid, const float* base, const float* gate, const RowPlan<ROWS, CH>& plan,
                                          int32_t k_left, RowRegs<ROWS, CH, GATE>& r) {
    using R = RowRegs<ROWS, CH, GATE>;
    const int kc = (tid % R::PER_ROW) * CH;             // the same in all of a thread's chunks
    uint32_t back;                                      // bytes from the chunk's place to where it is read
    if constexpr (CH == 4)
        back = uint32_t(max(kc + 4 - k_left, 0)) * 4u;  // from k_left - 4 at most: at least the row's first value, and k_left - 4 >= -3
    else
        back = kc < k_left ? 0u : uint32_t(kc) * 4u;    // k_left is a multiple of CH
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const uint32_t off = plan.off[h] - back;
#pragma unroll
        for (int u = 0; u < CH / 4; ++u) {
            r.v[h][u] = load4_at(base - 4, off + 16u * u);
            if (GATE) r.g[h][u] = load4_at(gate - 4, off + 16u * u);
        }
    }
}

// Masks, scales, splits and writes a stage's rows; first: of the tile's first stage. left: reduction steps from the stage's first on.
// scales[row] = {exponent, bits of the factor that the sums so far take}; whether any row of this wavefront took a smaller scale.
template <int ROWS, int CH, bool GATE>
__device__ __forceinline__ bool store_rows(int tid, RowRegs<ROWS, CH, GATE>& r, bool first, int32_t left, uint16_t* s, int2* scales) {
    using R = RowRegs<ROWS, CH, GATE>;
    const int kc = (tid % R::PER_ROW) * CH;
    bool grew = false;
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const int row = tile_row((tid + h * kThreads) / R::PER_ROW);
        float m = 0.f;
        float4 x[CH / 4];
#pragma unroll
        for (int u = 0; u < CH / 4; ++u) {
            x[u] = r.v[h][u];
            if (GATE) x[u] = gate4(x[u], r.g[h][u]);
            if (CH == 4 && left < BK && (left & 3))
                if (kc < left && kc + 4 > left) x[u] = moved_up(x[u], 4 - (left & 3));
            m = largest4(m, x[u]);
        }
        const int e = scale_exponent(largest_of_lanes<R::PER_ROW>(m), kFirst);
        int old = first ? e : r.e[h];
        const bool smaller = e < old - kRoom;
        const int now = smaller ? e : old;
        r.e[h] = now, grew = grew || smaller;
        if (kc == 0) scales[row] = make_int2(now, int(__float_as_uint(power_of_two(max(now - old, -126)))));
        const float sc = power_of_two(now);
        uint32_t hi[CH / 2], lo[CH / 2];
#pragma unroll
        for (int u = 0; u < CH / 4; ++u) {
            split_pair(x[u].x * sc, x[u].y * sc, hi[2 * u], lo[2 * u]);
            split_pair(x[u].z * sc, x[u].w * sc, hi[2 * u + 1], lo[2 * u + 1]);
        }
        uint16_t* dst = s + row * kPitch + kc;
        if constexpr (CH == 8) {
            *reinterpret_cast<uint4*>(dst) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4*>(dst + ROWS * kPitch) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        } else {
            *reinterpret_cast<uint2*>(dst) = make_uint2(hi[0], hi[1]);
            *reinterpret_cast<uint2*>(dst + ROWS * kPitch) = make_uint2(lo[0], lo[1]);
        }
    }
    return grew;
}

// ---- split weight copy: chunks of 8 elements, copied unchanged ----
// The copy is stored by tile and stage, [row tile][stage of BK reduction steps][term][row in tile][BK], so that what
// a workgroup fetches per step is one contiguous block (whole cache lines, one 1 KB run per wavefront load), and it
// is zero-padded to whole tiles and stages, so no chunk needs a bounds check.
constexpr int TERMS = 2;
template <int ROWS>
struct PrepRegs {
    static constexpr int PER_ROW = BK / 8;
    static constexpr int N = TERMS * ROWS * PER_ROW / kThreads;
    uint4 v[N];
};

template <int ROWS>
struct PrepPlan {
    static constexpr int PER_ROW = BK / 8;
    static constexpr int N = TERMS * ROWS * PER_ROW / kThreads;
    uint32_t off[N];     // bytes from the block's base
    __device__ __forceinline__ void init(int tid) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int c = tid + h * kThreads;
            const int p = c / (ROWS * PER_ROW), rc = c % (ROWS * PER_ROW);
            off[h] = uint32_t((p * ROWS + tile_row(rc / PER_ROW)) * BK + (rc % PER_ROW) * 8) * 2u;
        }
    }
};

template <int ROWS>
__device__ __forceinline__ void load_prep(const uint16_t* base, const PrepPlan<ROWS>& plan, PrepRegs<ROWS>& r) {
#pragma unroll
    for (int h = 0; h < PrepRegs<ROWS>::N; ++h) r.v[h] = load_at<uint4>(base, plan.off[h]);
}

template <int ROWS>
__device__ __forceinline__ void store_prep(int tid, const PrepRegs<ROWS>& r, uint16_t* s) {
    using R = PrepRegs<ROWS>;
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const int c = tid + h * kThreads;
        const int p = c / (ROWS * R::PER_ROW), rc = c % (ROWS * R::PER_ROW);
        *reinterpret_cast<uint4*>(s + p * ROWS * kPitch + tile_row(rc / R::PER_ROW) * kPitch + (rc % R::PER_ROW) * 8) = r.v[h];
    }
}

__device__ __forceinline__ halfx8 fragment(const uint16_t* s, int row, int koff) {
    return __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4*>(s + row * kPitch + koff));
}

template <int TMB, int TNB>
__device__ __forceinline__ void multiply(const halfx8 (&fa)[TMB], const halfx8 (&fb)[TNB], floatx16 (&acc)[TMB][TNB]) {
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fb[j], acc[i][j], 0, 0, 0);
}

// WM x WN wavefronts per tile, each TMB x TNB blocks of 32 x 32. A_CH: floats per chunk of A. GATE masks A.
template <int WM, int WN, int TMB, int TNB, int A_CH, bool GATE, bool FOUR>
__global__ __launch_bounds__(kThreads, 2) void gemm_half_kernel(HalfGemm g) {
    constexpr int BM = 32 * TMB * WM, BN = 32 * TNB * WN;
    __shared__ __attribute__((aligned(16))) uint16_t smem[TERMS * (BM + BN) * kPitch];
    __shared__ __attribute__((aligned(16))) int2 scales[BM];
    __shared__ int32_t smaller_at;                                // last stage in which a scale got smaller
    const int tid = threadIdx.x;
    uint16_t* const sa = smem;
    uint16_t* const sb = smem + TERMS * BM * kPitch;

    // workgroup -> tile: tiles that share streamed data go to one XCD (workgroups are dealt to the 8 XCDs
    // round-robin), so that the streamed operand is fetched into a single L2
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3;
    const int32_t in = within % g.inner, out = (within / g.inner) * 8 + xcd;
    if (out >= g.tiles_m) return;              // whole workgroup leaves together: no barrier is skipped
    const bool second = in >= g.tiles_n;       // this workgroup's tile belongs to the dual product
    const int32_t tm = out, tn = second ? in - g.tiles_n : in, steps = (g.k + BK - 1) / BK;
    const void* const b_ptr = second ? g.dual : g.b.ptr;
    const int32_t m0 = tm * BM, n0 = tn * BN;

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // uniform: addresses built from it stay scalar
    const int wm = (wave / WN) * (32 * TMB), wn = (wave % WN) * (32 * TNB);
    const int lrow = lane & 31, lk = lane >> 5;

    floatx16 acc[TMB][TNB], low[TMB][TNB];
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;
    if (tid == 0) smaller_at = -1;                // (whichever write of the first stage lasts: there are no sums yet)

    // staging registers and per-thread offsets
    RowRegs<BM, A_CH, GATE> ra;
    PrepRegs<BN> rb;
    RowPlan<BM, A_CH> plan_a;
    PrepPlan<BN> plan_b;
    plan_a.init(tid, m0, g.m, g.a.ld);
    plan_b.init(tid);

    auto fetch = [&](int32_t t) {
        const int32_t k0 = t * BK;
        const float* abase = static_cast<const float*>(g.a.ptr) + int64_t(m0) * g.a.ld + k0;
        const float* gbase = GATE ? g.a.gate + int64_t(m0) * g.a.ld + k0 : nullptr;
        const uint16_t* bbase = static_cast<const uint16_t*>(b_ptr) + (int64_t(tn) * (g.b.ld / BK) + t) * (TERMS * BN * BK);   // g.b.ld: padded reduction length
        load_rows<BM, A_CH, GATE>(tid, abase, gbase, plan_a, g.k - k0, ra);
        load_prep<BN>(bbase, plan_b, rb);
    };
    auto stash = [&](int32_t t) __attribute__((always_inline)) {
        if (store_rows<BM, A_CH, GATE>(tid, ra, t == 0, g.k - t * BK, sa, scales)) smaller_at = t;
        store_prep<BN>(tid, rb, sb);
    };
    // Half steps that hold padding only are left out: at most 16 values left means that only the first half multiplies.
    auto compute = [&](int32_t t) __attribute__((always_inline)) {
        const int32_t left = g.k - t * BK;
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            if (s * 16 >= left) break;
            const int koff = s * 16 + lk * 8;
            // (operands are read in the order of their use: two sets of sums leave few registers)
            halfx8 a0[TMB], b0[TNB];
#pragma unroll
            for (int i = 0; i < TMB; ++i) a0[i] = fragment(sa, wm + i * 32 + lrow, koff);
#pragma unroll
            for (int j = 0; j < TNB; ++j) b0[j] = fragment(sb, wn + j * 32 + lrow, koff);
            halfx8 b1[TNB];
#pragma unroll
            for (int j = 0; j < TNB; ++j) b1[j] = fragment(sb + BN * kPitch, wn + j * 32 + lrow, koff);
            multiply<TMB, TNB>(a0, b0, acc);
            multiply<TMB, TNB>(a0, b1, low);
            halfx8 a1[TMB];
#pragma unroll
            for (int i = 0; i < TMB; ++i) a1[i] = fragment(sa + BM * kPitch, wm + i * 32 + lrow, koff);
            multiply<TMB, TNB>(a1, b0, low);
            if constexpr (FOUR) {
#pragma unroll
                for (int i = 0; i < TMB; ++i) a1[i] *= _Float16(1.f / kHalfLow);
                multiply<TMB, TNB>(a1, b1, low);
            }
        }
    };
    // The sums so far follow rows that took a smaller scale with this stage.
    auto follow = [&](int32_t t) __attribute__((always_inline)) {
        if (__builtin_amdgcn_readfirstlane(smaller_at) != t) return;
#pragma unroll
        for (int i = 0; i < TMB; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float f = __uint_as_float(uint32_t(scales[wm + i * 32 + 8 * (v >> 2) + 4 * lk + (v & 3)].y));
#pragma unroll
                for (int j = 0; j < TNB; ++j) acc[i][j][v] *= f, low[i][j][v] *= f;
            }
    };

    // One LDS stage: a step's operands are fetched into registers while the previous step is multiplied, then
    // split and written once its fragments have been read. (A second register set, fetching two steps ahead,
    // was measured and changes nothing.)
    if (steps > 0) fetch(0);
    for (int32_t t = 0; t < steps; ++t) {
        stash(t);
        if (t + 1 < steps) fetch(t + 1);
        __syncthreads();
        follow(t);
        compute(t);
        __syncthreads();       // the stage's fragments have been read: the next one may overwrite them
    }
    if (steps == 0) return;
    // both sums, scales taken out
#pragma unroll
    for (int i = 0; i < TMB; ++i) {
        int e[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) e[v] = scales[wm + i * 32 + 8 * (v >> 2) + 4 * lk + (v & 3)].x;
#pragma unroll
        for (int j = 0; j < TNB; ++j) {
            const int eb = reinterpret_cast<const int32_t*>(static_cast<const uint16_t*>(b_ptr) + g.exps)[n0 + wn + j * 32 + lrow];
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = __builtin_ldexpf(acc[i][j][v] + low[i][j][v] * (1.f / kHalfLow), -(e[v] + eb));
        }
    }

    store_tile(acc, second ? g.c_dual : g.c, g.ldc, g.m, g.n, m0 + wm, n0 + wn, m0 + BM <= g.m && n0 + BN <= g.n, lane, g.accumulate != 0, false);
}

bool aligned_to(const void* p, uintptr_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

template <class F>
void with_flag(bool b, F&& f) {
    if (b)
        f(std::true_type{});
    else
        f(std::false_type{});
}

}  // namespace

bool varco_gemm_half_usable(const GemmArgs& ga) {
    if ((ga.f32_terms != 2 && ga.f32_terms != 3) || ga.m <= 0 || ga.n <= 0 || ga.k2 > 0 || ga.relu) return false;
    if (ga.a.dtype != VARCO_F32 || ga.c_dtype != VARCO_F32) return false;
    auto ok4 = [](const GemmOperand& o) { return aligned_to(o.ptr, 4) && aligned_to(o.gate, 4); };
    if (!ga.a.transposed) {   // NT: needs the library's split weight copy, padded to whole tiles
        if (!ga.b_halves || !ga.b_prep || !aligned_to(ga.b_prep, 16) || ga.b_prep_ld % BK != 0 || ga.b_prep_ld < ga.k ||
            ga.b_prep_plane != (int64_t(ga.n) + kPrepRows - 1) / kPrepRows * kPrepRows * ga.b_prep_ld)
            return false;
        if (ga.b.gate || ga.k < 4 || ga.split_k > 1 || !ok4(ga.a)) return false;
        return !ga.c_dual || (ga.b_dual_prep && aligned_to(ga.b_dual_prep, 16));
    }
    // TN: weight gradient
    if (ga.c_dual && (!ga.a_dual || !aligned_to(ga.a_dual, 4))) return false;
    if (ga.b.transposed || ga.b.dtype != VARCO_F32 || ga.a.gate) return false;
    return ok4(ga.a) && ok4(ga.b) && ga.m >= 4 && ga.n >= 4;
}

hipError_t varco_launch_gemm_half(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag) {
    const bool narrow = ga.n <= 64;
    const int bm = 128, bn = narrow ? 64 : 128;
    auto f32 = [](const void* p) { return static_cast<const float*>(p); };
    HalfGemm g{};
    g.m = ga.m, g.n = ga.n, g.k = ga.k;
    g.a = {ga.a.ptr, f32(ga.a.gate), ga.a.ld};
    g.b = {ga.b_prep, nullptr, ga.b_prep_ld};
    g.exps = 2 * ga.b_prep_plane;
    g.c = static_cast<float*>(ga.c), g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0;
    g.tiles_m = (ga.m + bm - 1) / bm, g.tiles_n = (ga.n + bn - 1) / bn;
    g.dual = ga.c_dual ? ga.b_dual_prep : nullptr;
    g.c_dual = static_cast<float*>(ga.c_dual);
    g.inner = g.tiles_n * (ga.c_dual ? 2 : 1);      // the dual product's tiles come right behind the first one's, on the same XCD
    const int64_t blocks = int64_t((g.tiles_m + 7) / 8 * 8) * g.inner;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid{unsigned(blocks)};

    tag.begin(stream);
    with_flag(narrow, [&](auto nr) {
        with_flag(ga.a.gate != nullptr, [&](auto gt) {
            with_flag(ga.k <= kShortSum, [&](auto fr) {
                constexpr bool NR = decltype(nr)::value, GT = decltype(gt)::value, FR = decltype(fr)::value;
                constexpr int WM = NR ? 4 : 2, WN = NR ? 1 : 2, TMB = NR ? 1 : 2, TNB = 2;
                if (ga.k % 8 == 0)
                    hipLaunchKernelGGL((gemm_half_kernel<WM, WN, TMB, TNB, 8, GT, FR>), grid, dim3(kThreads), 0, stream, g);
                else
                    hipLaunchKernelGGL((gemm_half_kernel<WM, WN, TMB, TNB, 4, GT, FR>), grid, dim3(kThreads), 0, stream, g);
            });
        });
    });
    tag.end(stream);
    return hipGetLastError();
}
