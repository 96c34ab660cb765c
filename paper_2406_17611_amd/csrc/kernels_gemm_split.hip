// Dense feature transform of eq. (2) for fp32-stored activations, computed on the bf16
// matrix cores from exact bf16 expansions of the fp32 operands:
//     x = x0 + x1 + x2,   x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1)
// (each difference is exact in fp32, and three 8-bit significands cover the 24 bits of x), so
//     a * b = a0 b0 + (a0 b1 + a1 b0) + (a1 b1 + a0 b2 + a2 b0) + terms below 2^-24 |a b|.
// The six kept products are exact in the fp32 accumulators of v_mfma_f32_32x32x16_bf16, which leaves the
// result with the accuracy of an fp32 product-sum; six bf16 instructions cost 6/16 of the fp32 matrix
// instructions that cover the same reduction steps. TERMS = 2 keeps x0 + x1 and three products (relative
// error about 2^-16 per product); the library does not use it by default.
// (The gradients take two fp16 terms and three products, kernels_gemm_half.hip, which is faster and no less accurate. The forward
// pass keeps this form and the order of its sums, so that a ReLU whose argument, or an argmax whose two logits, are within rounding
// of each other decide as they always did; that forgoes 0.7 of 3.30 ms for K = 2 x 256, N = 256 over 2,449,029 rows. Reductions of 65 to 256
// steps mostly go to kernels_gemm_split_rows.hip, which forms the same sums.)
//
// A workgroup of four wavefronts computes a 128 x 128 tile of C (128 x 64 for outputs at most 64 columns wide), a
// wavefront 64 x 64 (32 x 64); three workgroups are resident per compute unit (see the kernel). A stage of 32
// reduction steps is fetched into registers one step ahead, then expanded and written to LDS as TERMS planes of
// bf16 rows (one output index per row, reduction index contiguous, 64-byte pitch, pieces rotated). A has the reduction index contiguous and is
// expanded here; B is the library's own expanded copy of the weights (varco_launch_prep_weights), zero-padded
// to whole tiles and copied as is. The activation is applied in the epilogue.
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "gemm_tile.h"
#include "half_terms.h"
#include "prep_device.h"
#include "varco_internal.h"

namespace {

constexpr int BK = 32;
constexpr int kThreads = 256;
constexpr int kMaxChain = 4;     // products of a chain (gemm_split_kernel)
constexpr int kPitch = BK;       // bf16 elements per LDS row (64 bytes)
constexpr int kPrepRows = 128;   // expanded weight copies are padded to this many rows (the widest B tile) and to BK columns

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct SplitOperand {
    const void* ptr;      // fp32 matrix, or the expanded bf16 copy of a weight matrix
    int64_t ld;
};

struct SplitGemm {
    int32_t m, n, k, k2;
    SplitOperand a, b, a2, b2;
    float* c;
    int64_t ldc;
    int32_t accumulate, relu;
    int32_t tiles_m, tiles_n;
    int32_t taps;                          // CHAIN: products of k steps each
    const float* tap_a[kMaxChain];
    const uint16_t* tap_b[kMaxChain];
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// Two fp32 values rounded to bf16 (nearest even) by one packed conversion; `lo` in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    const floatx2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Expansion of two fp32 values: w[p] holds term p of both (x0 in the low half).
template <int TERMS>
__device__ __forceinline__ void expand_pair(float x0, float x1, uint32_t (&w)[TERMS]) {
#pragma unroll
    for (int p = 0; p < TERMS; ++p) {
        w[p] = pack_bf16(x0, x1);
        if (p + 1 < TERMS) {
            x0 -= __uint_as_float(w[p] << 16);
            x1 -= __uint_as_float(w[p] & 0xFFFF0000u);
        }
    }
}

// LDS rows are 64 bytes, four of them cover the banks once; the 16-byte pieces of every fourth row are rotated differently, so that
// the 16 rows whose fragments are read together lie in 16 different places.
__device__ __forceinline__ int lds_at(int row, int k) { return row * kPitch + (k ^ ((row << 1) & 24)); }      // (bits 2, 3 of the row)

// ---- fp32 operand with the reduction index contiguous: chunks of CH floats ----
// Addresses are a per-tile base (uniform) plus a 32-bit offset per chunk that does not change along the
// reduction. Rows beyond the matrix are clamped to its last row (their results are never stored); chunks
// beyond the reduction length re-read the tile's first chunk of the same row, and meet zeros in B.
template <int ROWS, int CH>
struct RowRegs {
    static constexpr int PER_ROW = BK / CH;
    static constexpr int N = ROWS * PER_ROW / kThreads;
    float4 v[N][CH / 4];
};

template <int ROWS, int CH>
struct RowPlan {
    static constexpr int PER_ROW = BK / CH;
    static constexpr int N = ROWS * PER_ROW / kThreads;
    uint32_t off[N];     // bytes from the tile base
    __device__ __forceinline__ void init(int tid, int32_t i0, int32_t extent, int64_t ld) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int c = tid + h * kThreads;
            const int32_t r = min(c / PER_ROW, extent - 1 - i0);
            off[h] = uint32_t(r * ld + (c % PER_ROW) * CH) * 4u;
        }
    }
};

template <int ROWS, int CH>
__device__ __forceinline__ void load_rows(int tid, const float* base, const RowPlan<ROWS, CH>& plan, int32_t k_left, RowRegs<ROWS, CH>& r) {
    using R = RowRegs<ROWS, CH>;
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const int kc = ((tid + h * kThreads) % R::PER_ROW) * CH;
        const uint32_t off = kc < k_left ? plan.off[h] : plan.off[h] - uint32_t(kc) * 4u;   // k_left is a multiple of CH
#pragma unroll
        for (int u = 0; u < CH / 4; ++u) r.v[h][u] = load4_at(base, off + 16u * u);
    }
}

template <int TERMS, int ROWS, int CH>
__device__ __forceinline__ void store_rows(int tid, const RowRegs<ROWS, CH>& r, uint16_t* s) {
    using R = RowRegs<ROWS, CH>;
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const int c = tid + h * kThreads;
        uint32_t w[CH / 2][TERMS];
#pragma unroll
        for (int u = 0; u < CH / 4; ++u) {
            const float4 x = r.v[h][u];
            expand_pair<TERMS>(x.x, x.y, w[2 * u]);
            expand_pair<TERMS>(x.z, x.w, w[2 * u + 1]);
        }
        uint16_t* dst = s + lds_at(c / R::PER_ROW, (c % R::PER_ROW) * CH);
#pragma unroll
        for (int p = 0; p < TERMS; ++p) {
            if constexpr (CH == 8)
                *reinterpret_cast<uint4*>(dst + p * ROWS * kPitch) = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
            else
                *reinterpret_cast<uint2*>(dst + p * ROWS * kPitch) = make_uint2(w[0][p], w[1][p]);
        }
    }
}

// ---- expanded bf16 weight copy: chunks of 8 elements, copied unchanged ----
// The copy is stored by tile and stage, [row tile][stage of BK reduction steps][term][row in tile][BK], so that what
// a workgroup fetches per step is one contiguous block (whole cache lines, one 1 KB run per wavefront load), and it
// is zero-padded to whole tiles and stages, so no chunk needs a bounds check.
template <int TERMS, int ROWS>
struct PrepRegs {
    static constexpr int PER_ROW = BK / 8;
    static constexpr int N = TERMS * ROWS * PER_ROW / kThreads;
    uint4 v[N];
};

template <int TERMS, int ROWS>
__device__ __forceinline__ void load_prep(int tid, const uint16_t* base, PrepRegs<TERMS, ROWS>& r) {
#pragma unroll
    for (int h = 0; h < PrepRegs<TERMS, ROWS>::N; ++h) r.v[h] = load_at<uint4>(base + h * kThreads * 8, uint32_t(tid) * 16u);
}

template <int TERMS, int ROWS>
__device__ __forceinline__ void store_prep(int tid, const PrepRegs<TERMS, ROWS>& r, uint16_t* s) {
    using R = PrepRegs<TERMS, ROWS>;
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const int c = tid + h * kThreads;
        const int p = c / (ROWS * R::PER_ROW), rc = c % (ROWS * R::PER_ROW);
        *reinterpret_cast<uint4*>(s + p * ROWS * kPitch + lds_at(rc / R::PER_ROW, (rc % R::PER_ROW) * 8)) = r.v[h];
    }
}

__device__ __forceinline__ bf16x8 fragment(const uint16_t* s, int row, int koff) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(s + lds_at(row, koff)));
}

template <int TMB, int TNB, int PA, int PB>
__device__ __forceinline__ void multiply(const bf16x8 (&fa)[3][TMB], const bf16x8 (&fb)[3][TNB], floatx16 (&acc)[TMB][TNB]) {
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA][i], fb[PB][j], acc[i][j], 0, 0, 0);
}

// WM x WN wavefronts per tile, each TMB x TNB blocks of 32 x 32. A_CH: floats per chunk of A.
//
// A workgroup is four wavefronts with one tile and one LDS stage (48 KB, rows without padding), so that three workgroups are
// resident on a compute unit and each SIMD holds one wavefront of each. On this device the vector ALU and the matrix
// unit of a SIMD do not run side by side (hardware counters: their busy times add up), so nothing is gained by
// steering one wavefront's conversions under the other's products; what matters is that the SIMD always has a
// wavefront that can issue, and that as few vector instructions as possible accompany the matrix instructions.
// Independent workgroups give the first: while one waits at a barrier, for its global loads, or stores its
// tile, the others multiply. (With rows padded to 80 bytes, two resident: the units idle 38 % of the time. 2,449,029 rows, 256 x 256
// 1,996 -> 1,895 us, 100 x 256 1,171 -> 1,086; 169,343 rows 146 -> 137, 77 -> 70; 50,021 rows, whose tiles end just past a round of three
// per unit, 47.6 -> 49.5.)
// CHAIN: the taps of a K-tap layer, act(((Y_0 H_0) + Y_1 H_1) + ..), each product summed by itself and added to the ones before it as launches
// that add to C would, bit for bit, without C being written and read between them: a second set of accumulators, two workgroups
// per compute unit where that takes 64 registers. Three taps over 60,013 rows, us, launch by launch / together: 64 -> 128 49 / 24, 128 -> 24
// 33 / 24.
template <int TERMS, int WM, int WN, int TMB, int TNB, int A_CH, bool CHAIN = false>
__global__ __launch_bounds__(kThreads, CHAIN && TMB * TNB > 2 ? 2 : 3) void gemm_split_kernel(SplitGemm g) {
    static_assert(TERMS == 2 || TERMS == 3, "two or three bf16 terms per operand");
    constexpr int BM = 32 * TMB * WM, BN = 32 * TNB * WN;
    __shared__ __attribute__((aligned(16))) uint16_t smem[TERMS * (BM + BN) * kPitch];
    const int tid = threadIdx.x;
    uint16_t* const sa = smem;
    uint16_t* const sb = smem + TERMS * BM * kPitch;

    // workgroup -> tile: tiles that share streamed data go to one XCD (workgroups are dealt to the 8 XCDs
    // round-robin), so that the streamed operand is fetched into a single L2
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3;
    const int32_t tn = within % g.tiles_n, tm = (within / g.tiles_n) * 8 + xcd;
    if (tm >= g.tiles_m) return;               // whole workgroup leaves together: no barrier is skipped
    const int32_t tiles1 = (g.k + BK - 1) / BK, tiles2 = (g.k2 + BK - 1) / BK, steps = CHAIN ? g.taps * tiles1 : tiles1 + tiles2;
    const int32_t m0 = tm * BM, n0 = tn * BN;

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // uniform: addresses built from it stay scalar
    const int wm = (wave / WN) * (32 * TMB), wn = (wave % WN) * (32 * TNB);
    const int lrow = lane & 31, lk = lane >> 5;

    floatx16 acc[TMB][TNB];
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    floatx16 total[CHAIN ? TMB : 1][CHAIN ? TNB : 1] = {};

    // staging registers and per-thread offsets
    RowRegs<BM, A_CH> ra;
    PrepRegs<TERMS, BN> rb;
    RowPlan<BM, A_CH> plan_a;
    plan_a.init(tid, m0, g.m, g.a.ld);            // a chained second product has the same leading dimensions

    auto fetch = [&](int32_t t) {
        if constexpr (CHAIN) {
            const int32_t tap = t / tiles1, stage = t - tap * tiles1;
            load_rows<BM, A_CH>(tid, g.tap_a[tap] + int64_t(m0) * g.a.ld + stage * BK, plan_a, g.k - stage * BK, ra);
            load_prep<TERMS, BN>(tid, g.tap_b[tap] + (int64_t(tn) * (g.b.ld / BK) + stage) * (TERMS * BN * BK), rb);
            return;
        }
        const bool first = t < tiles1;
        const int32_t k0 = (first ? t : t - tiles1) * BK, k_left = (first ? g.k : g.k2) - k0;
        const float* abase = static_cast<const float*>(first ? g.a.ptr : g.a2.ptr) + int64_t(m0) * g.a.ld + k0;
        const uint16_t* bbase = static_cast<const uint16_t*>(first ? g.b.ptr : g.b2.ptr) +
                                (int64_t(tn) * (g.b.ld / BK) + k0 / BK) * (TERMS * BN * BK);      // g.b.ld: padded reduction length
        load_rows<BM, A_CH>(tid, abase, plan_a, k_left, ra);
        load_prep<TERMS, BN>(tid, bbase, rb);
    };
    auto stash = [&]() {
        store_rows<TERMS, BM, A_CH>(tid, ra, sa);
        store_prep<TERMS, BN>(tid, rb, sb);
    };
    // Half steps that hold padding only are left out: at most 16 values left means that only the first half multiplies.
    // (K = 2 x 100, N = 256 over 2,449,029 rows: 2.04 ms for all of 2 x 128, 1.92 without, both with two workgroups resident.)
    auto compute = [&](int32_t t) {
        const int32_t left = CHAIN ? g.k - t % tiles1 * BK : t < tiles1 ? g.k - t * BK : g.k2 - (t - tiles1) * BK;
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            if (s * 16 >= left) break;
            const int koff = s * 16 + lk * 8;
            bf16x8 fa[3][TMB], fb[3][TNB];
#pragma unroll
            for (int p = 0; p < TERMS; ++p) {
#pragma unroll
                for (int i = 0; i < TMB; ++i) fa[p][i] = fragment(sa + p * BM * kPitch, wm + i * 32 + lrow, koff);
#pragma unroll
                for (int j = 0; j < TNB; ++j) fb[p][j] = fragment(sb + p * BN * kPitch, wn + j * 32 + lrow, koff);
            }
            multiply<TMB, TNB, 0, 0>(fa, fb, acc);
            multiply<TMB, TNB, 0, 1>(fa, fb, acc);
            multiply<TMB, TNB, 1, 0>(fa, fb, acc);
            if constexpr (TERMS == 3) {
                multiply<TMB, TNB, 1, 1>(fa, fb, acc);
                multiply<TMB, TNB, 0, 2>(fa, fb, acc);
                multiply<TMB, TNB, 2, 0>(fa, fb, acc);
            }
        }
    };

    // One LDS stage: a step's operands are fetched into registers while the previous step is multiplied, then
    // expanded and written once its fragments have been read. (A second register set, fetching two steps ahead,
    // was measured and changes nothing.)
    if (steps > 0) fetch(0);
    for (int32_t t = 0; t < steps; ++t) {
        stash();
        if (t + 1 < steps) fetch(t + 1);
        __syncthreads();
        compute(t);
        if constexpr (CHAIN)
            if ((t + 1) % tiles1 == 0)
#pragma unroll
                for (int i = 0; i < TMB; ++i)
#pragma unroll
                    for (int j = 0; j < TNB; ++j) total[i][j] = acc[i][j] + total[i][j], acc[i][j] = floatx16{};
        __syncthreads();       // the stage's fragments have been read: the next one may overwrite them
    }

    const bool inside = m0 + BM <= g.m && n0 + BN <= g.n;
    if constexpr (CHAIN)
        store_tile(total, g.c, g.ldc, g.m, g.n, m0 + wm, n0 + wn, inside, lane, false, g.relu != 0);
    else
        store_tile(acc, g.c, g.ldc, g.m, g.n, m0 + wm, n0 + wn, inside, lane, g.accumulate != 0, g.relu != 0);
}

// ---------------------------------------------------------------------------------------------------------
// Short reductions on the bf16 matrix units: C (+)= A B^T with at most 64 reduction steps and densely stored
// rows of A (an input gradient that reduces over few outputs; fp32 storage with 17 steps and more mostly goes to kernels_gemm_half.hip,
// half_takes_short). Rows of, say, 47
// elements are not 16-byte aligned, so a workgroup takes tiles of 64 rows of A, each one contiguous range of memory,
// with 16-byte loads, masks the values, expands them into TERMS bf16 terms once and writes them to LDS as rows of matrix
// operands (16 bytes of padding per row). Each wavefront owns 64 columns of C: their weights, expanded alike, sit in registers
// for the whole kernel, so workgroups are persistent over the tiles, and the next tile's range is requested before the
// current one is multiplied. The blocks are formed transposed (weights as the first matrix operand): a lane then holds four
// consecutive columns of a row, and a block of 32 rows leaves through LDS in whole lines.
// Bound by writing C. (One tile of 128 rows per workgroup, its values expanded by each wavefront from fp32 rows in LDS, which
// lay in few banks when the number of classes was a multiple of 8: 169,343 x 256 from 40 outputs 77 us, 57 now; 2,449,029
// x 2 x 256 from 47: 1.96 ms, 1.40 now.)
// With fp32 matrix instructions (still used when the context asks for them) the product is bound by those. TERMS = 1: bf16
// storage (the values are bf16 already; the weights are rounded to bf16 as for the other products of that storage type).
constexpr int kShortRows = 64;
constexpr int kEpiPitch = 68;      // floats per row of the epilogue's LDS block (64 + 4: rows start on different banks)

// Eight consecutive values as TERMS bf16 fragments.
template <int TERMS>
__device__ __forceinline__ void expand8(const float (&x)[8], bf16x8 (&f)[3]) {
    uint32_t w[4][TERMS];
#pragma unroll
    for (int q = 0; q < 4; ++q) expand_pair<TERMS>(x[2 * q], x[2 * q + 1], w[q]);
#pragma unroll
    for (int p = 0; p < TERMS; ++p) f[p] = __builtin_bit_cast(bf16x8, make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]));
}

template <typename T, int KS, bool GATE, int TERMS>
__global__ __launch_bounds__(kThreads, 2) void gemm_short_k_kernel(const T* __restrict__ a, const T* __restrict__ gate,
                                                                   const float* __restrict__ b, int64_t ldb, T* __restrict__ c,
                                                                   int64_t ldc, int32_t m, int32_t n, int32_t k,
                                                                   int32_t accumulate, const float* __restrict__ b_dual,
                                                                   T* __restrict__ c_dual) {
    if (blockIdx.z == 1) b = b_dual, c = c_dual;                  // second product of the same A
    constexpr int VE = 16 / int(sizeof(T));                       // elements per 16-byte load
    constexpr int kRow = 16 * KS + 8, kPlane = kShortRows * kRow; // elements per row and per term of the tile
    constexpr int N = (kShortRows * 16 * KS / VE + 1 + kThreads - 1) / kThreads;
    __shared__ __attribute__((aligned(16))) uint16_t tile[TERMS * kPlane];
    __shared__ __attribute__((aligned(16))) float epi[4 * 32 * kEpiPitch];      // a 32 x 64 block per wavefront
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lcol = lane & 31, lk = lane >> 5;
    // 64 columns to a wavefront; when there are fewer than four such groups, the blocks of 32 rows are dealt as well
    const int groups = n - int32_t(blockIdx.y) * 256 > 128 ? 4 : n - int32_t(blockIdx.y) * 256 > 64 ? 2 : 1;
    const int32_t c0 = blockIdx.y * 256 + wave % groups * 64;
    // rows of C can be written 4 elements at a time: whole vectors inside the matrix, aligned
    const bool vec_out = n % 4 == 0 && ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(c) & (4 * sizeof(T) - 1)) == 0;

    // weights of this wavefront's two column blocks: lane holds B[column][16 s + 8 lk .. + 7], expanded
    bf16x8 w[2][KS][3];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        const int32_t col = c0 + cb * 32 + lcol;
#pragma unroll
        for (int s2 = 0; s2 < KS; ++s2) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int kk = 16 * s2 + 8 * lk + e;
                x[e] = col < n && kk < k ? b[int64_t(col) * ldb + kk] : 0.f;
            }
            expand8<TERMS>(x, w[cb][s2]);
        }
    }
    for (int i = threadIdx.x; i < TERMS * kPlane / 8; i += kThreads) reinterpret_cast<uint4*>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);

    // A tile is read in 16-byte chunks on 16-byte boundaries (its range may start `skew` elements into a chunk; a tile is a
    // multiple of 16 bytes long, so every tile has the same skew, and so has the mask, checked by the launcher). A thread's
    // chunks are at the same places of every tile.
    const int32_t skew = int32_t((reinterpret_cast<uintptr_t>(a) & 15u) / sizeof(T));
    int32_t row[N], kk0[N];
#pragma unroll
    for (int h = 0; h < N; ++h) {
        const int32_t e = max((int32_t(threadIdx.x) + h * kThreads) * VE - skew, 0);
        row[h] = e / k, kk0[h] = e - row[h] * k;
    }
    uint4 raw[N], graw[GATE ? N : 1];
    const int32_t n_tiles = (m + kShortRows - 1) / kShortRows;
    auto chunk = [&](const T* src, int32_t e0, int32_t n_el) {
        if (e0 >= 0 && e0 + VE <= n_el) return *reinterpret_cast<const uint4*>(src + e0);
        uint32_t u[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < VE; ++i)
            if (e0 + i >= 0 && e0 + i < n_el) {
                if constexpr (sizeof(T) == 4)
                    u[i] = reinterpret_cast<const uint32_t*>(src)[e0 + i];
                else
                    u[i >> 1] |= uint32_t(reinterpret_cast<const uint16_t*>(src)[e0 + i]) << (16 * (i & 1));
            }
        return make_uint4(u[0], u[1], u[2], u[3]);
    };
    auto load = [&](int32_t t) {
        const int32_t r0 = t * kShortRows, n_el = min(kShortRows, m - r0) * k;
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int32_t e0 = (int32_t(threadIdx.x) + h * kThreads) * VE - skew;
            if (e0 < n_el) {
                raw[h] = chunk(a + int64_t(r0) * k, e0, n_el);
                if constexpr (GATE) graw[h] = chunk(gate + int64_t(r0) * k, e0, n_el);
            }
        }
    };
    auto value = [](const uint4& v, int i) {
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
        if constexpr (sizeof(T) == 4) return __uint_as_float(u[i]);
        return __uint_as_float((i & 1) ? (u[i >> 1] & 0xFFFF0000u) : (u[i >> 1] << 16));
    };

    int32_t t = blockIdx.x;
    if (t < n_tiles) load(t);
    __syncthreads();
    for (; t < n_tiles; t += gridDim.x) {
        const int32_t r0 = t * kShortRows, rows = min(kShortRows, m - r0), n_el = rows * k;
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int32_t e0 = (int32_t(threadIdx.x) + h * kThreads) * VE - skew;
            uint16_t* at = tile + row[h] * kRow + kk0[h];
            int32_t kk = kk0[h];
#pragma unroll
            for (int i = 0; i < VE; i += 2) {
                float x0 = value(raw[h], i), x1 = value(raw[h], i + 1);
                if constexpr (GATE) x0 = value(graw[h], i) > 0.f ? x0 : 0.f, x1 = value(graw[h], i + 1) > 0.f ? x1 : 0.f;
                uint32_t o[TERMS];
                expand_pair<TERMS>(x0, x1, o);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (e0 + i + q >= 0 && e0 + i + q < n_el) {
#pragma unroll
                        for (int p = 0; p < TERMS; ++p) at[p * kPlane] = uint16_t(o[p] >> (16 * q));
                        ++at, ++kk;
                        if (kk == k) kk = 0, at += kRow - k;
                    }
            }
        }
        __syncthreads();
        if (t + int32_t(gridDim.x) < n_tiles) load(t + gridDim.x);
        for (int rb = wave / groups; rb * 32 < rows && c0 < n; rb += 4 / groups) {
            floatx16 acc[2];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[cb][v] = 0.f;
#pragma unroll
            for (int s2 = 0; s2 < KS; ++s2) {
                bf16x8 fa[3];
#pragma unroll
                for (int p = 0; p < TERMS; ++p)
                    fa[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(tile + p * kPlane + (rb * 32 + lcol) * kRow + 16 * s2 + 8 * lk));
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    auto mul = [&](int pa, int pb) {
                        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[cb][s2][pb], fa[pa], acc[cb], 0, 0, 0);
                    };
                    mul(0, 0);
                    if constexpr (TERMS >= 2) {
                        mul(0, 1);
                        mul(1, 0);
                    }
                    if constexpr (TERMS == 3) {
                        mul(1, 1);
                        mul(0, 2);
                        mul(2, 0);
                    }
                }
            }
            // accumulator register v of a lane is element (row lane % 32, column 8 * (v / 4) + 4 * (lane / 32) + v % 4)
            float* ep = epi + wave * (32 * kEpiPitch);
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4*>(ep + lcol * kEpiPitch + cb * 32 + 8 * q + 4 * lk) =
                        make_float4(acc[cb][4 * q], acc[cb][4 * q + 1], acc[cb][4 * q + 2], acc[cb][4 * q + 3]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (vec_out) {
                const int er = lane >> 4, ec = (lane & 15) * 4;
                float4 old[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) old[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (accumulate) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int32_t r = min(rb * 32 + er + 4 * i, rows - 1);
                        if (c0 + ec < n) old[i] = Elem<T>::load4(c + int64_t(r0 + r) * ldc + c0 + ec);
                    }
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int32_t r = rb * 32 + er + 4 * i;
                    float4 x = *reinterpret_cast<const float4*>(ep + (er + 4 * i) * kEpiPitch + ec);
                    x.x += old[i].x, x.y += old[i].y, x.z += old[i].z, x.w += old[i].w;
                    if (r < rows && c0 + ec < n) Elem<T>::store4(c + int64_t(r0 + r) * ldc + c0 + ec, x);
                }
            } else if (c0 + lane < n) {
                T* out = c + int64_t(r0 + rb * 32) * ldc + c0 + lane;
                const int32_t here = min(32, rows - rb * 32);
                for (int i0 = 0; i0 < here; i0 += 8) {
                    float old[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) old[i] = accumulate ? Elem<T>::load(out + int64_t(min(i0 + i, here - 1)) * ldc) : 0.f;
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (i0 + i < here) Elem<T>::store(out + int64_t(i0 + i) * ldc, ep[(i0 + i) * kEpiPitch + lane] + old[i]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        __syncthreads();               // the tile has been read: the next one may overwrite it
    }
}

template <int CAP>               // the table travels with the launch: a single copy should not carry 3 KB of it
__global__ __launch_bounds__(kPrepThreads) void prep_weights_kernel(PrepJobs<CAP> jobs) {
    prep_weights(jobs, int32_t(blockIdx.x), int32_t(threadIdx.x));
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

hipError_t varco_launch_prep_weights(PrepJob* jobs, int n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    if (n > kMaxPrepJobs) return hipErrorInvalidValue;
    const int64_t blocks = varco_prep_blocks(jobs, n);
    if (blocks < 0) return hipErrorInvalidValue;
    if (blocks == 0) return hipSuccess;
    auto go = [&](auto cap) {
        PrepJobs<decltype(cap)::value> args{};
        for (int i = 0; i < n; ++i) args.job[i] = jobs[i];
        args.n = n;
        hipLaunchKernelGGL((prep_weights_kernel<decltype(cap)::value>), dim3(unsigned(blocks)), dim3(kPrepThreads), 0, stream, args);
    };
    if (n == 1)
        go(std::integral_constant<int, 1>{});
    else if (n <= kFewPrepJobs)
        go(std::integral_constant<int, kFewPrepJobs>{});
    else
        go(std::integral_constant<int, kMaxPrepJobs>{});
    return hipGetLastError();
}

int64_t varco_prep_blocks(PrepJob* jobs, int n) {
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        PrepJob& j = jobs[i];
        const bool plain = j.terms == 1 && j.rows_padded == j.rows && j.pitch >= j.cols;
        const bool tiled = (j.terms == 2 || j.terms == 3 || j.terms == kExactTerms || (j.terms == kHalfTerms && !j.transpose)) && j.rows_padded >= j.rows && j.rows_padded % kPrepRows == 0 && j.pitch >= j.cols && j.pitch % BK == 0;
        if (!plain && !tiled) return -1;
        j.first_block = int32_t(blocks);
        blocks += j.terms == kHalfTerms ? j.rows_padded / 32 : (int64_t(j.rows_padded) * j.pitch + kThreads - 1) / kThreads;
    }
    return blocks;
}

namespace {
template <typename U>
struct TypeTag {
    using type = U;
};
}  // namespace

// Short reductions (see gemm_short_k_kernel): terms = 1 for bf16 storage, 2 or 3 for fp32 storage.
hipError_t varco_launch_gemm_short_k(const GemmArgs& ga, int terms, hipStream_t stream) {
    const int64_t tiles = (ga.m + kShortRows - 1) / kShortRows, others = int64_t((ga.n + 255) / 256) * (ga.c_dual ? 2 : 1);
    const dim3 grid(unsigned(std::min<int64_t>(tiles, std::max<int64_t>(1, 512 / others))), unsigned((ga.n + 255) / 256), ga.c_dual ? 2 : 1);
    const int ks = (ga.k + 15) / 16;
    if (ks < 1 || ks > 4 || (ga.a.dtype == VARCO_F32 && ks % 2 == 0)) return hipErrorInvalidValue;
    auto go = [&](auto type, auto ksc, auto gt, auto tc) {
        using T = typename decltype(type)::type;
        hipLaunchKernelGGL((gemm_short_k_kernel<T, decltype(ksc)::value, decltype(gt)::value, decltype(tc)::value>), grid,
                           dim3(kThreads), 0, stream, static_cast<const T*>(ga.a.ptr), static_cast<const T*>(ga.a.gate),
                           static_cast<const float*>(ga.b.ptr), ga.b.ld, static_cast<T*>(ga.c), ga.ldc, ga.m, ga.n, ga.k,
                           ga.accumulate ? 1 : 0, static_cast<const float*>(ga.b_dual), static_cast<T*>(ga.c_dual));
    };
    auto with_ks = [&](auto type, auto gt, auto tc) {
        if (ks == 1) return go(type, std::integral_constant<int, 1>{}, gt, tc);
        if (ks == 3) return go(type, std::integral_constant<int, 3>{}, gt, tc);
        if constexpr (sizeof(typename decltype(type)::type) == 2) {      // (the others of fp32 storage go to kernels_gemm_half.hip)
            if (ks == 2) return go(type, std::integral_constant<int, 2>{}, gt, tc);
            return go(type, std::integral_constant<int, 4>{}, gt, tc);
        }
    };
    auto with_gate = [&](auto type, auto tc) {
        if (ga.a.gate)
            with_ks(type, std::true_type{}, tc);
        else
            with_ks(type, std::false_type{}, tc);
    };
    if (ga.a.dtype == VARCO_BF16)
        with_gate(TypeTag<bf16_t>{}, std::integral_constant<int, 1>{});
    else if (terms == 3)
        with_gate(TypeTag<float>{}, std::integral_constant<int, 3>{});
    else
        with_gate(TypeTag<float>{}, std::integral_constant<int, 2>{});
    return hipGetLastError();
}

bool varco_gemm_split_usable(const GemmArgs& ga) {
    if (ga.f32_terms != 2 && ga.f32_terms != 3) return false;
    if (ga.m <= 0 || ga.n <= 0) return false;
    if (ga.a.dtype != VARCO_F32 || ga.c_dtype != VARCO_F32 || ga.a.transposed || ga.a.gate || ga.b.gate || ga.c_dual || ga.split_k > 1 || ga.b_halves)
        return false;
    // needs the library's expanded weight copy [term][rows][pitch], padded to whole tiles
    auto prep_ok = [&](const void* p, int64_t ld, int64_t plane, int32_t k) {
        return p && aligned_to(p, 16) && ld % BK == 0 && ld >= k && plane == (int64_t(ga.n) + kPrepRows - 1) / kPrepRows * kPrepRows * ld;
    };
    if (!prep_ok(ga.b_prep, ga.b_prep_ld, ga.b_prep_plane, ga.k)) return false;
    // (Other reductions keep fp32 matrix instructions: the same sums in the same order as ever, so that a ReLU whose
    // argument is within rounding of zero opens as it did.)
    if (ga.k % 4 != 0 || !aligned_to(ga.a.ptr, 4)) return false;
    if (ga.k2 > 0) {   // a chained product shares the first one's leading dimensions
        if (!prep_ok(ga.b2_prep, ga.b2_prep_ld, ga.b2_prep_plane, ga.k2) || ga.b2_prep_ld != ga.b_prep_ld) return false;
        if (ga.k2 % 4 != 0 || !aligned_to(ga.a2.ptr, 4) || ga.a2.ld != ga.a.ld || ga.a2.gate || ga.a2.dtype != VARCO_F32 || ga.a2.transposed) return false;
    }
    return true;
}

bool varco_gemm_split_taps_usable(const GemmArgs* g, int n) {
    if (n < 2 || n > kMaxChain || g->accumulate || g->k2 > 0 || g->f32_terms != 3) return false;
    for (int i = 0; i < n; ++i)
        if (!varco_gemm_split_usable(g[i]) || g[i].m != g->m || g[i].n != g->n || g[i].k != g->k || g[i].k2 > 0 || g[i].a.ld != g->a.ld || g[i].b_prep_ld != g->b_prep_ld ||
            g[i].f32_terms != 3 || g[i].c != g->c || g[i].ldc != g->ldc || g[i].accumulate != (i > 0) || (g[i].relu && i + 1 < n))
            return false;
    return true;
}

namespace {
hipError_t launch_split(const GemmArgs* taps, int n, hipStream_t stream, const LaunchTag& tag) {
    const GemmArgs& ga = *taps;
    const bool narrow = ga.n <= 64;
    const int bm = 128, bn = narrow ? 64 : 128;
    const bool a8 = ga.k % 8 == 0 && (ga.k2 == 0 || ga.k2 % 8 == 0);

    SplitGemm g{};
    g.m = ga.m, g.n = ga.n, g.k = ga.k, g.k2 = ga.k2;
    g.a = {ga.a.ptr, ga.a.ld};
    g.a2 = {ga.a2.ptr, ga.a2.ld};
    g.b = {ga.b_prep, ga.b_prep_ld};
    g.b2 = {ga.b2_prep, ga.b2_prep_ld};
    g.c = static_cast<float*>(ga.c);
    g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0;
    g.relu = taps[n - 1].relu ? 1 : 0;
    g.taps = n;
    for (int i = 0; i < n; ++i) g.tap_a[i] = static_cast<const float*>(taps[i].a.ptr), g.tap_b[i] = static_cast<const uint16_t*>(taps[i].b_prep);
    g.tiles_m = (ga.m + bm - 1) / bm;
    g.tiles_n = (ga.n + bn - 1) / bn;
    const int64_t blocks = int64_t((g.tiles_m + 7) / 8 * 8) * g.tiles_n;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid{unsigned(blocks)};

    tag.begin(stream);
    with_flag(ga.f32_terms == 3, [&](auto t3) {
        with_flag(narrow, [&](auto nr) {
            with_flag(a8, [&](auto c8) {
                constexpr bool NR = decltype(nr)::value;
                if constexpr (decltype(t3)::value)
                    if (n > 1) {
                        hipLaunchKernelGGL((gemm_split_kernel<3, NR ? 4 : 2, NR ? 1 : 2, NR ? 1 : 2, 2, decltype(c8)::value ? 8 : 4, true>), grid, dim3(kThreads), 0, stream, g);
                        return;
                    }
                hipLaunchKernelGGL((gemm_split_kernel<decltype(t3)::value ? 3 : 2, NR ? 4 : 2, NR ? 1 : 2, NR ? 1 : 2, 2, decltype(c8)::value ? 8 : 4>), grid,
                                   dim3(kThreads), 0, stream, g);
            });
        });
    });
    tag.end(stream);
    return hipGetLastError();
}
}  // namespace

hipError_t varco_launch_gemm_split(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag) { return launch_split(&ga, 1, stream, tag); }
hipError_t varco_launch_gemm_split_taps(const GemmArgs* g, int n, hipStream_t stream, const LaunchTag& tag) { return launch_split(g, n, stream, tag); }
