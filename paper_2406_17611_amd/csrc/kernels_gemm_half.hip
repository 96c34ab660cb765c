// Gradients of the dense feature transform of eq. (2) for fp32-stored activations, on the fp16 matrix units. Operands are scaled by
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
// below zero on average, so every second slab of a weight gradient multiplies -B (its scale is negative) and changes sign in the epilogue.
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
// fp16 rows (one output index per row, reduction index contiguous, 80-byte pitch).
//   "NT" products (input gradient): A has the reduction index contiguous and is split here;
//        B is the library's own split copy of the weights (varco_launch_prep_weights), zero-padded
//        to whole tiles and copied as is.
//   "TN" products (weight gradient, reduction over nodes): both operands have the node index as the slow
//        one; a thread loads an 8 (nodes) x 4 (columns) block with eight 16-byte loads and splits the values of
//        two consecutive nodes of a column together, which yields the transposed (node index contiguous) words
//        directly; it writes four 16-byte LDS rows per plane. Half the threads serve A, half B.
// The ReLU mask of the backward pass is applied before the split. Bound by the vector ALU (about 8 instructions per pair of values) and the
// matrix unit, which take turns on a SIMD, and by what the memory delivers. Three bf16 terms / this, 2,449,029 rows: masked dZ
// (256 wide) times two 256 x 256 weights 4.47 / 3.50 ms, weight gradients of both taps 256 x 256 2.99 / 2.63 ms; 169,343 rows: one
// masked input gradient 161 / 133 us, one weight gradient 178 / 160 us.
// (Measured and not kept: 64 rows per workgroup, expanded once for all columns, weights straight from the L2 as operands: 3.0 to 3.9 ms
// for the first, bound by the vector memory path.)
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
    int32_t split_k, tiles_per_split;
    float* partial;
    int32_t tiles_m, tiles_n;
    int32_t inner, outer;            // tiles along the fast and the slow direction of the workgroup order
    const void* dual;                // second A (TN) or second split B (NT), or null
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

// ---- fp32 operand with the output index contiguous: one 8 (reduction) x 4 (output) block per thread ----
// Block b of an operand's tile covers reduction steps 8 * (b % 4) .. + 7 and output indices 4 * (b / 4) .. + 3:
// eight consecutive lanes then write two LDS rows that are four rows apart, all four 16-byte chunks of each,
// which touches every LDS bank once. Output indices beyond the matrix are clamped (their results are never
// stored), a group of four that crosses its end is moved up (rows of the 47 class columns of a last layer, of 75 input features;
// they need no alignment). In the last, partial tile of the reduction the node index is clamped and A is zeroed beyond it.
template <bool GATE>
struct ColRegs {
    float4 v[8];
    float4 g[GATE ? 8 : 1];
};

__device__ __forceinline__ uint32_t col_offset(int b, int32_t i0, int32_t extent) {
    return uint32_t(min(i0 + (b >> 2) * 4, extent - 4) - i0 + 4) * 4u;  // bytes from 4 floats before the tile's first column
}

template <bool GATE, bool TAIL, bool ZERO>
__device__ __forceinline__ void load_cols(const float* base, const float* gate, int b, uint32_t col_off, uint32_t ld_bytes,
                                          int32_t k_left, ColRegs<GATE>& r) {
    int kb = (b & 3) * 8;
    asm volatile("" : "+v"(kb));         // (offsets are formed anew for every stage: two sets of sums leave no registers for them)
    uint32_t off = uint32_t(TAIL ? min(kb, k_left - 1) : kb) * ld_bytes + col_off;
    uint32_t row_bytes = ld_bytes;
    asm volatile("" : "+s"(row_bytes));
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        r.v[kk] = load4_at(base, off);
        if (GATE) r.g[kk] = load4_at(gate, off);
        if (!TAIL || kb + kk + 1 < k_left) off += row_bytes;
        if (TAIL && ZERO && kb + kk >= k_left) r.v[kk] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// Masks, scales, splits and writes a stage's block of four columns; e: their scale exponents, kept from stage to stage (126 before the
// first value that is not zero). scales[column] = {exponent, bits of the factor that the sums so far take}; the four lanes that share
// the columns agree. Whether a scale got smaller.
template <int ROWS, bool GATE>
__device__ __forceinline__ bool store_cols(const ColRegs<GATE>& r, int b, int32_t i0, int32_t extent, float sign, int (&e)[4], uint16_t* s, int2* scales) {
    const bool crosses = (extent & 3) && i0 + (b >> 2) * 4 == (extent & ~3);
    float x[8][4], m[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        float4 v = r.v[kk];
        if constexpr (GATE) v = gate4(v, r.g[kk]);
        if (extent & 3) v = crosses ? moved_up(v, 4 - (extent & 3)) : v;
        x[kk][0] = v.x, x[kk][1] = v.y, x[kk][2] = v.z, x[kk][3] = v.w;
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) m[ii] = fmaxf(m[ii], fabsf(x[kk][ii]));
    }
    bool grew = false;
    int f[4];
    float sc[4];
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
        const int now = scale_exponent(largest_of_lanes<4>(m[ii]), kFirst), old = e[ii];
        const bool smaller = now < old - kRoom;
        if (smaller) e[ii] = now;
        grew = grew || smaller;
        f[ii] = int(__float_as_uint(power_of_two(max(e[ii] - old, -126))));
        sc[ii] = sign * power_of_two(e[ii]);
    }
    if ((b & 3) == 0) {
        int4* const at = reinterpret_cast<int4*>(scales + (b >> 2) * 4);
        at[0] = make_int4(e[0], f[0], e[1], f[1]), at[1] = make_int4(e[2], f[2], e[3], f[3]);
    }
    uint16_t* base = s + (b >> 2) * 4 * kPitch + (b & 3) * 8;
    // An LDS row holds one output index with its 8 reduction steps contiguous, two steps per 32-bit word: the two
    // values split together are steps 2 q and 2 q + 1 of one output index, which is the transposition itself.
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {                          // output index i + ii: its 8 reduction steps
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) split_pair(x[2 * q][ii] * sc[ii], x[2 * q + 1][ii] * sc[ii], hi[q], lo[q]);
        *reinterpret_cast<uint4*>(base + ii * kPitch) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        *reinterpret_cast<uint4*>(base + ROWS * kPitch + ii * kPitch) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    }
    return grew;
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

// All wavefronts of the workgroup meet here (same fences as __syncthreads); the two halves of a workgroup call
// it from different places, always the same number of times.
__device__ __forceinline__ void workgroup_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// TN: both operands stored with the output index contiguous (weight gradient), else A with the reduction
// index contiguous and B a split weight copy. WM x WN wavefronts per tile, each TMB x TNB blocks of
// 32 x 32. A_CH: floats per chunk of A (NT). GATE masks A (NT) or B (TN).
//
// A workgroup is four wavefronts with one tile and one LDS stage (40 KB), so that two workgroups are resident
// on a compute unit and each SIMD holds one wavefront of either. On this device the vector ALU and the matrix
// unit of a SIMD do not run side by side (hardware counters: their busy times add up), so nothing is gained by
// steering one wavefront's conversions under the other's products; what matters is that the SIMD always has a
// wavefront that can issue, and that as few vector instructions as possible accompany the matrix instructions.
// Two independent workgroups give the first: while one waits at a barrier, for its global loads, or stores its
// tile, the other multiplies. (Two groups in lock step inside one 512-thread workgroup, the previous form, left
// a tile's first fetch and epilogue uncovered and tied both groups to the slower one.)
template <bool TN, int WM, int WN, int TMB, int TNB, int A_CH, bool GATE, bool FOUR>
__global__ __launch_bounds__(kThreads, 2) void gemm_half_kernel(HalfGemm g) {
    constexpr int BM = 32 * TMB * WM, BN = 32 * TNB * WN;
    static_assert(BM + BN <= kThreads, "one 8 x 4 block per thread in the TN layout");
    __shared__ __attribute__((aligned(16))) uint16_t smem[TERMS * (BM + BN) * kPitch];
    __shared__ __attribute__((aligned(16))) int2 scales[TN ? BM + BN : BM];      // NT: of every row; TN: of the columns of A, then of B
    __shared__ int32_t smaller_at;                                // last stage in which a scale got smaller
    const int tid = threadIdx.x;
    uint16_t* const sa = smem;
    uint16_t* const sb = smem + TERMS * BM * kPitch;

    // workgroup -> tile: tiles that share streamed data go to one XCD (workgroups are dealt to the 8 XCDs
    // round-robin), so that the streamed operand is fetched into a single L2
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3;
    const int32_t in = within % g.inner, out = (within / g.inner) * 8 + xcd;
    if (out >= g.outer) return;                // whole workgroup leaves together: no barrier is skipped
    int32_t t_begin = 0, t_end = (g.k + BK - 1) / BK;
    int32_t tm, tn, z;
    bool second = false;             // this workgroup's tile belongs to the dual product
    if (g.split_k > 1 || TN) {
        t_begin = out * g.tiles_per_split;
        t_end = min(t_end, t_begin + g.tiles_per_split);
        const int32_t tiles = g.tiles_m * g.tiles_n;
        second = in >= tiles;
        const int32_t tile = second ? in - tiles : in;
        z = out, tm = tile / g.tiles_n, tn = tile % g.tiles_n;
    } else {
        second = in >= g.tiles_n;
        z = 0, tm = out, tn = second ? in - g.tiles_n : in;
    }
    const void* const a_ptr = TN && second ? g.dual : g.a.ptr;
    const void* const b_ptr = !TN && second ? g.dual : g.b.ptr;
    const float sign = TN && (z & 1) ? -1.f : 1.f;                // of the second operand of this slab (see the head of this file)
    const int32_t steps = max(t_end - t_begin, 0);
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

    // staging registers and per-thread offsets of the two layouts (only one set is used per instantiation)
    RowRegs<BM, A_CH, GATE && !TN> ra;
    PrepRegs<BN> rb;
    RowPlan<BM, A_CH> plan_a;
    PrepPlan<BN> plan_b;
    if constexpr (!TN) {
        plan_a.init(tid, m0, g.m, g.a.ld);
        plan_b.init(tid);
    }

    auto fetch = [&](int32_t t) {                 // NT
        const int32_t k0 = t * BK;
        const float* abase = static_cast<const float*>(a_ptr) + int64_t(m0) * g.a.ld + k0;
        const float* gbase = GATE ? g.a.gate + int64_t(m0) * g.a.ld + k0 : nullptr;
        const uint16_t* bbase = static_cast<const uint16_t*>(b_ptr) + (int64_t(tn) * (g.b.ld / BK) + t) * (TERMS * BN * BK);   // g.b.ld: padded reduction length
        if constexpr (!TN) {
            load_rows<BM, A_CH, GATE>(tid, abase, gbase, plan_a, g.k - k0, ra);
            load_prep<BN>(bbase, plan_b, rb);
        }
    };
    auto stash = [&](int32_t t) __attribute__((always_inline)) {                 // NT
        if constexpr (!TN) {
            if (store_rows<BM, A_CH, GATE>(tid, ra, t == t_begin, g.k - t * BK, sa, scales)) smaller_at = t;
            store_prep<BN>(tid, rb, sb);
        }
    };
    // Half steps that hold padding only are left out (NT): at most 16 values left means that only the first half multiplies.
    auto compute = [&](int32_t t) __attribute__((always_inline)) {
        const int32_t left = TN ? BK : g.k - t * BK;
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
    // The sums so far follow rows (NT) or columns (TN) that took a smaller scale with this stage.
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
        if constexpr (TN) {
#pragma unroll
            for (int j = 0; j < TNB; ++j) {
                const float f = __uint_as_float(uint32_t(scales[BM + wn + j * 32 + lrow].y));
#pragma unroll
                for (int i = 0; i < TMB; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] *= f, low[i][j][v] *= f;
            }
        }
    };

    // One LDS stage: a step's operands are fetched into registers while the previous step is multiplied, then
    // split and written once its fragments have been read. (A second register set, fetching two steps ahead,
    // was measured and changes nothing.)
    auto pipeline = [&](auto&& fetch_fn, auto&& stash_fn) __attribute__((always_inline)) {
        if (steps > 0) fetch_fn(t_begin);
        for (int32_t it = 0; it < steps; ++it) {
            stash_fn(t_begin + it);
            if (it + 1 < steps) fetch_fn(t_begin + it + 1);
            workgroup_barrier();
            follow(t_begin + it);
            compute(t_begin + it);
            workgroup_barrier();   // the stage's fragments have been read: the next one may overwrite them
        }
    };
    if constexpr (TN) {
        // Every wavefront serves 8 x 4 blocks of one operand only (BM and BN are multiples of 64), so the role is
        // a scalar and each role gets a loop of its own: one shared loop with per-thread role tests made the
        // compiler copy the 32 staging registers between the paths every step.
        const int role = __builtin_amdgcn_readfirstlane(tid < BM ? 0 : (tid < BM + BN ? 1 : 2));
        auto run = [&](auto is_a) {
            constexpr bool A = decltype(is_a)::value;
            constexpr bool G = GATE && !A;
            ColRegs<G> cr;
            const int b = A ? tid : tid - BM;
            const uint32_t col_off = A ? col_offset(b, m0, g.m) : col_offset(b, n0, g.n);
            const HalfOperand& op = A ? g.a : g.b;
            const uint32_t ld_bytes = uint32_t(op.ld) * 4u;
            auto fetch_cols = [&](int32_t t) {
                const int32_t k0 = t * BK, k_left = g.k - k0;
                const float* base = static_cast<const float*>(A ? a_ptr : op.ptr) + int64_t(k0) * op.ld + (A ? m0 : n0) - 4;
                const float* gbase = G ? op.gate + int64_t(k0) * op.ld + n0 - 4 : nullptr;
                if (k_left >= BK)
                    load_cols<G, false, A>(base, gbase, b, col_off, ld_bytes, k_left, cr);
                else
                    load_cols<G, true, A>(base, gbase, b, col_off, ld_bytes, k_left, cr);
            };
            int e[4] = {126, 126, 126, 126};
            pipeline(fetch_cols, [&](int32_t t) {
                if (store_cols<A ? BM : BN, G>(cr, b, A ? m0 : n0, A ? g.m : g.n, A ? 1.f : sign, e, A ? sa : sb, A ? scales : scales + BM)) smaller_at = t;
            });
        };
        if (role == 0)
            run(std::true_type{});
        else if (role == 1)
            run(std::false_type{});
        else
            pipeline([](int32_t) {}, [](int32_t) {});
    } else {
        pipeline(fetch, stash);
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
            int eb;
            if constexpr (TN)
                eb = scales[BM + wn + j * 32 + lrow].x;
            else
                eb = reinterpret_cast<const int32_t*>(static_cast<const uint16_t*>(b_ptr) + g.exps)[n0 + wn + j * 32 + lrow];
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = __builtin_ldexpf(sign * (acc[i][j][v] + low[i][j][v] * (1.f / kHalfLow)), -(e[v] + eb));
        }
    }

    const bool to_partial = g.split_k > 1;
    float* const base = to_partial ? g.partial + (int64_t(second ? g.split_k : 0) + z) * g.m * g.n : second ? g.c_dual : g.c;
    store_tile(acc, base, to_partial ? int64_t(g.n) : g.ldc, g.m, g.n, m0 + wm, n0 + wn, m0 + BM <= g.m && n0 + BN <= g.n, lane,
               !to_partial && g.accumulate, false);
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

hipError_t varco_launch_gemm_half(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag, int32_t* split_used) {
    const bool tn = ga.a.transposed;
    const bool narrow = ga.n <= 64;
    const int bm = 128, bn = narrow ? 64 : 128;
    const bool a8 = !tn && ga.k % 8 == 0;
    const bool gate = tn ? ga.b.gate != nullptr : ga.a.gate != nullptr;

    HalfGemm g{};
    g.m = ga.m, g.n = ga.n, g.k = ga.k;
    auto f32 = [](const void* p) { return static_cast<const float*>(p); };
    g.a = {ga.a.ptr, f32(ga.a.gate), ga.a.ld};
    if (tn) {
        g.b = {ga.b.ptr, f32(ga.b.gate), ga.b.ld};
    } else {
        g.b = {ga.b_prep, nullptr, ga.b_prep_ld};
        g.exps = 2 * ga.b_prep_plane;
    }
    g.c = static_cast<float*>(ga.c);
    g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0;
    g.tiles_m = (ga.m + bm - 1) / bm;
    g.tiles_n = (ga.n + bn - 1) / bn;
    const int32_t k_tiles = (ga.k + BK - 1) / BK;
    int32_t split = ga.split_k < 1 ? 1 : ga.split_k;
    if (split > k_tiles) split = k_tiles < 1 ? 1 : k_tiles;
    g.tiles_per_split = (k_tiles + split - 1) / split;
    split = g.tiles_per_split > 0 ? (k_tiles + g.tiles_per_split - 1) / g.tiles_per_split : 1;
    if (split < 1) split = 1;
    g.split_k = split;
    g.partial = ga.partial;
    if (split > 1 && !ga.partial) return hipErrorInvalidValue;
    g.dual = ga.c_dual ? (tn ? ga.a_dual : ga.b_dual_prep) : nullptr;
    g.c_dual = static_cast<float*>(ga.c_dual);
    const int32_t products = ga.c_dual ? 2 : 1;     // the dual product's tiles come right behind the first one's, on the same XCD
    if (split > 1 || tn) {
        g.inner = g.tiles_m * g.tiles_n * products;
        g.outer = split;
    } else {
        g.inner = g.tiles_n * products;
        g.outer = g.tiles_m;
    }
    const int64_t blocks = int64_t((g.outer + 7) / 8 * 8) * g.inner;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid{unsigned(blocks)};
    *split_used = split;

    tag.begin(stream);
    with_flag(narrow, [&](auto nr) {
        with_flag(gate, [&](auto gt) {
            with_flag(!tn && ga.k <= kShortSum, [&](auto fr) {
                constexpr bool NR = decltype(nr)::value, GT = decltype(gt)::value, FR = decltype(fr)::value;
                constexpr int WM = NR ? 4 : 2, WN = NR ? 1 : 2, TMB = NR ? 1 : 2, TNB = 2;
                if (tn) {
                    hipLaunchKernelGGL((gemm_half_kernel<true, WM, WN, TMB, TNB, 4, GT, false>), grid, dim3(kThreads), 0, stream, g);
                } else if (a8) {
                    hipLaunchKernelGGL((gemm_half_kernel<false, WM, WN, TMB, TNB, 8, GT, FR>), grid, dim3(kThreads), 0, stream, g);
                } else {
                    hipLaunchKernelGGL((gemm_half_kernel<false, WM, WN, TMB, TNB, 4, GT, FR>), grid, dim3(kThreads), 0, stream, g);
                }
            });
        });
    });
    tag.end(stream);
    return hipGetLastError();
}
