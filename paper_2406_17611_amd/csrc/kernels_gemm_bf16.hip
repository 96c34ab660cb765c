// Dense feature transform of eq. (2) and its input gradient for bf16-stored activations, on the bf16 matrix cores with
// fp32 accumulation (v_mfma_f32_32x32x16_bf16): X_out = act(M H1 + X H0), dM = dZ H1^T. Weights are kept in fp32 by the
// caller; the library hands this kernel a bf16 copy laid out [output index][reduction index] (see
// varco_launch_prep_weights). Weight gradients are in kernels_gemm_tn_bf16.hip.
//
// A workgroup of 4 wavefronts computes a 128 x 256 tile of C in stages of 64 reduction steps (rows of whole 128-byte lines
// from memory), or a 256 x 128 or 256 x 64 tile in stages of 32. A wavefront owns 64 x 128 (128 x 64, 64 x 64) of it as
// 32 x 32 blocks: at bf16 rates a wavefront tile smaller than that is limited by LDS reads of its fragments, not by
// the matrix cores. Operands are staged through LDS as rows of one output index with the reduction index contiguous (16
// bytes of padding per row: fragment reads without bank conflicts), copied 8 elements at a time unchanged. The narrower tiles
// keep two stages in LDS, one written while the other is read; the 128 x 256 tile keeps one (55 KB), so that two workgroups
// share a compute unit and one computes while the other waits or stores. The next stage's loads are in flight in both. The
// ReLU mask of the backward pass is applied when a stage is written to LDS, the activation in the epilogue.
#include <type_traits>

#include "elem.h"
#include "varco_internal.h"

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct OperandDev {
    const uint16_t* ptr;
    const uint16_t* gate;
    int64_t ld;
};

struct GemmDev {
    int32_t m, n, k, k2;
    OperandDev a, b, a2, b2;
    void* c;
    int64_t ldc;
    int32_t accumulate, relu;
    int32_t vec_c;                   // rows of C are whole, aligned 16-byte pieces
    int32_t tiles_n;
    int32_t inner, outer;
    const uint16_t* dual;            // second weight copy, or null
    void* c_dual;
};

// Two bf16 values packed in a word: keep each where the packed gate value is > 0.
__device__ __forceinline__ uint32_t gate_pair(uint32_t v, uint32_t g) {
    const uint32_t lo = __uint_as_float(g << 16) > 0.f ? 0x0000FFFFu : 0u;
    const uint32_t hi = __uint_as_float(g & 0xFFFF0000u) > 0.f ? 0xFFFF0000u : 0u;
    return v & (lo | hi);
}

// One operand's share of a stage: ROWS rows x BK reduction steps in chunks of 8 elements. A thread keeps its place in the
// stage, so its byte offsets into the operand are formed once and the stage's base stays in scalar registers. Rows past the
// matrix repeat its last one (their results are never stored); reduction steps past the end are zero. ANY: rows of any
// alignment and any length from 8 on (a chunk that crosses the end is loaded from before it and moved up, one past it repeats
// the row's last 8 elements: the last row may end the allocation), else padded ones.
template <int ROWS, bool GATE, bool ANY, int BK, int kThreads>
struct RowSlab {
    static constexpr int PER_ROW = BK / 8, kPitch = BK + 8;
    static constexpr int N = ROWS * PER_ROW / kThreads;
    uint4 v[N], g[GATE ? N : 1];
    uint32_t at[N];                                        // from 8 elements before the base: a chunk moved up may start before it
    __device__ __forceinline__ void place(int32_t rows_left, int64_t ld) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int c = int(threadIdx.x) + h * kThreads;
            at[h] = (uint32_t(min(c / PER_ROW, rows_left - 1)) * uint32_t(ld) + uint32_t(c % PER_ROW) * 8u + 8u) * 2u;
        }
    }
    // base (and gate): the tile's first row at the stage's first reduction step; left: reduction steps from there to the end
    __device__ __forceinline__ void load(const uint16_t* base, const uint16_t* gate, int32_t left) {
        const int32_t k = int32_t(threadIdx.x % PER_ROW) * 8, over = ANY ? max(k + 8 - left, 0) : 0;
        const char* const from = reinterpret_cast<const char*>(base - 8);
        const char* const mask = reinterpret_cast<const char*>(gate - 8);
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const uint32_t off = ANY ? at[h] - 2u * uint32_t(over) : k < left ? at[h] : 16u;
            v[h] = ANY ? load8_any(from + off) : *reinterpret_cast<const uint4*>(from + off);
            if constexpr (GATE) g[h] = load8_any(mask + off);
        }
    }
    __device__ __forceinline__ void store(uint16_t* s, int32_t left) const {
        const int32_t k = int32_t(threadIdx.x % PER_ROW) * 8;
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int c = int(threadIdx.x) + h * kThreads;
            uint4 x = v[h];
            if constexpr (GATE) x = make_uint4(gate_pair(x.x, g[h].x), gate_pair(x.y, g[h].y), gate_pair(x.z, g[h].z), gate_pair(x.w, g[h].w));
            if (left < BK) {
                if (ANY && (left & 7)) {
                    const uint4 y = moved_up8(x, 8 - (left & 7));
                    if (k < left && k + 8 > left) x = y;
                }
                if (k >= left) x = make_uint4(0u, 0u, 0u, 0u);
            }
            *reinterpret_cast<uint4*>(s + (c / PER_ROW) * kPitch + (c % PER_ROW) * 8) = x;
        }
    }
};

// A stage of the weights in TERMS terms: the copy holds every 32 of its steps in one piece, [term][row][32], padded to whole tiles and to 32 steps.
template <int ROWS, int TERMS, int BK, int kThreads>
struct TermSlab {
    static constexpr int kPitch = BK + 8, PART = TERMS * ROWS * 4, N = PART * (BK / 32) / kThreads;      // pieces of eight: of 32 steps, of a thread
    static_assert(PART % kThreads == 0, "a thread's pieces lie in the same 32 steps for the whole workgroup");
    uint4 v[N];
    __device__ __forceinline__ void place(int32_t, int64_t) {}
    __device__ __forceinline__ void load(const uint16_t* base, const uint16_t*, int32_t left) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            v[h] = make_uint4(0u, 0u, 0u, 0u);
            if (h * kThreads / PART * 32 < left) v[h] = *reinterpret_cast<const uint4*>(base + (uint32_t(threadIdx.x) + h * kThreads) * 8u);
        }
    }
    __device__ __forceinline__ void store(uint16_t* s, int32_t) const {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            const int c = int(threadIdx.x) + h * kThreads % PART;
            *reinterpret_cast<uint4*>(s + (c / 4) * kPitch + h * kThreads / PART * 32 + (c % 4) * 8) = v[h];
        }
    }
};

__device__ __forceinline__ bf16x8 fragment(const uint16_t* s) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(s)); }

// WM x WN wavefronts, each TMB x TNB blocks of 32 x 32. B is the library's own padded weight copy. GATE masks A.
// The blocks are formed transposed (the weights as the first matrix operand), which leaves four consecutive columns of a row
// in a lane: they are rounded in pairs, put through the wavefront's own part of LDS and stored 16 bytes per lane, whole lines
// at a time. Stored from the registers, 2 bytes per lane, the 128 store instructions of a thread kept the vector memory unit
// busy for as long as all matrix instructions of a K = 512 tile take.
// 169,343 rows, 512 x 512, masked: 208 us with the 256 x 128 tile, whose four column tiles read A and the mask four times
// through L2 in half lines (18 TB/s), 184 with 256 x 256, 164 with 128 x 256. One workgroup of 256 x 256 to a compute unit
// leaves its matrix cores idle while the tile's first stage arrives, at each barrier and while it stores; the smaller
// tile reads the weights, which L2 holds, twice as often instead. The plain product takes 94 us (108 with 256 x 256);
// 2,449,029 rows, 256 wide: 1.28 and, masked, 2.18 ms (1.44 and 2.31). Also tried, us at 512 wide plain / masked and ms at 256:
// 256 x 128 with one stage 95 / 197, 1.40 / 2.50; 128 x 128, three to a unit, 91 / 166, 1.31 / 2.34; 64 x 256 98 / 161,
// 1.47 / 2.25; workgroups that stay and fetch the next 256 x 256 tile behind the stores 108 / 197, 1.46 / 2.39.
// STAGES: stages of A and B kept in LDS, 2 or 1 (then a further barrier parts the reads of a stage from the next one's writes).
// TERMS = 3: the weights in three bf16 terms that add up to them exactly (kExactTerms), one product of each block of A with every term. Bound by the
// path of A into LDS: rows at odd addresses come in pieces of half a line in stages of 32 steps, most lines twice (the first three shapes of
// varco_gemm_bf16_usable 260, 283 and 229 us), in whole lines in stages of 64 (175, 178, 138). One stage in LDS, two workgroups to a compute unit.
// Elements that are not the correctly rounded fp64 result, of 100,000, fp32 instructions / this: 50,021 rows 75 -> 200 13 / 7, 20,011 rows 233 -> 47 21 / 12,
// 3,001 rows 511 -> 130 34 / 20.
template <int WM, int WN, int TMB, int TNB, int BK, int STAGES, bool GATE, int TERMS = 1>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm_bf16_kernel(GemmDev g) {
    constexpr int BM = 32 * TMB * WM, BN = 32 * TNB * WN, kThreads = WM * WN * 64, kPitch = BK + 8;
    static_assert(TERMS == 1 || !GATE, "the transform's weights only");
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];       // STAGES stages of A, then of B
    auto sa = [&](int buf) { return lds + buf * (BM * kPitch); };
    auto sb = [&](int buf) { return lds + STAGES * BM * kPitch + buf * (TERMS * BN * kPitch); };

    // workgroup -> tile: tiles that share streamed data go to one XCD (workgroups are dealt to the 8 XCDs
    // round-robin), so that the streamed operand is fetched into a single L2
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3;
    const int32_t in = within % g.inner, out = (within / g.inner) * 8 + xcd;
    if (out >= g.outer) return;        // whole workgroup leaves together: no barrier is skipped
    const bool second = in >= g.tiles_n;             // this workgroup's tile belongs to the dual product
    const int32_t m0 = out * BM, n0 = (second ? in - g.tiles_n : in) * BN;
    const uint16_t* const b_ptr = second ? g.dual : g.b.ptr;
    const int32_t tiles1 = (g.k + BK - 1) / BK, t_end = tiles1 + (g.k2 + BK - 1) / BK;

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = (wave / WN) * (32 * TMB), wn = (wave % WN) * (32 * TNB);
    const int lrow = lane & 31, lk = lane >> 5;

    floatx16 acc[TMB][TNB];
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    RowSlab<BM, GATE, true, BK, kThreads> ra;
    std::conditional_t<TERMS == 1, RowSlab<BN, false, false, BK, kThreads>, TermSlab<BN, TERMS, BK, kThreads>> rb;
    const uint16_t *pa = nullptr, *pg = nullptr, *pb = nullptr;     // the next stage's bases, and what is left of its product's steps
    int32_t left = 0;
    auto enter = [&](const OperandDev& a, const uint16_t* b, int64_t ldb, int32_t steps) {
        pa = a.ptr + int64_t(m0) * a.ld, pg = a.gate + int64_t(m0) * a.ld, pb = b + int64_t(n0) * ldb * TERMS;
        ra.place(g.m - m0, a.ld);
        rb.place(g.n - n0, ldb);
        left = steps;
    };
    int32_t held = 0;                                               // steps left of the stage that is in registers
    auto fetch = [&](int32_t t) {
        if (t == tiles1) enter(g.a2, g.b2.ptr, g.b2.ld, g.k2);
        ra.load(pa, pg, left);
        rb.load(pb, nullptr, left);
        held = left;
        pa += BK, pg += BK, pb += TERMS == 1 ? BK : TERMS * BN * BK, left -= BK;
    };
    auto stash = [&](int buf) {
        ra.store(sa(buf), held);
        rb.store(sb(buf), held);
    };

    if (t_end > 0) {
        enter(g.a, b_ptr, g.b.ld, g.k);
        fetch(0);
        if constexpr (STAGES == 2) stash(0);
    }
    if constexpr (STAGES == 2) __syncthreads();
    for (int32_t t = 0; t < t_end; ++t) {
        const int buf = STAGES == 2 ? t & 1 : 0;
        if constexpr (STAGES == 1) stash(0);
        if (t + 1 < t_end) fetch(t + 1);
        if constexpr (STAGES == 1) __syncthreads();
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            const int koff = s * 16 + lk * 8;
            bf16x8 fa[TMB], fb[TERMS][TNB];
#pragma unroll
            for (int i = 0; i < TMB; ++i) fa[i] = fragment(sa(buf) + (wm + i * 32 + lrow) * kPitch + koff);
#pragma unroll
            for (int p = 0; p < TERMS; ++p)
#pragma unroll
                for (int j = 0; j < TNB; ++j) fb[p][j] = fragment(sb(buf) + (p * BN + wn + j * 32 + lrow) * kPitch + koff);
#pragma unroll
            for (int p = 0; p < TERMS; ++p)
#pragma unroll
                for (int i = 0; i < TMB; ++i)
#pragma unroll
                    for (int j = 0; j < TNB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[p][j], fa[i], acc[i][j], 0, 0, 0);
        }
        if constexpr (STAGES == 2)
            if (t + 1 < t_end) stash(buf ^ 1);
        __syncthreads();
    }

    // accumulator register v of a lane is element (row lane % 32, column 8 * (v / 4) + 4 * (lane / 32) + v % 4)
    constexpr int kOut = 32 * TNB + 8;                     // elements per row of the wavefront's 32-row strip in LDS
    static_assert(kThreads / 64 * 32 * kOut <= STAGES * (BM + TERMS * BN) * kPitch, "a strip per wavefront");
    uint16_t* const strip = lds + wave * 32 * kOut;
    bf16_t* const base = static_cast<bf16_t*>(second ? g.c_dual : g.c);
    const bool vec = g.vec_c;
#pragma unroll
    for (int i = 0; i < TMB; ++i) {
        const int32_t row0 = m0 + wm + 32 * i;
        if (row0 >= g.m) break;
#pragma unroll
        for (int j = 0; j < TNB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = acc[i][j][4 * q + e];
                const int c = 32 * j + 8 * q + 4 * lk;
                if (g.accumulate) {                        // old values from clamped, always valid addresses
                    const bf16_t* old = base + int64_t(min(row0 + lrow, g.m - 1)) * g.ldc;
                    const int32_t col = n0 + wn + c;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] += Elem<bf16_t>::load(old + min(col + e, g.n - 1));
                }
                if (g.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = fmaxf(x[e], 0.f);
                }
                *reinterpret_cast<uint2*>(strip + lrow * kOut + c) = make_uint2(bf16_pair(x[0], x[1]), bf16_pair(x[2], x[3]));
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (vec) {                                         // rows of C are whole 16-byte pieces
            constexpr int PER = 4 * TNB, RPI = 64 / PER;   // pieces per row, rows per instruction
#pragma unroll
            for (int r = 0; r < 32; r += RPI) {
                const int rr = r + lane / PER, c = lane % PER * 8;
                if (row0 + rr < g.m && n0 + wn + c < g.n)
                    *reinterpret_cast<uint4*>(base + int64_t(row0 + rr) * g.ldc + n0 + wn + c) = *reinterpret_cast<const uint4*>(strip + rr * kOut + c);
            }
        } else {
            for (int r = 0; r < 32 && row0 + r < g.m; ++r)
                for (int c = lane; c < 32 * TNB; c += 64)
                    if (n0 + wn + c < g.n) base[int64_t(row0 + r) * g.ldc + n0 + wn + c].bits = strip[r * kOut + c];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
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

bool varco_gemm_bf16_usable(const GemmArgs& ga) {
    if (ga.m <= 0 || ga.n <= 0) return false;
    if (ga.a.transposed) return varco_gemm_tn_bf16_usable(ga);
    if (ga.a.dtype != VARCO_BF16) return false;
    if (ga.bf16_terms == kExactTerms) {
        // Rows of any length from 8 on, at any address of an element; weights that are not rounded, three products of each. fp32 instructions on
        // tiles of 128 x 128 (256 x 64) in stages of 16 steps / this, us: 819,353 rows two taps 135 -> 40 363 / 175, 911,699 rows 227 -> 40 added to C
        // 345 / 178, 323,741 rows 79 -> 272 239 / 138, 52,727 rows two taps 121 -> 168 93 / 36, 35,999 rows 221 -> 56 40 / 16. (Rows of at
        // most 16 elements, and of at most 32 for some outputs, keep the fp32 instructions: exact_terms.)
        auto ok3 = [&](const GemmOperand& o, const void* prep, int64_t pitch, int32_t k) {
            return o.dtype == VARCO_BF16 && !o.transposed && !o.gate && prep && aligned_to(prep, 16) && k >= 8 && pitch == (int64_t(k) + 31) / 32 * 32;
        };
        return ga.c_dtype == VARCO_BF16 && !ga.b.gate && !ga.c_dual && ga.split_k <= 1 && ok3(ga.a, ga.b_prep, ga.b_prep_ld, ga.k) &&
               (ga.k2 == 0 || ok3(ga.a2, ga.b2_prep, ga.b2_prep_ld, ga.k2));
    }
    // (Here the weights are rounded to bf16.)
    auto ok8 = [](const GemmOperand& o) { return aligned_to(o.ptr, 8) && aligned_to(o.gate, 8) && o.ld % 4 == 0; };
    // needs the library's bf16 weight copy [n][pitch], pitch a multiple of 8
    if (ga.c_dtype != VARCO_BF16 || !ga.b_prep || ga.b_prep_ld % 8 != 0 || !aligned_to(ga.b_prep, 16)) return false;
    if (ga.b.gate || ga.k < 8 || ga.k % 4 != 0 || !ok8(ga.a) || ga.split_k > 1) return false;
    if (ga.k2 > 0 && (!ga.b2_prep || ga.b2_prep_ld % 8 != 0 || !aligned_to(ga.b2_prep, 16) || ga.k2 < 8 || ga.k2 % 4 != 0 ||
                      !ok8(ga.a2) || ga.a2.gate || ga.a2.dtype != VARCO_BF16 || ga.a2.transposed))
        return false;
    return !ga.c_dual || (ga.k2 == 0 && ga.b_dual_prep && aligned_to(ga.b_dual_prep, 16));
}

hipError_t varco_launch_gemm_bf16(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag, int32_t* split_used) {
    if (ga.a.transposed) return varco_launch_gemm_tn_bf16(ga, stream, tag, split_used);
    // 128 x 256 where its tiles fill the device, two to a compute unit, and pad no more columns than 256 x 128
    const int64_t wide = int64_t((ga.m + 127) / 128) * ((ga.n + 255) / 256);
    const bool exact = ga.bf16_terms == kExactTerms;
    const int bn = ga.n <= 64 ? 64 : !exact && wide >= 512 && (ga.n + 255) / 256 * 2 == (ga.n + 127) / 128 ? 256 : 128;
    const int bm = bn == 256 || (exact && bn == 128) ? 128 : 256;
    const bool gate = ga.a.gate != nullptr;

    GemmDev g;
    g.m = ga.m, g.n = ga.n, g.k = ga.k, g.k2 = ga.k2;
    auto u16 = [](const void* p) { return static_cast<const uint16_t*>(p); };
    g.a = {u16(ga.a.ptr), u16(ga.a.gate), ga.a.ld};
    g.a2 = {u16(ga.a2.ptr), u16(ga.a2.gate), ga.a2.ld};
    g.b = {u16(ga.b_prep), nullptr, ga.b_prep_ld};
    g.b2 = {u16(ga.b2_prep), nullptr, ga.b2_prep_ld};
    g.c = ga.c;
    g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0;
    g.relu = ga.relu ? 1 : 0;
    g.vec_c = ga.n % 8 == 0 && ga.ldc % 8 == 0 && aligned_to(ga.c, 16) && aligned_to(ga.c_dual, 16) ? 1 : 0;
    g.tiles_n = (ga.n + bn - 1) / bn;
    g.dual = ga.c_dual ? u16(ga.b_dual_prep) : nullptr;
    g.c_dual = ga.c_dual;
    g.inner = g.tiles_n * (ga.c_dual ? 2 : 1);      // the dual product's tiles come right behind the first one's, on the same XCD
    g.outer = (ga.m + bm - 1) / bm;
    const int64_t blocks = int64_t((g.outer + 7) / 8 * 8) * g.inner;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid{unsigned(blocks)};
    *split_used = 1;

    hipError_t err = hipSuccess;
    auto launch = [&](auto wm, auto wn, auto tmb, auto tnb, auto bk, auto stages) {
        constexpr int WM = decltype(wm)::value, WN = decltype(wn)::value, TMB = decltype(tmb)::value, TNB = decltype(tnb)::value;
        constexpr int BK = decltype(bk)::value, STAGES = decltype(stages)::value;
        constexpr size_t bytes = size_t(STAGES) * 32 * (TMB * WM + TNB * WN) * (BK + 8) * 2;
        with_flag(gate, [&](auto gt) {
            const auto kernel = gemm_bf16_kernel<WM, WN, TMB, TNB, BK, STAGES, decltype(gt)::value>;
            if (bytes > 64 * 1024)
                err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
            if (err != hipSuccess) return;
            tag.begin(stream);
            hipLaunchKernelGGL(kernel, grid, dim3(WM * WN * 64), bytes, stream, g);
            tag.end(stream);
        });
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    using I32 = std::integral_constant<int, 32>;
    using I64 = std::integral_constant<int, 64>;
    if (exact) {
        auto go = [&](auto wm, auto wn, auto stages) {
            constexpr int WM = decltype(wm)::value, WN = decltype(wn)::value, STAGES = decltype(stages)::value;
            constexpr size_t bytes = size_t(STAGES) * 32 * (2 * WM + 3 * 2 * WN) * (64 + 8) * 2;
            const auto kernel = gemm_bf16_kernel<WM, WN, 2, 2, 64, STAGES, false, 3>;
            if (bytes > 64 * 1024)
                err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
            if (err != hipSuccess) return;
            tag.begin(stream);
            hipLaunchKernelGGL(kernel, grid, dim3(WM * WN * 64), bytes, stream, g);
            tag.end(stream);
        };
        if (bn == 128)
            go(I2{}, I2{}, I1{});
        else
            go(I4{}, I1{}, I1{});
    } else if (bn == 256)
        launch(I2{}, I2{}, I2{}, I4{}, I64{}, I1{});
    else if (bn == 128)
        launch(I2{}, I2{}, I4{}, I2{}, I32{}, I2{});
    else
        launch(I4{}, I1{}, I2{}, I2{}, I32{}, I2{});
    return err != hipSuccess ? err : hipGetLastError();
}
