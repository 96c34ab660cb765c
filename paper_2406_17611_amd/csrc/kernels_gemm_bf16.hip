// Dense feature transform of eq. (2) and its input gradient for bf16-stored activations, on the bf16 matrix cores with
// fp32 accumulation (v_mfma_f32_32x32x16_bf16): X_out = act(M H1 + X H0), dM = dZ H1^T. Weights are kept in fp32 by the
// caller; the library hands this kernel a bf16 copy laid out [output index][reduction index] (see
// varco_launch_prep_weights). Weight gradients are in kernels_gemm_tn_bf16.hip.
//
// One 256-thread workgroup (4 wavefronts) computes a 256 x 128 tile of C (256 x 64 for outputs at most 64
// columns wide). A wavefront owns 128 x 64 (or 64 x 64) of it as 32 x 32 blocks: at bf16 rates a wavefront
// tile smaller than that is limited by LDS reads of its fragments, not by the matrix cores. Operand tiles of
// 32 reduction steps are staged through LDS as rows of one output index with the reduction index contiguous
// (80-byte row pitch: 16-byte fragment reads without bank conflicts), double-buffered against the global
// loads of the next tile. Both operands have the reduction index contiguous in memory, so the global -> LDS copy moves
// 8 (or 4) elements at a time unchanged. The ReLU mask of the backward pass is applied when a tile is written to LDS, the
// activation in the epilogue.
#include <type_traits>

#include "elem.h"
#include "varco_internal.h"

namespace {

constexpr int BK = 32;
constexpr int kThreads = 256;
constexpr int kPitch = BK + 8;   // bf16 elements per LDS row (80 bytes)

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

// ---- operand with the reduction index contiguous in memory: chunks of CH elements, copied unchanged ----
template <int ROWS, int CH, bool GATE>
struct RowRegs {
    static constexpr int PER_ROW = BK / CH;
    static constexpr int N = ROWS * PER_ROW / kThreads;
    uint32_t v[N][CH / 2];
    uint32_t g[GATE ? N : 1][CH / 2];
    uint32_t inside;
};

template <int ROWS, int CH, bool GATE>
__device__ __forceinline__ void load_rows(const OperandDev& op, int32_t i0, int32_t extent, int32_t k0, int32_t kmax,
                                          RowRegs<ROWS, CH, GATE>& r) {
    using R = RowRegs<ROWS, CH, GATE>;
    using W = std::conditional_t<CH == 8, uint4, uint2>;
    r.inside = 0u;
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const int c = threadIdx.x + h * kThreads;
        const int32_t i = i0 + c / R::PER_ROW;
        const int32_t kk = k0 + (c % R::PER_ROW) * CH;
        const bool in = i < extent && kk < kmax;          // kmax is a multiple of CH: a chunk is wholly in or out
        const int64_t off = in ? int64_t(i) * op.ld + kk : 0;
        const W x = *reinterpret_cast<const W*>(op.ptr + off);
        r.v[h][0] = x.x, r.v[h][1] = x.y;
        if constexpr (CH == 8) r.v[h][2] = x.z, r.v[h][3] = x.w;
        if (GATE) {
            const W y = *reinterpret_cast<const W*>(op.gate + off);
            r.g[h][0] = y.x, r.g[h][1] = y.y;
            if constexpr (CH == 8) r.g[h][2] = y.z, r.g[h][3] = y.w;
        }
        r.inside |= in ? (1u << h) : 0u;
    }
}

template <int ROWS, int CH, bool GATE>
__device__ __forceinline__ void store_rows(const RowRegs<ROWS, CH, GATE>& r, uint16_t* s) {
    using R = RowRegs<ROWS, CH, GATE>;
#pragma unroll
    for (int h = 0; h < R::N; ++h) {
        const int c = threadIdx.x + h * kThreads;
        const bool in = (r.inside >> h) & 1u;
        uint32_t x[CH / 2];
#pragma unroll
        for (int u = 0; u < CH / 2; ++u) {
            x[u] = in ? r.v[h][u] : 0u;
            if (GATE) x[u] = gate_pair(x[u], r.g[h][u]);
        }
        uint16_t* dst = s + (c / R::PER_ROW) * kPitch + (c % R::PER_ROW) * CH;
        if constexpr (CH == 8)
            *reinterpret_cast<uint4*>(dst) = make_uint4(x[0], x[1], x[2], x[3]);
        else
            *reinterpret_cast<uint2*>(dst) = make_uint2(x[0], x[1]);
    }
}

__device__ __forceinline__ bf16x8 fragment(const uint16_t* s, int row, int koff) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(s + row * kPitch + koff));
}

// WM x WN wavefronts, each TMB x TNB blocks of 32 x 32. A_CH: elements per global load of A (B is the library's own padded
// weight copy, always 8). GATE masks A.
template <int WM, int WN, int TMB, int TNB, int A_CH, bool GATE>
__global__ __launch_bounds__(kThreads, 2) void gemm_bf16_kernel(GemmDev g) {
    constexpr int BM = 32 * TMB * WM, BN = 32 * TNB * WN;
    __shared__ __attribute__((aligned(16))) uint16_t sa[2][BM * kPitch];
    __shared__ __attribute__((aligned(16))) uint16_t sb[2][BN * kPitch];

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

    RowRegs<BM, A_CH, GATE> ra;
    RowRegs<BN, 8, false> rb;
    // operands of tile t are picked with selects, not branches, so that the loads stay straight-line code
    auto fetch = [&](int32_t t) {
        const bool first = t < tiles1;
        OperandDev oa, ob;
        oa.ptr = first ? g.a.ptr : g.a2.ptr, oa.gate = first ? g.a.gate : g.a2.gate, oa.ld = first ? g.a.ld : g.a2.ld;
        ob.ptr = first ? b_ptr : g.b2.ptr, ob.gate = first ? g.b.gate : g.b2.gate, ob.ld = first ? g.b.ld : g.b2.ld;
        const int32_t k0 = (first ? t : t - tiles1) * BK, kmax = first ? g.k : g.k2;
        load_rows(oa, m0, g.m, k0, kmax, ra);
        load_rows(ob, n0, g.n, k0, kmax, rb);
    };
    auto stash = [&](int buf) {
        store_rows(ra, sa[buf]);
        store_rows(rb, sb[buf]);
    };

    if (t_end > 0) {
        fetch(0);
        stash(0);
    }
    __syncthreads();
    for (int32_t t = 0; t < t_end; ++t) {
        const int buf = t & 1;
        if (t + 1 < t_end) fetch(t + 1);
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            const int koff = s * 16 + lk * 8;
            bf16x8 fa[TMB], fb[TNB];
#pragma unroll
            for (int i = 0; i < TMB; ++i) fa[i] = fragment(sa[buf], wm + i * 32 + lrow, koff);
#pragma unroll
            for (int j = 0; j < TNB; ++j) fb[j] = fragment(sb[buf], wn + j * 32 + lrow, koff);
#pragma unroll
            for (int i = 0; i < TMB; ++i)
#pragma unroll
                for (int j = 0; j < TNB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (t + 1 < t_end) stash(buf ^ 1);
        __syncthreads();
    }

    // epilogue: accumulator register v of a lane is element (8 * (v / 4) + 4 * (lane / 32) + v % 4, lane % 32).
    // A tile that lies wholly inside C takes a path without per-element tests, with addresses formed from one
    // 64-bit base per lane plus 32-bit multiples of the row pitch. When C is added to, the old values of a
    // block are fetched by loads that are all issued before the first one is used (from clamped, always valid
    // addresses), not one round trip per element.
    const int32_t col_base = n0 + wn + lrow;
    bf16_t* const base = static_cast<bf16_t*>(second ? g.c_dual : g.c);
    const bool add_old = g.accumulate, relu = g.relu;
    auto finish = [&](auto guard) {
        constexpr bool GUARD = decltype(guard)::value;
        bf16_t* const out0 = base + int64_t(m0 + wm) * g.ldc + col_base;          // interior tiles only
#pragma unroll
        for (int i = 0; i < TMB; ++i) {
#pragma unroll
            for (int j = 0; j < TNB; ++j) {
                bf16_t* ptr[16];
                bool ok[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int32_t r = i * 32 + 4 * lk + 8 * (v >> 2) + (v & 3);        // row inside the wavefront's part
                    if constexpr (GUARD) {
                        const int32_t row = m0 + wm + r, col = col_base + j * 32;
                        ok[v] = row < g.m && col < g.n;
                        ptr[v] = base + int64_t(min(row, g.m - 1)) * g.ldc + min(col, g.n - 1);
                    } else {
                        ok[v] = true;
                        ptr[v] = out0 + j * 32 + uint32_t(r) * uint32_t(g.ldc);        // a tile spans < 2^32 elements
                    }
                }
                float old[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) old[v] = 0.f;
                if (add_old) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) old[v] = Elem<bf16_t>::load(ptr[v]);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float x = acc[i][j][v] + old[v];
                    if (relu) x = fmaxf(x, 0.f);
                    if (ok[v]) Elem<bf16_t>::store(ptr[v], x);
                }
            }
        }
    };
    if (m0 + BM <= g.m && n0 + BN <= g.n)
        finish(std::false_type{});
    else
        finish(std::true_type{});
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
    auto ok8 = [](const GemmOperand& o) { return aligned_to(o.ptr, 8) && aligned_to(o.gate, 8) && o.ld % 4 == 0; };
    // needs the library's bf16 weight copy [n][pitch], pitch a multiple of 8
    if (ga.c_dtype != VARCO_BF16 || !ga.b_prep || ga.b_prep_ld % 8 != 0 || !aligned_to(ga.b_prep, 16)) return false;
    if (ga.b.gate || ga.k % 4 != 0 || !ok8(ga.a) || ga.split_k > 1) return false;
    if (ga.k2 > 0 && (!ga.b2_prep || ga.b2_prep_ld % 8 != 0 || !aligned_to(ga.b2_prep, 16) || ga.k2 % 4 != 0 ||
                      !ok8(ga.a2) || ga.a2.gate || ga.a2.dtype != VARCO_BF16 || ga.a2.transposed))
        return false;
    return !ga.c_dual || (ga.k2 == 0 && ga.b_dual_prep && aligned_to(ga.b_dual_prep, 16));
}

hipError_t varco_launch_gemm_bf16(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag, int32_t* split_used) {
    if (ga.a.transposed) return varco_launch_gemm_tn_bf16(ga, stream, tag, split_used);
    const bool narrow = ga.n <= 64;
    const int bm = 256, bn = narrow ? 64 : 128;
    auto chunk8 = [](const GemmOperand& o, int32_t k) {
        return !o.ptr || (aligned_to(o.ptr, 16) && aligned_to(o.gate, 16) && o.ld % 8 == 0 && k % 8 == 0);
    };
    const bool a8 = chunk8(ga.a, ga.k) && (ga.k2 == 0 || chunk8(ga.a2, ga.k2));
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
    g.tiles_n = (ga.n + bn - 1) / bn;
    g.dual = ga.c_dual ? u16(ga.b_dual_prep) : nullptr;
    g.c_dual = ga.c_dual;
    g.inner = g.tiles_n * (ga.c_dual ? 2 : 1);      // the dual product's tiles come right behind the first one's, on the same XCD
    g.outer = (ga.m + bm - 1) / bm;
    const int64_t blocks = int64_t((g.outer + 7) / 8 * 8) * g.inner;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid{unsigned(blocks)};
    *split_used = 1;

    tag.begin(stream);
    with_flag(narrow, [&](auto nr) {
        with_flag(gate, [&](auto gt) {
            constexpr bool NR = decltype(nr)::value, GT = decltype(gt)::value;
            constexpr int WM = NR ? 4 : 2, WN = NR ? 1 : 2, TMB = NR ? 2 : 4, TNB = 2;
            if (a8)
                hipLaunchKernelGGL((gemm_bf16_kernel<WM, WN, TMB, TNB, 8, GT>), grid, dim3(kThreads), 0, stream, g);
            else
                hipLaunchKernelGGL((gemm_bf16_kernel<WM, WN, TMB, TNB, 4, GT>), grid, dim3(kThreads), 0, stream, g);
        });
    });
    tag.end(stream);
    return hipGetLastError();
}
