// Graph-convolution aggregation M = S_q [X_loc ; X~_halo] (eq. (1)-(2) of the paper; Algorithm 1: local
// rows uncompressed, remote rows in compressed form) and its transpose for the backward pass.
//
// HBM-bound gather kernels. One wavefront (64 lanes) takes one work item = a run of consecutive CSR entries
// of one row, as long as the host's work list makes it (at most 128 entries in the forward block, 32 in the
// transposed ones); longer rows are split and their partial sums reduced in a second pass, so power-law hubs
// do not serialise on one wavefront and no floating-point atomics reach memory. The kernels are latency
// bound unless many loads are in flight, and a wavefront waits for the slowest load of a batch, so every
// gather loop first issues a block of independent loads and only then consumes them.
//
//   dense source rows (local rows; halo rows when k == width): a power-of-two group of lanes covers one
//     row with 16-byte loads, the groups of a wavefront take different edges and are summed at the end
//     with cross-lane shuffles (wavefront-level segmented reduction);
//   compressed halo rows (k < width): never decompressed to memory. The stored elements of several edges
//     are loaded side by side (lane = (edge, j)), their positions pi_v(j) are recomputed from the key,
//     and they are accumulated into a per-wavefront row in LDS.
//
// The forward kernel reads a per-entry record {source row, node id} that the library derives once from
// the caller's column indices, so that a halo entry needs no dependent index lookups before its data load.
#include <algorithm>

#include <type_traits>

#include "elem.h"
#include "gather_device.h"
#include "mask_device.h"
#include "prep_device.h"

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
// Threads per workgroup of spmm_kernel. With compressed rows a wavefront is a workgroup of its own: runs differ in
// length, and a workgroup keeps its LDS and wavefront slots until its last wavefront is done (bf16 configuration,
// forward aggregation 23.7 -> 22.8 ms per step). The dense-only kernels use no LDS and run faster four to a
// workgroup (large fp32 configuration, transposed local block 4.5 against 4.8 ms).
constexpr int agg_block(int mode) { return mode == 0 /* dense rows only */ ? kBlock : 64; }
// Independent row loads issued back to back by the kernels that also take compressed rows (dense rows here,
// compressed rows see sparse_phase): their register budget is the 64 of eight wavefronts per SIMD, or the 72 of
// seven; resident wavefronts, each a chain of dependent round trips, are what their rate is made of.
constexpr int kXcdRun = 32;       // consecutive workgroups of the work list that one XCD takes (see spmm_kernel)
constexpr int kHaloWaves = 7;
constexpr int kUnroll = 3;
constexpr int kUnrollDense = 4;   // dense-only kernels have registers to spare

template <int VEC>
using Vec = FloatVec<VEC>;

__device__ __forceinline__ void fma_vec(float4& acc, float w, const float4& v) {
    acc.x += w * v.x;
    acc.y += w * v.y;
    acc.z += w * v.z;
    acc.w += w * v.w;
}
__device__ __forceinline__ void fma_vec(float& acc, float w, const float& v) { acc += w * v; }
__device__ __forceinline__ void add_vec(float4& a, const float4& b) {
    a.x += b.x;
    a.y += b.y;
    a.z += b.z;
    a.w += b.w;
}
__device__ __forceinline__ void add_vec(float& a, const float& b) { a += b; }
__device__ __forceinline__ void add_vec(float2& a, const float2& b) {
    a.x += b.x;
    a.y += b.y;
}
__device__ __forceinline__ float4 shfl_xor_vec(const float4& v, int mask) {
    return make_float4(__shfl_xor(v.x, mask), __shfl_xor(v.y, mask), __shfl_xor(v.z, mask), __shfl_xor(v.w, mask));
}
__device__ __forceinline__ float shfl_xor_vec(const float& v, int mask) { return __shfl_xor(v, mask); }
__device__ __forceinline__ void zero_vec(float4& v) { v = make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ void zero_vec(float& v) { v = 0.f; }
__device__ __forceinline__ void zero_vec(float2& v) { v = make_float2(0.f, 0.f); }
__device__ __forceinline__ float elem(const float2& v, int i) { return i == 0 ? v.x : v.y; }
__device__ __forceinline__ float elem(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
__device__ __forceinline__ float elem(const float& v, int) { return v; }

template <typename T>
struct SpmmArgs {
    const SpmmItem* items;
    int32_t n_items;
    const VarcoEdge* edge;    // HALO kernels: one record per CSR entry
    const int32_t* colidx;    // dense-only kernels: column = source row
    const float* vals;
    const T* dense;
    const T* z;
    MaskRule rule;
    T* out;
    int32_t row_base;
    float* partial;           // partial sums of split rows stay in fp32
    int32_t lpr_log2;         // lanes per dense row = 1 << lpr_log2
    int32_t ku;               // loads per compressed row: k / ev, rounded up (the last one overlaps the one before)
    int32_t lpe_log2;         // lanes that share one compressed row = 1 << lpe_log2 (>= min(ku, 64))
    int32_t epi;              // compressed rows handled per instruction = private LDS rows per wavefront
    // kOwner: the messages themselves, written by the workgroups from `copy_block` to `prep_block` (see owner_messages)
    const int32_t *brow, *bgid;
    T* messages;
    uint32_t n_messages;      // elements: boundary rows x k
    int32_t copy_block, prep_block;
};

// N consecutive stored elements as they come from memory (bf16 stays packed until it is used).
template <typename T, int N>
struct Stored {
    using type = typename FloatVec<N>::type;
    static __device__ __forceinline__ float get(const type& v, int i) { return elem(v, i); }
};
template <>
struct Stored<bf16_t, 4> {
    using type = uint2;
    static __device__ __forceinline__ float get(const uint2& v, int i) {
        const uint32_t u = i < 2 ? v.x : v.y;
        return __uint_as_float((i & 1) ? (u & 0xFFFF0000u) : (u << 16));
    }
};
template <>
struct Stored<bf16_t, 2> {
    using type = uint32_t;
    static __device__ __forceinline__ float get(const uint32_t& v, int i) {
        return __uint_as_float(i ? (v & 0xFFFF0000u) : (v << 16));
    }
};
template <>
struct Stored<bf16_t, 1> {
    using type = uint16_t;
    static __device__ __forceinline__ float get(const uint16_t& v, int) { return bf16_to_float(v); }
};

// The four elements in the order rot, rot + 1, .. (mod 4); rot differs between lanes.
__device__ __forceinline__ uint2 rotated(const uint2& v, uint32_t rot) {
    const uint32_t sel = 0x03020100u + rot * 0x02020202u;           // bytes 2 rot .. 2 rot + 3, each mod 8
    return make_uint2(__builtin_amdgcn_perm(v.y, v.x, sel & 0x07070707u), __builtin_amdgcn_perm(v.y, v.x, (sel + 0x04040404u) & 0x07070707u));
}
__device__ __forceinline__ float4 rotated(const float4& v, uint32_t rot) {
    const bool one = rot & 1u, two = rot & 2u;
    const float4 s = make_float4(one ? v.y : v.x, one ? v.z : v.y, one ? v.w : v.z, one ? v.x : v.w);
    return make_float4(two ? s.z : s.x, two ? s.w : s.y, two ? s.x : s.z, two ? s.y : s.w);
}

// Scatter-accumulate the compressed rows of the wavefront's current batch: lanes [nd, nd + ns) hold one halo entry each (its
// row of z, weight, packed (a, b)). A group of `lpe` lanes takes one entry (lane = group of EV stored elements), `epi` entries
// are handled per instruction, and each of those lane groups adds into a private LDS row of its own: the positions of one
// entry are distinct, so plain read-add-write is race-free and no LDS atomics (which run at a small fraction of the plain LDS
// rate) are needed.
// The kernel issues vector instructions three quarters of the time, so their number is its time:
// Z32: every element of the compressed buffer lies below 2^32 bytes: `zoff` is the row's byte offset, an address is the
// (uniform) base plus 32 bits, one register per gather in flight; otherwise `zoff` is the row.
// POW2: positions are byte offsets (a and b come multiplied by 4) that wrap with the mask that also sets the row's base;
// otherwise they wrap with one unsigned minimum (q - width is huge when q < width).
// EV = 4: the lanes of one entry step through its stored elements four at a time, so at one instruction their positions would
// differ by multiples of 4 a: with 16 or more lanes per entry, lanes 8 apart would meet in one LDS bank at different
// addresses. Lane j therefore takes its four elements in the order r, r + 1, .. (mod 4), r = j / 8: lanes 8 apart then are at
// positions that differ by an odd number modulo 32. One byte permutation of the loaded words, against three instructions per
// element for folding position bits into the address, and the rows are read back as they are.
// (bf16, 512 wide, k = 128, a dozen entries per row: the forward aggregation took 314 us with the folded addresses, the
// multiplier table staged per wavefront and per-lane dense addresses; 176 us now.)
// REM: rows of any number of elements from EV on, at any address of an element. The last lane of an entry takes the row's last EV elements; those
// that its neighbour has as well it adds to a word behind the private rows that nobody reads (two lanes at one address would lose a sum).
template <typename T, int EV, bool Z32, bool POW2, bool REM>
__device__ __forceinline__ void sparse_phase(const SpmmArgs<T>& p, int lane, int nd, int ns, uint32_t zoff, float w, uint32_t mab,
                                             char* lrows) {
    constexpr bool ROT = EV == 4;
    using S = typename Stored<T, EV>::type;
    typedef S Any __attribute__((aligned(REM ? sizeof(T) : alignof(S))));
    // Gathers in flight per lane: six of at most 8 bytes (four bf16 or two fp32 elements), three of 16 bytes:
    // about the same registers either way. A wavefront waits for the slowest of its gathers, so fewer, larger
    // batches win even at the price of one resident wavefront (bf16 rows of 512 elements: 7 per SIMD, forward
    // aggregation 30.6 -> 24.8 ms per step; the fp32 kernel keeps 8: 13.8 -> 13.5 ms). Eight gathers, or four
    // of 16 bytes, cost more wavefronts than they gain (27.6 ms and 14.5 ms).
    constexpr int G = EV * sizeof(T) <= 8 ? 2 * kUnroll : kUnroll;
    const uint32_t width = p.rule.width;
    const int sub = lane >> p.lpe_log2;
    const int jl = lane & ((1 << p.lpe_log2) - 1);
    const bool lane_ok = sub < p.epi && jl < p.ku;
    using lds_float = __attribute__((address_space(3))) float;
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lrows)) + uint32_t(sub) * width * 4u;
    const uint32_t mask = (width - 1u) * 4u;
    const uint32_t rot = ROT ? uint32_t(jl >> 3) & 3u : 0u;
    const uint32_t nowhere = base + uint32_t(p.epi - sub) * width * 4u;
    for (int j0 = 0; j0 < p.ku; j0 += 64) {          // more than one pass only when an entry needs > 64 lanes
        const int ju = j0 + jl;
        const bool j_ok = lane_ok && ju < p.ku;
        const uint32_t j = REM ? min(uint32_t(ju) * EV, p.rule.k - EV) : uint32_t(ju) * EV, j_bytes = j * uint32_t(sizeof(T));
        const uint32_t again = REM ? uint32_t(ju) * EV - j : 0u;         // of the lane's elements, so many are its neighbour's
        // `count` entries per lane group from entry r0 on. All gathers are issued first, with the entries' weights and rules
        // fetched from their lanes behind them; the positions are computed after the wait, so that more gathers fit the
        // registers of a wavefront. Straight-line code: a branch per entry would wait for every fetch by itself.
        auto batch = [&](int r0, auto count) {
            constexpr int N = decltype(count)::value;
            S v[N];
            float wi[N];
            uint32_t ab[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int es = r0 + u * p.epi + sub;
                const uint32_t r = lane_value(zoff, 4 * (nd + es));
                // lanes without an entry re-read the start of the buffer (never used, but no branch around the load)
                if constexpr (Z32)
                    v[u] = *reinterpret_cast<const Any*>(reinterpret_cast<const char*>(p.z) + (j_ok && es < ns ? r + j_bytes : 0u));
                else
                    v[u] = *reinterpret_cast<const Any*>(p.z + (j_ok && es < ns ? int64_t(r) * p.rule.k + j : int64_t(0)));
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int at = 4 * (nd + r0 + u * p.epi + sub);
                wi[u] = __uint_as_float(lane_value(__float_as_uint(w), at));
                ab[u] = lane_value(mab, at);
            }
            __builtin_amdgcn_sched_barrier(0);       // keep the work below behind the loads
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (j_ok && r0 + u * p.epi + sub < ns) {
                    const uint32_t a = ab[u] & 0xFFFFu;
                    uint32_t q = __umul24(a, j + rot) + (ab[u] >> 16);
                    uint32_t at[EV];
                    float cur[EV];
                    if constexpr (POW2) {
                        at[0] = (q & mask) | base;
                        const uint32_t back = a * uint32_t(1 - EV);          // from element 3 to element 0
#pragma unroll
                        for (int i = 1; i < EV; ++i) at[i] = ((at[i - 1] + (ROT && rot == uint32_t(EV - i) ? back : a)) & mask) | base;
                    } else {
                        q = varco_mod_width(q, width, p.rule.width_magic);
                        at[0] = q * 4u + base;
                        uint32_t back = 0u;
                        if constexpr (ROT) {
                            back = 2u * a, back = min(back, back - width);
                            back += a, back = min(back, back - width);
                            back = width - back;                             // -3 a mod width (width itself for 0)
                        }
#pragma unroll
                        for (int i = 1; i < EV; ++i) {
                            q += ROT && rot == uint32_t(EV - i) ? back : a;
                            q = min(q, q - width);
                            at[i] = q * 4u + base;
                        }
                    }
                    if constexpr (REM)
#pragma unroll
                        for (int i = 0; i < EV; ++i) at[i] = ((uint32_t(i) + rot) & uint32_t(EV - 1)) < again ? nowhere : at[i];
                    S x = v[u];
                    if constexpr (ROT) x = rotated(x, rot);
#pragma unroll
                    for (int i = 0; i < EV; ++i) cur[i] = *(const lds_float*)(uintptr_t(at[i]));   // distinct positions of one entry
#pragma unroll
                    for (int i = 0; i < EV; ++i) *(lds_float*)(uintptr_t(at[i])) = cur[i] + wi[u] * Stored<T, EV>::get(x, i);
                }
        };
        constexpr int kHalf = G / 2;
        int r0 = 0;
        for (; r0 + p.epi * kHalf < ns; r0 += p.epi * G) batch(r0, std::integral_constant<int, G>{});
        if (r0 + p.epi < ns)
            batch(r0, std::integral_constant<int, (kHalf > 1 ? kHalf : 2)>{});
        else if (r0 < ns)
            batch(r0, std::integral_constant<int, 1>{});
    }
}

// The same sums, in the same order, from the owners' rows of x instead of the compressed ones: `xoff` is a row's byte offset, mab its (a, b).
// An element is a load of its own, behind its position: for launches whose chain of round trips costs less than the launch that writes the
// compressed rows first (varco_spmm_owners_pay).
template <typename T, int EV>
__device__ __forceinline__ void owner_phase(const SpmmArgs<T>& p, int lane, int nd, int ns, uint32_t xoff, float w, uint32_t mab, float* lrows) {
    constexpr int G = EV == 4 ? 2 : EV == 2 ? 4 : 6;       // loads in flight: 8, 8, 6 per lane
    using S = typename Stored<T, 1>::type;
    const uint32_t width = p.rule.width;
    const int sub = lane >> p.lpe_log2, jl = lane & ((1 << p.lpe_log2) - 1);
    float* const mine = lrows + sub * width;
    for (int j0 = 0; j0 < p.ku; j0 += 64) {
        const bool j_ok = sub < p.epi && jl < p.ku && j0 + jl < p.ku;
        const uint32_t j = uint32_t(j0 + jl) * EV;
        for (int r0 = 0; r0 < ns; r0 += p.epi * G) {
            S v[G][EV];
            uint32_t q[G][EV];
            float wi[G];
            bool ok[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int es = r0 + u * p.epi + sub, at = 4 * (nd + es);
                ok[u] = j_ok && es < ns;
                const uint32_t row = lane_value(xoff, at), ab = lane_value(mab, at);
                wi[u] = __uint_as_float(lane_value(__float_as_uint(w), at));
                const uint32_t a = ab & 0xFFFFu;
                q[u][0] = varco_mod_width(__umul24(a, j) + (ab >> 16), width, p.rule.width_magic);
#pragma unroll
                for (int i = 1; i < EV; ++i) q[u][i] = q[u][i - 1] + a, q[u][i] = min(q[u][i], q[u][i] - width);
#pragma unroll
                for (int i = 0; i < EV; ++i)       // lanes without an entry read the first element, unused
                    v[u][i] = *reinterpret_cast<const S*>(reinterpret_cast<const char*>(p.dense) + (ok[u] ? row + q[u][i] * uint32_t(sizeof(T)) : 0u));
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (ok[u]) {
                    float cur[EV];
#pragma unroll
                    for (int i = 0; i < EV; ++i) cur[i] = mine[q[u][i]];          // distinct positions of one entry
#pragma unroll
                    for (int i = 0; i < EV; ++i) mine[q[u][i]] = cur[i] + wi[u] * Stored<T, 1>::get(v[u][i], 0);
                }
        }
    }
}

// Elements [256 block, 256 block + 256) of the messages, by one wavefront.
template <typename T>
__device__ __forceinline__ void owner_messages(const SpmmArgs<T>& p, uint32_t block, int lane) {
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t t = (4 * block + i) * 64 + uint32_t(lane);
        if (t >= p.n_messages) continue;
        const uint32_t b = t / p.rule.k, j = t - b * p.rule.k;
        const MaskAffine m = varco_affine(p.rule, uint32_t(p.bgid[b]));
        p.messages[t] = p.dense[uint32_t(p.brow[b]) * p.rule.width + varco_position(p.rule, m, j)];
    }
}

// T: storage type of the dense rows, the compressed rows and the output (sums are kept in fp32);
// VEC: elements per lane per load of a dense row (16 bytes, or fewer when the width or the bases do not allow it);
// NV: such loads per lane per row (0: fewer than 64 lanes cover a row, see gather_rows);
// MODE: kDenseOnly: all rows are dense; forward aggregation: kFull: halo rows are complete; kSparse / kSparseZ32: compressed,
// EV elements per lane and load, power-of-two width or not, the latter mode with 32-bit offsets (see sparse_phase); kOwner: kept elements come from
// the owners' rows and the launch writes the messages as well (owner_phase, owner_messages). One
// kernel per form: the constants of forms that do not run would take registers, i.e. resident wavefronts, from the one
// that does.
// ANY: rows of any length from VEC elements on, at any address of an element (gather_rows); the lane at the end of a row stores what its
// neighbour stores as well.
constexpr int kDenseOnly = 0, kFull = 1, kSparse = 2, kSparseZ32 = 3, kOwner = 4;
template <typename T, int VEC, int NV, int MODE, int EV, bool POW2, bool ANY, bool REM>
__device__ __forceinline__ void spmm_rows(const SpmmArgs<T>& p) {
    constexpr bool HALO = MODE != kDenseOnly, SPARSE = MODE >= kSparse, Z32 = MODE == kSparseZ32;
    constexpr int kAggBlock = agg_block(MODE), kAggWaves = kAggBlock / 64;
    constexpr int U = NV >= 4 ? 1 : (NV == 2 ? 2 : (HALO ? kUnroll : kUnrollDense)), NR = loads_per_row(NV);
    extern __shared__ __attribute__((aligned(16))) float lds[];     // HALO: the workgroup's (one wavefront's) private rows of compressed-row sums
    static_assert(!HALO || kAggWaves == 1, "the private rows start at the workgroup's LDS");
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int32_t width = int32_t(p.rule.width);

    // Workgroups are dealt to the 8 XCDs round-robin; an XCD takes the work list in runs of kXcdRun consecutive
    // workgroups (the grid is a multiple of 8 runs), so that rows next to each other - which on a graph with any
    // locality share source rows - are aggregated through the same L2 at about the same time, while every XCD still
    // sees the same mix of long and short rows (contiguous eighths put all split rows on one XCD: twice as slow).
    const int32_t xcd = int32_t(blockIdx.x & 7u), seq = int32_t(blockIdx.x >> 3);
    const int32_t block = ((seq / kXcdRun) * 8 + xcd) * kXcdRun + seq % kXcdRun;
    const int32_t idx = block * kAggWaves + __builtin_amdgcn_readfirstlane(wave);   // uniform: the item sits in scalar registers
    if (idx >= p.n_items) return;       // no barriers: wavefronts are independent
    const SpmmItem it = p.items[idx];
    VarcoEdge ed{0, -1};                // the current batch's records: one entry per lane
    int32_t col = 0;
    float w = 0.f;
    auto load_records = [&](int32_t base) {
        ed = VarcoEdge{0, -1}, col = 0, w = 0.f;
        if (base + lane < it.e1) {
            if (HALO)
                ed = p.edge[base + lane];
            if (!HALO || MODE == kOwner)
                col = p.colidx[base + lane];
            w = p.vals[base + lane];
        }
    };
    load_records(it.e0);
    if constexpr (SPARSE)
        for (int c = 4 * lane; c < p.epi * width; c += 256) *reinterpret_cast<float4*>(lds + c) = make_float4(0.f, 0.f, 0.f, 0.f);

    float acc[NR][VEC];
#pragma unroll
    for (int m = 0; m < NR; ++m)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[m][i] = 0.f;
    bool any_sparse = false;
    int dense = 0;                      // entries of whole rows
    const uint32_t key0 = SPARSE ? varco_key0(p.rule) : 0u, key1 = SPARSE ? varco_key1(p.rule) : 0u;

    for (int32_t base = it.e0; base < it.e1; base += 64) {
        if (base != it.e0) load_records(base);
        const bool is_halo = HALO && ed.gid >= 0;
        uint32_t zoff = 0, shift = 0, unit = 0;
        if (SPARSE && is_halo) {         // the multiplier table (at most 2 KB) comes from the cache, used behind the first rows
            zoff = MODE == kOwner ? uint32_t(col) * (uint32_t(width) * uint32_t(sizeof(T))) : Z32 ? uint32_t(ed.src) * (p.rule.k * uint32_t(sizeof(T))) : uint32_t(ed.src);
            const uint32_t h1 = varco_mix32(uint32_t(ed.gid) ^ key0);
            unit = p.rule.units[__umulhi(varco_mix32(h1 ^ key1), p.rule.n_units)];
            shift = __umulhi(h1, p.rule.width) << 16;
        }
        const T* const from = MODE == kFull && is_halo ? p.z : p.dense;
        const uint64_t addr = reinterpret_cast<uint64_t>(from + int64_t(HALO ? ed.src : col) * width);
        const uint64_t hmask = SPARSE ? __ballot(is_halo) : 0ull;
        const int cnt = min(64, it.e1 - base);
        const int ns = SPARSE ? __popcll(hmask) : 0;
        const int nd = cnt - ns;        // columns ascend within a row, so dense entries sit in lanes [0, nd)
        dense += nd;
        gather_rows<T, VEC, NV, U, ANY>(addr, w, nd, width, lane, p.lpr_log2, acc);
        if constexpr (SPARSE) {
            if (ns > 0) {
                if (!any_sparse) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // the rows are cleared
                any_sparse = true;
                if constexpr (MODE == kOwner)
                    owner_phase<T, EV>(p, lane, nd, ns, zoff, w, unit | shift, lds);
                else
                    sparse_phase<T, EV, Z32, POW2, REM>(p, lane, nd, ns, zoff, w, (unit | shift) << (POW2 ? 2 : 0), reinterpret_cast<char*>(lds));
            }
        }
    }

    sum_groups<VEC, NV>(p.lpr_log2, dense, acc);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (NV == 0 && lane >= (1 << p.lpr_log2)) return;
#pragma unroll
    for (int m = 0; m < NR; ++m) {
        if (VEC * (lane + 64 * m) < width) {
            const int c = row_column<VEC, ANY>(VEC * (lane + 64 * m), width);
            if (SPARSE && any_sparse)
                for (int sub = 0; sub < p.epi; ++sub) add_floats<VEC, ANY>(lds + sub * width + c, acc[m]);
            if (it.dst < 0)
                Packed<T, VEC>::template put<ANY>(p.out + int64_t(it.row - p.row_base) * width + c, acc[m]);
            else
                put_floats<VEC, ANY>(p.partial + int64_t(it.dst) * width + c, acc[m]);
        }
    }
}

template <typename T, int VEC, int NV, int MODE, int EV = 1, bool POW2 = false, bool ANY = false, bool REM = false>
__global__ __launch_bounds__(agg_block(MODE), MODE >= kSparse && VEC * NV <= 8 ? kHaloWaves : 1) void spmm_kernel(SpmmArgs<T> p) {
    spmm_rows<T, VEC, NV, MODE, EV, POW2, ANY, REM>(p);
}
// kOwner, then the messages, then weight copies, a workgroup of which is four here. Bound by the launch, 3 us of a small step for the
// copies alone: forward passes with / without a launch of theirs, us, 2,000 nodes 16-32-8 21.8 / 19.7, 16,000 nodes 32-64-8 42.4 / 39.9,
// 40,000 nodes of 6 neighbours 64-128-24 89.3 / 87.1.
template <typename T, int NV, int EV>
__global__ __launch_bounds__(64, kHaloWaves) void spmm_owner_kernel(SpmmArgs<T> p, PrepJobs<kFewPrepJobs> copies) {
    const int32_t block = int32_t(blockIdx.x), lane = int32_t(threadIdx.x);
    if (block < p.copy_block)
        spmm_rows<T, 4, NV, kOwner, EV, false, false, false>(p);
    else if (block < p.prep_block)
        owner_messages(p, uint32_t(block - p.copy_block), lane);
    else
        prep_weights(copies, (block - p.prep_block) >> 2, ((block - p.prep_block) & 3) * 64 + lane);
}

// Dense-only blocks whose rows are very short (the transposed local block of a finely partitioned graph has
// one or two entries per row): a wavefront per row would leave the device waiting on each wavefront's chain of
// dependent loads (row extent -> entry records -> source row), with nothing else in flight in that wavefront.
// Here a wavefront takes four consecutive rows and walks them in step: the extents, then the entry records,
// then the i-th source row of all four are each fetched by loads issued together. Rows longer than `max_len`
// are left to spmm_kernel (whose work list then holds only those).
template <typename T>
struct ShortRowArgs {
    const int32_t* rowptr;    // CSR row pointer of the block's matrix (absolute entry offsets)
    const int32_t* colidx;
    const float* vals;
    const T* dense;
    T* out;
    int32_t r0, n_rows;       // rows r0 .. r0 + n_rows - 1
    int32_t row_base;         // out row = row - row_base
    int32_t max_len;          // at most 64
    int32_t width;
};

template <typename T, int VEC, int NV>
__global__ __launch_bounds__(kBlock) void spmm_short_rows_kernel(ShortRowArgs<T> p) {
    using V = typename Vec<VEC>::type;
    constexpr int R = 4;
    const int lane = threadIdx.x & 63;
    const int32_t first = p.r0 + (blockIdx.x * kWaves + (threadIdx.x >> 6)) * R;
    const int32_t n_here = min(R, p.r0 + p.n_rows - first);
    if (n_here <= 0) return;           // wavefronts are independent: no barrier below

    const int32_t ptr = lane <= n_here ? p.rowptr[first + lane] : 0;
    int32_t e0[R], len[R];
    bool mine[R];
    int32_t longest = 0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        e0[q] = __shfl(ptr, q);
        const int32_t l = __shfl(ptr, q + 1) - e0[q];
        mine[q] = q < n_here && l <= p.max_len;
        len[q] = mine[q] ? l : 0;
        longest = max(longest, len[q]);
    }
    int32_t col[R];
    float wt[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {      // lane j holds entry j of every row
        const bool has = lane < len[q];
        col[q] = has ? p.colidx[e0[q] + lane] : 0;
        wt[q] = has ? p.vals[e0[q] + lane] : 0.f;
    }
    V acc[R][NV];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int m = 0; m < NV; ++m) zero_vec(acc[q][m]);
    for (int32_t i = 0; i < longest; ++i) {
        V v[R][NV];
        float wi[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const bool on = i < len[q];
            const int32_t r = __shfl(col[q], i);
            wi[q] = on ? __shfl(wt[q], i) : 0.f;
            const T* src = p.dense + int64_t(r) * p.width;
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                const int c = VEC * (lane + 64 * m);
                zero_vec(v[q][m]);
                if (on && c < p.width) v[q][m] = load_vec<T, VEC>(src + c);
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int m = 0; m < NV; ++m) fma_vec(acc[q][m], wi[q], v[q][m]);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (!mine[q]) continue;
        T* dst = p.out + int64_t(first + q - p.row_base) * p.width;
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            const int c = VEC * (lane + 64 * m);
            if (c < p.width) store_vec<T, VEC>(dst + c, acc[q][m]);
        }
    }
}

// out[row] = sum of the partial rows of a split row, in slot order (fixed order: reproducible bits).
template <typename T>
__global__ __launch_bounds__(kBlock) void spmm_fixup_kernel(const SpmmSplit* splits, int32_t n_splits,
                                                            const float* partial, T* out, int32_t row_base,
                                                            int32_t width) {
    const int32_t s = blockIdx.x;
    if (s >= n_splits) return;
    const SpmmSplit sp = splits[s];
    for (int c = threadIdx.x; c < width; c += kBlock) {
        const float* src = partial + int64_t(sp.first) * width + c;
        float acc = 0.f;
        int i = 0;
        for (; i + 8 <= sp.count; i += 8) {      // eight loads in flight; the additions keep slot order
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[int64_t(i + u) * width];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
        for (; i < sp.count; ++i) acc += src[int64_t(i) * width];
        Elem<T>::store(out + int64_t(sp.row - row_base) * width + c, acc);
    }
}

// The same for rows whose width is a multiple of 4: a launch ends with its longest split row (a hub's hundreds of
// partial rows, one dependent chain per thread above), so here the four wavefronts of the workgroup each sum a
// contiguous quarter of the slots, 4 columns per lane and 8 loads in flight, and the quarters are added in wavefront
// order: a fixed order as well, with a chain a quarter as long.
template <typename T>
__global__ __launch_bounds__(kBlock) void spmm_fixup4_kernel(const SpmmSplit* splits, int32_t n_splits,
                                                             const float* partial, T* out, int32_t row_base,
                                                             int32_t width) {
    __shared__ float4 part[kWaves][64];
    const int32_t s = blockIdx.x;
    if (s >= n_splits) return;          // whole workgroup
    const SpmmSplit sp = splits[s];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t per = (sp.count + kWaves - 1) / kWaves;
    const int32_t i0 = min(wave * per, sp.count), i1 = min(i0 + per, sp.count);
    for (int32_t c0 = 0; c0 < width; c0 += 256) {
        const int32_t c = c0 + 4 * lane;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c < width) {
            const float* src = partial + int64_t(sp.first) * width + c;
            int32_t i = i0;
            for (; i + 8 <= i1; i += 8) {
                float4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(src + int64_t(i + u) * width);
#pragma unroll
                for (int u = 0; u < 8; ++u) add_vec(acc, v[u]);
            }
            for (; i < i1; ++i) add_vec(acc, *reinterpret_cast<const float4*>(src + int64_t(i) * width));
        }
        part[wave][lane] = acc;
        __syncthreads();
        if (wave == 0 && c < width) {
            float4 x = part[0][lane];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) add_vec(x, part[w][lane]);
            store_vec<T, 4>(out + int64_t(sp.row - row_base) * width + c, x);
        }
        __syncthreads();                // the next column group reuses the block
    }
}

// ---------------------------------------------------------------------------------------------------------
// Transposed aggregation for halo rows, produced directly in compressed form:
//     dz_halo[s, j] = sum over local rows i of S[i, halo s] * dM[i, pi_v(j)],  j < k,  v = node of slot s.
// Gathering the k scattered columns of every dM row an entry refers to would pull whole cache lines for
// 4 useful bytes each, once per entry. Instead the work is done in two streaming passes:
//   1. row order: a wavefront stages dM[i, :] in LDS once, and for each halo entry of row i writes the k
//      products w * dM[i, pi_v(j)] as one contiguous row of a product buffer (elements of the storage type),
//      at the entry's position in the transposed order (prow, derived once at registration);
//   2. transposed order: the products of one halo slot are now consecutive rows; they are summed in entry
//      order (fixed order: reproducible bits) into dz_halo.
// ---------------------------------------------------------------------------------------------------------
template <typename T>
struct ProductArgs {
    const SpmmItem* items;      // work list of the forward row block
    int32_t n_items;
    const VarcoEdge* edge;
    const float* vals;
    const int32_t* prow;        // per entry: row of the product buffer (halo entries only)
    const T* dm;                // n_local x width
    MaskRule rule;
    T* prod;                    // (halo entries) x pitch, in the storage type
    int32_t pitch;              // elements per row: k, or k rounded up to whole 16-byte or 64-byte pieces (see varco_product_pitch)
    int32_t ku;                 // stores per entry = k / (elements per store)
    int32_t lpe_log2;           // lanes per entry
};

// EV elements per lane and store (16 bytes where k and the alignment allow it: with 8 bf16 values per lane a 128-element
// message takes 16 lanes, and what is done once per lane and entry - fetching its record from another lane, the store
// address, the first position - is shared by twice as many elements as with 4; this pass issues vector instructions all
// the time, so their number is its time). Positions are kept as byte offsets into the LDS row; they wrap with a mask for
// power-of-two widths and with one unsigned minimum otherwise (q - width is huge when q < width).
// SWZ: lanes of one entry step by EV positions, which meet in few LDS banks; position bits 6-8 folded into bits 0-2 of the
// address (the same map as when the row was staged) spread them.
constexpr uint32_t swizzled(uint32_t q_bytes) { return q_bytes ^ ((q_bytes >> 6) & 0x1Cu); }

// The product rows are read back by another kernel, long after they have left the caches: streaming stores.
template <typename T, int EV>
__device__ __forceinline__ void store_products(T* row, const float (&x)[EV]) {
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    typedef uint32_t words2 __attribute__((ext_vector_type(2)));
    auto* const dst = (__attribute__((address_space(1))) T*)row;
    constexpr int N = EV * int(sizeof(T)) / 4;
    uint32_t u[N > 0 ? N : 1];
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < EV; ++i) u[i] = __float_as_uint(x[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) u[i] = bf16_pair(x[2 * i], x[2 * i + 1]);
    }
    if constexpr (N == 4)
        __builtin_nontemporal_store(words4{u[0], u[1], u[2], u[3]}, (__attribute__((address_space(1))) words4*)dst);
    else if constexpr (N == 2)
        __builtin_nontemporal_store(words2{u[0], u[1]}, (__attribute__((address_space(1))) words2*)dst);
    else if constexpr (N == 1)
        __builtin_nontemporal_store(u[0], (__attribute__((address_space(1))) uint32_t*)dst);
    else
        Elem<T>::store(row, x[0]);
}

// `row`: LDS byte address of the wavefront's row of dM; dst: every entry's row of the product buffer (its lane's).
template <typename T, int EV, bool POW2, bool SWZ>
__device__ __forceinline__ void product_phase(const ProductArgs<T>& p, int lane, int first, int ns, uint64_t dst, float w,
                                              uint32_t mab, uint32_t row) {
    using lds_float = __attribute__((address_space(3))) float;
    const uint32_t width = p.rule.width, row_bytes = width * 4u;
    const int epi = 64 >> p.lpe_log2;
    const int sub = lane >> p.lpe_log2;
    const int jl = lane & ((1 << p.lpe_log2) - 1);
    for (int j0 = 0; j0 < p.ku; j0 += 64) {
        const int ju = j0 + jl;
        const bool j_ok = ju < p.ku;
        const int j = ju * EV;
        for (int r0 = 0; r0 < ns; r0 += epi) {
            const int at = 4 * (first + r0 + sub);
            const uint64_t to = (uint64_t(lane_value(uint32_t(dst >> 32), at)) << 32) | lane_value(uint32_t(dst), at);
            const float wi = __uint_as_float(lane_value(__float_as_uint(w), at));
            const uint32_t ab = lane_value(mab, at);
            if (j_ok && r0 + sub < ns) {
                const uint32_t a = ab & 0xFFFFu, a4 = a * 4u;
                uint32_t q = __umul24(a, uint32_t(j)) + (ab >> 16);
                q = (POW2 ? q & (width - 1u) : varco_mod_width(q, width, p.rule.width_magic)) * 4u;
                float out[EV];
#pragma unroll
                for (int i = 0; i < EV; ++i) {
                    out[i] = wi * *(const lds_float*)(uintptr_t((SWZ ? swizzled(q) : q) + row));
                    q += a4;
                    q = POW2 ? q & (row_bytes - 1u) : min(q, q - row_bytes);
                }
                store_products<T, EV>(reinterpret_cast<T*>(to) + j, out);
            }
        }
    }
}

// A wavefront takes kProductItems consecutive items of the work list. Its time per item is a chain - records of the entries
// and the row of dM, the hash, LDS, the stores - so the next item's records and row are requested before the current item's
// products are formed: on a graph with 10 halo entries per row an item is 1.3 KB of stores, far too little to cover that
// chain by resident wavefronts alone. ROWV: 4-element loads per lane that hold a row of dM in registers ahead of its turn
// (width <= 256 ROWV, rows aligned to 4 elements); 0: the row is copied to LDS when its turn comes.
constexpr int kProductItems = 4;
template <typename T, int EV, bool POW2, bool SWZ, int ROWV>
__global__ __launch_bounds__(kBlock) void halo_products_kernel(ProductArgs<T> p) {
    extern __shared__ float lds[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int32_t width = int32_t(p.rule.width);
    float* lrow = lds + wave * width;
    const uint32_t lrow_at = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)lrow));
    uint16_t* lunits = reinterpret_cast<uint16_t*>(lds + kWaves * width);
    int32_t idx = (blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(wave)) * kProductItems;   // uniform: items sit in scalar registers
    const int32_t end = min(idx + kProductItems, p.n_items);
    auto item_at = [&](int32_t i) {
        SpmmItem it{};                  // empty range past the end
        if (i < end) it = p.items[i];
        return it;
    };
    // The records of a batch (entry, weight, product row) are loaded together and for every entry, halo or
    // not, so that one memory round trip serves all three.
    VarcoEdge ed{0, -1};
    float w = 0.f;
    int32_t pr = 0;
    auto load_batch = [&](const SpmmItem& it, int32_t base) {
        const int32_t e = base + lane;
        ed = VarcoEdge{0, -1}, w = 0.f, pr = 0;
        if (e < it.e1) ed = p.edge[e], w = p.vals[e], pr = p.prow[e];
    };
    using R = typename Stored<T, 4>::type;
    R ahead[ROWV > 0 ? ROWV : 1];
    auto load_row = [&](const SpmmItem& it) {
        if constexpr (ROWV > 0) {
            const T* src = p.dm + int64_t(it.row) * width;
#pragma unroll
            for (int m = 0; m < ROWV; ++m) {
                const int c = 4 * (lane + 64 * m);
                ahead[m] = R{};
                if (it.e0 < it.e1 && c < width) ahead[m] = *reinterpret_cast<const R*>(src + c);
            }
        }
    };
    auto stash_row = [&](const SpmmItem& it) {
        if constexpr (ROWV > 0) {
#pragma unroll
            for (int m = 0; m < ROWV; ++m) {
                const int c = 4 * (lane + 64 * m);
                if (c < width) {
                    float4 x = make_float4(Stored<T, 4>::get(ahead[m], 0), Stored<T, 4>::get(ahead[m], 1), Stored<T, 4>::get(ahead[m], 2),
                                           Stored<T, 4>::get(ahead[m], 3));
                    if constexpr (SWZ) {    // position i of the group of four goes to i ^ (s & 3) of the group with index bit 2 flipped by s & 4
                        const int s = (c >> 6) & 7;
                        const float e[4] = {x.x, x.y, x.z, x.w};
                        x = make_float4(e[s & 3], e[1 ^ (s & 3)], e[2 ^ (s & 3)], e[3 ^ (s & 3)]);
                        *reinterpret_cast<float4*>(lrow + (c ^ (s & 4))) = x;
                    } else {
                        *reinterpret_cast<float4*>(lrow + c) = x;
                    }
                }
            }
        } else if (it.e0 < it.e1) {
            const T* src = p.dm + int64_t(it.row) * width;
            for (int c = lane; c < width; c += 64) lrow[SWZ ? swizzled(4u * c) / 4u : uint32_t(c)] = Elem<T>::load(src + c);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };

    SpmmItem it = item_at(idx);
    load_batch(it, it.e0);
    load_row(it);
    for (uint32_t i = threadIdx.x; i < p.rule.n_units; i += kBlock) lunits[i] = p.rule.units[i];
    __syncthreads();                    // no block-wide barrier below
    for (; idx < end; ++idx) {
        stash_row(it);
        const SpmmItem nx = item_at(idx + 1);
        load_row(nx);
        if (it.e0 >= it.e1) load_batch(nx, nx.e0);
        for (int32_t base = it.e0; base < it.e1; base += 64) {
            const bool is_halo = ed.gid >= 0;
            const uint64_t hmask = __ballot(is_halo);
            uint32_t mab = 0;
            if (is_halo) {
                const uint32_t h1 = varco_mix32(uint32_t(ed.gid) ^ varco_key0(p.rule));
                const uint32_t h2 = varco_mix32(h1 ^ varco_key1(p.rule));
                mab = uint32_t(lunits[__umulhi(h2, p.rule.n_units)]) | (__umulhi(h1, p.rule.width) << 16);
            }
            const int cnt = min(64, it.e1 - base);
            const int ns = __popcll(hmask);
            const int first = cnt - ns;     // columns ascend within a row: halo entries sit in the last lanes
            const float wb = w;
            const uint64_t dst = reinterpret_cast<uint64_t>(p.prod + int64_t(pr) * p.pitch);
            if (base + 64 < it.e1)
                load_batch(it, base + 64);
            else
                load_batch(nx, nx.e0);
            if (ns > 0) product_phase<T, EV, POW2, SWZ>(p, lane, first, ns, dst, wb, mab, lrow_at);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // the row has been read: the next one may overwrite it
        it = nx;
    }
}

template <typename T>
struct SegsumArgs {
    const SpmmItem* items;      // work list of the transposed halo rows (entry ranges in transposed order)
    int32_t n_items;
    const T* prod;
    int32_t prod_base;          // transposed position of the first halo entry (= product row 0)
    int32_t k;
    T* out;
    int32_t row_base;
    float* partial;
    int32_t ev, ku, lpe_log2;
};

template <typename T, int EV>
__device__ __forceinline__ void segsum_body(const SegsumArgs<T>& p, const SpmmItem& it, int jl, int lpe) {
    using V = typename Vec<EV>::type;
    for (int ju = jl; ju < p.ku; ju += lpe) {
        const T* src = p.prod + int64_t(it.e0 - p.prod_base) * p.k + ju * EV;
        V acc;
        zero_vec(acc);
        int32_t n = it.e1 - it.e0;
        for (; n >= 4; n -= 4) {
            const V v0 = load_vec<T, EV>(src), v1 = load_vec<T, EV>(src + p.k);
            const V v2 = load_vec<T, EV>(src + 2 * int64_t(p.k));
            const V v3 = load_vec<T, EV>(src + 3 * int64_t(p.k));
            add_vec(acc, v0), add_vec(acc, v1), add_vec(acc, v2), add_vec(acc, v3);
            src += 4 * int64_t(p.k);
        }
        if (n > 0) {   // up to three rows left: fetched together (rows past the end re-read the first), added in order
            const V v0 = load_vec<T, EV>(src), v1 = load_vec<T, EV>(src + (n > 1 ? p.k : 0));
            const V v2 = load_vec<T, EV>(src + (n > 2 ? 2 * int64_t(p.k) : 0));
            add_vec(acc, v0);
            if (n > 1) add_vec(acc, v1);
            if (n > 2) add_vec(acc, v2);
        }
        if (it.dst < 0)
            store_vec<T, EV>(p.out + int64_t(it.row - p.row_base) * p.k + ju * EV, acc);
        else
            *reinterpret_cast<V*>(p.partial + int64_t(it.dst) * p.k + ju * EV) = acc;
    }
}

// bf16 rows, 8 elements (16 bytes) per lane and load: half as many, twice as wide loads as the 4-element form.
struct Float8 {
    float4 lo, hi;
};
__device__ __forceinline__ Float8 load8(const bf16_t* p) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    Float8 v;
    v.lo = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xFFFF0000u));
    v.hi = make_float4(__uint_as_float(u.z << 16), __uint_as_float(u.z & 0xFFFF0000u), __uint_as_float(u.w << 16),
                       __uint_as_float(u.w & 0xFFFF0000u));
    return v;
}
__device__ __forceinline__ void add8(Float8& a, const Float8& b) {
    add_vec(a.lo, b.lo);
    add_vec(a.hi, b.hi);
}
__device__ __forceinline__ void segsum_body8(const SegsumArgs<bf16_t>& p, const SpmmItem& it, int jl, int lpe) {
    for (int ju = jl; ju < p.ku; ju += lpe) {
        const bf16_t* src = p.prod + int64_t(it.e0 - p.prod_base) * p.k + ju * 8;
        Float8 acc;
        zero_vec(acc.lo), zero_vec(acc.hi);
        int32_t n = it.e1 - it.e0;
        for (; n >= 4; n -= 4) {
            const Float8 v0 = load8(src), v1 = load8(src + p.k), v2 = load8(src + 2 * int64_t(p.k)), v3 = load8(src + 3 * int64_t(p.k));
            add8(acc, v0), add8(acc, v1), add8(acc, v2), add8(acc, v3);
            src += 4 * int64_t(p.k);
        }
        if (n > 0) {   // up to three rows left: fetched together (rows past the end re-read the first), added in order
            const Float8 v0 = load8(src), v1 = load8(src + (n > 1 ? p.k : 0)), v2 = load8(src + (n > 2 ? 2 * int64_t(p.k) : 0));
            add8(acc, v0);
            if (n > 1) add8(acc, v1);
            if (n > 2) add8(acc, v2);
        }
        if (it.dst < 0) {
            bf16_t* dst = p.out + int64_t(it.row - p.row_base) * p.k + ju * 8;
            Elem<bf16_t>::store4(dst, acc.lo);
            Elem<bf16_t>::store4(dst + 4, acc.hi);
        } else {
            float* dst = p.partial + int64_t(it.dst) * p.k + ju * 8;
            *reinterpret_cast<float4*>(dst) = acc.lo;
            *reinterpret_cast<float4*>(dst + 4) = acc.hi;
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void halo_segsum_kernel(SegsumArgs<T> p) {
    const int lpe = 1 << p.lpe_log2;
    const int64_t gidx = (int64_t(blockIdx.x) * kBlock + threadIdx.x) >> p.lpe_log2;
    if (gidx >= p.n_items) return;
    const SpmmItem it = p.items[gidx];
    const int jl = threadIdx.x & (lpe - 1);
    if constexpr (std::is_same_v<T, bf16_t>) {
        if (p.ev == 8) {
            segsum_body8(p, it, jl, lpe);
            return;
        }
    }
    if (p.ev == 4)
        segsum_body<T, 4>(p, it, jl, lpe);
    else if (p.ev == 2)
        segsum_body<T, 2>(p, it, jl, lpe);
    else
        segsum_body<T, 1>(p, it, jl, lpe);
}

// prow[e] of a halo entry e = (local row i, halo column c): its position among the halo entries in the
// transposed order, found by searching i in the ascending row list of transposed row c. One thread per row.
__global__ __launch_bounds__(kBlock) void build_prow_kernel(const int32_t* rowptr, const int32_t* colidx, int32_t n_local,
                                                            const int32_t* t_rowptr, const int32_t* t_colidx,
                                                            int32_t* prow) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_local) return;
    const int32_t base = t_rowptr[n_local];
    for (int32_t e = rowptr[i]; e < rowptr[i + 1]; ++e) {
        const int32_t c = colidx[e];
        int32_t pos = -1;
        if (c >= n_local) {
            int32_t lo = t_rowptr[c], hi = t_rowptr[c + 1] - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi) >> 1;
                if (t_colidx[mid] < i) lo = mid + 1; else hi = mid;
            }
            pos = lo - base;
        }
        prow[e] = pos;
    }
}

// Per-entry records of a partition's row block: local column -> {row, -1}; halo column -> {row of the
// node in the concatenated compressed buffer, node id}.
__global__ __launch_bounds__(kBlock) void build_edges_kernel(const int32_t* colidx, int64_t nnz, int32_t n_local,
                                                             const int32_t* halo_zrow, const int32_t* halo_gid,
                                                             VarcoEdge* edge) {
    const int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (e >= nnz) return;
    const int32_t c = colidx[e];
    VarcoEdge ed;
    if (c < n_local) {
        ed.src = c, ed.gid = -1;
    } else {
        ed.src = halo_zrow[c - n_local], ed.gid = halo_gid[c - n_local];
    }
    edge[e] = ed;
}

// Checks of a partition's index arrays at registration, so that no later kernel can be led out of bounds or to
// silently wrong sums by a malformed descriptor. Every failed check sets a bit of *flags.
//   rows:  columns of each row strictly ascending and inside [0, n_local + n_halo)
//   trows: row indices of each transposed row strictly ascending and inside [0, n_local), and every transposed
//          entry (c, i, v) present in forward row i with the same value (with equal entry counts and distinct
//          entries on both sides: the two structures hold the same triplets)
// One thread per (transposed) row; row pointers were checked on the host.
__global__ __launch_bounds__(kBlock) void validate_rows_kernel(const int32_t* rowptr, const int32_t* colidx, int32_t n_local,
                                                               int32_t n_cols, int32_t* flags) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_local) return;
    int32_t prev = -1, bad = 0;
    for (int32_t e = rowptr[i]; e < rowptr[i + 1]; ++e) {
        const int32_t c = colidx[e];
        if (c < 0 || c >= n_cols) bad |= VARCO_BAD_COLUMN_RANGE;
        if (c <= prev) bad |= VARCO_BAD_COLUMN_ORDER;
        prev = c;
    }
    if (bad) atomicOr(flags, bad);
}
__global__ __launch_bounds__(kBlock) void validate_trows_kernel(const int32_t* rowptr, const int32_t* colidx, const float* vals,
                                                                int32_t n_local, int32_t n_cols, const int32_t* t_rowptr,
                                                                const int32_t* t_colidx, const float* t_vals, int32_t* flags) {
    const int32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= n_cols) return;
    int32_t prev = -1, bad = 0;
    for (int32_t pos = t_rowptr[c]; pos < t_rowptr[c + 1]; ++pos) {
        const int32_t i = t_colidx[pos];
        if (i < 0 || i >= n_local) {
            bad |= VARCO_BAD_TROW_RANGE;
            continue;
        }
        if (i <= prev) bad |= VARCO_BAD_TROW_ORDER;
        prev = i;
        int32_t lo = rowptr[i], hi = rowptr[i + 1];     // first entry of row i with column >= c (rows may be unsorted
        while (lo < hi) {                               // if the other kernel flags them: the search stays in bounds)
            const int32_t mid = lo + ((hi - lo) >> 1);
            if (colidx[mid] < c) lo = mid + 1; else hi = mid;
        }
        if (lo >= rowptr[i + 1] || colidx[lo] != c || __float_as_uint(vals[lo]) != __float_as_uint(t_vals[pos]))
            bad |= VARCO_BAD_TRANSPOSE;
    }
    if (bad) atomicOr(flags, bad);
}
// Non-negative ids (a: n values), strictly ascending rows inside [0, limit) when ascending != 0.
__global__ __launch_bounds__(kBlock) void validate_ids_kernel(const int32_t* a, int64_t n, int32_t limit, int ascending,
                                                              int32_t bit, int32_t* flags) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    const int32_t v = a[i];
    bool bad = v < 0 || (limit > 0 && v >= limit);
    if (ascending && i > 0 && a[i - 1] >= v) bad = true;
    if (bad) atomicOr(flags, bit);
}

template <typename T, int VEC, int MODE, int EV, bool POW2, bool ANY, bool REM>
hipError_t launch_spmm_nv(int nv, const SpmmArgs<T>& a, dim3 grid, size_t lds_bytes, hipStream_t stream) {
    auto go = [&](auto n) {
        constexpr int NV = decltype(n)::value;
        hipLaunchKernelGGL((spmm_kernel<T, VEC, NV, MODE, EV, POW2, ANY, REM>), grid, dim3(agg_block(MODE)), lds_bytes, stream, a);
        return hipGetLastError();
    };
    switch (nv) {
        case 0:
            if constexpr (VEC < 8 && !(ANY && sizeof(T) == 4)) return go(std::integral_constant<int, 0>{});
            break;
        case 1:
            if constexpr (VEC > 1 || sizeof(T) == 4 || MODE >= kSparse) return go(std::integral_constant<int, 1>{});
            break;
        case 2:
            if constexpr (VEC >= 4 || (VEC == 1 && sizeof(T) == 2 && MODE >= kSparse)) return go(std::integral_constant<int, 2>{});
            break;
        case 4:
            if constexpr (VEC >= 4 && !ANY) return go(std::integral_constant<int, 4>{});
            break;
        case 8:
            if constexpr (VEC == 4 && !ANY) return go(std::integral_constant<int, 8>{});
    }
    return hipErrorInvalidValue;
}
template <typename T, int VEC, int MODE, bool ANY>
hipError_t launch_spmm_vec(int nv, int ev, bool rem, const SpmmArgs<T>& a, dim3 grid, size_t lds_bytes, hipStream_t stream) {
    if constexpr (MODE < kSparse) {
        return launch_spmm_nv<T, VEC, MODE, 1, false, ANY, false>(nv, a, grid, lds_bytes, stream);
    } else {
        const bool pow2 = (a.rule.width & (a.rule.width - 1)) == 0;
        auto with_ev = [&](auto e) {
            constexpr int EV = decltype(e)::value;
            auto go = [&](auto rm) {
                constexpr bool REM = decltype(rm)::value;
                if constexpr (VEC > 1 && !ANY)
                    if (pow2) return launch_spmm_nv<T, VEC, MODE, EV, true, false, REM>(nv, a, grid, lds_bytes, stream);
                return launch_spmm_nv<T, VEC, MODE, EV, false, ANY, REM>(nv, a, grid, lds_bytes, stream);
            };
            if constexpr (EV > 1 && VEC > 1)
                if (rem) return go(std::true_type{});
            return go(std::false_type{});
        };
        return ev == 4 ? with_ev(std::integral_constant<int, 4>{}) : ev == 2 ? with_ev(std::integral_constant<int, 2>{})
                                                                             : with_ev(std::integral_constant<int, 1>{});
    }
}

bool aligned_to(const void* p, size_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

template <typename T>
hipError_t spmm_t(const SpmmPlan& plan, const VarcoEdge* edge, const int32_t* colidx, const float* vals, const void* dense_v,
                  const void* z_v, int64_t z_rows, const MaskRule& rule, void* out_v, int32_t row_base, float* partial,
                  const SpmmOwners* owners, hipStream_t stream, const LaunchTag& tag) {
    const T* dense = static_cast<const T*>(dense_v);
    const T* z = static_cast<const T*>(z_v);
    T* out = static_cast<T*>(out_v);
    const int32_t width = int32_t(rule.width);
    const bool full = rule.k == rule.width;
    const bool halo = edge != nullptr;
    auto vec_ok = [&](int v) {
        return width % v == 0 && aligned_to(dense, v * sizeof(T)) && aligned_to(out, v * sizeof(T)) && aligned_to(partial, 16) &&
               (!(halo && full) || aligned_to(z, v * sizeof(T)));
    };
    const bool vec4 = vec_ok(4);
    // bf16: 16-byte loads where a row then still takes all lanes. (Narrower rows would have twice as many lane groups, and the
    // forward sums another order.)
    // Compressed messages beside bf16 rows of at most 128 elements that are not aligned: one element to a load, in small launches up to 64. (With four, up
    // to 64 private rows are added up four columns to a lane. One / four, us, 400,003 nodes of 10 neighbours: 5 wide, no messages, 167 / 368, 13 wide, 5 kept,
    // 164 / 244, 63 wide, 8 kept, 164 / 212, 75 wide, 25 kept, 203 / 231, 127 wide, 16 kept, 208 / 231, but 135 wide, 17 kept, 278 / 231, and 20,011 nodes 13
    // wide, 5 kept, 15.0 / 20.8, 63 wide, 8 kept, 18.1 / 19.4, 75 wide, 9 kept, 22.2 / 19.8, 127 wide, 43 kept, 34 / 27. Whole messages, 400,003 nodes: 13
    // wide 130 / 111, 127 wide 252 / 217.)
    const bool narrow = sizeof(T) == 2 && !vec4 && (width < 4 || (halo && !full && (width <= 64 || (width <= 128 && plan.n_items > 65'536))));
    const int vec = sizeof(T) == 2 && width > 256 && vec_ok(8) ? 8 : vec4 ? 4 : narrow ? 1 : sizeof(T) == 2 ? 4 : width <= 64 ? 1 : width <= 128 ? 2 : 4;
    // Rows whose length is no multiple of 4, or whose base is not aligned, are loaded from any address of an element as well. fp32: as many
    // elements to a load as let a row take all lanes with one load (two above 256 elements). One row after the other is added up, so the bits
    // are those of loads of one element. bf16: four, and narrow rows in groups of lanes as aligned ones. One element to a load / this, us: fp32 116,187
    // nodes 147 wide 110 / 78, 265,139 nodes 209 wide, 105 kept, 276 / 218, 771,643 nodes 94 wide 444 / 398, 50,021 nodes 75 wide 49 / 45; bf16 (with the
    // messages below) 35,999 nodes 221 wide 73 / 49, 819,353 nodes 135 wide 524 / 465, 52,727 nodes 121 wide 53 / 44.
    const bool any = !vec4 && vec > 1;
    const int per_row = (width + vec - 1) / vec;   // loads of VEC elements that cover a row
    int lpr_log2 = 0;
    while ((1 << lpr_log2) < per_row && lpr_log2 < 6) ++lpr_log2;
    int nv = lpr_log2 < 6 ? 0 : 1;
    while (nv && nv * 64 < per_row) nv <<= 1;
    if (nv > 8 || (any && nv > 2)) return hipErrorInvalidValue;

    SpmmArgs<T> a{};
    a.items = plan.items;
    a.n_items = plan.n_items;
    a.edge = edge;
    a.colidx = owners ? owners->arow : colidx;
    a.vals = vals;
    a.dense = dense;
    a.z = z;
    a.rule = rule;
    a.out = out;
    a.row_base = row_base;
    a.partial = partial;
    a.lpr_log2 = lpr_log2;
    // Compressed rows: `ev` stored elements per lane and load, lpe = pow2 >= k / ev lanes per row, epi = 64 / lpe
    // rows per instruction, each with a private LDS row. Prefer wide loads, but keep the private rows of
    // a wavefront within 4 KB so that LDS does not limit the number of resident wavefronts.
    const int epi_cap = std::max(1, 1024 / width);
    int ev = 1;
    for (int c : {4, 2}) {
        if (rule.k % c != 0 || !aligned_to(z, c * sizeof(T))) continue;
        int lg = 0;
        while ((1 << lg) < int(rule.k) / c && lg < 6) ++lg;
        if ((64 >> lg) <= epi_cap) {
            ev = c;
            break;
        }
    }
    // Numbers of kept elements that are no multiple of that (or rows at other addresses): two or four per lane only where an entry takes all lanes either
    // way (65 elements and more), so that as many entries share a private row, and the sums are those of an aligned message of that many loads. (With one
    // element per lane such an entry takes two passes, its last elements behind the first of the 64 entries around it: the same sums in another order.)
    // bf16 rows of odd lengths: as above. One per lane / this, us: 50,021 nodes 200 fp32 columns, 67 kept, 107 / 76.
    // (Not taken for aligned bf16 rows of at most 64 kept elements, which would share private rows otherwise.)
    bool rem = false;
    if (halo && !full && !owners && vec > 1) {
        const int k = int(rule.k);
        if (sizeof(T) == 4 || !any) {
            const int wide = k <= 64 ? 1 : k <= 128 ? 2 : 4;
            rem = wide > ev && (ev == 1 || k > 128);
            if (rem) ev = wide;
        } else {
            for (int c : {4, 2}) {
                int lg = 0;
                while ((1 << lg) < (k + c - 1) / c && lg < 6) ++lg;
                if (c <= ev || k < c) break;
                if ((64 >> lg) > epi_cap) continue;
                ev = c, rem = true;
                break;
            }
        }
    }
    a.ku = (int32_t(rule.k) + ev - 1) / ev;
    a.lpe_log2 = 0;
    while ((1 << a.lpe_log2) < a.ku && a.lpe_log2 < 6) ++a.lpe_log2;
    a.epi = std::max(1, std::min(64 >> a.lpe_log2, epi_cap));
    const int agg_waves = agg_block(halo ? kFull : kDenseOnly) / 64;
    const int32_t per_round = 8 * kXcdRun;                                         // see the kernel's XCD mapping
    dim3 grid(((plan.n_items + agg_waves - 1) / agg_waves + per_round - 1) / per_round * per_round);
    PrepJobs<kFewPrepJobs> copies{};
    if (owners) {
        a.brow = owners->brow, a.bgid = owners->bgid;
        a.messages = static_cast<T*>(const_cast<void*>(z_v));
        a.n_messages = uint32_t(z_rows) * rule.k;
        a.copy_block = int32_t(grid.x);
        a.prep_block = a.copy_block + int32_t((a.n_messages + 255) / 256);
        const int64_t blocks = varco_prep_blocks(owners->jobs, owners->n_jobs);
        if (blocks < 0 || owners->n_jobs > kFewPrepJobs) return hipErrorInvalidValue;
        for (int i = 0; i < owners->n_jobs; ++i) copies.job[i] = owners->jobs[i];
        copies.n = owners->n_jobs;
        grid.x = unsigned(a.prep_block + 4 * blocks);
    }
    size_t lds_bytes = 0;
    if (halo && !full)
        lds_bytes = (size_t(a.epi) * width * sizeof(float) + 15) / 16 * 16 + (rem ? 16 : 0);
    tag.begin(stream);
    hipError_t err = hipErrorInvalidValue;
    // compressed buffer below 4 GiB: 32-bit row offsets (z_rows = 0: size unknown)
    const bool z32 = halo && !full && z_rows > 0 && z_rows * int64_t(rule.k) * int64_t(sizeof(T)) < (int64_t(1) << 32);
    auto with_vec = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
        if constexpr (sizeof(T) == 2)
            if (vec == 8) return launch_spmm_vec<T, 8, MODE, false>(nv, ev, rem, a, grid, lds_bytes, stream);
        if constexpr (sizeof(T) == 4)
            if (vec == 2) return launch_spmm_vec<T, 2, MODE, true>(nv, ev, rem, a, grid, lds_bytes, stream);
        if (any) return launch_spmm_vec<T, 4, MODE, true>(nv, ev, rem, a, grid, lds_bytes, stream);
        return vec4 ? launch_spmm_vec<T, 4, MODE, false>(nv, ev, rem, a, grid, lds_bytes, stream) : launch_spmm_vec<T, 1, MODE, false>(nv, ev, rem, a, grid, lds_bytes, stream);
    };
    if (owners) {
        auto with_ev = [&](auto e) {
            constexpr int EV = decltype(e)::value;
            const auto kernel = nv == 0 ? spmm_owner_kernel<T, 0, EV> : spmm_owner_kernel<T, 1, EV>;
            hipLaunchKernelGGL(kernel, grid, dim3(64), lds_bytes, stream, a, copies);
            return hipGetLastError();
        };
        if (vec4 && vec == 4 && nv <= 1 && halo && !full)
            err = ev == 4 ? with_ev(std::integral_constant<int, 4>{}) : ev == 2 ? with_ev(std::integral_constant<int, 2>{}) : with_ev(std::integral_constant<int, 1>{});
    } else if (halo && full)
        err = with_vec(std::integral_constant<int, kFull>{});
    else if (halo && z32)
        err = with_vec(std::integral_constant<int, kSparseZ32>{});
    else if (halo)
        err = with_vec(std::integral_constant<int, kSparse>{});
    else
        err = with_vec(std::integral_constant<int, kDenseOnly>{});
    tag.end(stream);
    if (err != hipSuccess) return err;
    if (plan.n_splits > 0) {
        // the split records, every fp32 partial row once, every split row written once
        tag.begin_as(VARCO_K_REDUCE, stream, 16.0 * plan.n_splits + 4.0 * double(plan.n_partials) * width +
                                                 double(sizeof(T)) * plan.n_splits * width);
        if (vec4)
            hipLaunchKernelGGL(spmm_fixup4_kernel<T>, dim3(plan.n_splits), dim3(kBlock), 0, stream, plan.splits, plan.n_splits,
                               partial, out, row_base, width);
        else
            hipLaunchKernelGGL(spmm_fixup_kernel<T>, dim3(plan.n_splits), dim3(kBlock), 0, stream, plan.splits, plan.n_splits,
                               partial, out, row_base, width);
        tag.end(stream);
        err = hipGetLastError();
    }
    return err;
}

// The short rows of a dense-only block (see spmm_short_rows_kernel); the block's other rows are on plan.items.
template <typename T>
hipError_t spmm_short_t(const SpmmPlan& plan, const int32_t* colidx, const float* vals, const void* dense_v, void* out_v,
                        int32_t width, int32_t row_base, hipStream_t stream, const LaunchTag& tag) {
    ShortRowArgs<T> a;
    a.rowptr = plan.short_rowptr;
    a.colidx = colidx;
    a.vals = vals;
    a.dense = static_cast<const T*>(dense_v);
    a.out = static_cast<T*>(out_v);
    a.r0 = plan.short_r0, a.n_rows = plan.short_rows, a.row_base = row_base;
    a.max_len = plan.short_max_len;
    a.width = width;
    const bool vec4 = width % 4 == 0 && aligned_to(a.dense, 4 * sizeof(T)) && aligned_to(a.out, 4 * sizeof(T));
    const int per_row = vec4 ? width / 4 : width;
    int nv = 1;
    while (nv * 64 < per_row) nv <<= 1;
    if (nv > 8) return hipErrorInvalidValue;
    const int32_t n_waves = (plan.short_rows + 3) / 4;
    const dim3 grid((n_waves + kWaves - 1) / kWaves), block(kBlock);
    tag.begin(stream);
    auto go = [&](auto vec, auto nvc) {
        hipLaunchKernelGGL((spmm_short_rows_kernel<T, decltype(vec)::value, decltype(nvc)::value>), grid, block, 0, stream, a);
    };
    auto with_nv = [&](auto vec) {
        switch (nv) {
            case 1: go(vec, std::integral_constant<int, 1>{}); break;
            case 2: go(vec, std::integral_constant<int, 2>{}); break;
            case 4: go(vec, std::integral_constant<int, 4>{}); break;
            default: go(vec, std::integral_constant<int, 8>{}); break;
        }
    };
    if (vec4)
        with_nv(std::integral_constant<int, 4>{});
    else
        with_nv(std::integral_constant<int, 1>{});
    tag.end(stream);
    return hipGetLastError();
}

// First pass: see halo_products_kernel.
template <typename T>
hipError_t halo_products_t(const SpmmPlan& fwd_plan, const VarcoEdge* edge, const float* vals, const int32_t* prow, const void* dm,
                           const MaskRule& rule, void* prod_v, int32_t pitch, hipStream_t stream, const LaunchTag& tag) {
    T* prod = static_cast<T*>(prod_v);
    const int32_t width = int32_t(rule.width);
    int ev = 1;
    for (int c : {int(16 / sizeof(T)), 4, 2})
        if (pitch % c == 0 && aligned_to(prod, c * sizeof(T))) {
            ev = c;
            break;
        }
    ProductArgs<T> a;
    a.items = fwd_plan.items;
    a.n_items = fwd_plan.n_items;
    a.edge = edge;
    a.vals = vals;
    a.prow = prow;
    a.dm = static_cast<const T*>(dm);
    a.rule = rule;
    a.prod = prod;
    a.pitch = pitch;
    a.ku = pitch / ev, a.lpe_log2 = 0;      // elements beyond k are products as well, and are not read
    while ((1 << a.lpe_log2) < a.ku && a.lpe_log2 < 6) ++a.lpe_log2;
    const size_t lds_bytes = size_t(kWaves) * width * sizeof(float) + size_t(rule.n_units) * sizeof(uint16_t);
    const bool pow2 = (width & (width - 1)) == 0;
    const dim3 grid((fwd_plan.n_items + kWaves * kProductItems - 1) / (kWaves * kProductItems));
    const int rowv = width % 4 != 0 || !aligned_to(dm, 4 * sizeof(T)) || width > 512 ? 0 : width > 256 ? 2 : 1;
    auto go = [&](auto evc, auto p2, auto swz) {
        constexpr int EV = decltype(evc)::value;
        constexpr bool P2 = decltype(p2)::value, SW = decltype(swz)::value;
        if (rowv == 1)
            hipLaunchKernelGGL((halo_products_kernel<T, EV, P2, SW, 1>), grid, dim3(kBlock), lds_bytes, stream, a);
        else if (rowv == 2)
            hipLaunchKernelGGL((halo_products_kernel<T, EV, P2, SW, 2>), grid, dim3(kBlock), lds_bytes, stream, a);
        else
            hipLaunchKernelGGL((halo_products_kernel<T, EV, P2, SW, 0>), grid, dim3(kBlock), lds_bytes, stream, a);
    };
    auto with_wrap = [&](auto evc) {
        constexpr bool kSwz = (decltype(evc)::value >= 8);
        if (pow2 && kSwz && width >= 512)
            go(evc, std::true_type{}, std::integral_constant<bool, kSwz>{});
        else if (pow2)
            go(evc, std::true_type{}, std::false_type{});
        else
            go(evc, std::false_type{}, std::false_type{});
    };
    tag.begin(stream);
    if constexpr (sizeof(T) == 2)
        if (ev == 8) with_wrap(std::integral_constant<int, 8>{});
    if (ev == 4)
        with_wrap(std::integral_constant<int, 4>{});
    else if (ev == 2)
        with_wrap(std::integral_constant<int, 2>{});
    else if (ev == 1)
        with_wrap(std::integral_constant<int, 1>{});
    tag.end(stream);
    return hipGetLastError();
}

template <typename T>
hipError_t halo_grad_t(const SpmmPlan& fwd_plan, const SpmmPlan& t_halo_plan, const VarcoEdge* edge, const float* vals,
                       const int32_t* prow, int32_t prod_base, const void* dm, const MaskRule& rule, void* prod_v,
                       void* out_v, int32_t row_base, float* partial, hipStream_t stream, const LaunchTag& tag,
                       const LaunchTag& sum_tag) {
    hipError_t err = halo_products_t<T>(fwd_plan, edge, vals, prow, dm, rule, prod_v, int32_t(rule.k), stream, tag);
    if (err != hipSuccess) return err;
    T* out = static_cast<T*>(out_v);
    T* prod = static_cast<T*>(prod_v);
    int ev = 1;
    for (int c : {4, 2})
        if (rule.k % c == 0 && aligned_to(prod, c * sizeof(T)) && aligned_to(out, c * sizeof(T)) && aligned_to(partial, 4 * c)) {
            ev = c;
            break;
        }
    const int ku = int(rule.k) / ev;
    int lpe_log2 = 0;
    while ((1 << lpe_log2) < ku && lpe_log2 < 6) ++lpe_log2;
    SegsumArgs<T> b;
    b.items = t_halo_plan.items;
    b.n_items = t_halo_plan.n_items;
    b.prod = prod;
    b.prod_base = prod_base;
    b.k = int32_t(rule.k);
    b.out = out;
    b.row_base = row_base;
    b.partial = partial;
    b.ev = ev, b.ku = ku, b.lpe_log2 = lpe_log2;
    if (std::is_same_v<T, bf16_t> && rule.k % 8 == 0 && aligned_to(prod, 16) && aligned_to(out, 16) && aligned_to(partial, 16)) {
        b.ev = 8, b.ku = int(rule.k) / 8;      // the sums read 16 bytes per lane (as the products above are written)
        b.lpe_log2 = 0;
        while ((1 << b.lpe_log2) < b.ku && b.lpe_log2 < 6) ++b.lpe_log2;
    }
    const int64_t threads = int64_t(t_halo_plan.n_items) << b.lpe_log2;
    sum_tag.begin(stream);
    hipLaunchKernelGGL(halo_segsum_kernel<T>, dim3(unsigned((threads + kBlock - 1) / kBlock)), dim3(kBlock), 0, stream, b);
    sum_tag.end(stream);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    if (t_halo_plan.n_splits > 0) {
        tag.begin_as(VARCO_K_REDUCE, stream, 16.0 * t_halo_plan.n_splits + 4.0 * double(t_halo_plan.n_partials) * rule.k +
                                                 double(sizeof(T)) * t_halo_plan.n_splits * rule.k);
        if (ev == 4)
            hipLaunchKernelGGL(spmm_fixup4_kernel<T>, dim3(t_halo_plan.n_splits), dim3(kBlock), 0, stream, t_halo_plan.splits,
                               t_halo_plan.n_splits, partial, out, row_base, int32_t(rule.k));
        else
            hipLaunchKernelGGL(spmm_fixup_kernel<T>, dim3(t_halo_plan.n_splits), dim3(kBlock), 0, stream, t_halo_plan.splits,
                               t_halo_plan.n_splits, partial, out, row_base, int32_t(rule.k));
        tag.end(stream);
        err = hipGetLastError();
    }
    return err;
}

}  // namespace

hipError_t varco_launch_build_edges(const int32_t* colidx, int64_t nnz, int32_t n_local, const int32_t* halo_zrow,
                                    const int32_t* halo_gid, VarcoEdge* edge, hipStream_t stream) {
    if (nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(build_edges_kernel, dim3(unsigned((nnz + kBlock - 1) / kBlock)), dim3(kBlock), 0, stream, colidx,
                       nnz, n_local, halo_zrow, halo_gid, edge);
    return hipGetLastError();
}

hipError_t varco_launch_validate_partition(const varco_partition_desc& d, int32_t* flags, hipStream_t stream) {
    const int32_t n_cols = d.n_local + d.n_halo;
    auto blocks = [](int64_t n) { return dim3(unsigned((n + kBlock - 1) / kBlock)); };
    if (d.n_local > 0 && d.nnz > 0)
        hipLaunchKernelGGL(validate_rows_kernel, blocks(d.n_local), dim3(kBlock), 0, stream, d.rowptr, d.colidx, d.n_local,
                           n_cols, flags);
    if (n_cols > 0 && d.nnz > 0)
        hipLaunchKernelGGL(validate_trows_kernel, blocks(n_cols), dim3(kBlock), 0, stream, d.rowptr, d.colidx, d.vals,
                           d.n_local, n_cols, d.t_rowptr, d.t_colidx, d.t_vals, flags);
    struct Ids { const int32_t* a; int64_t n; int32_t limit; int ascending; int32_t bit; };
    const Ids lists[] = {{d.local_gid, d.n_local, 0, 0, VARCO_BAD_ID}, {d.halo_gid, d.n_halo, 0, 0, VARCO_BAD_ID},
                         {d.halo_zrow, d.n_halo, 0, 0, VARCO_BAD_ID}, {d.halo_src_row, d.n_halo, 0, 0, VARCO_BAD_ID},
                         {d.boundary_rows, d.n_boundary, d.n_local, 1, VARCO_BAD_BOUNDARY},
                         {d.ret_src, d.ret_src ? d.n_returned : 0, 0, 0, VARCO_BAD_RETURN_MAP}};
    for (const Ids& l : lists)
        if (l.n > 0 && l.a)
            hipLaunchKernelGGL(validate_ids_kernel, blocks(l.n), dim3(kBlock), 0, stream, l.a, l.n, l.limit, l.ascending, l.bit, flags);
    return hipGetLastError();
}

// The launch saved is worth 2 to 4 us and the reading of x by it. Against it: an entry touches a cache line per kept element, up to the whole row of
// its owner, where the compressed row is a line or two (all cross entries: at most 64 MB here), and where an entry takes all lanes the runs of long rows
// become chains of round trips. Forward pass, messages first / together, us (62 networks of 2,000 to 100,000 nodes: 0.99 to 1.29 of the speed):
//   2,000 nodes 16-32-8, ratio 4 28.1 / 21.8     16,000 nodes 32-64-8, 8 partitions 48.5 / 42.4     100,000 nodes of 6 neighbours 16-32-8 165 / 156
//   2,000 nodes of 30 neighbours 128-256-256-40, ratio 8 96 / 90.5     16,000 of 8, bf16 125 / 115
// beyond the lines: 40,000 nodes of 20 neighbours 128-256-256-40 262 / 363, 64-128-24 103 / 110; 43 and 86 kept elements, 6,000 nodes 86 / 91
bool varco_spmm_owners_pay(int dtype, const SpmmPlan& plan, const MaskRule& rule, int64_t rows, int64_t cross, int64_t boundary, const void* dense,
                           const void* out, const void* partial) {
    const int64_t es = dtype == VARCO_BF16 ? 2 : 4, row = (int64_t(rule.width) * es + 127) / 128;
    if (rule.k == 0 || rule.k >= rule.width || rule.width % 4 != 0 || rule.width > 256 || boundary <= 0 || plan.n_items <= 0) return false;
    if (!aligned_to(dense, 4 * es) || !aligned_to(out, 4 * es) || !aligned_to(partial, 16)) return false;
    if (rows * rule.width * es >= int64_t(1) << 32) return false;          // 32-bit offsets
    const uint32_t loads = rule.k % 4 == 0 ? rule.k / 4 : rule.k % 2 == 0 ? rule.k / 2 : rule.k;       // lanes of an entry
    return rule.k <= 64 && loads <= 32 && cross * std::min<int64_t>(rule.k, row) * 128 <= int64_t(1) << 26;
}

hipError_t varco_launch_spmm(int dtype, const SpmmPlan& plan, const VarcoEdge* edge, const int32_t* colidx,
                             const float* vals, const void* dense, const void* z, int64_t z_rows, const MaskRule& rule,
                             void* out, int32_t row_base, float* partial, hipStream_t stream, const LaunchTag& tag, const SpmmOwners* owners) {
    hipError_t err = hipSuccess;
    if (plan.n_items > 0)
        err = dtype == VARCO_BF16
                  ? spmm_t<bf16_t>(plan, edge, colidx, vals, dense, z, z_rows, rule, out, row_base, partial, owners, stream, tag)
                  : spmm_t<float>(plan, edge, colidx, vals, dense, z, z_rows, rule, out, row_base, partial, owners, stream, tag);
    if (err != hipSuccess || plan.short_rows == 0) return err;
    if (edge) return hipErrorInvalidValue;     // short-row plans are built for dense-only blocks
    LaunchTag rest = tag;                      // the block's bytes are booked once
    if (plan.n_items > 0) rest.bytes = 0, rest.flops = 0;
    return dtype == VARCO_BF16
               ? spmm_short_t<bf16_t>(plan, colidx, vals, dense, out, int32_t(rule.width), row_base, stream, rest)
               : spmm_short_t<float>(plan, colidx, vals, dense, out, int32_t(rule.width), row_base, stream, rest);
}

hipError_t varco_launch_build_prow(const int32_t* rowptr, const int32_t* colidx, int32_t n_local,
                                   const int32_t* t_rowptr, const int32_t* t_colidx, int32_t* prow, hipStream_t stream) {
    if (n_local == 0) return hipSuccess;
    hipLaunchKernelGGL(build_prow_kernel, dim3(unsigned((n_local + kBlock - 1) / kBlock)), dim3(kBlock), 0, stream, rowptr,
                       colidx, n_local, t_rowptr, t_colidx, prow);
    return hipGetLastError();
}

hipError_t varco_launch_halo_products(int dtype, const SpmmPlan& fwd_plan, const VarcoEdge* edge, const float* vals, const int32_t* prow,
                                      const void* dm, const MaskRule& rule, void* prod, int32_t pitch, hipStream_t stream, const LaunchTag& tag) {
    if (fwd_plan.n_items == 0) return hipSuccess;
    return dtype == VARCO_BF16 ? halo_products_t<bf16_t>(fwd_plan, edge, vals, prow, dm, rule, prod, pitch, stream, tag)
                               : halo_products_t<float>(fwd_plan, edge, vals, prow, dm, rule, prod, pitch, stream, tag);
}

hipError_t varco_launch_halo_grad(int dtype, const SpmmPlan& fwd_plan, const SpmmPlan& t_halo_plan, const VarcoEdge* edge,
                                  const float* vals, const int32_t* prow, int32_t prod_base, const void* dm,
                                  const MaskRule& rule, void* prod, void* out, int32_t row_base, float* partial,
                                  hipStream_t stream, const LaunchTag& tag, const LaunchTag& sum_tag) {
    if (t_halo_plan.n_items == 0 || fwd_plan.n_items == 0) return hipSuccess;
    return dtype == VARCO_BF16 ? halo_grad_t<bf16_t>(fwd_plan, t_halo_plan, edge, vals, prow, prod_base, dm, rule, prod, out,
                                                     row_base, partial, stream, tag, sum_tag)
                               : halo_grad_t<float>(fwd_plan, t_halo_plan, edge, vals, prow, prod_base, dm, rule, prod, out,
                                                    row_base, partial, stream, tag, sum_tag);
}
