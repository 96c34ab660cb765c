// Kernels of the calls that serve all partitions of one device at once (varco_network_*).
//
// Backward aggregation by node. One device holds every partition, so the errors that the consumers of a node compute need
// not be summed per consumer, written, read back by the owner and added to the owner's gradient row in a pass of its own:
// node v's gradient row is
//     dX[v, :] = sum over local entries (i, v) of S[i, v] dM[i, :]
//              + its kept positions of the sum over all cross entries (i, v) (rows i of other partitions) of S[i, v] dM[i, :]
// and one wavefront forms it from both kinds of entries and writes it once. The cross entries come in one of two forms:
//   products  the k kept products of every cross entry were written by the row-order pass (halo_products_kernel) at the
//             entry's place in node order, so a node's rows of k values are one contiguous stream: 2 k elements of traffic
//             per entry at the rate of a copy;
//   masked    the whole rows dM[i, :] are gathered and everything outside the kept positions is dropped once, from the
//             sum: width elements of traffic per entry at the rate of a gather, no buffer. The better form when k is more
//             than about a third of the width (a gather moves 7 TB/s on this device, write + read back 4.8 TB/s), and
//             for rows of at most 320 to 768 bytes whatever k is: a product costs its place in memory however short it is
//             (products_pay).
// Against the per-partition calls this saves the per-consumer rows (written and read), one read-modify-write of every
// gradient row and, for the sums over short consumer lists (a few entries per halo row on fine partitions), most of the
// fixed cost per row; all partitions share one launch.
#include <algorithm>
#include <type_traits>

#include "gather_device.h"
#include "mask_device.h"

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kXcdRun = 32;      // consecutive workgroups that one XCD takes, as in the aggregation kernels

template <typename T>
struct NodeArgs {
    const NodeItem* nodes;      // of this launch
    int32_t n_nodes;
    const SpmmItem* pieces;     // taken by the launch's first wavefronts
    int32_t n_pieces;
    const uint2* t_local;
    const uint2* t_cross;
    const T* dm;
    const T* prod;
    MaskRule rule;
    T* out;
    int32_t add_old;
    float* partial;           // one width-float row per piece
    int32_t lpr_log2;         // lanes per dense row = 1 << lpr_log2
    int32_t pitch;            // elements between product rows
    int32_t ku, lpe_log2;     // loads per product row, lanes per product row = 1 << lpe_log2
};

// acc += the rows of dM of entries [e0, e1).
template <typename T, int VEC, int NV>
__device__ __forceinline__ void gather_entries(const NodeArgs<T>& p, const uint2* pairs, int32_t e0, int32_t e1, int lane,
                                               float (&acc)[loads_per_row(NV)][VEC]) {
    constexpr int U = NV >= 4 ? 1 : (NV == 2 ? 2 : 4);
    const int32_t width = int32_t(p.rule.width);
    for (int32_t base = e0; base < e1; base += 64) {
        uint2 mine = make_uint2(0u, 0u);
        if (base + lane < e1) mine = pairs[base + lane];
        const uint64_t addr = reinterpret_cast<uint64_t>(p.dm + int64_t(int32_t(mine.x)) * width);
        gather_rows<T, VEC, NV, U>(addr, __uint_as_float(mine.y), min(64, e1 - base), width, lane, p.lpr_log2, acc);
    }
}

// The same over rows of fp32 partial sums (pieces of a long range), slot order.
template <int VEC, int NV>
__device__ __forceinline__ void add_partials(const float* partial, int32_t width, int32_t s0, int32_t s1, int lane, int lpr_log2,
                                             float (&acc)[loads_per_row(NV)][VEC]) {
    if constexpr (NV > 0) {
        for (int32_t s = s0; s < s1; ++s)
#pragma unroll
            for (int m = 0; m < NV; ++m)
                if (VEC * (lane + 64 * m) < width) add_floats<VEC>(partial + int64_t(s) * width + VEC * (lane + 64 * m), acc[m]);
    } else {
        const int c = VEC * (lane & ((1 << lpr_log2) - 1));
        for (int32_t s = s0 + (lane >> lpr_log2); s < s1; s += 64 >> lpr_log2)
            if (c < width) add_floats<VEC>(partial + int64_t(s) * width + c, acc[0]);
    }
}

template <int VEC, int NR>
__device__ __forceinline__ void clear(float (&acc)[NR][VEC]) {
#pragma unroll
    for (int m = 0; m < NR; ++m)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[m][i] = 0.f;
}

// Sum of the rows [c0, c1) of `src` (pitch `pitch` elements of type S), elements j0 .. j0 + EV - 1 of every row; lane
// groups take different rows, six rows of a group in flight (fewer at the end of the range); the groups' sums are added at the
// end, so that the lanes of the first group (sub = 0) hold the totals, and no others.
template <typename S, int EV>
__device__ __forceinline__ void sum_rows(const S* src, int64_t pitch, int32_t c0, int32_t c1, int j0, bool on, int sub, int n_sub,
                                         int lpe_log2, float (&acc)[EV]) {
    using P = Packed<S, EV>;
#pragma unroll
    for (int i = 0; i < EV; ++i) acc[i] = 0.f;
    const uint32_t mine = (uint32_t(sub) * uint32_t(pitch) + uint32_t(j0)) * uint32_t(sizeof(S));
    auto batch = [&](int32_t r, auto count) {
        constexpr int N = decltype(count)::value;
        typename P::type v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int32_t first = r + u * n_sub;      // uniform: the rows' base is a scalar
            v[u] = typename P::type{};
            if (on && first + sub < c1) v[u] = load_packed<S, EV>(reinterpret_cast<uint64_t>(src + int64_t(first) * pitch), mine);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            float x[EV];
            P::get(v[u], x);
#pragma unroll
            for (int i = 0; i < EV; ++i) acc[i] += x[i];
        }
    };
    int32_t r = c0;
    for (; r + 2 * n_sub < c1; r += 6 * n_sub) batch(r, std::integral_constant<int, 6>{});
    if (r + n_sub < c1)
        batch(r, std::integral_constant<int, 2>{});
    else if (r < c1)
        batch(r, std::integral_constant<int, 1>{});
    add_lanes(acc, lpe_log2, min(c1 - c0, 64) << lpe_log2);
}

// Partial sum of a piece of a long range (hub nodes): a dense row of width floats, or k floats of summed products.
template <typename T, int VEC, int NV, int CROSS, int EV>
__device__ __forceinline__ void node_piece(const NodeArgs<T>& p, const SpmmItem& it, int lane) {
    const int32_t width = int32_t(p.rule.width);
    float* dst = p.partial + int64_t(it.dst) * width;
    if (it.row == 1 && CROSS == kCrossNone) return;
    if (it.row == 1 && CROSS == kCrossProducts) {
        const int sub = lane >> p.lpe_log2, n_sub = 64 >> p.lpe_log2, jl = lane & ((1 << p.lpe_log2) - 1);
        for (int u0 = 0; u0 < p.ku; u0 += 64) {
            const int ju = u0 + jl;
            const bool on = ju < p.ku;
            float s[EV];
            sum_rows<T, EV>(p.prod, p.pitch, it.e0, it.e1, ju * EV, on, sub, n_sub, p.lpe_log2, s);
            if (on && sub == 0)
#pragma unroll
                for (int i = 0; i < EV; ++i) dst[ju * EV + i] = s[i];
        }
        return;
    }
    float acc[loads_per_row(NV)][VEC];
    clear(acc);
    gather_entries<T, VEC, NV>(p, it.row == 0 ? p.t_local : p.t_cross, it.e0, it.e1, lane, acc);
    sum_groups<VEC, NV>(p.lpr_log2, it.e1 - it.e0, acc);
    if (NV == 0 && lane >= (1 << p.lpr_log2)) return;
#pragma unroll
    for (int m = 0; m < loads_per_row(NV); ++m) {
        const int c = VEC * (lane + 64 * m);
        if (c < width) put_floats<VEC>(dst + c, acc[m]);
    }
}

// One wavefront per item. SPLIT = false: the pieces of the long ranges, then the nodes without one (the pieces are the longest
// items and go first; a launch of their own left most of the device idle: 4,096 pieces took 58 us beside 258 us for 169,343
// nodes of 512 bf16 elements). SPLIT = true: the nodes whose ranges were cut, from the partial sums.
template <typename T, int VEC, int NV, int CROSS, int EV, bool SPLIT>
__global__ __launch_bounds__(kBlock) void node_sum_kernel(NodeArgs<T> p) {
    constexpr int NR = loads_per_row(NV);
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int lane = threadIdx.x & 63;
    const int32_t xcd = int32_t(blockIdx.x & 7u), seq = int32_t(blockIdx.x >> 3);
    const int32_t block = ((seq / kXcdRun) * 8 + xcd) * kXcdRun + seq % kXcdRun;
    int32_t idx = block * kWaves + __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6));
    if constexpr (!SPLIT) {                  // no barrier below: wavefronts are independent
        if (idx < p.n_pieces) {
            node_piece<T, VEC, NV, CROSS, EV>(p, p.pieces[idx], lane);
            return;
        }
        idx -= p.n_pieces;
    }
    if (idx >= p.n_nodes) return;
    const NodeItem it = p.nodes[idx];
    const int32_t width = int32_t(p.rule.width);
    const bool local_split = SPLIT && (it.flags & VARCO_NODE_LOCAL_SPLIT), cross_split = SPLIT && (it.flags & VARCO_NODE_CROSS_SPLIT);

    float acc[NR][VEC];
    clear(acc);
    if (local_split)
        add_partials<VEC, NV>(p.partial, width, it.l0, it.l1, lane, p.lpr_log2, acc);
    else
        gather_entries<T, VEC, NV>(p, p.t_local, it.l0, it.l1, lane, acc);

    const bool cross = CROSS != kCrossNone && it.c1 > it.c0;
    float* lrow = lds + (threadIdx.x >> 6) * ((width + 3) & ~3);
    if constexpr (CROSS == kCrossFull) {
        if (cross_split)
            add_partials<VEC, NV>(p.partial, width, it.c0, it.c1, lane, p.lpr_log2, acc);
        else
            gather_entries<T, VEC, NV>(p, p.t_cross, it.c0, it.c1, lane, acc);
    }
    sum_groups<VEC, NV>(p.lpr_log2, CROSS == kCrossFull ? it.l1 - it.l0 + (it.c1 - it.c0) : it.l1 - it.l0, acc);
    const int first = NV == 0 ? VEC * (lane & ((1 << p.lpr_log2) - 1)) : VEC * lane;     // first column of this lane
    if constexpr (CROSS == kCrossMasked) {
        if (cross) {
            float far[NR][VEC];
            clear(far);
            if (cross_split)
                add_partials<VEC, NV>(p.partial, width, it.c0, it.c1, lane, p.lpr_log2, far);
            else
                gather_entries<T, VEC, NV>(p, p.t_cross, it.c0, it.c1, lane, far);
            sum_groups<VEC, NV>(p.lpr_log2, it.c1 - it.c0, far);
            const MaskAffine ma = varco_affine(p.rule, it.gid);
#pragma unroll
            for (int m = 0; m < NR; ++m) {
                const int c = first + VEC * 64 * m;
#pragma unroll
                for (int i = 0; i < VEC; ++i)
                    if (c < width && varco_inverse_position(p.rule, ma, uint32_t(c + i)) < p.rule.k) acc[m][i] += far[m][i];
            }
        }
    }
    if constexpr (CROSS == kCrossProducts) {
        if (cross) {
            for (int c = 4 * lane; c < width; c += 256) *reinterpret_cast<float4*>(lrow + c) = make_float4(0.f, 0.f, 0.f, 0.f);
            const MaskAffine ma = varco_affine(p.rule, it.gid);
            const int sub = lane >> p.lpe_log2, n_sub = 64 >> p.lpe_log2, jl = lane & ((1 << p.lpe_log2) - 1);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int u0 = 0; u0 < p.ku; u0 += 64) {
                const int ju = u0 + jl;
                const bool on = ju < p.ku;
                float s[EV];
                if (cross_split) {          // fp32 partial rows, EV elements at a time as well (rows are width floats apart)
#pragma unroll
                    for (int i = 0; i < EV; ++i) s[i] = 0.f;
                    for (int32_t r = it.c0 + sub; r < it.c1; r += n_sub)
                        if (on)
#pragma unroll
                            for (int i = 0; i < EV; ++i) s[i] += p.partial[int64_t(r) * width + ju * EV + i];
                    add_lanes(s, p.lpe_log2);
                } else {
                    sum_rows<T, EV>(p.prod, p.pitch, it.c0, it.c1, ju * EV, on, sub, n_sub, p.lpe_log2, s);
                }
                if (on && sub == 0) {
                    uint32_t q = varco_position(p.rule, ma, uint32_t(ju * EV));
#pragma unroll
                    for (int i = 0; i < EV; ++i) {
                        if (i == 0 || uint32_t(ju * EV + i) < p.rule.k) lrow[q] = s[i];
                        q += ma.a;
                        q = min(q, q - p.rule.width);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    if (NV == 0 && lane >= (1 << p.lpr_log2)) return;
    T* dst = p.out + int64_t(it.row) * width;
#pragma unroll
    for (int m = 0; m < NR; ++m) {
        const int c = first + VEC * 64 * m;
        if (c < width) {
            if (CROSS == kCrossProducts && cross) add_floats<VEC>(lrow + c, acc[m]);
            if (p.add_old) {
                float old[VEC];
                Packed<T, VEC>::get(Packed<T, VEC>::load(dst + c), old);
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[m][i] += old[i];
            }
            Packed<T, VEC>::put(dst + c, acc[m]);
        }
    }
}

bool aligned_to(const void* p, size_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }
template <int N>
using Int = std::integral_constant<int, N>;

template <typename T>
hipError_t node_sum_t(const NodePlan& plan, const uint2* t_local, const uint2* t_cross, const void* dm, const void* prod,
                      int32_t pitch, const MaskRule& rule, VarcoCross cross, void* out, bool add_old, float* partial, hipStream_t stream,
                      const LaunchTag& tag) {
    NodeArgs<T> a;
    a.pieces = plan.pieces, a.n_pieces = plan.n_pieces;
    a.t_local = t_local, a.t_cross = t_cross;
    a.dm = static_cast<const T*>(dm), a.prod = static_cast<const T*>(prod);
    a.rule = rule;
    a.out = static_cast<T*>(out);
    a.add_old = add_old ? 1 : 0;
    a.partial = partial;
    const int32_t width = int32_t(rule.width);
    auto vec_ok = [&](int v) {
        return width % v == 0 && aligned_to(dm, v * sizeof(T)) && aligned_to(out, v * sizeof(T)) && aligned_to(partial, 16);
    };
    const int vec = sizeof(T) == 2 && vec_ok(8) ? 8 : vec_ok(4) ? 4 : 1;
    const int per_row = width / vec;
    a.lpr_log2 = 0;
    while ((1 << a.lpr_log2) < per_row && a.lpr_log2 < 6) ++a.lpr_log2;
    int nv = a.lpr_log2 < 6 ? 0 : 1;
    while (nv && nv * 64 < per_row) nv <<= 1;
    if (nv > 8) return hipErrorInvalidValue;
    a.pitch = pitch;
    constexpr int ev = 16 / sizeof(T);
    if (cross == kCrossProducts && (a.pitch % ev != 0 || !aligned_to(prod, 16) || width * int(sizeof(T)) <= kProductRowBytes)) return hipErrorInvalidValue;
    a.ku = (int32_t(rule.k) + ev - 1) / ev;
    a.lpe_log2 = 0;
    while ((1 << a.lpe_log2) < a.ku && a.lpe_log2 < 6) ++a.lpe_log2;

    auto grid_for = [](int32_t n) {
        const int32_t per_round = 8 * kXcdRun;
        return dim3(unsigned(((n + kWaves - 1) / kWaves + per_round - 1) / per_round * per_round));
    };
    const size_t lds_bytes = cross == kCrossProducts ? size_t(kWaves) * ((width + 3) / 4 * 4) * sizeof(float) : 0;
    auto launch = [&](auto vec, auto nvc, auto cr, auto evc) {
        constexpr int VEC = decltype(vec)::value, NV = decltype(nvc)::value, CR = decltype(cr)::value, EV = decltype(evc)::value;
        a.nodes = plan.nodes, a.n_nodes = plan.n_whole;
        tag.begin(stream);
        hipLaunchKernelGGL((node_sum_kernel<T, VEC, NV, CR, EV, false>), grid_for(plan.n_pieces + plan.n_whole), dim3(kBlock), lds_bytes, stream, a);
        tag.end(stream);
        if (plan.n_nodes > plan.n_whole) {
            a.nodes = plan.nodes + plan.n_whole, a.n_nodes = plan.n_nodes - plan.n_whole;
            tag.begin_as(VARCO_K_REDUCE, stream, 0.0);
            hipLaunchKernelGGL((node_sum_kernel<T, VEC, NV, CR, EV, true>), grid_for(a.n_nodes), dim3(kBlock), lds_bytes, stream, a);
            tag.end(stream);
        }
    };
    auto with_cross = [&](auto vec, auto nvc) {
        switch (cross) {
            case kCrossNone: launch(vec, nvc, Int<kCrossNone>{}, Int<1>{}); break;
            case kCrossMasked: launch(vec, nvc, Int<kCrossMasked>{}, Int<1>{}); break;
            case kCrossFull: launch(vec, nvc, Int<kCrossFull>{}, Int<1>{}); break;
            default:
                // (loads of this kind that cover only rows too short for products: never asked for)
                if constexpr ((decltype(nvc)::value > 0 ? 64 * decltype(nvc)::value : 32) * decltype(vec)::value * int(sizeof(T)) > kProductRowBytes)
                    launch(vec, nvc, Int<kCrossProducts>{}, Int<ev>{});
        }
    };
    auto with_nv = [&](auto vec) {
        constexpr int VEC = decltype(vec)::value;
        switch (nv) {
            case 0: with_cross(vec, Int<0>{}); break;
            case 1: with_cross(vec, Int<1>{}); break;
            case 2: with_cross(vec, Int<2>{}); break;
            case 4: with_cross(vec, Int<4>{}); break;
            default:
                if constexpr (VEC < 8) with_cross(vec, Int<8>{});
        }
    };
    if constexpr (sizeof(T) == 2)
        if (vec == 8) {
            with_nv(Int<8>{});
            return hipGetLastError();
        }
    if (vec == 4)
        with_nv(Int<4>{});
    else
        with_nv(Int<1>{});
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Set-up: the partitions' arrays joined into one block (varco_link_partitions). H = row of the concatenated halo rows.
// ---------------------------------------------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void link_halo_kernel(LinkPartition p, int32_t* halo_len, int32_t* halo_gid, int32_t* halo_zrow) {
    const int32_t s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= p.d.n_halo) return;
    const int64_t h = int64_t(p.d.halo_row_offset) + s;
    halo_len[h] = p.d.t_rowptr[p.d.n_local + s + 1] - p.d.t_rowptr[p.d.n_local + s];
    halo_gid[h] = p.d.halo_gid[s];
    halo_zrow[h] = p.d.halo_zrow[s];
}

// Owner p: which arena row every returned halo row belongs to, and how many cross entries each of its rows has. The
// consumers' halo rows must all be of this boundary node, and of its row of the compressed buffer.
__global__ __launch_bounds__(kBlock) void link_owner_kernel(LinkPartition p, int64_t halo_total, const int32_t* halo_len,
                                                            const int32_t* halo_gid, const int32_t* halo_zrow, int32_t* owner_row,
                                                            int32_t* cross_len, int32_t* brow, int32_t* bgid, int32_t* zrow_of,
                                                            int32_t* flags) {
    const int32_t b = blockIdx.x * kBlock + threadIdx.x;
    if (b >= p.d.n_boundary) return;
    const int32_t i = p.d.boundary_rows[b], gid = p.d.local_gid[i], row = int32_t(p.row_off) + i, zrow = p.d.z_row_offset + b;
    int32_t total = 0;
    bool bad = false;
    for (int32_t e = p.d.ret_ptr[b]; e < p.d.ret_ptr[b + 1]; ++e) {
        const int32_t h = p.d.ret_src[e];
        if (h < 0 || h >= halo_total) {
            bad = true;
            continue;
        }
        if (halo_gid[h] != gid || halo_zrow[h] != zrow || atomicExch(owner_row + h, row) != -1) bad = true;
        total += halo_len[h];
    }
    brow[zrow] = row, bgid[zrow] = gid, zrow_of[row] = zrow;
    cross_len[row] = total;
    if (bad) atomicOr(flags, VARCO_BAD_LINK);
}

__global__ __launch_bounds__(kBlock) void link_starts_kernel(LinkPartition p, const int32_t* halo_len, const int32_t* cross_ptr,
                                                             int32_t* prod_start) {
    const int32_t b = blockIdx.x * kBlock + threadIdx.x;
    if (b >= p.d.n_boundary) return;
    int32_t at = cross_ptr[p.row_off + p.d.boundary_rows[b]];
    for (int32_t e = p.d.ret_ptr[b]; e < p.d.ret_ptr[b + 1]; ++e) {
        const int32_t h = p.d.ret_src[e];
        prod_start[h] = at;
        at += halo_len[h];
    }
}

__global__ __launch_bounds__(kBlock) void link_edges_kernel(LinkPartition p, const int32_t* prow_part, const int32_t* owner_row,
                                                            const int32_t* prod_start, VarcoEdge* edges, int32_t* arow, float* vals,
                                                            int32_t* prow) {
    const int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (e >= p.d.nnz) return;
    const int32_t c = p.d.colidx[e], nl = p.d.n_local;
    const int64_t o = p.ent_off + e;
    vals[o] = p.d.vals[e];
    if (c < nl) {
        const int32_t r = int32_t(p.row_off) + c;
        edges[o] = VarcoEdge{r, -1};
        arow[o] = r;
        prow[o] = -1;
    } else {
        const int32_t s = c - nl;
        const int64_t h = int64_t(p.d.halo_row_offset) + s;
        edges[o] = VarcoEdge{p.d.halo_zrow[s], p.d.halo_gid[s]};
        arow[o] = owner_row[h];
        prow[o] = prod_start[h] + (prow_part[e] + p.d.t_rowptr[nl] - p.d.t_rowptr[c]);
    }
}

// Transposed entries in node order; one thread per row of the partition's transpose.
__global__ __launch_bounds__(kBlock) void link_transposed_kernel(LinkPartition p, const int32_t* prod_start, uint2* t_local,
                                                                 uint2* t_cross) {
    const int32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= p.d.n_local + p.d.n_halo) return;
    const int32_t e0 = p.d.t_rowptr[c], e1 = p.d.t_rowptr[c + 1];
    uint2* dst = c < p.d.n_local ? t_local + p.local_off + e0 : t_cross + prod_start[int64_t(p.d.halo_row_offset) + c - p.d.n_local];
    for (int32_t e = e0; e < e1; ++e) dst[e - e0] = make_uint2(uint32_t(int32_t(p.row_off) + p.d.t_colidx[e]), __float_as_uint(p.d.t_vals[e]));
}

__global__ __launch_bounds__(kBlock) void link_items_kernel(const SpmmItem* in, int32_t n, int32_t row_off, int32_t ent_off,
                                                            int32_t slot_off, SpmmItem* out) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    SpmmItem it = in[i];
    it.row += row_off, it.e0 += ent_off, it.e1 += ent_off;
    if (it.dst >= 0) it.dst += slot_off;
    out[i] = it;
}
__global__ __launch_bounds__(kBlock) void link_splits_kernel(const SpmmSplit* in, int32_t n, int32_t row_off, int32_t slot_off,
                                                             SpmmSplit* out) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    SpmmSplit s = in[i];
    s.row += row_off, s.first += slot_off;
    out[i] = s;
}

dim3 blocks_for(int64_t n) { return dim3(unsigned((n + kBlock - 1) / kBlock)); }

}  // namespace

hipError_t varco_launch_node_sum(int dtype, const NodePlan& plan, const uint2* t_local, const uint2* t_cross, const void* dm,
                                 const void* prod, int32_t pitch, const MaskRule& rule, VarcoCross cross, void* out, bool add_old,
                                 float* partial, hipStream_t stream, const LaunchTag& tag) {
    if (plan.n_nodes == 0) return hipSuccess;
    return dtype == VARCO_BF16 ? node_sum_t<bf16_t>(plan, t_local, t_cross, dm, prod, pitch, rule, cross, out, add_old, partial, stream, tag)
                               : node_sum_t<float>(plan, t_local, t_cross, dm, prod, pitch, rule, cross, out, add_old, partial, stream, tag);
}

hipError_t varco_launch_link_halo(const LinkPartition& p, int32_t* halo_len, int32_t* halo_gid, int32_t* halo_zrow, hipStream_t stream) {
    if (p.d.n_halo == 0) return hipSuccess;
    hipLaunchKernelGGL(link_halo_kernel, blocks_for(p.d.n_halo), dim3(kBlock), 0, stream, p, halo_len, halo_gid, halo_zrow);
    return hipGetLastError();
}
hipError_t varco_launch_link_owner(const LinkPartition& p, int64_t halo_total, const int32_t* halo_len, const int32_t* halo_gid,
                                   const int32_t* halo_zrow, int32_t* owner_row, int32_t* cross_len, int32_t* brow, int32_t* bgid,
                                   int32_t* zrow_of, int32_t* flags, hipStream_t stream) {
    if (p.d.n_boundary == 0) return hipSuccess;
    hipLaunchKernelGGL(link_owner_kernel, blocks_for(p.d.n_boundary), dim3(kBlock), 0, stream, p, halo_total, halo_len, halo_gid,
                       halo_zrow, owner_row, cross_len, brow, bgid, zrow_of, flags);
    return hipGetLastError();
}
hipError_t varco_launch_link_starts(const LinkPartition& p, const int32_t* halo_len, const int32_t* cross_ptr, int32_t* prod_start,
                                    hipStream_t stream) {
    if (p.d.n_boundary == 0) return hipSuccess;
    hipLaunchKernelGGL(link_starts_kernel, blocks_for(p.d.n_boundary), dim3(kBlock), 0, stream, p, halo_len, cross_ptr, prod_start);
    return hipGetLastError();
}
hipError_t varco_launch_link_edges(const LinkPartition& p, const int32_t* prow_part, const int32_t* owner_row, const int32_t* prod_start,
                                   VarcoEdge* edges, int32_t* arow, float* vals, int32_t* prow, hipStream_t stream) {
    if (p.d.nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(link_edges_kernel, blocks_for(p.d.nnz), dim3(kBlock), 0, stream, p, prow_part, owner_row, prod_start, edges, arow,
                       vals, prow);
    return hipGetLastError();
}
hipError_t varco_launch_link_transposed(const LinkPartition& p, const int32_t* prod_start, uint2* t_local, uint2* t_cross,
                                        hipStream_t stream) {
    const int64_t n = int64_t(p.d.n_local) + p.d.n_halo;
    if (n == 0 || p.d.nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(link_transposed_kernel, blocks_for(n), dim3(kBlock), 0, stream, p, prod_start, t_local, t_cross);
    return hipGetLastError();
}
hipError_t varco_launch_link_items(const SpmmPlan& part, int32_t row_off, int32_t ent_off, int32_t slot_off, int32_t item_off,
                                   int32_t split_off, const SpmmPlan& out, hipStream_t stream) {
    if (part.n_items > 0)
        hipLaunchKernelGGL(link_items_kernel, blocks_for(part.n_items), dim3(kBlock), 0, stream, part.items, part.n_items, row_off, ent_off,
                           slot_off, out.items + item_off);
    if (part.n_splits > 0)
        hipLaunchKernelGGL(link_splits_kernel, blocks_for(part.n_splits), dim3(kBlock), 0, stream, part.splits, part.n_splits, row_off,
                           slot_off, out.splits + split_off);
    return hipGetLastError();
}
