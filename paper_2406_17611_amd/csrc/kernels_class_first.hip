// A layer that applies its weights before the aggregation (varco_set_layer_order; bf16 storage, at most 64 outputs), for
// all partitions of a device at once. Every consumer of a node receives the same compressed row, so on one device that row
// is transformed once (b_total rows instead of one per consumer), and the errors of all its consumers are summed before they
// are taken back through the weights:
//   Y = [X H ; X~_z H]                    rows of the arena, then the compressed boundary rows        (pitch kClassPitch)
//   X_out[i] = sum of S[i, v] Y[v]        narrow gather below
//   G_loc[v], G_z[v] = sums of S[i, v] dZ[i] over v's local and cross entries (narrow gather)
//   dH += X^T G_loc + X~_z^T G_z          GEMM and halo_transform_wgrad_kernel
//   dX[v] = G_loc[v] H^T + kept positions of (G_z[v] H^T)                                             class_dgrad_kernel
// Rows of Y, G and of the copy of dZ take kClassPitch = 64 elements, 128 bytes: one cache line per gathered row, read by
// eight lanes with 16-byte loads, eight rows per instruction (rows of 47 elements, unaligned, took a 2-byte load per lane and
// one row per instruction).
#include <algorithm>
#include <type_traits>

#include "gather_device.h"
#include "mask_device.h"

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int P = kClassPitch;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ void add_row(float (&acc)[8], float w, const uint4& v) {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[2 * i] += w * __uint_as_float(u[i] << 16), acc[2 * i + 1] += w * __uint_as_float(u[i] & 0xFFFF0000u);
}

// Sum of the rows of a range of entries, column `lane` of it in every lane. Lane t of a group of eight takes columns 8 t ..
// 8 t + 7, the groups take different entries; at the end the groups exchange halves of what they hold until one column is left
// per lane (7 exchanges and additions instead of 24 in a butterfly of whole rows). record(e): {row of src, weight bits}.
__device__ __forceinline__ float add_halves32(float a, float b) {      // lanes below 32: a of both halves; above: b of both
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_halves16(float a, float b) {      // the same for the two 16-lane rows of each half
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <class F>
__device__ __forceinline__ float narrow_sum(const uint16_t* src, int32_t e0, int32_t e1, int lane, F&& record) {
    const int t = lane & 7, g = lane >> 3;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    for (int32_t base = e0; base < e1; base += 64) {
        uint2 mine = make_uint2(0u, 0u);
        if (base + lane < e1) mine = record(base + lane);
        const int cnt = min(64, e1 - base);
        auto batch = [&](int i0, auto count) {
            constexpr int N = decltype(count)::value;
            uint4 v[N];
            uint32_t w[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int i = i0 + 8 * u + g;
                const uint32_t r = lane_value(mine.x, 4 * i);
                w[u] = lane_value(mine.y, 4 * i);
                v[u] = *reinterpret_cast<const uint4*>(src + int64_t(i < cnt ? r : 0u) * P + 8 * t);
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (i0 + 8 * u + g < cnt) add_row(acc, __uint_as_float(w[u]), v[u]);
        };
        int i0 = 0;
        for (; i0 + 16 < cnt; i0 += 32) batch(i0, std::integral_constant<int, 4>{});
        if (i0 + 8 < cnt)
            batch(i0, std::integral_constant<int, 2>{});
        else if (i0 < cnt)
            batch(i0, std::integral_constant<int, 1>{});
    }
    // columns 8 t + 4 (lane / 32) + 2 (lane / 16 % 2) + (lane / 8 % 2) of the sums
    float h[4], q[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = add_halves32(acc[i], acc[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) q[i] = add_halves16(h[i], h[i + 2]);
    const bool odd = lane & 8;
    const float keep = odd ? q[1] : q[0], give = odd ? q[0] : q[1];
    return keep + __shfl_xor(give, 8);
}
__device__ __forceinline__ int my_column(int lane) { return 8 * (lane & 7) + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1); }

// X_out rows from the forward work list; pieces of split rows go to `partial` (P floats each).
__global__ __launch_bounds__(kBlock) void narrow_forward_kernel(const SpmmItem* items, int32_t n_items, const VarcoEdge* edge, const float* vals,
                                                                const uint16_t* y, int32_t rows, bf16_t* out, int32_t fo, float* partial) {
    const int lane = threadIdx.x & 63;
    const int32_t idx = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6));
    if (idx >= n_items) return;
    const SpmmItem it = items[idx];
    const float x = narrow_sum(y, it.e0, it.e1, lane, [&](int32_t e) {
        const VarcoEdge ed = edge[e];
        return make_uint2(uint32_t(ed.gid < 0 ? ed.src : rows + ed.src), __float_as_uint(vals[e]));
    });
    const int c = my_column(lane);
    if (it.dst >= 0)
        partial[int64_t(it.dst) * P + c] = x;
    else if (c < fo)
        Elem<bf16_t>::store(out + int64_t(it.row) * fo + c, x);
}
__global__ __launch_bounds__(kBlock) void narrow_fixup_kernel(const SpmmSplit* splits, int32_t n_splits, const float* partial, bf16_t* out,
                                                              int32_t fo) {
    const int32_t s = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (s >= n_splits) return;
    const SpmmSplit sp = splits[s];
    const int c = threadIdx.x & 63;
    float x = 0.f;
    for (int32_t i = 0; i < sp.count; ++i) x += partial[int64_t(sp.first + i) * P + c];
    if (c < fo) Elem<bf16_t>::store(out + int64_t(sp.row) * fo + c, x);
}

// G_loc[row] and G_z[zrow of row] (zeros beyond fo). SPLIT = false: partial sums of the pieces of long ranges (the launch's
// first wavefronts) and the nodes without pieces; SPLIT = true: the others, from the partial sums.
template <bool SPLIT>
__global__ __launch_bounds__(kBlock) void narrow_backward_kernel(const NodeItem* nodes, int32_t n, const SpmmItem* pieces, int32_t n_pieces,
                                                                 const uint2* t_local, const uint2* t_cross, const uint16_t* dz,
                                                                 const int32_t* zrow_of, bf16_t* g_loc, bf16_t* g_z, int32_t fo, float* partial) {
    const int lane = threadIdx.x & 63, c = my_column(lane);
    int32_t idx = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6));
    if constexpr (!SPLIT) {
        if (idx < n_pieces) {
            const SpmmItem it = pieces[idx];
            const uint2* pairs = it.row == 0 ? t_local : t_cross;
            partial[int64_t(it.dst) * P + c] = narrow_sum(dz, it.e0, it.e1, lane, [&](int32_t e) { return pairs[e]; });
            return;
        }
        idx -= n_pieces;
    }
    if (idx >= n) return;
    const NodeItem it = nodes[idx];
    auto range = [&](const uint2* pairs, int32_t e0, int32_t e1, bool split) {
        float x = 0.f;
        if (SPLIT && split)
            for (int32_t s = e0; s < e1; ++s) x += partial[int64_t(s) * P + c];
        else
            x = narrow_sum(dz, e0, e1, lane, [&](int32_t e) { return pairs[e]; });
        return c < fo ? x : 0.f;
    };
    const int32_t zr = zrow_of[it.row];
    Elem<bf16_t>::store(g_loc + int64_t(it.row) * P + c, range(t_local, it.l0, it.l1, it.flags & VARCO_NODE_LOCAL_SPLIT));
    if (g_z && zr >= 0) Elem<bf16_t>::store(g_z + int64_t(zr) * P + c, range(t_cross, it.c0, it.c1, it.flags & VARCO_NODE_CROSS_SPLIT));
}

// Rows of fo elements -> rows of P elements, zeros beyond fo.
__global__ __launch_bounds__(kBlock) void pad_rows_kernel(const uint16_t* __restrict__ in, int64_t n, int32_t fo, uint16_t* __restrict__ out) {
    const int64_t stride = int64_t(gridDim.x) * kWaves;
    const int c = threadIdx.x & 63;
    for (int64_t r = int64_t(blockIdx.x) * kWaves + (threadIdx.x >> 6); r < n; r += stride) out[r * P + c] = c < fo ? in[r * fo + c] : uint16_t(0);
}

// dX[v] = G_loc[v] H^T + kept positions of (G_z[v] H^T). A workgroup walks tiles of 32 rows; wavefront w holds the weights of
// positions 128 w .. 128 w + 127 ([position][column], at most 64 columns) as matrix operands in registers, forms both
// products, drops the second at positions that the row's message did not carry, and the tile leaves through LDS in 16-byte
// pieces. Bound by writing dX.
constexpr int kTile = 32, kMaxWidth = 512, kPitch = kMaxWidth + 8, kPitchG = P + 8;
__global__ __launch_bounds__(kBlock, 2) void class_dgrad_kernel(const uint16_t* __restrict__ g_loc, const uint16_t* __restrict__ g_z,
                                                                const int32_t* __restrict__ zrow_of, const int32_t* __restrict__ bgid, int32_t n,
                                                                MaskRule rule, int32_t fo, const uint16_t* __restrict__ wr, int32_t cpitch,
                                                                uint16_t* __restrict__ dx) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[kTile * kPitch];
    __shared__ __attribute__((aligned(16))) uint16_t ga[2][kTile * kPitchG];
    __shared__ uint2 rows_ab[kTile];              // {a_inv, b}; a_inv = 0 and b = width: nothing kept
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lrow = lane & 31, lk = lane >> 5;
    const int32_t width = int32_t(rule.width);
    const int ksteps = (fo + 15) / 16;
    auto frag = [](const uint16_t* p) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p)); };
    bf16x8 wf[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int32_t pos = wave * 128 + b * 32 + lrow;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            wf[b][s] = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
            const int32_t c0 = 16 * s + 8 * lk;
            if (s < ksteps && pos < width && c0 + 8 <= cpitch) wf[b][s] = frag(wr + int64_t(pos) * cpitch + c0);
        }
    }
    const int32_t n_tiles = (n + kTile - 1) / kTile;
    const int fr = threadIdx.x >> 3, fc = (threadIdx.x & 7) * 8;      // this thread's 16-byte piece of a tile of G: row, first column
    uint4 nl, nz;
    int32_t nzr = -1;
    auto fetch = [&](int32_t t) {
        const int32_t row = min(t * kTile + fr, n - 1);
        nl = *reinterpret_cast<const uint4*>(g_loc + int64_t(row) * P + fc);
        nzr = g_z ? zrow_of[row] : -1;
        nz = make_uint4(0u, 0u, 0u, 0u);
        if (nzr >= 0) nz = *reinterpret_cast<const uint4*>(g_z + int64_t(nzr) * P + fc);
    };
    if (int32_t(blockIdx.x) < n_tiles) fetch(blockIdx.x);
    for (int32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const int32_t row0 = t * kTile, rows = min(kTile, n - row0);
        *reinterpret_cast<uint4*>(&ga[0][fr * kPitchG + fc]) = nl;
        *reinterpret_cast<uint4*>(&ga[1][fr * kPitchG + fc]) = nz;
        if ((threadIdx.x & 7) == 0) {
            uint2 ab = make_uint2(0u, 0u);
            if (nzr >= 0 && rule.k < rule.width) {
                const MaskAffine m = varco_affine(rule, uint32_t(bgid[nzr]));
                ab = make_uint2(m.a_inv, m.b);
            }
            rows_ab[fr] = ab;
        }
        __syncthreads();
        if (t + int32_t(gridDim.x) < n_tiles) fetch(t + gridDim.x);
        bf16x8 fl[4], fz[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            fl[s] = frag(&ga[0][lrow * kPitchG + 16 * s + 8 * lk]);
            fz[s] = frag(&ga[1][lrow * kPitchG + 16 * s + 8 * lk]);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int32_t pos = wave * 128 + b * 32 + lrow;
            if (wave * 128 + b * 32 >= width) break;
            floatx16 al, az;
#pragma unroll
            for (int v = 0; v < 16; ++v) al[v] = az[v] = 0.f;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (s < ksteps) {
                    al = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fl[s], wf[b][s], al, 0, 0, 0);
                    az = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fz[s], wf[b][s], az, 0, 0, 0);
                }
            // accumulator register v of a lane is element (8 * (v / 4) + 4 * (lane / 32) + v % 4, lane % 32)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v >> 2) + 4 * lk + (v & 3);
                const uint2 ab = rows_ab[r];
                bool kept = rule.k == rule.width;
                if (!kept) {
                    const uint32_t d = uint32_t(pos) >= ab.y ? uint32_t(pos) - ab.y : uint32_t(pos) + rule.width - ab.y;
                    kept = varco_mod_width(ab.x * d, rule.width, rule.width_magic) < rule.k;
                }
                if (pos < width) tile[r * kPitch + pos] = float_to_bf16(al[v] + (kept ? az[v] : 0.f));
            }
        }
        __syncthreads();
        const int per_row = width / 8;                 // width is a multiple of 16
        for (int e = threadIdx.x; e < rows * per_row; e += kBlock) {
            const int r = e / per_row, c = (e - r * per_row) * 8;
            *reinterpret_cast<uint4*>(dx + int64_t(row0 + r) * width + c) = *reinterpret_cast<const uint4*>(&tile[r * kPitch + c]);
        }
    }
}

dim3 waves_for(int64_t n) { return dim3(unsigned((n + kWaves - 1) / kWaves)); }

}  // namespace

hipError_t varco_launch_narrow_forward(const SpmmPlan& plan, const VarcoEdge* edge, const float* vals, const void* y, int32_t rows, void* out,
                                       int32_t fo, float* partial, hipStream_t stream, const LaunchTag& tag) {
    if (plan.n_items == 0) return hipSuccess;
    tag.begin(stream);
    hipLaunchKernelGGL(narrow_forward_kernel, waves_for(plan.n_items), dim3(kBlock), 0, stream, plan.items, plan.n_items, edge, vals,
                       static_cast<const uint16_t*>(y), rows, static_cast<bf16_t*>(out), fo, partial);
    tag.end(stream);
    if (plan.n_splits > 0) {
        tag.begin_as(VARCO_K_REDUCE, stream, 4.0 * plan.n_partials * P);
        hipLaunchKernelGGL(narrow_fixup_kernel, waves_for(plan.n_splits), dim3(kBlock), 0, stream, plan.splits, plan.n_splits, partial,
                           static_cast<bf16_t*>(out), fo);
        tag.end(stream);
    }
    return hipGetLastError();
}

hipError_t varco_launch_narrow_backward(const NodePlan& plan, const uint2* t_local, const uint2* t_cross, const void* dz, int64_t rows,
                                        const int32_t* zrow_of, void* dz_padded, void* g_loc, void* g_z, int32_t fo, float* partial,
                                        hipStream_t stream, const LaunchTag& tag) {
    if (plan.n_nodes == 0) return hipSuccess;
    tag.begin(stream);
    hipLaunchKernelGGL(pad_rows_kernel, dim3(unsigned(std::min<int64_t>((rows + kWaves - 1) / kWaves, 256 * 32))), dim3(kBlock), 0, stream,
                       static_cast<const uint16_t*>(dz), rows, fo, static_cast<uint16_t*>(dz_padded));
    const uint16_t* src = static_cast<const uint16_t*>(dz_padded);
    hipLaunchKernelGGL(narrow_backward_kernel<false>, waves_for(int64_t(plan.n_pieces) + plan.n_whole), dim3(kBlock), 0, stream, plan.nodes, plan.n_whole,
                       plan.pieces, plan.n_pieces, t_local, t_cross, src, zrow_of, static_cast<bf16_t*>(g_loc), static_cast<bf16_t*>(g_z), fo, partial);
    if (plan.n_nodes > plan.n_whole)
        hipLaunchKernelGGL(narrow_backward_kernel<true>, waves_for(plan.n_nodes - plan.n_whole), dim3(kBlock), 0, stream, plan.nodes + plan.n_whole,
                           plan.n_nodes - plan.n_whole, plan.pieces, 0, t_local, t_cross, src, zrow_of, static_cast<bf16_t*>(g_loc),
                           static_cast<bf16_t*>(g_z), fo, partial);
    tag.end(stream);
    return hipGetLastError();
}

hipError_t varco_launch_class_dgrad(const void* g_loc, const void* g_z, const int32_t* zrow_of, const int32_t* bgid, int64_t rows,
                                    const MaskRule& rule, int32_t fo, const void* wr, int32_t cpitch, void* dx, hipStream_t stream,
                                    const LaunchTag& tag) {
    if (rows == 0) return hipSuccess;
    if (rule.width % 16 != 0 || rule.width > uint32_t(kMaxWidth) || fo > P || cpitch < fo || cpitch % 8 != 0 || (reinterpret_cast<uintptr_t>(dx) & 15u))
        return hipErrorInvalidValue;
    tag.begin(stream);
    const int64_t tiles = (rows + kTile - 1) / kTile;
    hipLaunchKernelGGL(class_dgrad_kernel, dim3(unsigned(std::min<int64_t>(tiles, 512))), dim3(kBlock), 0, stream, static_cast<const uint16_t*>(g_loc),
                       static_cast<const uint16_t*>(g_z), zrow_of, bgid, int32_t(rows), rule, fo, static_cast<const uint16_t*>(wr), cpitch,
                       static_cast<uint16_t*>(dx));
    tag.end(stream);
    return hipGetLastError();
}
