// A layer that applies its weights before the aggregation (varco_set_layer_order; bf16 storage, at most 64 outputs), and the input
// gradient of any class layer (at most 64 outputs, either storage type), for
// all partitions of a device at once. Every consumer of a node receives the same compressed row, so on one device that row
// is transformed once (b_total rows instead of one per consumer), and the errors of all its consumers are summed before they
// are taken back through the weights:
//   Y = [X H ; X~_z H]                    rows of the arena, then the compressed boundary rows        (pitch kClassPitch)
//   X_out[i] = sum of S[i, v] Y[v]        narrow gather below
//   G_loc[v], G_z[v] = sums of S[i, v] dZ[i] over v's local and cross entries (narrow gather)
//   dH += X^T G_loc + X~_z^T G_z          GEMM and halo_transform_wgrad_kernel
//   dX[v] = G_loc[v] H^T + kept positions of (G_z[v] H^T)                                             class_dgrad_kernel,
//                                                                                                     class_dgrad_f32_kernel
// Rows of Y, G and of a copy of dZ take kClassPitch = 64 elements (32 with fp32 storage and at most 32 outputs): whole cache lines
// per gathered row, read by 8 or 16 lanes with 16-byte loads, eight or four rows per instruction (rows of 47 elements, unaligned, took
// an element load per lane and one row per instruction). Rows of dZ that are whole 16-byte pieces are gathered where they are: they touch
// as many lines as padded ones, and the copy is a launch (3 us on 2,000 nodes, 10 us on 169,343 of 40 outputs).
#include <algorithm>
#include <type_traits>

#include "gather_device.h"
#include "half_terms.h"
#include "mask_device.h"

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int P = kClassPitch;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The columns of a row that a lane holds, and the row's weighted sum.
template <typename T>
struct Columns;
template <>
struct Columns<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void add(float (&acc)[8], float w, const uint4& v) {
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[2 * i] += w * __uint_as_float(u[i] << 16), acc[2 * i + 1] += w * __uint_as_float(u[i] & 0xFFFF0000u);
    }
};
template <>
struct Columns<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void add(float (&acc)[4], float w, const uint4& v) {
        acc[0] += w * __uint_as_float(v.x), acc[1] += w * __uint_as_float(v.y);
        acc[2] += w * __uint_as_float(v.z), acc[3] += w * __uint_as_float(v.w);
    }
};

__device__ __forceinline__ uint32_t bits_of(float x) { return __float_as_uint(x); }
__device__ __forceinline__ uint32_t bits_of(bf16_t x) { return x.bits; }

// A piece that was loaded `by` elements early, moved up; zeros follow.
template <typename T>
__device__ __forceinline__ uint4 moved_up(uint4 x, int by) {
    if constexpr (sizeof(T) == 2) return moved_up8(x, by);
    if (by & 2) x = make_uint4(x.z, x.w, 0u, 0u);
    if (by & 1) x = make_uint4(x.y, x.z, x.w, 0u);
    return x;
}

// Sum of the rows (ROW elements each) of a range of entries, column my_column() of it in every lane. A group of lanes covers a row
// with 16-byte loads, the groups take different entries; at the end the groups exchange halves of what they hold until one column is
// left per lane (bf16: 7 exchanges and additions instead of 24 in a butterfly of whole rows). record(e): {row of src, weight bits}.
__device__ __forceinline__ float add_halves32(float a, float b) {      // lanes below 32: a of both halves; above: b of both
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_halves16(float a, float b) {      // the same for the two 16-lane rows of each half
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Rows are `ld` elements apart and have `cols` of them, whole 16-byte pieces; a lane beyond them adds zeros.
template <typename T, int ROW, class F>
__device__ __forceinline__ float narrow_sum(const T* src, int32_t ld, int32_t cols, int32_t e0, int32_t e1, int lane, F&& record) {
    constexpr int C = Columns<T>::N, LANES = ROW / C, ROWS = 64 / LANES, MOST = 32 / ROWS;      // 32 rows in flight
    static_assert(LANES == 8 || LANES == 16, "a row is covered by 8 or 16 lanes");
    const int t = lane % LANES, g = lane / LANES;
    const bool in = C * t < cols;
    float acc[C];
#pragma unroll
    for (int i = 0; i < C; ++i) acc[i] = 0.f;
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
                const int i = i0 + ROWS * u + g;
                const uint32_t r = lane_value(mine.x, 4 * i);
                w[u] = lane_value(mine.y, 4 * i);
                v[u] = make_uint4(0u, 0u, 0u, 0u);
                if (in) v[u] = *reinterpret_cast<const uint4*>(src + int64_t(i < cnt ? r : 0u) * ld + C * t);
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (i0 + ROWS * u + g < cnt) Columns<T>::add(acc, __uint_as_float(w[u]), v[u]);
        };
        int i0 = 0;
        for (; i0 + 16 < cnt; i0 += 32) batch(i0, std::integral_constant<int, MOST>{});
        if (i0 + 8 < cnt)
            batch(i0, std::integral_constant<int, MOST / 2>{});
        else if (i0 < cnt)
            batch(i0, std::integral_constant<int, MOST / 4>{});
    }
    float h[C / 2], q[C / 4];
#pragma unroll
    for (int i = 0; i < C / 2; ++i) h[i] = add_halves32(acc[i], acc[i + C / 2]);
#pragma unroll
    for (int i = 0; i < C / 4; ++i) q[i] = add_halves16(h[i], h[i + C / 4]);
    if constexpr (C == 8) {
        const bool odd = lane & 8;
        const float keep = odd ? q[1] : q[0], give = odd ? q[0] : q[1];
        return keep + __shfl_xor(give, 8);
    }
    return LANES == 8 ? q[0] + __shfl_xor(q[0], 8) : q[0];      // (eight lanes to an fp32 row: every column twice)
}
template <typename T, int ROW>
__device__ __forceinline__ int my_column(int lane) {
    if constexpr (sizeof(T) == 2) return 8 * (lane & 7) + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1);
    return 4 * (lane % (ROW / 4)) + 2 * (lane >> 5) + ((lane >> 4) & 1);
}

// X_out rows from the forward work list; pieces of split rows go to `partial` (P floats each).
__global__ __launch_bounds__(kBlock) void narrow_forward_kernel(const SpmmItem* items, int32_t n_items, const VarcoEdge* edge, const float* vals,
                                                                const bf16_t* y, int32_t rows, bf16_t* out, int32_t fo, float* partial) {
    const int lane = threadIdx.x & 63;
    const int32_t idx = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6));
    if (idx >= n_items) return;
    const SpmmItem it = items[idx];
    const float x = narrow_sum<bf16_t, P>(y, P, P, it.e0, it.e1, lane, [&](int32_t e) {
        const VarcoEdge ed = edge[e];
        return make_uint2(uint32_t(ed.gid < 0 ? ed.src : rows + ed.src), __float_as_uint(vals[e]));
    });
    const int c = my_column<bf16_t, P>(lane);
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

// G_loc[row] and G_z[zrow of row] (zeros beyond fo), rows g_ld apart. SPLIT = false: partial sums of the pieces of long ranges (the
// launch's first wavefronts) and the nodes without pieces; SPLIT = true: the others, from the partial sums. bf16 rows of 2 ROW elements
// hold a sum as two terms, x = g[c] + g[ROW + c]: 16 of its bits.
template <typename T, int ROW, bool SPLIT>
__global__ __launch_bounds__(kBlock) void narrow_backward_kernel(const NodeItem* nodes, int32_t n, const SpmmItem* pieces, int32_t n_pieces,
                                                                 const uint2* t_local, const uint2* t_cross, const T* dz, int32_t ld,
                                                                 const int32_t* zrow_of, T* g_loc, T* g_z, int32_t g_ld, int32_t fo, float* partial) {
    const int lane = threadIdx.x & 63, c = my_column<T, ROW>(lane);
    const int32_t cols = min(ld, ROW);                 // rows that are not padded have no more
    int32_t idx = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6));
    if constexpr (!SPLIT) {
        if (idx < n_pieces) {
            const SpmmItem it = pieces[idx];
            const uint2* pairs = it.row == 0 ? t_local : t_cross;
            partial[int64_t(it.dst) * ROW + c] = narrow_sum<T, ROW>(dz, ld, cols, it.e0, it.e1, lane, [&](int32_t e) { return pairs[e]; });
            return;
        }
        idx -= n_pieces;
    }
    if (idx >= n) return;
    const NodeItem it = nodes[idx];
    auto range = [&](const uint2* pairs, int32_t e0, int32_t e1, bool split) {
        float x = 0.f;
        if (SPLIT && split)
            for (int32_t s = e0; s < e1; ++s) x += partial[int64_t(s) * ROW + c];
        else
            x = narrow_sum<T, ROW>(dz, ld, cols, e0, e1, lane, [&](int32_t e) { return pairs[e]; });
        return c < fo ? x : 0.f;
    };
    auto put = [&](T* at, float x) {
        Elem<T>::store(at, x);
        if constexpr (sizeof(T) == 2) {
            const float high = bf16_to_float(float_to_bf16(x));
            if (g_ld > ROW) Elem<T>::store(at + ROW, fabsf(high) < __builtin_inff() ? x - high : 0.f);      // (infinities and NaN are the first term's)
        }
    };
    const int32_t zr = zrow_of[it.row];
    put(g_loc + int64_t(it.row) * g_ld + c, range(t_local, it.l0, it.l1, it.flags & VARCO_NODE_LOCAL_SPLIT));
    if (g_z && zr >= 0) put(g_z + int64_t(zr) * g_ld + c, range(t_cross, it.c0, it.c1, it.flags & VARCO_NODE_CROSS_SPLIT));
}

// Rows of fo elements -> rows of ROW elements, zeros beyond fo. A thread writes 16 bytes; a piece that crosses a row's end is loaded
// from before it and moved up. (2,449,029 rows of 47 bf16 elements: 85 us, 212 element by element.)
template <typename T, int ROW>
__global__ __launch_bounds__(kBlock) void pad_rows_kernel(const T* __restrict__ in, int64_t n, int32_t fo, T* __restrict__ out) {
    constexpr int C = Columns<T>::N, PIECES = ROW / C;
    const int64_t total = n * PIECES, stride = int64_t(gridDim.x) * kBlock;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < total; i += stride) {
        const int64_t row = i / PIECES;
        const int c = int(i % PIECES) * C, over = c + C - fo;
        const T* const from = in + row * fo;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (over < C) {
            if (fo >= C) {
                v = load8_any(reinterpret_cast<const char*>(from + (over > 0 ? fo - C : c)));
                if (over > 0) v = moved_up<T>(v, over);
            } else {
                uint32_t u[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < C; ++j)
                    if (j < fo) u[j * 4 / C] |= bits_of(from[j]) << (32 * 4 / C * (j % (C / 4)) & 31);
                v = make_uint4(u[0], u[1], u[2], u[3]);
            }
        }
        reinterpret_cast<uint4*>(out)[i] = v;
    }
}

// dX[v] = G_loc[v] H^T + kept positions of (G_z[v] H^T). A workgroup of eight wavefronts walks tiles of 64 rows; a wavefront holds the
// weights of 64 positions ([position][column], at most 64 columns) as matrix operands in registers, the groups of positions are
// dealt to the wavefronts and, with fewer than eight groups, the two blocks of 32 rows as well. The weights are the first matrix
// operand, which leaves positions of one row in a lane: its rule is read once, the places of positions next to each other differ by a_inv
// (an addition and a wrap instead of a multiplication and a division by the width for each), and four results are packed at a time.
// They leave through the wavefront's own strip of LDS as whole lines. One barrier per tile; the rows of the next tile, and the
// places of the one after it, are on their way meanwhile. Bound by writing dX: 2,449,029 x 512 from 47 outputs 606 us (rows of the
// result first, four wavefronts of 128 positions, the rule worked out for each element: 1,530), 169,343 x 512 from 40 47 us (104).
// Sums in two terms take one LDS buffer and a second barrier per tile: 756 us, and narrow_backward_kernel before it 2,527 instead of 2,391.
constexpr int kWide = 512, kMaxWidth = 512, kTile = 64, kPitchG = P + 8, kStrip = 64 + 8;
template <int TERMS>
struct alignas(16) ClassLds {
    static constexpr int BUFS = 3 - TERMS;        // as many as leave room for two workgroups
    uint16_t strips[kWide / 64][32 * kStrip];
    uint16_t g[BUFS][2 * TERMS][kTile * kPitchG];      // [buffer][terms of G_loc, of G_z]
    uint2 rows_ab[BUFS][kTile];                   // {a_inv, b}; a_inv = 0: every position kept (nothing came back, or everything)
};
template <int TERMS>
__global__ __launch_bounds__(kWide, 4) void class_dgrad_kernel(const uint16_t* __restrict__ g_loc, const uint16_t* __restrict__ g_z,
                                                               const int32_t* __restrict__ zrow_of, const int32_t* __restrict__ bgid, int32_t n,
                                                               MaskRule rule, int32_t fo, const uint16_t* __restrict__ wr, int32_t cpitch,
                                                               uint16_t* __restrict__ dx) {
    extern __shared__ __attribute__((aligned(16))) char class_lds[];
    using Lds = ClassLds<TERMS>;
    Lds& lds = *reinterpret_cast<Lds*>(class_lds);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6)), lrow = lane & 31, lk = lane >> 5;
    const int32_t width = int32_t(rule.width);
    const int ksteps = (fo + 15) / 16;
    const int groups = width > 256 ? 8 : width > 128 ? 4 : width > 64 ? 2 : 1;
    const int32_t first = wave % groups * 64;
    auto frag = [](const uint16_t* p) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p)); };
    bf16x8 wf[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int32_t pos = first + b * 32 + lrow;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            wf[b][s] = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
            const int32_t c0 = 16 * s + 8 * lk;
            if (s < ksteps && pos < width && c0 + 8 <= cpitch) wf[b][s] = frag(wr + int64_t(pos) * cpitch + c0);
        }
    }
    const int32_t n_tiles = (n + kTile - 1) / kTile, step = int32_t(gridDim.x);
    const int fr = threadIdx.x >> 3, fc = (threadIdx.x & 7) * 8;      // this thread's 16-byte piece of a tile of G: row, first column
    auto row_of = [&](int32_t t) { return min(t * kTile + fr, n - 1); };
    uint4 nl, nz, nl2, nz2;                       // (the last two: second terms)
    int32_t nzr = -1, ngid = 0;
    int32_t after = g_z && int32_t(blockIdx.x) < n_tiles ? zrow_of[row_of(blockIdx.x)] : -1;
    auto fetch = [&](int32_t t) {
        nzr = after;
        const uint16_t* const gl = g_loc + int64_t(row_of(t)) * (TERMS * P) + fc;
        nl = *reinterpret_cast<const uint4*>(gl), nz = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (TERMS == 2) nl2 = *reinterpret_cast<const uint4*>(gl + P), nz2 = nz;
        if (nzr >= 0) {
            const uint16_t* const gz = g_z + int64_t(nzr) * (TERMS * P) + fc;
            nz = *reinterpret_cast<const uint4*>(gz), ngid = bgid[nzr];
            if constexpr (TERMS == 2) nz2 = *reinterpret_cast<const uint4*>(gz + P);
        }
        if (g_z && t + step < n_tiles) after = zrow_of[row_of(t + step)];
    };
    if (int32_t(blockIdx.x) < n_tiles) fetch(blockIdx.x);
    int buf = 0;
    for (int32_t t = blockIdx.x; t < n_tiles; t += step, buf ^= Lds::BUFS - 1) {      // (of two buffers, one is written again behind the next tile's barrier)
        *reinterpret_cast<uint4*>(&lds.g[buf][0][fr * kPitchG + fc]) = nl;
        *reinterpret_cast<uint4*>(&lds.g[buf][TERMS][fr * kPitchG + fc]) = nz;
        if constexpr (TERMS == 2) {
            *reinterpret_cast<uint4*>(&lds.g[buf][1][fr * kPitchG + fc]) = nl2;
            *reinterpret_cast<uint4*>(&lds.g[buf][3][fr * kPitchG + fc]) = nz2;
        }
        if (fc == 0) {
            uint2 ab = make_uint2(0u, 0u);
            if (nzr >= 0 && rule.k < rule.width) {
                const MaskAffine m = varco_affine(rule, uint32_t(ngid));
                ab = make_uint2(m.a_inv, m.b);
            }
            lds.rows_ab[buf][fr] = ab;
        }
        __syncthreads();
        if (t + step < n_tiles) fetch(t + step);
        for (int rb = wave / groups; rb < kTile / 32 && first < width; rb += 8 / groups) {
            const int32_t row0 = t * kTile + rb * 32, rows = min(32, n - row0);
            if (rows <= 0) break;
            const uint2 ab = lds.rows_ab[buf][rb * 32 + lrow];
            const uint32_t p0 = uint32_t(first + 4 * lk), a8 = varco_mod_width(8u * ab.x, rule.width, rule.width_magic);
            uint32_t q8 = varco_mod_width(ab.x * (p0 + rule.width - ab.y), rule.width, rule.width_magic);
            uint16_t* const strip = lds.strips[wave];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                floatx16 al, az;
#pragma unroll
                for (int v = 0; v < 16; ++v) al[v] = az[v] = 0.f;
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (s < ksteps) {
                        const int at = (rb * 32 + lrow) * kPitchG + 16 * s + 8 * lk;
#pragma unroll
                        for (int m = 0; m < TERMS; ++m) {
                            al = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[b][s], frag(&lds.g[buf][m][at]), al, 0, 0, 0);
                            az = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[b][s], frag(&lds.g[buf][TERMS + m][at]), az, 0, 0, 0);
                        }
                    }
                // accumulator register v of a lane is position 8 * (v / 4) + 4 * (lane / 32) + v % 4 of row lane % 32
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float x[4];
                    uint32_t q = q8;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        x[i] = al[4 * g + i] + (q < rule.k ? az[4 * g + i] : 0.f);
                        q += ab.x, q = min(q, q - rule.width);
                    }
                    q8 += a8, q8 = min(q8, q8 - rule.width);
                    *reinterpret_cast<uint2*>(strip + lrow * kStrip + 32 * b + 8 * g + 4 * lk) = make_uint2(bf16_pair(x[0], x[1]), bf16_pair(x[2], x[3]));
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int sr = lane >> 3, sc = (lane & 7) * 8;                // width is a multiple of 16
            if (first + sc < width)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (sr + 8 * i < rows)
                        *reinterpret_cast<uint4*>(dx + int64_t(row0 + sr + 8 * i) * width + first + sc) =
                            *reinterpret_cast<const uint4*>(strip + (sr + 8 * i) * kStrip + sc);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if constexpr (Lds::BUFS == 1) __syncthreads();
    }
}

// The same for fp32 storage, with the self tap of a SAGE layer: dX[v] = G_loc[v] H1^T + kept positions of (G_z[v] H1^T) (+ dZ[v] H0^T)
// from two scaled fp16 terms per operand (kernels_gemm_half.hip), three where at most 16 columns are summed: there the rounding of the
// terms does not average out (128 positions from 3 columns: Frobenius error 9.2e-8 with two, 7.0e-8 with three, 8.4e-8 for sums over
// products formed in fp32). A workgroup of eight wavefronts walks tiles of ROWS rows; a wavefront holds the weights of 32 positions as
// matrix operands in registers. 16 or 8 lanes take a row of each source, agree on its scale and write the terms to LDS once for all
// wavefronts. The cross product comes first and is cleared where nothing came back, so that all three are summed in the same registers;
// 128 of them hold everything of two workgroups per compute unit. Sources of a row, and taps of a position, share a scale unless one is
// more than 2^8 smaller than the largest; that one is scaled by itself, sources up to 2^64 and taps up to 2^24 further (then its error is
// 2^-108, 2^-68 of the largest), and the sums follow from scale to scale. (One scale for all lost the errors of a node's own partition
// at positions that larger remote ones do not reach: 2^35 between them, relative error 4e-4.) Bound by
// writing dX and reading the three sources: 2,449,029 x 256 from 47 outputs with both taps 0.96 ms (1.45 with rows of the result first,
// one workgroup per compute unit and dependent loads at each tile), 169,343 x 256 from 40 outputs 61 us (74).
// Wavefronts per SIMD: two workgroups are resident where 128 registers hold the weights, the sums and the next tile (and the LDS allows).
constexpr int class_waves(int ks, int rows, bool self) { return !self || ks < (rows == 32 ? 4 : 3) ? 4 : 2; }
constexpr int kStripF = 32 + 4;
template <int KS, int ROWS, bool SELF>
struct alignas(16) ClassLdsF32 {
    static constexpr int TERMS = KS == 1 ? 3 : 2, kTile = (SELF ? 3 : 2) * TERMS * ROWS * (16 * KS + 8), kStrips = kWide / 64 * 32 * kStripF;
    static constexpr int BUFS = 2 * 2 * kTile + 4 * kStrips + 32 * ROWS + 4 * 256 <= 80 * 1024 ? 2 : 1;      // two where two workgroups still fit
    float strips[kWide / 64][32 * kStripF];
    uint16_t tile[BUFS][kTile];                   // [source][term][row][column]
    // {a_inv, b, scale of the last source, steps of the scale to the second and the third source (16 bits each)};
    // a_inv = 0: every position kept (nothing came back, or everything)
    uint4 rows[BUFS][ROWS];
    int32_t eb[kWide / 64][32];                   // of each position's weights: scale of the last tap (16 bits), step of the scale to it
};
// Scale of a source or tap beside the largest one's. Sums are below 2^38 at the scale of the largest (three sources of 64 products of
// 2^30), so that the furthest steps of both together keep them finite.
constexpr int kApart = 8, kSourceSteps = 64, kTapSteps = 24;
__device__ __forceinline__ int own_scale(float largest, int shared, int most) {
    const int e = scale_exponent(largest, kHalfTop);
    return largest > 0.f && e > shared + kApart ? min(e, shared + most) : shared;
}
template <int KS, int ROWS, int ROW, bool SELF>
__global__ __launch_bounds__(kWide, class_waves(KS, ROWS, SELF)) void class_dgrad_f32_kernel(const float* __restrict__ g_loc, const float* __restrict__ g_z,
                                                                    const float* __restrict__ dz, int32_t dz_ld, const int32_t* __restrict__ zrow_of,
                                                                    const int32_t* __restrict__ bgid, int32_t n, MaskRule rule, int32_t fo,
                                                                    const float* __restrict__ h1, const float* __restrict__ h0, float* __restrict__ dx, bool vec) {
    constexpr int S = SELF ? 3 : 2, kRow = 16 * KS + 8, kPlane = ROWS * kRow;         // sources: G_loc, G_z, dZ
    constexpr int LANES = ROW / 4, kPass = kWide / LANES, N = (ROWS + kPass - 1) / kPass;      // rows per pass, passes
    static_assert(LANES == 8 || LANES == 16, "rows of 32 or 64 values");
    using Lds = ClassLdsF32<KS, ROWS, SELF>;
    constexpr int BUFS = Lds::BUFS, TERMS = Lds::TERMS;
    extern __shared__ __attribute__((aligned(16))) char class_lds[];
    Lds& lds = *reinterpret_cast<Lds*>(class_lds);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6)), lcol = lane & 31, lk = lane >> 5;
    const int32_t width = int32_t(rule.width), first = int32_t(blockIdx.y) * 256;
    // groups of 32 positions; with fewer than eight the blocks of rows are dealt as well
    const int groups = width - first > 128 ? 8 : width - first > 64 ? 4 : width - first > 32 ? 2 : 1;
    const int32_t pos0 = first + wave % groups * 32, pos = pos0 + lcol;

    // operands: lane holds H[position][16 s + 8 lk .. + 7], both terms
    uint4 w[SELF ? 2 : 1][KS][TERMS];
    bool taps_apart;
    {
        float x[SELF ? 2 : 1][KS][8], m[2] = {0.f, 0.f};
#pragma unroll
        for (int tap = 0; tap < (SELF ? 2 : 1); ++tap)
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int k = 16 * s + 8 * lk + i;
                    x[tap][s][i] = pos < width && k < fo ? (tap ? h0 : h1)[int64_t(pos) * fo + k] : 0.f;
                    m[tap] = fmaxf(m[tap], fabsf(x[tap][s][i]));
                }
        int32_t eb[2];
        {
            m[0] = fmaxf(m[0], __shfl_xor(m[0], 32)), m[1] = fmaxf(m[1], __shfl_xor(m[1], 32));
            const int32_t shared = scale_exponent(fmaxf(m[0], m[1]), kHalfTop);
            eb[0] = own_scale(m[0], shared, kTapSteps), eb[1] = own_scale(m[1], shared, kTapSteps);
        }
        const int32_t last = SELF ? eb[1] : eb[0], by = last - eb[0];
        if (lk == 0) lds.eb[wave][lcol] = (last & 0xFFFF) | by << 16;      // (read by this wavefront only, behind the first tile's barrier)
        taps_apart = __any(by != 0);
#pragma unroll
        for (int tap = 0; tap < (SELF ? 2 : 1); ++tap)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const float sc = power_of_two(eb[tap]);
                uint32_t hi[4], lo[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) split_pair(x[tap][s][2 * i] * sc, x[tap][s][2 * i + 1] * sc, hi[i], lo[i]);
                w[tap][s][0] = make_uint4(hi[0], hi[1], hi[2], hi[3]), w[tap][s][1] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                if constexpr (TERMS == 3) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) lo[i] = third_pair(x[tap][s][2 * i] * sc, x[tap][s][2 * i + 1] * sc, hi[i], lo[i]);
                    w[tap][s][2] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                }
            }
    }

    const int32_t n_tiles = (n + ROWS - 1) / ROWS, step = int32_t(gridDim.x);
    const int fr = threadIdx.x / LANES, fc = (threadIdx.x % LANES) * 4;               // rows fr + kPass h, columns fc .. fc + 3
    auto row_of = [&](int32_t t, int h) { return uint32_t(min(min(fr + kPass * h, ROWS - 1), n - 1 - t * ROWS)); };     // within the tile
    float4 next[N][S];
    int32_t next_gid[N], after[N];
    auto places = [&](int32_t t) {
#pragma unroll
        for (int h = 0; h < N; ++h) after[h] = g_z ? (zrow_of + t * ROWS)[row_of(t, h)] : -1;
    };
    auto fetch = [&](int32_t t) {
#pragma unroll
        for (int h = 0; h < N; ++h) {
            uint32_t row = row_of(t, h);
            asm volatile("" : "+v"(row));
            next_gid[h] = -1;
            next[h][0] = *reinterpret_cast<const float4*>(g_loc + int64_t(t) * (ROWS * ROW) + (row * ROW + uint32_t(fc)));
            next[h][1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (after[h] >= 0) next[h][1] = *reinterpret_cast<const float4*>(g_z + int64_t(after[h]) * ROW + fc), next_gid[h] = bgid[after[h]];
            if constexpr (SELF) {
                next[h][2] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (fc < dz_ld) next[h][2] = *reinterpret_cast<const float4*>(dz + int64_t(t) * ROWS * dz_ld + (row * uint32_t(dz_ld) + uint32_t(fc)));
            }
        }
        if (t + step < n_tiles) places(t + step);
    };
    if (int32_t(blockIdx.x) < n_tiles) {
        places(blockIdx.x);
        fetch(blockIdx.x);
    }
    int buf = 0;
    for (int32_t t = blockIdx.x; t < n_tiles; t += step, buf ^= BUFS - 1) {    // (a second buffer is written again behind the next tile's barrier)
        uint16_t* const tile = lds.tile[buf];
#pragma unroll
        for (int h = 0; h < N; ++h) {
            float m[S], most = 0.f;
#pragma unroll
            for (int s = 0; s < S; ++s) {                    // (all lanes of a row are here)
                m[s] = largest_of_lanes<LANES>(fmaxf(fmaxf(fabsf(next[h][s].x), fabsf(next[h][s].y)), fmaxf(fabsf(next[h][s].z), fabsf(next[h][s].w))));
                m[s] = m[s] < __builtin_inff() ? m[s] : 0.f;         // an infinite source says nothing about the others' scale, and is NaN at any
                most = fmaxf(most, m[s]);
            }
            int e[S];
#pragma unroll
            for (int s = 0; s < S; ++s) e[s] = own_scale(m[s], scale_exponent(most, kHalfTop), kSourceSteps);
            const int r = fr + kPass * h;
            if (r < ROWS && fc < 16 * KS) {
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const float sc = power_of_two(e[s]);
                    uint32_t hi[2], lo[2];
                    split_pair(next[h][s].x * sc, next[h][s].y * sc, hi[0], lo[0]);
                    split_pair(next[h][s].z * sc, next[h][s].w * sc, hi[1], lo[1]);
                    *reinterpret_cast<uint2*>(&tile[(TERMS * s) * kPlane + r * kRow + fc]) = make_uint2(hi[0], hi[1]);
                    *reinterpret_cast<uint2*>(&tile[(TERMS * s + 1) * kPlane + r * kRow + fc]) = make_uint2(lo[0], lo[1]);
                    if constexpr (TERMS == 3)
                        *reinterpret_cast<uint2*>(&tile[(TERMS * s + 2) * kPlane + r * kRow + fc]) =
                            make_uint2(third_pair(next[h][s].x * sc, next[h][s].y * sc, hi[0], lo[0]), third_pair(next[h][s].z * sc, next[h][s].w * sc, hi[1], lo[1]));
                }
            }
            if (r < ROWS && fc == 0) {
                uint2 ab = make_uint2(0u, 0u);
                if (next_gid[h] >= 0 && rule.k < rule.width) {
                    const MaskAffine a = varco_affine(rule, uint32_t(next_gid[h]));
                    ab = make_uint2(a.a_inv, a.b);
                }
                lds.rows[buf][r] = make_uint4(ab.x, ab.y, uint32_t(e[SELF ? 2 : 0]), (uint32_t(e[0] - e[1]) & 0xFFFFu) | uint32_t(e[SELF ? 2 : 0] - e[0]) << 16);
            }
        }
        __syncthreads();
        if (t + step < n_tiles) fetch(t + step);
        for (int rb = wave / groups; rb < ROWS / 32 && pos0 < width; rb += 8 / groups) {
            const int32_t row0 = t * ROWS + rb * 32, rows = min(32, n - row0);
            if (rows <= 0) break;
            floatx16 sum, low;
            int me = lane;
            asm volatile("" : "+v"(me));              // addresses are formed where they are used
            const int lcol = me & 31, lk = me >> 5;
            const int frag_at = (rb * 32 + lcol) * kRow + 8 * lk;
            auto frag = [&](int source, int term, int s) {
                return __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4*>(&tile[(TERMS * source + term) * kPlane + frag_at + 16 * s]));
            };
            auto product = [&](int source, int tap) {
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const halfx8 a0 = frag(source, 0, s), a1 = frag(source, 1, s);
                    const halfx8 b0 = __builtin_bit_cast(halfx8, w[tap][s][0]), b1 = __builtin_bit_cast(halfx8, w[tap][s][1]);
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(b0, a0, sum, 0, 0, 0);
                    low = __builtin_amdgcn_mfma_f32_32x32x16_f16(b1, a0, low, 0, 0, 0);
                    low = __builtin_amdgcn_mfma_f32_32x32x16_f16(b0, a1, low, 0, 0, 0);
                    if constexpr (TERMS == 3) {
                        const halfx8 a2 = frag(source, 2, s), b2 = __builtin_bit_cast(halfx8, w[tap][s][2]);
                        low = __builtin_amdgcn_mfma_f32_32x32x16_f16(b1 * _Float16(1.f / kHalfLow), a1, low, 0, 0, 0);
                        low = __builtin_amdgcn_mfma_f32_32x32x16_f16(b2, a0, low, 0, 0, 0);
                        low = __builtin_amdgcn_mfma_f32_32x32x16_f16(b0, a2, low, 0, 0, 0);
                    }
                }
            };
            // accumulator register v of a lane is position 8 * (v / 4) + 4 * (lane / 32) + v % 4 of row lane % 32
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[v] = low[v] = 0.f;
            const int32_t steps = int32_t(lds.rows[buf][rb * 32 + lcol].w);      // of the scale of the row's sums
            if (g_z) {                                // first, and dropped where the row's message did not carry it
                product(1, 0);
                const uint2 ab = *reinterpret_cast<const uint2*>(&lds.rows[buf][rb * 32 + lcol]);
                const uint32_t a_inv = ab.x, at = ab.y, p0 = uint32_t(pos0 + 4 * lk);
                const uint32_t a8 = varco_mod_width(8u * a_inv, rule.width, rule.width_magic);
                uint32_t q8 = varco_mod_width(a_inv * (p0 >= at ? p0 - at : p0 + rule.width - at), rule.width, rule.width_magic);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint32_t q = q8;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (q >= rule.k) sum[4 * g + i] = low[4 * g + i] = 0.f;
                        q += a_inv, q = min(q, q - rule.width);
                    }
                    q8 += a8, q8 = min(q8, q8 - rule.width);
                }
                if (__any(int16_t(steps))) {
                    const float f = power_of_two(int16_t(steps));
#pragma unroll
                    for (int v = 0; v < 16; ++v) sum[v] *= f, low[v] *= f;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            product(0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (SELF) {
                if (taps_apart || __any(steps >> 16)) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float f = power_of_two((steps >> 16) + (lds.eb[wave][8 * (v >> 2) + 4 * lk + (v & 3)] >> 16));
                        sum[v] *= f, low[v] *= f;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                product(2, 1);
            }
            float* const strip = lds.strips[wave];
            const int32_t row_scale = int32_t(lds.rows[buf][rb * 32 + lcol].z);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int4 eb = *reinterpret_cast<const int4*>(&lds.eb[wave][8 * g + 4 * lk]);
                const int32_t e[4] = {int16_t(eb.x), int16_t(eb.y), int16_t(eb.z), int16_t(eb.w)};
                float y[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    y[i] = __builtin_ldexpf(sum[4 * g + i] + low[4 * g + i] * (1.f / kHalfLow), -(row_scale + e[i]));
                *reinterpret_cast<float4*>(strip + lcol * kStripF + 8 * g + 4 * lk) = make_float4(y[0], y[1], y[2], y[3]);
                __builtin_amdgcn_sched_barrier(0);            // (a group's scales are read when it is its turn)
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            float* const out = dx + int64_t(row0) * width + pos0;
            if (vec) {                                // a scalar per row and one offset per lane
                const int sr = me >> 3, sc = (me & 7) * 4;
                const uint32_t lane_off = uint32_t(sr) * uint32_t(width) + uint32_t(sc);
                if (pos0 + sc < width)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (sr + 8 * i < rows)
                            *reinterpret_cast<float4*>(out + int64_t(8 * i) * width + lane_off) = *reinterpret_cast<const float4*>(strip + (sr + 8 * i) * kStripF + sc);
            } else if (pos < width) {
                for (int r = lk; r < rows; r += 2) out[int64_t(r) * width + lcol] = strip[r * kStripF + lcol];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if constexpr (BUFS == 1) __syncthreads();
    }
}

dim3 waves_for(int64_t n) { return dim3(unsigned((n + kWaves - 1) / kWaves)); }

}  // namespace

hipError_t varco_launch_narrow_forward(const SpmmPlan& plan, const VarcoEdge* edge, const float* vals, const void* y, int32_t rows, void* out,
                                       int32_t fo, float* partial, hipStream_t stream, const LaunchTag& tag) {
    if (plan.n_items == 0) return hipSuccess;
    tag.begin(stream);
    hipLaunchKernelGGL(narrow_forward_kernel, waves_for(plan.n_items), dim3(kBlock), 0, stream, plan.items, plan.n_items, edge, vals,
                       static_cast<const bf16_t*>(y), rows, static_cast<bf16_t*>(out), fo, partial);
    tag.end(stream);
    if (plan.n_splits > 0) {
        tag.begin_as(VARCO_K_REDUCE, stream, 4.0 * plan.n_partials * P);
        hipLaunchKernelGGL(narrow_fixup_kernel, waves_for(plan.n_splits), dim3(kBlock), 0, stream, plan.splits, plan.n_splits, partial,
                           static_cast<bf16_t*>(out), fo);
        tag.end(stream);
    }
    return hipGetLastError();
}

namespace {
template <typename T, int ROW>
hipError_t narrow_backward(const NodePlan& plan, const uint2* t_local, const uint2* t_cross, const void* dz, int64_t rows, const int32_t* zrow_of,
                           void* dz_padded, void* g_loc, void* g_z, int32_t g_ld, int32_t fo, float* partial, hipStream_t stream) {
    const T* const src = static_cast<const T*>(dz_padded);
    const int32_t ld = dz_padded == dz ? fo : ROW;
    if (dz_padded != dz)
        hipLaunchKernelGGL((pad_rows_kernel<T, ROW>), dim3(unsigned(std::min<int64_t>((rows * ROW / Columns<T>::N + kBlock - 1) / kBlock, 256 * 32))), dim3(kBlock), 0, stream,
                           static_cast<const T*>(dz), rows, fo, static_cast<T*>(dz_padded));
    hipLaunchKernelGGL((narrow_backward_kernel<T, ROW, false>), waves_for(int64_t(plan.n_pieces) + plan.n_whole), dim3(kBlock), 0, stream, plan.nodes,
                       plan.n_whole, plan.pieces, plan.n_pieces, t_local, t_cross, src, ld, zrow_of, static_cast<T*>(g_loc), static_cast<T*>(g_z), g_ld, fo, partial);
    if (plan.n_nodes > plan.n_whole)
        hipLaunchKernelGGL((narrow_backward_kernel<T, ROW, true>), waves_for(plan.n_nodes - plan.n_whole), dim3(kBlock), 0, stream,
                           plan.nodes + plan.n_whole, plan.n_nodes - plan.n_whole, plan.pieces, 0, t_local, t_cross, src, ld, zrow_of,
                           static_cast<T*>(g_loc), static_cast<T*>(g_z), g_ld, fo, partial);
    return hipGetLastError();
}
}  // namespace

hipError_t varco_launch_narrow_backward(int dtype, const NodePlan& plan, const uint2* t_local, const uint2* t_cross, const void* dz, int64_t rows,
                                        const int32_t* zrow_of, void* dz_padded, void* g_loc, void* g_z, bool two_terms, int32_t fo, float* partial,
                                        hipStream_t stream, const LaunchTag& tag) {
    if (plan.n_nodes == 0) return hipSuccess;
    if (two_terms && dtype != VARCO_BF16) return hipErrorInvalidValue;
    tag.begin(stream);
    const int32_t g_ld = varco_class_pitch(dtype, fo) * (two_terms ? 2 : 1);
    auto go = [&](auto fn) { return fn(plan, t_local, t_cross, dz, rows, zrow_of, dz_padded, g_loc, g_z, g_ld, fo, partial, stream); };
    const hipError_t e = dtype == VARCO_BF16 ? go(narrow_backward<bf16_t, 64>) : varco_class_pitch(dtype, fo) == 32 ? go(narrow_backward<float, 32>) : go(narrow_backward<float, 64>);
    tag.end(stream);
    return e;
}

hipError_t varco_launch_class_dgrad(const void* g_loc, const void* g_z, bool two_terms, const int32_t* zrow_of, const int32_t* bgid, int64_t rows,
                                    const MaskRule& rule, int32_t fo, const void* wr, int32_t cpitch, void* dx, hipStream_t stream,
                                    const LaunchTag& tag) {
    if (rows == 0) return hipSuccess;
    if (rule.width % 16 != 0 || rule.width > uint32_t(kMaxWidth) || fo > P || cpitch < fo || cpitch % 8 != 0 || (reinterpret_cast<uintptr_t>(dx) & 15u))
        return hipErrorInvalidValue;
    auto go = [&](auto terms) {
        using Lds = ClassLds<decltype(terms)::value>;
        const auto kernel = class_dgrad_kernel<decltype(terms)::value>;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(sizeof(Lds)));
        if (e != hipSuccess) return e;
        tag.begin(stream);
        const int64_t tiles = (rows + kTile - 1) / kTile;
        hipLaunchKernelGGL(kernel, dim3(unsigned(std::min<int64_t>(tiles, 512))), dim3(kWide), sizeof(Lds), stream, static_cast<const uint16_t*>(g_loc),
                           static_cast<const uint16_t*>(g_z), zrow_of, bgid, int32_t(rows), rule, fo, static_cast<const uint16_t*>(wr), cpitch,
                           static_cast<uint16_t*>(dx));
        tag.end(stream);
        return hipGetLastError();
    };
    return two_terms ? go(std::integral_constant<int, 2>{}) : go(std::integral_constant<int, 1>{});
}

hipError_t varco_launch_class_dgrad_f32(const void* g_loc, const void* g_z, const void* dz, int32_t dz_ld, const int32_t* zrow_of, const int32_t* bgid, int64_t rows,
                                        const MaskRule& rule, int32_t fo, const void* h1, const void* h0, void* dx, hipStream_t stream,
                                        const LaunchTag& tag) {
    if (rows == 0) return hipSuccess;
    if (fo < 1 || fo > 64) return hipErrorInvalidValue;
    tag.begin(stream);
    hipError_t err = hipSuccess;
    const bool vec = rule.width % 4 == 0 && (reinterpret_cast<uintptr_t>(dx) & 15u) == 0;
    auto go = [&](auto ks, auto tile, auto row, auto self) {
        constexpr int ROWS = decltype(tile)::value;
        const int64_t tiles = (rows + ROWS - 1) / ROWS, slices = (rule.width + 255) / 256;
        const dim3 grid{unsigned(std::min<int64_t>(tiles, std::max<int64_t>(1, 128 * class_waves(decltype(ks)::value, ROWS, decltype(self)::value) / slices))), unsigned(slices)};
        using Lds = ClassLdsF32<decltype(ks)::value, ROWS, decltype(self)::value>;
        const auto kernel = class_dgrad_f32_kernel<decltype(ks)::value, ROWS, decltype(row)::value, decltype(self)::value>;
        if (sizeof(Lds) > 64 * 1024) err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(sizeof(Lds)));
        if (err != hipSuccess) return;
        hipLaunchKernelGGL(kernel, grid, dim3(kWide), sizeof(Lds), stream,
                           static_cast<const float*>(g_loc), static_cast<const float*>(g_z), static_cast<const float*>(dz), dz_ld, zrow_of, bgid, int32_t(rows),
                           rule, fo, static_cast<const float*>(h1), static_cast<const float*>(h0), static_cast<float*>(dx), vec);
    };
    using std::integral_constant;
    auto with_self = [&](auto ks, auto tile, auto row) {
        if (h0)
            go(ks, tile, row, std::true_type{});
        else
            go(ks, tile, row, std::false_type{});
    };
    auto with_tile = [&](auto ks, auto row) {        // at most 128 positions occupy half of the wavefronts: tiles of two blocks of rows then
        if (rule.width > 128)
            with_self(ks, integral_constant<int, 32>{}, row);
        else
            with_self(ks, integral_constant<int, 64>{}, row);
    };
    switch ((fo + 15) / 16) {
        case 1: with_tile(integral_constant<int, 1>{}, integral_constant<int, 32>{}); break;
        case 2: with_tile(integral_constant<int, 2>{}, integral_constant<int, 32>{}); break;
        case 3: with_tile(integral_constant<int, 3>{}, integral_constant<int, 64>{}); break;
        default: with_tile(integral_constant<int, 4>{}, integral_constant<int, 64>{}); break;
    }
    tag.end(stream);
    return err != hipSuccess ? err : hipGetLastError();
}
