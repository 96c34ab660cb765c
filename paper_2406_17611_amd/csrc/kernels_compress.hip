// Encoder and decoder of Definition 1 / Appendix "Compression Mechanism": keep k keyed-random elements of
// each node vector; decode by writing them in place and zero elsewhere (no rescale). Pure data movement:
// HBM-bound, no index bytes are stored or read. A power-of-two group of lanes serves one row, so that
// narrow messages (k of 4..32) still fill the 64-wide wavefront with several rows.
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "mask_device.h"

namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ float vec_elem(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
__device__ __forceinline__ float vec_elem(const float2& v, int i) { return i == 0 ? v.x : v.y; }
__device__ __forceinline__ float vec_elem(const float& v, int) { return v; }

__device__ __forceinline__ int64_t group_row(int g_log2) {
    return (int64_t(blockIdx.x) * kBlock + threadIdx.x) >> g_log2;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void compress_kernel(MaskRule rule, const int32_t* __restrict__ gids,
                                                          const int32_t* __restrict__ rows, int64_t n_rows,
                                                          const T* __restrict__ x, int64_t ldx,
                                                          T* __restrict__ z, int g_log2) {
    const uint32_t g = 1u << g_log2;
    const uint32_t gl = threadIdx.x & (g - 1);
    const int64_t stride = (int64_t(gridDim.x) * kBlock) >> g_log2;
    for (int64_t row = group_row(g_log2); row < n_rows; row += stride) {
        const int64_t src = rows ? int64_t(rows[row]) : row;
        const T* xr = x + src * ldx;
        T* zr = z + row * int64_t(rule.k);
        const MaskAffine m = varco_affine(rule, uint32_t(gids[row]));
        for (uint32_t j = gl; j < rule.k; j += g) zr[j] = xr[varco_position(rule, m, j)];
    }
}

// Encoder and decoder through LDS. Kept positions are spread over the whole row, so a row's cache lines all travel whether
// 4 bytes of a line are wanted or 128, and element-wise accesses (64 scattered addresses per instruction) cost the vector
// memory unit about a cycle each: instead a wavefront moves whole rows with 16-byte accesses, a group of them at a
// time, and picks (encoder) or places (decoder) the kept elements in LDS. 450,000 rows
// of 256, element-wise -> through LDS: decoder 265 -> 116 us (fp32, k = 32), 197 -> 64 (bf16, k = 64); encoder 197 -> 133
// (fp32, k = 128), 136 -> 46 (bf16, k = 64); decoder with sum 224 -> 196 (fp32, k = 32), 194 -> 135
// (bf16, k = 128). Where the element-wise kernels win (few kept elements, narrow or unaligned rows): codec_rows_pay.
// Two forms. codec_rows_kernel: persistent workgroups of four wavefronts that walk the range, the next group's rows already requested.
// codec_wide_rows_kernel: a wavefront is a workgroup and takes one group of rows; workgroups start in the order of the rows, so that
// what is in flight lies close together in memory, which drifting wavefronts lose (a plain copy: 6.2 against 4.8 TB/s). Which one: codec_rows_wide.
//   MODE 0: z[i, j] = x[row_i, pi(j)];  1: x[row_i, :] = 0 except x[row_i, pi(j)] = z[i, j];  2: x[row_i, pi(j)] += z[i, j],
//   in LDS on the old row, which is written back whole: what is not added to keeps its bits
// S: the storage word (fp32 or bf16 bits); V: elements per access to x (16 bytes, or 1 for unaligned rows); PE: elements of z
// per lane (2 for bf16 pairs); U: rows of a group (codec_rows_kernel: kRowsInFlight); ONE: a row is at most one access per lane.
constexpr int kRowsInFlight = 4;         // of codec_rows_kernel
constexpr int kCodecBlock = 64;          // of codec_wide_rows_kernel
constexpr int64_t kCodecGrid = int64_t(1) << 24;      // a launch holds fewer than 2^32 threads
template <typename S>
__device__ __forceinline__ S add_words(S x, S z) {
    if constexpr (sizeof(S) == 4)
        return __float_as_uint(__uint_as_float(x) + __uint_as_float(z));
    else
        return float_to_bf16(bf16_to_float(x) + bf16_to_float(z));
}

template <typename S, int MODE, int V, int PE, bool ONE>
__global__ __launch_bounds__(kBlock) void codec_rows_kernel(MaskRule rule, const int32_t* __restrict__ gids, const int32_t* __restrict__ rows,
                                                            int64_t n_rows, S* x, int64_t ldx, S* z, int lpe_log2) {
    constexpr int U = kRowsInFlight;
    typedef S Vec __attribute__((ext_vector_type(V)));
    typedef S Pair __attribute__((ext_vector_type(PE)));
    extern __shared__ __attribute__((aligned(16))) unsigned char codec_lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t width = int32_t(rule.width), k = int32_t(rule.k);
    const int32_t pitch = (width + 7) & ~7;
    S* const buf = reinterpret_cast<S*>(codec_lds) + wave * U * pitch;
    const int lpe = 1 << lpe_log2, sub = lane >> lpe_log2, jl = lane & (lpe - 1), n_sub = 64 >> lpe_log2;
    auto clear = [&]() {
        for (int u = 0; u < U; ++u)
            for (int c = lane * V; c < width; c += 64 * V) *reinterpret_cast<Vec*>(buf + u * pitch + c) = Vec(S(0));
    };
    if (MODE == 1) clear();
    const int64_t stride = int64_t(gridDim.x) * (kBlock / 64) * U;
    int64_t r0 = (int64_t(blockIdx.x) * (kBlock / 64) + wave) * U;
    if (r0 >= n_rows) return;                        // wavefronts are independent: no barrier
    // Software pipeline over groups of U rows: the rows' ids are fetched two groups ahead, their data one group ahead.
    int32_t gid = 0, src = 0;                        // lane u: of row u of a group (past the end: the last row)
    auto load_ids = [&](int64_t r) {
        const int64_t i = min(r + (lane & (U - 1)), n_rows - 1);
        gid = gids[i];
        if (rows) src = rows[i];
    };
    int64_t at[U];                                   // element offset of the group's rows in x
    uint32_t ab = 0;
    auto resolve = [&](int64_t r) {
        const MaskAffine m = varco_affine(rule, uint32_t(gid));
        ab = m.a | (m.b << 16);
#pragma unroll
        for (int u = 0; u < U; ++u) at[u] = (rows ? int64_t(__shfl(src, u)) : min(r + u, n_rows - 1)) * ldx;
    };
    Vec v[U];
    const int own = min(lane * V, width - V);        // lanes past the row repeat its last access (never stored)
    auto load_rows = [&]() {
        if constexpr (ONE && MODE != 1) {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const Vec*>(x + at[u] + own);
        }
    };
    load_ids(r0);
    resolve(r0);
    load_rows();
    if (r0 + stride < n_rows) load_ids(r0 + stride);
    for (; r0 < n_rows; r0 += stride) {
        const int n_here = int(min(int64_t(U), n_rows - r0));
        const uint32_t ab_now = ab;
        int64_t at_now[U];
#pragma unroll
        for (int u = 0; u < U; ++u) at_now[u] = at[u];
        if constexpr (MODE != 1) {
            if constexpr (ONE) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (lane * V < width) *reinterpret_cast<Vec*>(buf + u * pitch + lane * V) = v[u];
            } else {
                for (int c = lane * V; c < width; c += 64 * V)
#pragma unroll
                    for (int u = 0; u < U; ++u) *reinterpret_cast<Vec*>(buf + u * pitch + c) = *reinterpret_cast<const Vec*>(x + at_now[u] + c);
            }
        }
        if (r0 + stride < n_rows) {
            resolve(r0 + stride);
            load_rows();
            if (r0 + 2 * stride < n_rows) load_ids(r0 + 2 * stride);
        }
        __builtin_amdgcn_wave_barrier();
        // the kept elements: a group of lanes serves one row, the groups different rows
        for (int u0 = 0; u0 < n_here; u0 += n_sub) {
            const int u = u0 + sub;
            const uint32_t m = __shfl(ab_now, u & (U - 1)), a = m & 0xFFFFu;
            if (u < n_here) {
                S* const row = buf + u * pitch;
                for (int j = jl * PE; j < k; j += lpe * PE) {
                    uint32_t q = varco_mod_width(__umul24(a, uint32_t(j)) + (m >> 16), rule.width, rule.width_magic);
                    Pair* const zp = reinterpret_cast<Pair*>(z + (r0 + u) * k + j);
                    Pair e;
                    if constexpr (MODE != 0) e = *zp;
#pragma unroll
                    for (int i = 0; i < PE; ++i) {
                        if constexpr (MODE == 0)
                            e[i] = row[q];
                        else
                            row[q] = MODE == 1 ? e[i] : add_words<S>(row[q], e[i]);
                        q += a;
                        q = min(q, q - rule.width);
                    }
                    if (MODE == 0) *zp = e;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (MODE == 0) continue;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u >= n_here) break;
            for (int c = lane * V; c < width; c += 64 * V) *reinterpret_cast<Vec*>(x + at_now[u] + c) = *reinterpret_cast<const Vec*>(buf + u * pitch + c);
        }
        if (MODE == 1) clear();
        __builtin_amdgcn_wave_barrier();
    }
}
// The other form: one group of rows per wavefront.
template <typename S, int MODE, int U, int V, int PE, bool ONE>
__global__ __launch_bounds__(kCodecBlock) void codec_wide_rows_kernel(MaskRule rule, const int32_t* __restrict__ gids, const int32_t* __restrict__ rows,
                                                                 int64_t n_rows, S* x, int64_t ldx, S* z, int lpe_log2) {
    typedef S Vec __attribute__((ext_vector_type(V)));
    typedef S Pair __attribute__((ext_vector_type(PE)));
    extern __shared__ __attribute__((aligned(16))) unsigned char codec_lds[];
    const int lane = threadIdx.x;
    const int32_t width = int32_t(rule.width), k = int32_t(rule.k);
    const int32_t pitch = (width + 7) & ~7;
    S* const buf = reinterpret_cast<S*>(codec_lds);
    const int lpe = 1 << lpe_log2, sub = lane >> lpe_log2, jl = lane & (lpe - 1), n_sub = 64 >> lpe_log2;
    for (int64_t r0 = int64_t(blockIdx.x) * U; r0 < n_rows; r0 += int64_t(gridDim.x) * U) {      // (once, up to kCodecGrid workgroups)
        const int n_here = int(min(int64_t(U), n_rows - r0));
        if constexpr (MODE == 1) {
            for (int u = 0; u < U; ++u)
                for (int c = lane * V; c < width; c += 64 * V) *reinterpret_cast<Vec*>(buf + u * pitch + c) = Vec(S(0));
        }
        const int64_t i = min(r0 + (lane & (U - 1)), n_rows - 1);      // lane u: row u of the group (past the end: the last row)
        const int32_t gid = gids[i], src = rows ? rows[i] : 0;
        const MaskAffine rm = varco_affine(rule, uint32_t(gid));
        const uint32_t ab = rm.a | (rm.b << 16);
        int64_t at[U];                                   // element offset of the group's rows in x
#pragma unroll
        for (int u = 0; u < U; ++u) at[u] = (rows ? int64_t(__shfl(src, u)) : min(r0 + u, n_rows - 1)) * ldx;
        if constexpr (MODE != 1 && ONE) {
            Vec v[U];
            const int own = min(lane * V, width - V);    // lanes past the row repeat its last access (never stored)
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const Vec*>(x + at[u] + own);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (lane * V < width) *reinterpret_cast<Vec*>(buf + u * pitch + lane * V) = v[u];
        } else if constexpr (MODE != 1) {
            for (int c = lane * V; c < width; c += 64 * V)
#pragma unroll
                for (int u = 0; u < U; ++u) *reinterpret_cast<Vec*>(buf + u * pitch + c) = *reinterpret_cast<const Vec*>(x + at[u] + c);
        }
        __builtin_amdgcn_wave_barrier();
        // the kept elements: a group of lanes serves one row, the groups different rows
        for (int u0 = 0; u0 < n_here; u0 += n_sub) {
            const int u = u0 + sub;
            const uint32_t m = __shfl(ab, u & (U - 1)), a = m & 0xFFFFu;
            if (u < n_here) {
                S* const row = buf + u * pitch;
                for (int j = jl * PE; j < k; j += lpe * PE) {
                    uint32_t q = varco_mod_width(__umul24(a, uint32_t(j)) + (m >> 16), rule.width, rule.width_magic);
                    Pair* const zp = reinterpret_cast<Pair*>(z + (r0 + u) * k + j);
                    Pair e;
                    if constexpr (MODE != 0) e = *zp;
#pragma unroll
                    for (int i = 0; i < PE; ++i) {
                        if constexpr (MODE == 0)
                            e[i] = row[q];
                        else
                            row[q] = MODE == 1 ? e[i] : add_words<S>(row[q], e[i]);
                        q += a;
                        q = min(q, q - rule.width);
                    }
                    if (MODE == 0) *zp = e;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (MODE == 0) continue;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u >= n_here) break;
            for (int c = lane * V; c < width; c += 64 * V) *reinterpret_cast<Vec*>(x + at[u] + c) = *reinterpret_cast<const Vec*>(buf + u * pitch + c);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Owner-side sum of returned errors: rows are distinct within a call and positions are distinct within a
// row, so plain read-modify-write is race-free and the result does not depend on scheduling.
template <typename T>
__global__ __launch_bounds__(kBlock) void decompress_add_kernel(MaskRule rule, const int32_t* __restrict__ gids,
                                                                const int32_t* __restrict__ rows, int64_t n_rows,
                                                                const T* __restrict__ z, T* __restrict__ x,
                                                                int64_t ldx, int g_log2) {
    const uint32_t g = 1u << g_log2;
    const uint32_t gl = threadIdx.x & (g - 1);
    const int64_t stride = (int64_t(gridDim.x) * kBlock) >> g_log2;
    for (int64_t row = group_row(g_log2); row < n_rows; row += stride) {
        const int64_t dst = rows ? int64_t(rows[row]) : row;
        T* xr = x + dst * ldx;
        const T* zr = z + row * int64_t(rule.k);
        const MaskAffine m = varco_affine(rule, uint32_t(gids[row]));
        for (uint32_t j = gl; j < rule.k; j += g) {
            T* dstp = xr + varco_position(rule, m, j);
            Elem<T>::store(dstp, Elem<T>::load(dstp) + Elem<T>::load(zr + j));
        }
    }
}

// Owner-side sum over all consumers: a group of lanes (one per EV stored elements) owns one boundary row,
// adds up the rows returned for it (coalesced reads of k consecutive values each, four in flight), and
// touches the wide gradient row once.
template <typename T, int EV>
__global__ __launch_bounds__(kBlock) void accumulate_returned_kernel(MaskRule rule, const int32_t* __restrict__ gids,
                                                                     const int32_t* __restrict__ rows, int64_t n_rows,
                                                                     const int32_t* __restrict__ ptr,
                                                                     const int32_t* __restrict__ src,
                                                                     const T* __restrict__ returned,
                                                                     T* __restrict__ x, int64_t ldx, int g_log2) {
    using V = typename FloatVec<EV>::type;
    const uint32_t g = 1u << g_log2;
    const uint32_t gl = threadIdx.x & (g - 1);
    const int64_t stride = (int64_t(gridDim.x) * kBlock) >> g_log2;
    const int64_t k = rule.k;
    const uint32_t ku = rule.k / EV;
    for (int64_t b = group_row(g_log2); b < n_rows; b += stride) {
        const int32_t e0 = ptr[b], e1 = ptr[b + 1];
        if (e0 == e1) continue;
        T* xr = x + int64_t(rows[b]) * ldx;
        MaskAffine m{1, 0, 1};
        if (rule.k != rule.width) m = varco_affine(rule, uint32_t(gids[b]));
        for (uint32_t ju = gl; ju < ku; ju += g) {
            const uint32_t j = ju * EV;
            float acc[EV];
#pragma unroll
            for (int i = 0; i < EV; ++i) acc[i] = 0.f;
            for (int32_t e = e0; e < e1; e += 4) {          // rows past the end re-read row e0 and are dropped
                V v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = load_vec<T, EV>(returned + int64_t(src[e + u < e1 ? e + u : e0]) * k + j);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (e + u < e1) {
#pragma unroll
                        for (int i = 0; i < EV; ++i) acc[i] += vec_elem(v[u], i);
                    }
            }
            uint32_t pos = rule.k == rule.width ? j : varco_position(rule, m, j);
#pragma unroll
            for (int i = 0; i < EV; ++i) {
                Elem<T>::store(xr + pos, Elem<T>::load(xr + pos) + acc[i]);
                pos += rule.k == rule.width ? 1u : m.a;
                if (pos >= rule.width) pos -= rule.width;
            }
        }
    }
}

__global__ __launch_bounds__(kBlock) void calibration_copy_kernel(const float4* __restrict__ src,
                                                                  float4* __restrict__ dst, int64_t n) {
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

__global__ __launch_bounds__(kBlock) void sum_gradients_kernel(float* __restrict__ dst, const float* __restrict__ src,
                                                               int64_t n) {
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) dst[i] += src[i];
}

__device__ __forceinline__ uint64_t mix64_device(uint64_t x) {   // splitmix64 output function
    x ^= x >> 30;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 27;
    x *= 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x;
}

// One workgroup of 256 threads, thread t = tap address t.
__global__ __launch_bounds__(kBlock) void step_table_kernel(uint64_t* d_step, uint32_t* table, uint64_t key, int set,
                                                            uint64_t value) {
    const uint64_t step = set ? value : *d_step + 1;
    __syncthreads();                       // every thread has read the old step before it is replaced
    if (threadIdx.x == 0) *d_step = step;
    const uint64_t inner = mix64_device(step + 0x9E3779B97F4A7C15ull * uint64_t(threadIdx.x + 1));
    const uint64_t s = mix64_device(key ^ inner);
    table[2 * threadIdx.x] = uint32_t(s & 0xFFFFFFFFull);
    table[2 * threadIdx.x + 1] = uint32_t(s >> 32);
}

int group_log2(uint32_t elems) {
    int l = 0;
    while ((1u << l) < elems && l < 6) ++l;
    return l;
}

unsigned grid_for(int64_t n_rows, int g_log2) {
    const int64_t threads = n_rows << g_log2;
    int64_t blocks = (threads + kBlock - 1) / kBlock;
    const int64_t cap = int64_t(1) << 22;  // a launch holds fewer than 2^32 threads; workgroups that each take one place start in memory order
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return unsigned(blocks);
}
// For kernels that move an element per lane: 16 resident workgroups on each of the 256 compute units, which walk on. One place each, as
// for 16-byte accesses, costs them 5 to 10 % (216,537 rows of 188 bf16 values, 23 of them kept, encoder 33.5 -> 35.7 us; 129,597 rows of 118 fp32
// values, 39 kept, decoder with sum 32.2 -> 33.7).
unsigned walking_grid(int64_t n_rows, int g_log2) { return std::min(grid_for(n_rows, g_log2), 256u * 16u); }

// Per halo row: its position rule (element j sits at position (a j + b) mod width) and its row in the compressed
// buffer, for the kernels that transform halo rows from their received elements.
__global__ __launch_bounds__(kBlock) void halo_rows_kernel(MaskRule rule, const int32_t* __restrict__ gids,
                                                           const int32_t* __restrict__ zrow, int32_t n,
                                                           uint2* __restrict__ out) {
    const int32_t s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= n) return;
    uint32_t ab = 1u << 16;                       // every element kept: position c holds element c
    if (rule.k < rule.width) {
        const MaskAffine m = varco_affine(rule, uint32_t(gids[s]));
        ab = (m.a << 16) | m.b;
    }
    out[s] = make_uint2(ab, uint32_t(zrow ? zrow[s] : s));
}

// Whether whole rows through LDS beat element-wise accesses (measured over widths 75 to 512 and ratios 2 to 64). The decoder
// writes whole rows either way. The encoder's element-wise form costs per kept element, the other one per row: the line lies
// at an eighth (fp32) or a sixteenth (bf16) of the row, at a quarter for rows that take one element per access. Adding
// element-wise also spares the write-back of untouched sectors, so the line is higher for rows that leave half of a
// wavefront's 16-byte accesses unused.
template <typename T, int MODE>
bool codec_rows_pay(const MaskRule& rule, const void* x, int64_t ldx) {
    if (rule.k >= rule.width) return false;
    if (MODE == 1) return true;
    constexpr uint32_t V16 = 16 / sizeof(T);
    const bool vec = rule.width % V16 == 0 && ldx % V16 == 0 && (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    uint32_t part = MODE == 0 ? (vec ? (sizeof(T) == 4 ? 8 : 16) : 4) : 2;
    if (MODE == 2 && vec) part = rule.width * sizeof(T) >= 512 ? (sizeof(T) == 4 ? 16 : 8) : (sizeof(T) == 4 ? 4 : 2);
    return rule.k * part >= rule.width;
}

// Everything is kept: rows are copied (TO_Z: x -> z, else z -> x) or added to x, V elements per access.
template <typename S, int V, bool TO_Z, bool ADD>
__global__ __launch_bounds__(kBlock) void whole_rows_kernel(const int32_t* __restrict__ rows, int64_t n_rows, S* x, int64_t ldx, S* z, int32_t width,
                                                            int g_log2) {
    typedef S Vec __attribute__((ext_vector_type(V)));
    const int g = 1 << g_log2, gl = threadIdx.x & (g - 1);
    const int64_t stride = (int64_t(gridDim.x) * kBlock) >> g_log2;
    for (int64_t row = group_row(g_log2); row < n_rows; row += stride) {
        S* const xr = x + (rows ? int64_t(rows[row]) : row) * ldx;
        S* const zr = z + row * width;
        for (int c = gl * V; c < width; c += g * V) {
            if constexpr (TO_Z) {
                *reinterpret_cast<Vec*>(zr + c) = *reinterpret_cast<const Vec*>(xr + c);
            } else {
                Vec v = *reinterpret_cast<const Vec*>(zr + c);
                if constexpr (ADD) {
                    const Vec old = *reinterpret_cast<const Vec*>(xr + c);
#pragma unroll
                    for (int i = 0; i < V; ++i) v[i] = add_words<S>(old[i], v[i]);
                }
                *reinterpret_cast<Vec*>(xr + c) = v;
            }
        }
    }
}

template <typename T, bool TO_Z, bool ADD>
hipError_t launch_whole_rows(const MaskRule& rule, const int32_t* rows, int64_t n_rows, void* x, int64_t ldx, void* z, hipStream_t stream) {
    using S = std::conditional_t<sizeof(T) == 2, uint16_t, uint32_t>;
    constexpr int V16 = 16 / int(sizeof(S));
    // (adding fp32 rows is bound by the copy rate and ran 5 % slower with wide accesses)
    const bool vec = !(ADD && sizeof(S) == 4) && rule.width % V16 == 0 && ldx % V16 == 0 &&
                     ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(z)) & 15u) == 0;
    const int gl = group_log2(vec ? rule.width / V16 : rule.width);
    auto go = [&](auto vc) {
        hipLaunchKernelGGL((whole_rows_kernel<S, decltype(vc)::value, TO_Z, ADD>), dim3(vec ? grid_for(n_rows, gl) : walking_grid(n_rows, gl)), dim3(kBlock), 0,
                           stream, rows, n_rows, static_cast<S*>(x), ldx, static_cast<S*>(z), int32_t(rule.width), gl);
    };
    if (vec)
        go(std::integral_constant<int, V16>{});
    else
        go(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

// Which of the two forms, by what a call does and by the bytes of a row and of all rows. Measured at 34 widths of fp32 and 21 of bf16, ratios 2 to 32, 3 to 460 MB of
// rows; walking / one group per wavefront, us (or the latter's gain or loss).
// Adding decoder: one group for 1,024 bytes, an access of every lane, and from 1,536 on. 460 MB: 256 fp32 values, ratio 2 234 / 218, 8 197 / 185, 16 190 / 178, 1,024 values, ratio 4
//   263 / 213, bf16 rows of 512, ratio 8 -7 %; 14 MB, 512 fp32 values, ratio 2 9.6 / 6.6; the worst, 180 MB, 256 values, ratio 12 55.6 / 59.0. Between, where a second access has few lanes, from
//   memory or from the L2 caches (320 values, ratio 4 460 MB 207 / 203, 14 MB -13 %, but 230 MB 90.5 / 95.5, 90 MB, ratio 16 29.4 / 30.4). Below: 128 values, ratio 4 206 / 225,
//   192 values, 90 MB 33.6 / 34.9, bf16 rows of 256, ratio 8 +17 %.
// Encoder: from 1,536 bytes on (460 MB, 384 fp32 values, ratio 4 110 / 107, 1,536 values 183 / 140; 230 MB, 384 values, ratio 8 +4 %, the worst), from 1,024 bytes on where the rows
//   come from memory: 256 values, ratio 8 460 MB 103 / 97, 340 MB 72 / 69, 280 MB 48.8 / 49.2, 180 MB 30.3 / 31.3, 90 MB 16.5 / 17.0; bf16 rows of 640 102 / 98, 180 MB +4 %.
// Decoder, rows written and not read: into the cache, one group (14 MB, 256 values, ratio 4 6.4 / 6.1, 1,024 values, ratio 2 -25 %; 90 MB, 512 values, ratio 8 -5 %, 256 values
//   17.5 / 17.3, 230 MB 256 values, ratio 2 +9 %). To memory, walking where little is kept, a fill (460 MB, 384 values, ratio 32 93 / 103, 16 110 / 108, 512 values 91 / 100, 104 / 109), unless
//   rows are long (896 values, ratio 16 149 / 131, 32 level; 800 values +3, +7 %), and where a short row takes many picks (256 values, ratio 2 147 / 162, 4 121 / 126, 320 values 161 / 177,
//   146 / 147); between, one group (256 values, ratio 6 134 / 135, 8 112 / 109, 12 114 / 115, 320 values 126 / 122, 128 / 118, 115 / 107, bf16 rows of 640, ratio 8 129 / 119; 352 values, ratio 8 129 / 133).
// Rows that are no whole 16-byte pieces, 64 values to an access: 301 fp32 values, ratio 2, 460 MB +5, +5, +3 %, 385 values +3, -4, -6 %, 505 values 147 / 146, 242 / 228, 309 / 255; bf16 rows of
//   516, 180 MB, ratio 2 62 / 65, 83 / 80, 115 / 131, ratio 8 43 / 43, 51 / 46; of 772 level, -4 %, level.
constexpr int64_t kCachedBytes = int64_t(320) << 20;      // rows in all of which the last-level cache (256 MB) serves a part
template <typename T, int MODE>
bool codec_rows_wide(const MaskRule& rule, int64_t n_rows, bool vec) {
    const int64_t bytes = int64_t(rule.width) * int64_t(sizeof(T)), all = n_rows * bytes;
    if (bytes < 1024) return false;
    const bool longer = bytes >= 1536, few = rule.k * 12 < rule.width, many = rule.k * 5 > rule.width;
    if (MODE == 0) return longer || (vec && all > kCachedBytes);
    if (MODE == 2) return longer || (vec && (bytes == 1024 || all > kCachedBytes || 8 * all <= kCachedBytes));
    if (!vec) return rule.width >= 384;
    return longer ? !few || all <= kCachedBytes || bytes >= 3584 : (!few && !many) || 2 * all <= kCachedBytes;
}

// Rows of a group of codec_wide_rows_kernel: two where rows are read and written, else four. The adding decoder with two / four, us: 460 MB of rows, 512 fp32
// values, ratio 2 224 / 251, 256 values, ratio 8 185 / 193, 768 bf16 values, ratio 4 202 / 210; 14 MB, 512 fp32 values, ratio 4 6.0 / 7.3, 256 values 6.1 / 6.5.
template <typename T, int MODE, int U = MODE == 2 ? 2 : 4>
hipError_t launch_codec_rows(const MaskRule& rule, const int32_t* gids, const int32_t* rows, int64_t n_rows, void* x, int64_t ldx, void* z,
                             hipStream_t stream) {
    using S = std::conditional_t<sizeof(T) == 2, uint16_t, uint32_t>;
    constexpr int V16 = 16 / int(sizeof(S));
    const bool vec = rule.width % V16 == 0 && ldx % V16 == 0 && (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    const bool pair = sizeof(S) == 2 && rule.k % 2 == 0 && (reinterpret_cast<uintptr_t>(z) & 3u) == 0;
    const bool one = int(rule.width) <= 64 * (vec ? V16 : 1);
    const int lpe = group_log2(pair ? rule.k / 2 : rule.k);
    constexpr int W = kBlock / 64;
    const bool wide = codec_rows_wide<T, MODE>(rule, n_rows, vec);
    const size_t row = size_t((rule.width + 7) & ~7u) * sizeof(S);
    const int64_t blocks = wide ? std::min((n_rows + U - 1) / U, kCodecGrid) : std::min<int64_t>((n_rows + W * kRowsInFlight - 1) / (W * kRowsInFlight), 256 * 32);
    auto go = [&](auto vc, auto pc, auto oc) {
        constexpr int V = decltype(vc)::value, PE = decltype(pc)::value;
        constexpr bool ONE = decltype(oc)::value;
        if (wide)
            hipLaunchKernelGGL((codec_wide_rows_kernel<S, MODE, U, V, PE, ONE>), dim3(unsigned(blocks)), dim3(kCodecBlock), U * row, stream, rule, gids, rows,
                               n_rows, static_cast<S*>(x), ldx, static_cast<S*>(z), lpe);
        else
            hipLaunchKernelGGL((codec_rows_kernel<S, MODE, V, PE, ONE>), dim3(unsigned(blocks)), dim3(kBlock), W * kRowsInFlight * row, stream, rule, gids,
                               rows, n_rows, static_cast<S*>(x), ldx, static_cast<S*>(z), lpe);
    };
    auto with_one = [&](auto vc, auto pc) {
        if (one)
            go(vc, pc, std::true_type{});
        else
            go(vc, pc, std::false_type{});
    };
    auto with_pair = [&](auto vc) {
        if constexpr (sizeof(S) == 2)
            if (pair) return with_one(vc, std::integral_constant<int, 2>{});
        with_one(vc, std::integral_constant<int, 1>{});
    };
    if (vec)
        with_pair(std::integral_constant<int, V16>{});
    else
        with_pair(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

template <typename T>
hipError_t launch_compress_t(const MaskRule& rule, const int32_t* gids, const int32_t* rows, int64_t n_rows, const void* x,
                             int64_t ldx, void* z, hipStream_t stream) {
    if (rule.k == rule.width) return launch_whole_rows<T, true, false>(rule, rows, n_rows, const_cast<void*>(x), ldx, z, stream);
    if (codec_rows_pay<T, 0>(rule, x, ldx)) return launch_codec_rows<T, 0>(rule, gids, rows, n_rows, const_cast<void*>(x), ldx, z, stream);
    const int gl = group_log2(rule.k);
    hipLaunchKernelGGL(compress_kernel<T>, dim3(walking_grid(n_rows, gl)), dim3(kBlock), 0, stream, rule, gids, rows, n_rows,
                       static_cast<const T*>(x), ldx, static_cast<T*>(z), gl);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_decompress_t(const MaskRule& rule, const int32_t* gids, const int32_t* rows, int64_t n_rows,
                               const void* z, void* x, int64_t ldx, int accumulate, hipStream_t stream) {
    void* const zw = const_cast<void*>(z);
    if (rule.k == rule.width)
        return accumulate ? launch_whole_rows<T, false, true>(rule, rows, n_rows, x, ldx, zw, stream)
                          : launch_whole_rows<T, false, false>(rule, rows, n_rows, x, ldx, zw, stream);
    if (!accumulate) return launch_codec_rows<T, 1>(rule, gids, rows, n_rows, x, ldx, zw, stream);
    if (codec_rows_pay<T, 2>(rule, x, ldx)) return launch_codec_rows<T, 2>(rule, gids, rows, n_rows, x, ldx, zw, stream);
    const int gl = group_log2(rule.k);
    hipLaunchKernelGGL(decompress_add_kernel<T>, dim3(walking_grid(n_rows, gl)), dim3(kBlock), 0, stream, rule, gids, rows, n_rows,
                       static_cast<const T*>(z), static_cast<T*>(x), ldx, gl);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_accumulate_t(const MaskRule& rule, const int32_t* gids, const int32_t* rows, int64_t n_rows,
                               const int32_t* ptr, const int32_t* src, const void* returned, void* x, int64_t ldx,
                               hipStream_t stream) {
    // wide loads only while at least 32 lanes still share a row: fewer lanes per row means more rows per
    // wavefront, whose differing numbers of returned rows then serialise
    int ev = 1;
    for (int c : {4, 2})
        if (rule.k % c == 0 && rule.k / c >= 32 && (reinterpret_cast<uintptr_t>(returned) & (c * sizeof(T) - 1)) == 0) {
            ev = c;
            break;
        }
    const int gl = group_log2(rule.k / ev);
    const dim3 grid(walking_grid(n_rows, gl)), block(kBlock);
    const T* ret = static_cast<const T*>(returned);
    T* xt = static_cast<T*>(x);
    if (ev == 4)
        hipLaunchKernelGGL((accumulate_returned_kernel<T, 4>), grid, block, 0, stream, rule, gids, rows, n_rows, ptr, src, ret,
                           xt, ldx, gl);
    else if (ev == 2)
        hipLaunchKernelGGL((accumulate_returned_kernel<T, 2>), grid, block, 0, stream, rule, gids, rows, n_rows, ptr, src, ret,
                           xt, ldx, gl);
    else
        hipLaunchKernelGGL((accumulate_returned_kernel<T, 1>), grid, block, 0, stream, rule, gids, rows, n_rows, ptr, src, ret,
                           xt, ldx, gl);
    return hipGetLastError();
}

}  // namespace

hipError_t varco_launch_compress(int dtype, const MaskRule& rule, const int32_t* gids, const int32_t* rows, int64_t n_rows,
                                 const void* x, int64_t ldx, void* z, hipStream_t stream, const LaunchTag& tag) {
    if (n_rows == 0) return hipSuccess;
    tag.begin(stream);
    const hipError_t e = dtype == VARCO_BF16 ? launch_compress_t<bf16_t>(rule, gids, rows, n_rows, x, ldx, z, stream)
                                             : launch_compress_t<float>(rule, gids, rows, n_rows, x, ldx, z, stream);
    tag.end(stream);
    return e;
}

hipError_t varco_launch_decompress(int dtype, const MaskRule& rule, const int32_t* gids, const int32_t* rows,
                                   int64_t n_rows, const void* z, void* x, int64_t ldx, int accumulate,
                                   hipStream_t stream, const LaunchTag& tag) {
    if (n_rows == 0) return hipSuccess;
    tag.begin(stream);
    const hipError_t e = dtype == VARCO_BF16
                             ? launch_decompress_t<bf16_t>(rule, gids, rows, n_rows, z, x, ldx, accumulate, stream)
                             : launch_decompress_t<float>(rule, gids, rows, n_rows, z, x, ldx, accumulate, stream);
    tag.end(stream);
    return e;
}

hipError_t varco_launch_accumulate_returned(int dtype, const MaskRule& rule, const int32_t* gids, const int32_t* rows,
                                            int64_t n_rows, const int32_t* ptr, const int32_t* src, const void* returned,
                                            void* x, int64_t ldx, hipStream_t stream, const LaunchTag& tag) {
    if (n_rows == 0) return hipSuccess;
    tag.begin(stream);
    const hipError_t e = dtype == VARCO_BF16
                             ? launch_accumulate_t<bf16_t>(rule, gids, rows, n_rows, ptr, src, returned, x, ldx, stream)
                             : launch_accumulate_t<float>(rule, gids, rows, n_rows, ptr, src, returned, x, ldx, stream);
    tag.end(stream);
    return e;
}

hipError_t varco_launch_halo_rows(const MaskRule& rule, const int32_t* gids, const int32_t* zrow, int32_t n, uint2* out,
                                  hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(halo_rows_kernel, dim3(unsigned((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, stream, rule, gids, zrow,
                       n, out);
    return hipGetLastError();
}

hipError_t varco_launch_calibration_copy(void* dst, const void* src, int64_t bytes, hipStream_t stream) {
    if (bytes == 0) return hipSuccess;
    hipLaunchKernelGGL(calibration_copy_kernel, dim3(256 * 32), dim3(kBlock), 0, stream, static_cast<const float4*>(src),
                       static_cast<float4*>(dst), bytes / 16);
    return hipGetLastError();
}

hipError_t varco_launch_sum_gradients(float* dst, const float* src, int64_t n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int64_t want = (n + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(sum_gradients_kernel, dim3(unsigned(want < 256 * 16 ? want : 256 * 16)), dim3(kBlock), 0, stream, dst,
                       src, n);
    return hipGetLastError();
}

hipError_t varco_launch_step_table(uint64_t* d_step, uint32_t* table, uint64_t key, int set, uint64_t value,
                                   hipStream_t stream) {
    hipLaunchKernelGGL(step_table_kernel, dim3(1), dim3(kBlock), 0, stream, d_step, table, key, set, value);
    return hipGetLastError();
}
