// Sums of gathered dense rows by one wavefront, shared by the forward aggregation and the node sums of the backward pass.
#pragma once

#include <type_traits>

#include "elem.h"

// N consecutive stored elements, packed as they lie in memory until they are used: load(), get() converts, put() rounds and
// stores.
template <typename T, int N>
struct Packed;
template <int N>
struct Packed<float, N> {
    typedef float type __attribute__((ext_vector_type(N)));
    static __device__ __forceinline__ type load(const float* p) { return *reinterpret_cast<const type*>(p); }
    static __device__ __forceinline__ void get(const type& v, float (&x)[N]) {
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = v[i];
    }
    template <bool ANY = false>
    static __device__ __forceinline__ void put(float* p, const float (&x)[N]) {
        typedef type stored __attribute__((aligned(ANY ? sizeof(float) : sizeof(type))));
        type v;
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = x[i];
        *reinterpret_cast<stored*>(p) = v;
    }
};
template <>
struct Packed<float, 1> {
    using type = float;
    static __device__ __forceinline__ type load(const float* p) { return *p; }
    static __device__ __forceinline__ void get(const type& v, float (&x)[1]) { x[0] = v; }
    template <bool ANY = false>
    static __device__ __forceinline__ void put(float* p, const float (&x)[1]) { *p = x[0]; }
};
template <int N>
struct Packed<bf16_t, N> {
    typedef uint32_t type __attribute__((ext_vector_type(N / 2)));
    static __device__ __forceinline__ type load(const bf16_t* p) { return *reinterpret_cast<const type*>(p); }
    static __device__ __forceinline__ void get(const type& v, float (&x)[N]) {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) x[2 * i] = __uint_as_float(v[i] << 16), x[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
    }
    template <bool ANY = false>
    static __device__ __forceinline__ void put(bf16_t* p, const float (&x)[N]) {
        typedef type stored __attribute__((aligned(ANY ? sizeof(bf16_t) : sizeof(type))));
        type v;
#pragma unroll
        for (int i = 0; i < N / 2; ++i) v[i] = bf16_pair(x[2 * i], x[2 * i + 1]);
        *reinterpret_cast<stored*>(p) = v;
    }
};
template <>
struct Packed<bf16_t, 2> {
    using type = uint32_t;
    static __device__ __forceinline__ type load(const bf16_t* p) { return *reinterpret_cast<const uint32_t*>(p); }
    static __device__ __forceinline__ void get(const type& v, float (&x)[2]) { x[0] = __uint_as_float(v << 16), x[1] = __uint_as_float(v & 0xFFFF0000u); }
    template <bool ANY = false>
    static __device__ __forceinline__ void put(bf16_t* p, const float (&x)[2]) {
        typedef uint32_t any __attribute__((aligned(2)));
        if constexpr (ANY)
            *reinterpret_cast<any*>(p) = bf16_pair(x[0], x[1]);
        else
            *reinterpret_cast<uint32_t*>(p) = bf16_pair(x[0], x[1]);
    }
};
template <>
struct Packed<bf16_t, 1> {
    using type = uint16_t;
    static __device__ __forceinline__ type load(const bf16_t* p) { return p->bits; }
    static __device__ __forceinline__ void get(const type& v, float (&x)[1]) { x[0] = bf16_to_float(v); }
    template <bool ANY = false>
    static __device__ __forceinline__ void put(bf16_t* p, const float (&x)[1]) { p->bits = float_to_bf16(x[0]); }
};

// Load from an address in global memory that was handled as a number (a generic address would go through the LDS check). ANY: from the
// address of any element (the device loads up to 16 bytes from there just as well).
template <typename T, int N, bool ANY = false>
__device__ __forceinline__ typename Packed<T, N>::type load_packed(uint64_t address, uint32_t byte_offset) {
    using V = typename Packed<T, N>::type;
    if constexpr (ANY) {
        typedef V any __attribute__((aligned(sizeof(T))));
        return *(const __attribute__((address_space(1))) any*)((const __attribute__((address_space(1))) char*)address + byte_offset);
    }
    return *(const __attribute__((address_space(1))) V*)((const __attribute__((address_space(1))) char*)address + byte_offset);
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int byte_lane) { return uint32_t(__builtin_amdgcn_ds_bpermute(byte_lane, int(v))); }

// acc += sum over i < n of w_i * row_i: lane i holds entry i's weight and the address of its row. NV > 0: a row of `width`
// elements takes all 64 lanes, NV loads of VEC elements each; NV = 0: it takes one load of 1 << lpr_log2 lanes, and the groups
// of lanes take different entries (sum_groups adds them). U rows of a group are requested before the first is used.
// These kernels issue vector instructions most of the time on graphs of ordinary degree (a wavefront has a dozen entries), so
// what is the same for the whole wavefront stays in scalar registers: with all lanes on one row its address and weight come by
// v_readlane and the load takes a scalar base; the last batch leaves out by scalar branches what
// is not there.
// ANY: rows of any length from VEC elements on; the lane that would reach past the end of its row takes the row's last VEC elements instead,
// and adds to them what its neighbour adds.
constexpr int loads_per_row(int nv) { return nv > 0 ? nv : 1; }
template <int VEC, bool ANY>
__device__ __forceinline__ int32_t row_column(int32_t c, int32_t width) { return ANY ? min(c, width - VEC) : c; }
template <typename T, int VEC, int NV, int U, bool ANY = false>
__device__ __forceinline__ void gather_rows(uint64_t addr, float w, int n, int32_t width, int lane, int lpr_log2, float (&acc)[loads_per_row(NV)][VEC]) {
    using P = Packed<T, VEC>;
    uint32_t lo = uint32_t(addr), hi = uint32_t(addr >> 32), wb = __float_as_uint(w);
    // v_readlane reads lanes that are switched off, too: their values must be formed here, where every lane is on, and not (as
    // the compiler is free to do) where the loads of the lanes below `width` are issued.
    asm volatile("" : "+v"(lo), "+v"(hi), "+v"(wb));
    if constexpr (NV > 0) {
        uint32_t off[NV];                        // lanes beyond the row re-read its start (their sums are never stored)
#pragma unroll
        for (int m = 0; m < NV; ++m) off[m] = VEC * (lane + 64 * m) < width ? uint32_t(sizeof(T)) * uint32_t(row_column<VEC, ANY>(VEC * (lane + 64 * m), width)) : 0u;
        auto batch = [&](int i0, auto partial) {
            constexpr bool PART = decltype(partial)::value;
            typename P::type v[U][NV];
            float wi[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (!PART || u == 0 || i0 + u < n) {
                    const uint64_t row = (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(hi), i0 + u))) << 32) |
                                         uint32_t(__builtin_amdgcn_readlane(int(lo), i0 + u));
                    wi[u] = __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(wb), i0 + u)));
#pragma unroll
                    for (int m = 0; m < NV; ++m) v[u][m] = load_packed<T, VEC, ANY>(row, off[m]);
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (!PART || u == 0 || i0 + u < n)
#pragma unroll
                    for (int m = 0; m < NV; ++m) {
                        float x[VEC];
                        P::get(v[u][m], x);
#pragma unroll
                        for (int i = 0; i < VEC; ++i) acc[m][i] += wi[u] * x[i];
                    }
        };
        int i0 = 0;
        for (; i0 + U <= n; i0 += U) batch(i0, std::false_type{});
        if (i0 < n) batch(i0, std::true_type{});
    } else {
        const int lpr = 1 << lpr_log2, ng = 64 >> lpr_log2, c = VEC * (lane & (lpr - 1)), g = lane >> lpr_log2;
        const uint32_t off = c < width ? uint32_t(row_column<VEC, ANY>(c, width)) * uint32_t(sizeof(T)) : 0u;
        auto batch = [&](int i0, auto count, auto partial) {
            constexpr int N = decltype(count)::value;
            constexpr bool PART = decltype(partial)::value;
            typename P::type v[N];
            uint32_t wi[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int i = i0 + u * ng + g;
                const uint64_t row = (uint64_t(lane_value(hi, 4 * i)) << 32) | lane_value(lo, 4 * i);
                wi[u] = lane_value(wb, 4 * i);
                if (!PART || i < n) v[u] = load_packed<T, VEC, ANY>(row, off);
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (!PART || i0 + u * ng + g < n) {
                    float x[VEC];
                    P::get(v[u], x);
#pragma unroll
                    for (int i = 0; i < VEC; ++i) acc[0][i] += __uint_as_float(wi[u]) * x[i];
                }
        };
        int i0 = 0;
        for (; i0 + ng * U <= n; i0 += ng * U) batch(i0, std::integral_constant<int, U>{}, std::false_type{});
        if (i0 + ng < n)
            batch(i0, std::integral_constant<int, U>{}, std::true_type{});
        else if (i0 < n)
            batch(i0, std::integral_constant<int, 1>{}, std::true_type{});
    }
}

// Every lane gets the sums over the lanes whose number differs from its own in bits log2 to 5 (log2 is the same in all lanes, all of them are on): lane l
// and l ^ off are added for off = 1 << log2, .., 32 in turn, by data paths of the vector ALU. (__shfl_xor goes through LDS: an instruction there and a
// round trip for every value. Node sums with it / with this, us, bf16: 819,353 nodes 40 wide, 12 kept, 599 / 487, 911,699 nodes 40 wide, 5 kept, 722 /
// 551, 35,999 nodes 56 wide 39 / 31; fp32 rows of 256 elements, three steps of four values a node, level at 153.)
// lanes (the same in all of them): from that lane on there are zeros, and only the first 1 << log2 lanes are looked at afterwards: steps that add nothing
// to those are left out.
template <int N>
__device__ __forceinline__ void add_lanes(float (&x)[N], int log2, int lanes = 64) {
    auto moved = [](float v, auto ctrl, auto banks) __attribute__((always_inline)) {       // v where `banks` are not
        const int u = __builtin_bit_cast(int, v);
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(u, u, decltype(ctrl)::value, 0xF, decltype(banks)::value, false));
    };
    using std::integral_constant;
    using All = integral_constant<int, 0xF>;
    // (nested: a wide row, whose few groups take the last steps only, passes one test)
    if (log2 <= 4) {
        if (log2 <= 2) {
            if (log2 <= 0 && lanes > 1)
#pragma unroll
                for (int i = 0; i < N; ++i) x[i] += moved(x[i], integral_constant<int, 0xB1>{}, All{});        // quad_perm 1 0 3 2
            if (log2 <= 1 && lanes > 2)
#pragma unroll
                for (int i = 0; i < N; ++i) x[i] += moved(x[i], integral_constant<int, 0x4E>{}, All{});        // quad_perm 2 3 0 1
            if (lanes > 4)
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const float up = moved(x[i], integral_constant<int, 0x104>{}, integral_constant<int, 0x5>{});      // lanes 0-3 and 8-11 from four lanes
                    const int u = __builtin_bit_cast(int, x[i]);                                                       // above, the others from four below
                    x[i] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, up), u, 0x114, 0xF, 0xA, false));
                }
        }
        if (log2 <= 3 && lanes > 8)
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] += moved(x[i], integral_constant<int, 0x128>{}, All{});       // row_ror 8
        if (lanes > 16)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i]), false, false);
                x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            }
    }
    if (log2 <= 5 && lanes > 32)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i]), false, false);
            x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
}

// The lanes of the first group get the sums over the groups, which took at most n entries.
template <int VEC, int NV>
__device__ __forceinline__ void sum_groups(int lpr_log2, int n, float (&acc)[loads_per_row(NV)][VEC]) {
    if constexpr (NV == 0) add_lanes(acc[0], lpr_log2, min(n, 64) << lpr_log2);
}

// Rows of fp32 in LDS or memory, VEC at a time (ANY: from the address of any element).
template <int VEC, bool ANY = false>
__device__ __forceinline__ void add_floats(const float* p, float (&x)[VEC]) {
    constexpr int W = ANY ? 1 : VEC < 4 ? VEC : 4;
#pragma unroll
    for (int i = 0; i < VEC; i += W) {
        const typename FloatVec<W>::type v = *reinterpret_cast<const typename FloatVec<W>::type*>(p + i);
        const float* e = reinterpret_cast<const float*>(&v);
#pragma unroll
        for (int q = 0; q < W; ++q) x[i + q] += e[q];
    }
}
template <int VEC, bool ANY = false>
__device__ __forceinline__ void put_floats(float* p, const float (&x)[VEC]) {
    constexpr int W = ANY ? 1 : VEC < 4 ? VEC : 4;
#pragma unroll
    for (int i = 0; i < VEC; i += W) {
        typename FloatVec<W>::type v;
        float* e = reinterpret_cast<float*>(&v);
#pragma unroll
        for (int q = 0; q < W; ++q) e[q] = x[i + q];
        *reinterpret_cast<typename FloatVec<W>::type*>(p + i) = v;
    }
}
