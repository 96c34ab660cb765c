// The rest of Algorithm 1's iteration around the layer calls: the cross-entropy loss of Section II on a
// partition's labelled rows with its gradient with respect to the logits, fixed-order sums of the per-row
// results, and the gradient step (SGD). Memory-bound elementwise / row-wise kernels.
#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "varco_internal.h"

namespace {

constexpr int kBlock = 256;

template <typename U>
struct Tag {
    using type = U;
};
template <int N>
using Int = std::integral_constant<int, N>;

// loss_i = logsumexp(z_i) - z_i[y_i], dz_i = scale * (softmax(z_i) - onehot(y_i)), correct_i = [argmax z_i == y_i] (lowest
// index on ties); rows whose y_i is not a class (negative: not a training node; n_classes or above: never read as an index)
// give 0 everywhere. A group of G lanes takes a row, E elements per lane held in registers (G E >= n_classes; E = 0: rows are
// re-read, for more than 512 classes), so that the rows of 47 logits of a class layer fill a wavefront four at a time: with a
// wavefront per row the kernel was bound by its shuffles, not by memory. 410,003 rows of 47: 119 -> 29 us, and the sum of the rows 121 -> 5 us.
// A workgroup's sums of its rows go to block_sums (null: not wanted), its rows in a fixed order.
// dlogits may be the logits themselves (same rows): every element is read by the lane that replaces it, and the label's logit
// before that, so neither pointer promises to be the only one.
template <typename T, int G, int E>
__global__ __launch_bounds__(kBlock) void softmax_xent_kernel(const T* logits, int64_t ld,
                                                              const int32_t* __restrict__ labels, int64_t n_rows,
                                                              int32_t n_classes, float scale, T* dlogits,
                                                              int64_t ldd, float* __restrict__ row_loss,
                                                              int32_t* __restrict__ row_correct, float2* __restrict__ block_sums) {
    constexpr int kRows = kBlock / G;            // rows of a workgroup at a time
    const int t = threadIdx.x & (G - 1);
    float sum_loss = 0.f, sum_correct = 0.f;
    for (int64_t row = int64_t(blockIdx.x) * kRows + threadIdx.x / G; row < n_rows; row += int64_t(gridDim.x) * kRows) {
        const int32_t y = labels[row];
        const T* z = logits + row * ld;
        float v[E > 0 ? E : 1];
        float vmax = -INFINITY;
        int32_t imax = 0x7FFFFFFF;
        if constexpr (E > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = t + e * G < n_classes ? Elem<T>::load(z + t + e * G) : -INFINITY;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (v[e] > vmax) vmax = v[e], imax = t + e * G;      // ascending class within a lane: the first maximum is kept
        } else {
            for (int c = t; c < n_classes; c += G) {
                const float x = Elem<T>::load(z + c);
                if (x > vmax) vmax = x, imax = c;
            }
        }
        float gmax = vmax;
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) gmax = fmaxf(gmax, __shfl_xor(gmax, off));
        int32_t cand = vmax == gmax ? imax : 0x7FFFFFFF;
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) cand = min(cand, __shfl_xor(cand, off));
        float se = 0.f;
        if constexpr (E > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                v[e] = t + e * G < n_classes ? expf(v[e] - gmax) : 0.f;
                se += v[e];
            }
        } else {
            for (int c = t; c < n_classes; c += G) se += expf(Elem<T>::load(z + c) - gmax);
        }
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) se += __shfl_xor(se, off);
        const bool on = y >= 0 && y < n_classes;
        float loss = 0.f;
        if (on) loss = gmax + logf(se) - Elem<T>::load(z + y);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // before any lane of the row writes dlogits
        if (dlogits) {
            T* d = dlogits + row * ldd;
            const float inv = scale / se;
            if constexpr (E > 0) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int c = t + e * G;
                    if (c < n_classes) Elem<T>::store(d + c, on ? v[e] * inv - (c == y ? scale : 0.f) : 0.f);
                }
            } else {
                for (int c = t; c < n_classes; c += G) {
                    float g = 0.f;
                    if (on) g = expf(Elem<T>::load(z + c) - gmax) * inv - (c == y ? scale : 0.f);
                    Elem<T>::store(d + c, g);
                }
            }
        }
        if (t == 0) {
            const int32_t correct = on && cand == y ? 1 : 0;
            row_loss[row] = loss;
            row_correct[row] = correct;
            sum_loss += loss, sum_correct += float(correct);
        }
    }
    if (!block_sums) return;
    __shared__ float2 part[kRows];
    if (t == 0) part[threadIdx.x / G] = make_float2(sum_loss, sum_correct);
    __syncthreads();
    for (int s = kRows / 2; s > 0; s >>= 1) {
        if (int(threadIdx.x) < s) part[threadIdx.x].x += part[threadIdx.x + s].x, part[threadIdx.x].y += part[threadIdx.x + s].y;
        __syncthreads();
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = part[0];
}

// totals[0] += scale * sum(loss), totals[1] += count of correct rows, over n rows or block sums; one workgroup, fixed order.
__device__ __forceinline__ void add_totals(float l, float c, float scale, float* totals) {
    __shared__ float sl[1024];
    __shared__ float sc[1024];
    sl[threadIdx.x] = l, sc[threadIdx.x] = c;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if (int(threadIdx.x) < s) sl[threadIdx.x] += sl[threadIdx.x + s], sc[threadIdx.x] += sc[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) totals[0] += scale * sl[0], totals[1] += sc[0];
}
__global__ __launch_bounds__(1024) void sum_rows_kernel(const float* __restrict__ row_loss,
                                                        const int32_t* __restrict__ row_correct, int64_t n, float scale,
                                                        float* __restrict__ totals) {
    float l = 0.f, c = 0.f;
    for (int64_t i = threadIdx.x; i < n; i += 1024) l += row_loss[i], c += float(row_correct[i]);
    add_totals(l, c, scale, totals);
}
__global__ __launch_bounds__(1024) void sum_blocks_kernel(const float2* __restrict__ sums, int32_t n, float scale, float* __restrict__ totals) {
    float l = 0.f, c = 0.f;
    for (int32_t i = threadIdx.x; i < n; i += 1024) l += sums[i].x, c += sums[i].y;
    add_totals(l, c, scale, totals);
}

__global__ __launch_bounds__(kBlock) void sgd_kernel(float* __restrict__ w, const float* __restrict__ dw, int64_t n,
                                                     float lr) {
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) w[i] -= lr * dw[i];
}

}  // namespace

hipError_t varco_launch_softmax_xent(int dtype, const void* logits, int64_t ld, const int32_t* labels, int64_t n_rows,
                                     int32_t n_classes, float scale, void* dlogits, int64_t ldd, float* row_loss,
                                     int32_t* row_correct, float* totals, float* block_sums, hipStream_t stream) {
    if (n_rows == 0) return hipSuccess;
    float2* const sums = totals ? reinterpret_cast<float2*>(block_sums) : nullptr;
    unsigned blocks = 0;
    auto go = [&](auto type, auto gc, auto ec) {
        using T = typename decltype(type)::type;
        constexpr int G = decltype(gc)::value;
        blocks = unsigned(std::min<int64_t>((n_rows + kBlock / G - 1) / (kBlock / G), kLossBlocks));
        hipLaunchKernelGGL((softmax_xent_kernel<T, G, decltype(ec)::value>), dim3(blocks), dim3(kBlock), 0, stream, static_cast<const T*>(logits),
                           ld, labels, n_rows, n_classes, scale, static_cast<T*>(dlogits), ldd, row_loss, row_correct, sums);
    };
    auto with_size = [&](auto type) {
        if (n_classes <= 8)
            go(type, Int<4>{}, Int<2>{});
        else if (n_classes <= 16)
            go(type, Int<8>{}, Int<2>{});
        else if (n_classes <= 64)
            go(type, Int<16>{}, Int<4>{});
        else if (n_classes <= 512)
            go(type, Int<64>{}, Int<8>{});
        else
            go(type, Int<64>{}, Int<0>{});
    };
    if (dtype == VARCO_BF16)
        with_size(Tag<bf16_t>{});
    else
        with_size(Tag<float>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !totals) return e;
    if (sums)
        hipLaunchKernelGGL(sum_blocks_kernel, dim3(1), dim3(1024), 0, stream, sums, int32_t(blocks), scale, totals);
    else
        hipLaunchKernelGGL(sum_rows_kernel, dim3(1), dim3(1024), 0, stream, row_loss, row_correct, n_rows, scale, totals);
    return hipGetLastError();
}

hipError_t varco_launch_sgd(float* w, const float* dw, int64_t n, float lr, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int64_t want = (n + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(sgd_kernel, dim3(unsigned(want < 256 * 16 ? want : 256 * 16)), dim3(kBlock), 0, stream, w, dw, n, lr);
    return hipGetLastError();
}
