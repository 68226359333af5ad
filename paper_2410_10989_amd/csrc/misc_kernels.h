// Last step of a dX product: partial results summed, rows put back in place, loss summed.
#pragma once
#include "flce_device.h"
#include "rowreduce.h"

namespace flce {

// Row i of a chunk's dX, for the chunk's `rows` rows (or *live of them):
//     out[idx ? idx[i] : i] (+)= sum_s src[s][i]        in the fixed order s = 0, 1, ...
// src: fp32 partial results of the K ranges (split_stride elements apart, dyn_nsplit their number
// when only the device knows it), or with nsplit = 1 the product's rows in the storage type.
// With ADD the row is added to what out holds (dX summed over heads).  One wavefront per row, 4
// elements per lane and access with VEC4 (n, split_stride and the pointers are multiples of 4).
// The workgroup past the rows sums the chunk's losses (row_loss not null).
// Latency bound at small sizes: one launch where the sum over K ranges, the scatter, the loss sum
// and its finalisation were four of 4-5 us each.
template <typename T, typename SrcT, bool ADD, bool VEC4>
__global__ __launch_bounds__(256) void finish_dx_kernel(const SrcT* __restrict__ src, int64_t split_stride, int nsplit,
                                                        const int* __restrict__ dyn_nsplit,
                                                        const int* __restrict__ idx, const int* __restrict__ live,
                                                        int rows, int n, T* __restrict__ out,
                                                        const float* __restrict__ row_loss, DeviceHeader* hdr,
                                                        LossOut loss) {
    const int row_groups = (rows + 3) / 4;
    if ((int)blockIdx.x == row_groups) {
        if (row_loss) loss_accumulate(row_loss, rows, hdr, loss);
        return;
    }
    const int i = (int)blockIdx.x * 4 + (int)threadIdx.x / WAVE;
    if (i >= (live ? min(rows, *live) : rows)) return;
    if (dyn_nsplit) nsplit = *dyn_nsplit;
    const SrcT* from = src + (int64_t)i * n;
    T* to = out + (int64_t)(idx ? idx[i] : i) * n;
    constexpr int E = VEC4 ? 4 : 1;
    struct alignas(E * sizeof(SrcT)) In { SrcT e[E]; };
    struct alignas(E * sizeof(T)) Out { T e[E]; };
    for (int j = ((int)threadIdx.x & (WAVE - 1)) * E; j < n; j += WAVE * E) {
        float v[E];
        const In a = *reinterpret_cast<const In*>(from + j);
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = to_f32(a.e[e]);
        Out o{};
        if constexpr (ADD) {
            o = *reinterpret_cast<const Out*>(to + j);
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] += to_f32(o.e[e]);
        }
#pragma unroll 4
        for (int s = 1; s < nsplit; ++s) {
            const In b = *reinterpret_cast<const In*>(from + (int64_t)s * split_stride + j);
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] += to_f32(b.e[e]);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) o.e[e] = from_f32<T>(v[e]);
        *reinterpret_cast<Out*>(to + j) = o;
    }
}

}  // namespace flce
