// Last step of a dX product: partial results summed, rows put back in place, loss summed.
#pragma once
#include <type_traits>

#include "flce_device.h"
#include "rowreduce.h"

namespace flce {

// Row i of a chunk's dX, for the chunk's `rows` rows (or *live of them):
//     out[idx ? idx[i] : i] (+)= sum_s src[s][i]        in the fixed order s = 0, 1, ...
// src: fp32 partial results of the K ranges (split_stride elements apart, dyn_nsplit their number
// when only the device knows it), or with nsplit = 1 the product's rows in the storage type.
// With ADD the row is added to what out holds (dX summed over heads).  One wavefront per segment, 4
// elements per lane and access with VEC4 (n, split_stride and the pointers are multiples of 4).
// The first workgroup sums the chunk's losses (row_loss not null).
// Latency bound at small sizes: one launch where the sum over K ranges, the scatter, the loss sum
// and its finalisation were four of 4-5 us each; in front of a dW product on small tiles its
// workgroups ride along with that launch instead (nothing in it waits for the other).
struct FinishArgs {
    const void* src;
    int src_f32;            // src: fp32 partial results, or rows in the storage type
    int64_t split_stride;
    int nsplit;
    const int* dyn_nsplit;
    const int* idx;
    const int* live;
    int rows, n;
    void* out;
    int add;
    const float* row_loss;
    DeviceHeader* hdr;
    LossOut loss;
    int segs;               // FIN_SEG elements of a row per wavefront
    int blocks;             // workgroups: one per 4 segments and one for the losses, rounded up to a multiple of 8
};
// (Rows are cut into segments so that a few long rows with many partial results fill the chip too:
// 180 rows of 4096 with 16 ranges took 45 us with a wavefront per row.)
constexpr int FIN_SEG = 512;
// K ranges whose loads a wavefront has in flight, twice as many where there are more (and no more loads than
// ranges where there are few: 7776 x 2880 with 2 ranges 33 us, 55 with groups of 8): with 62 ranges, one wait for
// memory after the other, this launch was a quarter of the call (whole calls, 4 one by one / 8 together, us: 19 x
// 448 x 32000 50.9 / 42.6, 58 x 320 x 44288 56.9 / 48.8, 94 x 384 x 23460 43.1 / 38.1, 2 heads of 218 x 312 x
// 104206 200 / 188).
constexpr int FIN_AHEAD = 8;
inline int finish_segs(int64_t n) { return (int)((n + FIN_SEG - 1) / FIN_SEG); }
inline int64_t finish_blocks(int64_t rows, int64_t n) { return ((rows * finish_segs(n) + 3) / 4 + 1 + 7) / 8 * 8; }

template <typename T, typename SrcT, bool ADD, int E, bool MANY>
__device__ __forceinline__ void finish_row(const FinishArgs& f, int i, int j0, int lane) {
    const int nsplit = f.dyn_nsplit ? *f.dyn_nsplit : f.nsplit;
    const SrcT* from = static_cast<const SrcT*>(f.src) + (int64_t)i * f.n;
    T* to = static_cast<T*>(f.out) + (int64_t)(f.idx ? f.idx[i] : i) * f.n;
    struct alignas(E * sizeof(SrcT)) In { SrcT e[E]; };
    struct alignas(E * sizeof(T)) Out { T e[E]; };
    const int j1 = min(f.n, j0 + FIN_SEG);
#pragma unroll 2
    for (int j = j0 + lane * E; j < j1; j += WAVE * E) {
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
        if constexpr (std::is_same<SrcT, float>::value) {   // (rows in the storage type are whole sums)
            // all of a group's loads before the first sum: a wavefront waits for memory once per group (past the last
            // range a group repeats it)
            [[maybe_unused]] auto add_group = [&](auto ahead_, int s0) {
                constexpr int AHEAD = decltype(ahead_)::value;
                In b[AHEAD];
#pragma unroll
                for (int k = 0; k < AHEAD; ++k)
                    b[k] = *reinterpret_cast<const In*>(from + (int64_t)min(s0 + k, nsplit - 1) * f.split_stride + j);
#pragma unroll
                for (int k = 0; k < AHEAD; ++k)
#pragma unroll
                    for (int e = 0; e < E; ++e) v[e] = s0 + k < nsplit ? v[e] + to_f32(b[k].e[e]) : v[e];
            };
            int s = 1;
            if constexpr (MANY) {
                for (; nsplit - s > FIN_AHEAD; s += 2 * FIN_AHEAD) add_group(std::integral_constant<int, 2 * FIN_AHEAD>{}, s);
                if (nsplit - s > FIN_AHEAD / 2) {
                    add_group(std::integral_constant<int, FIN_AHEAD>{}, s);
                    s += FIN_AHEAD;
                }
            }
#pragma unroll 4
            for (; s < nsplit; ++s) {
                const In b = *reinterpret_cast<const In*>(from + (int64_t)s * f.split_stride + j);
#pragma unroll
                for (int e = 0; e < E; ++e) v[e] += to_f32(b.e[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) o.e[e] = from_f32<T>(v[e]);
        *reinterpret_cast<Out*>(to + j) = o;
    }
}
// One workgroup of 256 threads; part: 32 bytes of LDS.  MANY: for more than FIN_AHEAD ranges (its registers cost
// launches that only move rows 10 %).
template <typename T, int E, bool MANY = true>
__device__ __forceinline__ void finish_dx(const FinishArgs& f, int block, void* part) {
    if (block == 0) {   // (first: it takes longer than a few rows do)
        if (f.row_loss) loss_accumulate(f.row_loss, f.rows, f.hdr, f.loss, static_cast<double*>(part));
        return;
    }
    const int u = (block - 1) * 4 + (int)threadIdx.x / WAVE, lane = (int)threadIdx.x & (WAVE - 1);
    const int i = u / f.segs, j0 = (u - i * f.segs) * FIN_SEG;
    if (i >= (f.live ? min(f.rows, *f.live) : f.rows)) return;
    if (f.src_f32) {
        if (f.add) finish_row<T, float, true, E, MANY>(f, i, j0, lane); else finish_row<T, float, false, E, MANY>(f, i, j0, lane);
    } else if (E == 4 && sizeof(T) == 2 && f.n % 8 == 0) {   // whole rows in the storage type: 16 bytes per lane
        constexpr int E8 = E == 4 ? 8 : E;                   // (dX and the workspace are 16-byte aligned)
        if (f.add) finish_row<T, T, true, E8, false>(f, i, j0, lane); else finish_row<T, T, false, E8, false>(f, i, j0, lane);
    } else {
        if (f.add) finish_row<T, T, true, E, false>(f, i, j0, lane); else finish_row<T, T, false, E, false>(f, i, j0, lane);
    }
}
template <typename T, bool VEC4, bool MANY>
__global__ __launch_bounds__(256) void finish_dx_kernel(FinishArgs f) {
    __shared__ double part[4];
    finish_dx<T, VEC4 ? 4 : 1, MANY>(f, (int)blockIdx.x, part);
}

// One launch for the gradients of a chunk on small tiles: dX's tiles and K ranges (dx_blocks, a multiple of
// 8) and dW's tiles, which do not depend on one another; without K ranges also a workgroup for the losses
// (8 ids, in front), and every workgroup puts the rows of its own tile of dX in place, so that no launch follows
// (fin.idx null: they stay in the chunk's block, for the RMSNorm backward, which also sums the losses).
// (With K ranges finish_dx_kernel follows.  Having the last workgroup of a tile add its ranges up instead
// costs 15 us: partial results written through to memory and 64 KB of each read back by one workgroup;
// 1024 x 512 x 8192 with 8 ranges 58 -> 73 us, 209 x 448 x 2179 with 4 ranges 27 -> 41.)
struct GradArgs {
    FinishArgs fin;    // src, idx, n, out, add, and the losses (row_loss null: not here)
    int dx_blocks;
    // dW's workgroups where theirs are the longer K loops and they come first, else 0 (a launch that ends in its
    // longest workgroups: 7005 x 3392 x 448 200 -> 207 us, 3195 x 2560 x 829 62.5 -> 65.2)
    int dw_first;
};

// Rows of the TILE x TILE tile at (m0, n0) of dX, which this workgroup (256 threads) has just written to
// f.src, to their places (see finish_dx).
template <typename T, int TILE>
__device__ __forceinline__ void place_tile(const FinishArgs& f, int m0, int n0, int rows) {
    const int tid = threadIdx.x;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the L1 is write-through)
    __syncthreads();
    constexpr int LANES = TILE / 4, RPP = 256 / LANES;   // threads per row, rows at a time
    const int col = n0 + tid % LANES * 4;
    if (col >= f.n) return;   // (n % 4 == 0)
    struct alignas(4 * sizeof(T)) Quad { T e[4]; };
    const T* src = static_cast<const T*>(f.src);
#pragma unroll 8
    for (int r = tid / LANES; r < rows; r += RPP) {
        const int i = m0 + r;
        Quad q = *reinterpret_cast<const Quad*>(src + (int64_t)i * f.n + col);
        Quad* to = reinterpret_cast<Quad*>(static_cast<T*>(f.out) + (int64_t)f.idx[i] * f.n + col);
        if (f.add) {
            const Quad o = *to;
#pragma unroll
            for (int e = 0; e < 4; ++e) q.e[e] = from_f32<T>(to_f32(q.e[e]) + to_f32(o.e[e]));
        }
        *to = q;
    }
}

}  // namespace flce
