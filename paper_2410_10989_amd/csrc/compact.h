// Rows whose target is ignore_index take no part in the result: their loss is not
// counted, their dlogits are zero, so they add nothing to dW and their dX row is
// zero.  Instead of projecting them and multiplying zeros, the chunk loop runs over
// the VALID rows: chunk c gathers the next (at most) C valid rows of the batch into a
// dense block, all three products and the row kernel run on the block, and dX is
// scattered back; ignored rows of dX are zeroed once.  Where a chunk ends in the
// batch and how many live rows it holds is known on the device only: a two-word
// device array carries the row cursor and the live row count from kernel to kernel
// ("dynamic rows"), so the host never waits and the launches are sized for the worst
// case (no row ignored).  Every output element is computed by the same arithmetic as
// without compaction; only dW sums the same non-zero terms in other groups of K.
#pragma once
#include "flce_device.h"
#include "rowreduce.h"
#include "scheduler.h"

namespace flce {

// Which batches one launch per chunk (select_rows_kernel) counts, collects, copies and clears; the
// others count once and walk the batch with a cursor (the kernels below it).  Every workgroup of the
// one launch looks at all targets, 8 BT bytes from L2, once per chunk; the cursor needs three more
// launches, two of them once per batch.  Whole calls at V = 64, H = 64, cursor / one launch per chunk, us:
//   BT 4096   1 chunk 65 / 57, 4 chunks 142 / 130, 16 chunks 437 / 410
//   BT 8192   1 chunk 106 / 92, 4 chunks 181 / 170, 16 chunks 482 / 472
//   BT 12288  1 chunk 147 / 129, 4 chunks 222 / 215, 16 chunks 526 / 541
//   BT 16384  1 chunk 188 / 166, 4 chunks 258 / 252, 16 chunks 567 / 606, 64 chunks 1797 / 2015
//   BT 24576  2 chunks 293 / 271, 4 chunks 335 / 335, 16 chunks 661 / 744
//   BT 32768  1 chunk 346 / 307, 2 chunks 376 / 347, 4 chunks 424 / 416, 16 chunks 713 / 865
// (with H = 4096 the same differences in us): break-even at about 4, 5, 8 and 12 chunks.
constexpr int64_t SEL_MAX_ROWS = 32768, SEL_ANY_CHUNKS_ROWS = 8192, SEL_MAX_SCANS = 131072;
inline bool one_launch_selects(int64_t BT, int64_t nchunks) {
    return BT <= SEL_ANY_CHUNKS_ROWS || (BT <= SEL_MAX_ROWS && BT * nchunks <= SEL_MAX_SCANS);
}
constexpr int SEL_GRID = 1024;   // workgroups at most: 4 rows each up to 4096, 32 at SEL_MAX_ROWS

constexpr int CP_THREADS = 1024;
constexpr int CP_PER = 8;   // consecutive rows per thread and round

// Words of the device array that carries the chunk loop's state from kernel to kernel.
enum { DYN_CURSOR = 0,      // first batch row the next chunk looks at
       DYN_LIVE = 1,        // rows of the current chunk
       DYN_FIRST_LIVE = 2,  // index of the first chunk launch that holds rows
       DYN_DX_RANGES = 3 }; // K ranges of the current chunk's dX product
static_assert(DYN_DX_RANGES < (int)DYN_WORDS, "room for the words");

// How the N valid rows of a batch are dealt to the launches (see compact_chunk_kernel).
struct RowDeal {
    int first_live, quota;
};
__device__ __forceinline__ RowDeal deal_rows(int n_valid, int C, int nchunks) {
    const int n_live = max(1, (n_valid + C - 1) / C);
    return {nchunks - n_live, min(C, ((n_valid + n_live - 1) / n_live + 255) / 256 * 256)};
}
// K ranges of a chunk's dX product (dx_max_ranges = 1: not cut, or not chosen here)
__device__ __forceinline__ int dx_ranges_of(int rows, int dx_tiles_n, int dx_ksteps, int dx_max_ranges) {
    return dx_max_ranges > 1
        ? choose_ksplit((int64_t)((rows + 255) / 256) * dx_tiles_n, dx_ksteps, dx_max_ranges) : 1;
}

// Launch `c` of `nchunks` for a batch of at most SEL_MAX_ROWS rows: what compact_chunk_kernel,
// count_valid_kernel, gather_rows_kernel and zero_ignored_rows_kernel do, in one launch, or as the first
// workgroups of the logits launch (select_in_logits).
// Workgroup b owns batch rows b R .. b R + R - 1 (R <= 64 rows); it counts the valid rows in front
// of them and in the whole batch (every workgroup reads all targets), which gives each of its
// rows its place in the chunk.  One wavefront per row copies it to Xg (X not null; with gamma it
// writes the RMS-normalised row and rstd = 1 / RMS instead, see rmsnorm_fwd_kernel), or clears its
// gradient row (zero_out not null, row ignored).  Workgroup 0 writes the header (c = 0) and dyn.
// Measured, 1024 rows of 512 bf16: 4 launches, 19 us -> one of 5; 4096 x 4096: 32 -> 15 us.
template <typename T>
struct SelectArgs {
    const int64_t* targets;
    int BT;
    int64_t ignore_index;
    float weight;
    int C, c, nchunks;
    int dx_tiles_n, dx_ksteps, dx_max_ranges;
    DeviceHeader* hdr;
    const T* X;
    int n;
    T* Xg;
    T* zero_out;
    int* idx;
    int64_t* tv;
    int* dyn;
    const T* gamma;
    float eps;
    float* rstd;
    int blocks;
};
// (The pointers are parameters for their __restrict__, which local copies of a struct's do not have: without
// it the copies of a wavefront wait for one another, 13947 x 3648 bf16 64 us instead of 51.)
template <typename T>
__device__ __forceinline__ void select_rows_of(const SelectArgs<T>& s, int block, int (*part)[2],   // part: [4][2] in LDS
                                               const int64_t* __restrict__ targets, const T* __restrict__ X,
                                               T* __restrict__ Xg, T* __restrict__ zero_out, int* __restrict__ idx,
                                               int64_t* __restrict__ tv, int* __restrict__ dyn,
                                               const T* __restrict__ gamma, float* __restrict__ rstd) {
    const int64_t ignore_index = s.ignore_index;
    const int BT = s.BT, C = s.C, c = s.c, nchunks = s.nchunks, n = s.n;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int R = (BT + s.blocks - 1) / s.blocks;
    const int r0 = min(BT, block * R), r1 = min(BT, r0 + R);
    int before = 0, n_valid = 0;
#pragma unroll 8
    for (int i = tid; i < BT; i += 256) {
        const int v = targets[i] != ignore_index;
        n_valid += v;
        before += (i < r0) ? v : 0;
    }
    before = wave_sum(before);
    n_valid = wave_sum(n_valid);
    if (lane == 0) {
        part[wave][0] = before;
        part[wave][1] = n_valid;
    }
    __syncthreads();
    before = part[0][0] + part[1][0] + part[2][0] + part[3][0];
    n_valid = part[0][1] + part[1][1] + part[2][1] + part[3][1];
    const RowDeal deal = deal_rows(n_valid, C, nchunks);
    const int begin = (c - deal.first_live) * deal.quota;   // of this chunk among the valid rows
    const int count = c < deal.first_live ? 0 : max(0, min(deal.quota, n_valid - begin));
    if (block == 0 && tid == 0) {
        if (c == 0) write_header(s.hdr, n_valid, s.weight);
        dyn[DYN_LIVE] = count;
        dyn[DYN_FIRST_LIVE] = deal.first_live;
        dyn[DYN_DX_RANGES] = dx_ranges_of(count, s.dx_tiles_n, s.dx_ksteps, s.dx_max_ranges);
    }
    const int64_t t = (r0 + lane < r1) ? targets[r0 + lane] : ignore_index;
    const unsigned long long mask = __ballot(t != ignore_index);
    const int at = before + __popcll(mask & ((1ull << lane) - 1)) - begin;   // place of row r0 + lane, if valid
    constexpr int VEC = 16 / sizeof(T);
    const int nv = n / VEC;
    for (int j = wave; j < r1 - r0; j += 4) {
        const int place = __shfl(at, j, WAVE);
        const bool valid = (mask >> j) & 1;
        const int r = r0 + j;
        if (!valid) {
            if (!zero_out) continue;
            const u32x4 zero = {0u, 0u, 0u, 0u};
            u32x4* dst = reinterpret_cast<u32x4*>(zero_out + (int64_t)r * n);
            for (int v = lane; v < nv; v += WAVE) dst[v] = zero;
        } else if (place >= 0 && place < count) {
            if (lane == 0) {
                idx[place] = r;
                tv[place] = targets[r];
            }
            if (!X) continue;
            const u32x4* src = reinterpret_cast<const u32x4*>(X + (int64_t)r * n);
            u32x4* dst = reinterpret_cast<u32x4*>(Xg + (int64_t)place * n);
            if (!gamma) {
#pragma unroll 8
                for (int v = lane; v < nv; v += WAVE) dst[v] = src[v];
                continue;
            }
            const u32x4* gr = reinterpret_cast<const u32x4*>(gamma);
            float ss = 0.f;
#pragma unroll 8
            for (int v = lane; v < nv; v += WAVE) {
                float x[VEC];
                RowVec<T>::unpack(src[v], x);
#pragma unroll
                for (int e = 0; e < VEC; ++e) ss += x[e] * x[e];
            }
            ss = wave_sum(ss);
            const float scale = 1.0f / sqrtf(ss / (float)n + s.eps);
            if (lane == 0) rstd[place] = scale;
#pragma unroll 4
            for (int v = lane; v < nv; v += WAVE) {   // (the row comes from cache this time)
                float x[VEC], g[VEC];
                RowVec<T>::unpack(src[v], x);
                RowVec<T>::unpack(gr[v], g);
#pragma unroll
                for (int e = 0; e < VEC; ++e) x[e] = x[e] * scale * g[e];
                dst[v] = RowVec<T>::pack(x);
            }
        }
    }
}
template <typename T>
__device__ __forceinline__ void select_rows(const SelectArgs<T>& s, int block, int (*part)[2]) {
    select_rows_of<T>(s, block, part, s.targets, s.X, s.Xg, s.zero_out, s.idx, s.tv, s.dyn, s.gamma, s.rstd);
}

template <typename T>
__global__ __launch_bounds__(256) void select_rows_kernel(SelectArgs<T> s) {
    __shared__ int part[4][2];
    select_rows(s, (int)blockIdx.x, part);
}

// The selection inside the logits launch of a batch that is one chunk: its workgroups come first and leave
// what the later launches read; the product's workgroups do not wait for them, each finds the rows of
// its tile by itself.
//
// Valid rows of the batch, and which ones have the places m0 .. m0 + count - 1 among them: begin() by all
// wavefronts of a workgroup, then place().  Wavefront w looks at its share of the batch, 64 rows at a time, and
// keeps these masks for place(): at most MAX_ROWS rows.
template <int WAVES>
struct TileRows {
    static constexpr int KEEP = 8, MAX_ROWS = KEEP * WAVE * WAVES;
    const int64_t* __restrict__ targets;
    int64_t ignore_index;
    int r0, r1, before;   // the wavefront's share, and the valid rows in front of it
    unsigned long long kept[KEEP];

    __device__ __forceinline__ unsigned long long look(int r) const {   // r: of the first of 64 rows
        const int mine = r + (int)(threadIdx.x & (WAVE - 1));
        return __ballot(targets[min(mine, r1 - 1)] != ignore_index && mine < r1);   // (no branch around the load)
    }
    __device__ __forceinline__ int begin(const int64_t* t, int BT, int64_t ignore, int* totals) {   // totals: [WAVES] in LDS
        targets = t;
        ignore_index = ignore;
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
        const int per = (BT + WAVES * WAVE - 1) / (WAVES * WAVE) * WAVE;
        r0 = min(BT, wave * per);
        r1 = min(BT, r0 + per);
        int n = 0;
        if (r0 < r1) {
#pragma unroll
            for (int g = 0; g < KEEP; ++g) kept[g] = look(r0 + g * WAVE);
#pragma unroll
            for (int g = 0; g < KEEP; ++g) n += __popcll(kept[g]);
        }
        if ((threadIdx.x & (WAVE - 1)) == 0) totals[wave] = n;
        __syncthreads();
        int all = 0;
        before = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            before += w < wave ? totals[w] : 0;
            all += totals[w];
        }
        return __builtin_amdgcn_readfirstlane(all);
    }
    __device__ __forceinline__ void place(int m0, int count, int* rows) const {   // rows: [count] in LDS
        const int lane = threadIdx.x & (WAVE - 1);
        int at = before - m0;
        auto put = [&](int r, unsigned long long mask) {
            const int mine = at + __popcll(mask & ((1ull << lane) - 1));
            if (mask >> lane & 1 && mine >= 0 && mine < count) rows[mine] = r + lane;
            at += __popcll(mask);
        };
        if (r0 < r1) {
#pragma unroll
            for (int g = 0; g < KEEP; ++g) put(r0 + g * WAVE, kept[g]);
        }
        __syncthreads();
    }
};

// One workgroup; launch `c` of `nchunks`, each sized for `C` rows.  The N valid rows of
// the batch (N = hdr->n_valid, counted before the loop) are dealt evenly to the LAST
// n = max(1, ceil(N / C)) launches, ceil_256(ceil(N / n)) rows each (the last one takes
// what is left), so no launch ends up with a handful of rows and a batch with many
// ignored rows runs fewer chunks: launches before the first live one hold no rows, and
// the dW product, which keeps fp32 partial sums from the first live chunk to the last
// launch, skips them altogether.  The last launch is always live (with N = 0 it holds
// zero rows and writes a zero dW).  For a live launch this collects the next valid rows
// of the batch starting at the row cursor:
//   idx[i] = row of the i-th collected row (ascending), tv[i] = its target
//   dyn[DYN_LIVE] = rows collected, dyn[DYN_CURSOR] = the row after the last one looked at
//   dyn[DYN_DX_RANGES] = K ranges of the dX product for that many rows (dx_tiles_n tile
//   columns, dx_ksteps K steps, at most dx_max_ranges ranges)
__global__ __launch_bounds__(CP_THREADS) void compact_chunk_kernel(
    const int64_t* __restrict__ targets, int BT, int64_t ignore_index, int C, int c, int nchunks,
    const DeviceHeader* __restrict__ hdr, int dx_tiles_n, int dx_ksteps, int dx_max_ranges,
    int* __restrict__ idx, int64_t* __restrict__ tv, int* __restrict__ dyn) {
    __shared__ int wave_total[CP_THREADS / WAVE];
    __shared__ int s_next;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int n_valid = hdr->n_valid;
    const RowDeal deal = deal_rows(n_valid, C, nchunks);
    const int cap = c < deal.first_live ? 0 : deal.quota;
    int cursor = c == 0 ? 0 : dyn[DYN_CURSOR];
    int found = 0;
    while (cursor < BT && found < cap) {   // uniform: every thread sees the same values
        const int r0 = min(BT, cursor + tid * CP_PER), r1 = min(BT, r0 + CP_PER);
        int n = 0;
        for (int r = r0; r < r1; ++r) n += (targets[r] != ignore_index);
        int incl = n;   // inclusive prefix sum over the workgroup
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const int up = __shfl_up(incl, o, WAVE);
            if (lane >= o) incl += up;
        }
        if (tid == 0) s_next = -1;
        __syncthreads();   // also: wave_total and s_next of the previous round are no longer read
        if (lane == WAVE - 1) wave_total[wave] = incl;
        __syncthreads();
        int base = 0, total = 0;
        for (int w = 0; w < CP_THREADS / WAVE; ++w) {
            if (w < wave) base += wave_total[w];
            total += wave_total[w];
        }
        int at = found + base + incl - n;
        for (int r = r0; r < r1; ++r) {
            const int64_t t = targets[r];
            if (t != ignore_index) {
                if (at < cap) {
                    idx[at] = r;
                    tv[at] = t;
                    if (at == cap - 1) s_next = r + 1;   // the chunk is full after this row
                }
                ++at;
            }
        }
        __syncthreads();
        if (found + total >= cap) {
            found = cap;
            cursor = s_next;
        } else {
            found += total;
            cursor = min(BT, cursor + CP_THREADS * CP_PER);
        }
    }
    if (tid == 0) {
        dyn[DYN_CURSOR] = cursor;
        dyn[DYN_LIVE] = found;
        dyn[DYN_FIRST_LIVE] = deal.first_live;
        dyn[DYN_DX_RANGES] = dx_ranges_of(found, dx_tiles_n, dx_ksteps, dx_max_ranges);
    }
}

// out[i][:] = in[idx[i]][:] for the live rows i; one workgroup per row, rows are n
// 16-byte vectors long.
__global__ __launch_bounds__(256) void gather_rows_kernel(const u32x4* __restrict__ in,
                                                          const int* __restrict__ idx,
                                                          const int* __restrict__ live, int n,
                                                          u32x4* __restrict__ out) {
    const int i = blockIdx.x;
    if (i >= *live) return;
    const u32x4* src = in + (int64_t)idx[i] * n;
    u32x4* dst = out + (int64_t)i * n;
    for (int v = threadIdx.x; v < n; v += 256) dst[v] = src[v];
}

// Rows with an ignored target get a zero gradient.  Workgroups stride over the rows of
// the batch.
template <typename T>
__global__ __launch_bounds__(256) void zero_ignored_rows_kernel(const int64_t* __restrict__ targets,
                                                                int64_t BT, int64_t ignore_index,
                                                                int n, T* __restrict__ out) {
    constexpr int VEC = 16 / sizeof(T);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int64_t r = blockIdx.x; r < BT; r += gridDim.x) {
        if (targets[r] != ignore_index) continue;   // uniform per workgroup
        u32x4* dst = reinterpret_cast<u32x4*>(out + r * n);
        for (int v = threadIdx.x; v < n / VEC; v += 256) dst[v] = zero;
    }
}

}  // namespace flce
