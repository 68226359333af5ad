// Row-wise softmax cross entropy with the gradient written over the logits
// (paper section 3.2, CE paragraph: online softmax, in-place dlogits).
//
// One workgroup per row.  Sweep 1 keeps a running (max, sum of exp) pair per
// thread and merges the pairs across the wavefront and the workgroup; the loss
// of the row is lse - z[target] ("safe log": log is only taken of a sum that is
// at least 1).  Sweep 2 rewrites the row as (exp(z - lse) - onehot) / N, or as
// zeros for an ignored row.  N arrives through the device header as 1/N.
#pragma once
#include "flce_device.h"

namespace flce {

struct MaxSum {
    float m, s;   // running maximum and sum of exp(z - m)
};
__device__ __forceinline__ MaxSum ms_merge(MaxSum a, MaxSum b) {
    const float m = fmaxf(a.m, b.m);
    // exp(-inf - finite) = 0 handles empty partners; both -inf cannot occur for
    // the partner that holds at least one element, guard it anyway
    const float sa = (a.m == -INFINITY) ? 0.f : a.s * __expf(a.m - m);
    const float sb = (b.m == -INFINITY) ? 0.f : b.s * __expf(b.m - m);
    return {m, sa + sb};
}

// The arithmetic per logit decides the speed of these kernels as much as the memory
// traffic does (a CU retires 64 plain and 16 transcendental lane operations per
// cycle), so both sweeps work on whole 16-byte vectors and exponentials are taken as
// exp2(fma(z, log2 e, c)): one multiply-add and one v_exp_f32 per logit.
constexpr float RR_LOG2E = 1.4426950408889634f;

template <typename T> struct RowVec;
template <> struct RowVec<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void unpack(const u32x4& raw, float (&f)[4]) {
#pragma unroll
        for (int w = 0; w < 4; ++w) f[w] = __uint_as_float(raw[w]);
    }
    static __device__ __forceinline__ u32x4 pack(const float (&f)[4]) {
        u32x4 r;
#pragma unroll
        for (int w = 0; w < 4; ++w) r[w] = __float_as_uint(f[w]);
        return r;
    }
};
template <> struct RowVec<bf16_t> {
    static constexpr int N = 8;
    // a bf16 is the upper half of the float with the same value
    static __device__ __forceinline__ void unpack(const u32x4& raw, float (&f)[8]) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            f[2 * w] = __uint_as_float(raw[w] << 16);
            f[2 * w + 1] = __uint_as_float(raw[w] & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ u32x4 pack(const float (&f)[8]) {
        u32x4 r;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const bf16x2 p = {(bf16_t)f[2 * w], (bf16_t)f[2 * w + 1]};   // round to nearest even
            r[w] = __builtin_bit_cast(uint32_t, p);
        }
        return r;
    }
};

// exp(z - ref).  bf16 logits: exp2(fma(z, log2 e, -ref log2 e)), the rounding of the
// constant (half an ulp of |ref| log2 e) is far below what bf16 resolves.  fp32
// logits: the difference is taken first, which stays exact for large |z|.
template <typename T> struct RowExp;
template <> struct RowExp<bf16_t> {
    float c;
    __device__ __forceinline__ explicit RowExp(float ref) : c(-ref * RR_LOG2E) {}
    __device__ __forceinline__ float operator()(float z) const {
        return __builtin_amdgcn_exp2f(fmaf(z, RR_LOG2E, c));
    }
};
template <> struct RowExp<float> {
    float ref;
    __device__ __forceinline__ explicit RowExp(float r) : ref(r) {}
    __device__ __forceinline__ float operator()(float z) const {
        return __builtin_amdgcn_exp2f((z - ref) * RR_LOG2E);
    }
};

// Online softmax update with N logits at once: one rescale of the running sum per
// vector instead of one decision per logit.
template <typename T, int N>
__device__ __forceinline__ void ms_push_vec(MaxSum& a, const float (&f)[N]) {
    float vm = f[0];
#pragma unroll
    for (int j = 1; j < N; ++j) vm = fmaxf(vm, f[j]);
    const float m_new = fmaxf(a.m, vm);
    // a row may start with -inf logits: keep the reference finite
    const RowExp<T> ex((m_new == -INFINITY) ? 0.f : m_new);
    float s = a.s * ex(a.m);   // a.m = -inf: s was 0 and stays 0
#pragma unroll
    for (int j = 0; j < N; ++j) s += ex(f[j]);
    a.m = m_new;
    a.s = s;
}
template <typename T>
__device__ __forceinline__ void ms_push(MaxSum& a, float x) {
    const float f[1] = {x};
    ms_push_vec<T, 1>(a, f);
}

// (softmax - onehot) / N of one vector: exp(z - lse) * inv_n; the one-hot term only
// touches the vector that holds the target column.
template <typename T>
__device__ __forceinline__ u32x4 ce_gradient_vec(const u32x4& raw, int i, int tcol,
                                                 const RowExp<T>& ex, float inv_n) {
    constexpr int N = RowVec<T>::N;
    float f[N];
    RowVec<T>::unpack(raw, f);
#pragma unroll
    for (int j = 0; j < N; ++j) f[j] = ex(f[j]) * inv_n;
    if (i == tcol / N) {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (j == tcol % N) f[j] -= inv_n;
    }
    return RowVec<T>::pack(f);
}
template <typename T>
__device__ __forceinline__ T ce_gradient_one(T z, int v, int tcol, const RowExp<T>& ex, float inv_n) {
    float g = ex(to_f32(z)) * inv_n;
    if (v == tcol) g -= inv_n;
    return from_f32<T>(g);
}

// A row's loss.  THROUGH: to memory, for a workgroup on another XCD in the same launch (the launch that sums
// the losses otherwise finds them in the L2s: 2 us less).
template <bool THROUGH>
__device__ __forceinline__ void store_loss(float* p, float loss) {
    if constexpr (THROUGH) __hip_atomic_store(p, loss, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = loss;
}

// Merges the per-thread pairs of a workgroup of NW wavefronts; thread 0 then holds
// the row's log-sum-exp, publishes it and the row's loss.  Ends with a barrier, so
// z[target] has been read before any thread overwrites the row.
template <typename T, int NW, bool THROUGH>
__device__ __forceinline__ float row_lse(MaxSum a, const T* z, int64_t t, int row,
                                         float* __restrict__ row_loss, MaxSum* part, float* s_lse) {
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        MaxSum b = {__shfl_xor(a.m, o, WAVE), __shfl_xor(a.s, o, WAVE)};
        a = ms_merge(a, b);
    }
    if (lane == 0) part[wave] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        MaxSum r = part[0];
        for (int w = 1; w < NW; ++w) r = ms_merge(r, part[w]);
        const float l = r.m + logf(r.s);
        *s_lse = l;
        store_loss<THROUGH>(row_loss + row, l - to_f32(z[t]));
    }
    __syncthreads();
    return *s_lse;
}

// Row kernel: one workgroup of THREADS threads per row holds the first THREADS * NV 16-byte
// vectors of the row in registers between the two sweeps, so that part of the row is read from
// HBM once instead of twice; what is beyond is swept twice.  All of a thread's loads are issued
// before the first is consumed.  Rows may start anywhere (a vocabulary of odd size in a dense
// matrix): the vectors lie between a head and a tail of a few scalars.
// What bounds it: HBM, and next to it the arithmetic (about 16 lane operations per logit).
// Three shapes: 256 threads x 12 vectors for rows up to 48 KB and 512 x 12 up to 112 KB, where
// several workgroups fit a CU and overlap one another's memory, reduction and barrier phases;
// 1024 x 16 (256 KB) beyond, where 16 wavefronts keep the per-thread ALU phases short.  TB/s of
// algorithmic traffic, kernel alone, 256 x 12 / 512 x 12 / 1024 x 16: 7.1 / 4.5 / 2.2 at 16 KB rows
// (16384 of them), - / 7.2 / 4.9 at 64 KB (4096), - / 5.3 / 4.8 at 100 KB, - / - / 5.2 at 240 KB.  From 96 to 112 KB
// (seven row lengths of bf16, four of fp32) whole calls of 512 x 12 against 1024 x 16 take 17.7 / 21.4 us (300
// rows), 41 / 51 (1024), 150 / 170 (4096) at 97 KB and 20.5 / 23.5, 46 / 56, 161 / 188 at 112 KB; 64 rows 12.8 / 12.5.
// NL: that many more vectors per thread stay in LDS (9 x 1024: 144 KB; one such workgroup fits a CU by
// its registers anyway).  Used beyond 400 KB rows, without / with, us: 5734 x 256000 bf16 1164 / 1085, 3328 x
// 152064 fp32 843 / 775, 2048 x 204807 bf16 (400 KB) 320 / 313; at 297 KB rows 348 / 368, where the little
// that is swept twice comes from cache.
// NT (nontemporal accesses) where the logits exceed the 256 MB memory-side cache, ordinary / NT:
// 8192 x 128256 bf16 803 / 717 us, 4096 x 122880 bf16 387 / 356, 4096 x 81920 fp32 525 / 419; below it
// they would push out what the next product reads: 4096 x 32000 bf16 73 / 89.  Only for logits that
// another program made: right behind the logits product, which leaves its last output in the
// caches, they cost more than they save (8192 x 128256: 790 / 850 us).
// Rows of 50257 bf16 at odd addresses (4096 of them): 451 us with 2-byte accesses in two sweeps
// before, 155 / 150 (NT) now.
constexpr int RC_THREADS = 1024;
constexpr int RC_NV = 16;
constexpr int RC_NL = 9;
constexpr int RM_THREADS = 512;   // rows up to 112 KB
constexpr int RM_NV = 12;
constexpr int RS_THREADS = 256;   // rows up to 48 KB
constexpr int RS_NV = 12;

// 16-byte accesses of a row; NT: nontemporal, for logits that no cache will keep anyway.
template <bool NT>
__device__ __forceinline__ u32x4 row_load(const u32x4* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT>
__device__ __forceinline__ void row_store(u32x4* p, u32x4 v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Valid rows among targets[0 .. n), the same value returned to every thread of the workgroup.
template <int THREADS>
__device__ __forceinline__ int count_rows(const int64_t* __restrict__ targets, int n, int64_t ignore_index, int* part) {
    int c = 0;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += THREADS) c += (targets[i] != ignore_index);
    c = wave_sum(c);
    if ((threadIdx.x & (WAVE - 1)) == 0) part[threadIdx.x / WAVE] = c;
    __syncthreads();
    int total = 0;
    for (int w = 0; w < THREADS / WAVE; ++w) total += part[w];
    return total;
}
__device__ __forceinline__ void write_header(DeviceHeader* hdr, int n_valid, float weight) {
    hdr->n_valid = n_valid;
    hdr->inv_n = n_valid > 0 ? weight / (float)n_valid : 0.f;
    hdr->loss_sum = 0.0;
}
// A batch of at most this many rows is counted by every workgroup of the row kernel itself (about 1
// us per row and workgroup slot, from L2) instead of by a launch of its own in front of it, which
// takes 4-5 us whatever it does: as many rows as run in two rounds of the CUs in the row length's
// shape (1, 2 or 3 and more workgroups per CU).
inline int64_t ce_count_rows(int64_t row_bytes) {
    return row_bytes > 112 * 1024 ? 512 : row_bytes > 48 * 1024 ? 1024 : 1536;
}
// Counters of finished workgroups: workgroup b counts itself in word b % DONE_GROUPS, the last one of a group
// in the word behind them.  One word takes an arrival every 10-12 ns (1068 rows of one call 14.3 -> 22.5 us
// with a single word); the words lie in lines of their own.
//
// A word holds the launch's ticket and, in its low bits, the count.  It is zero between launches, but launches
// that overlapped on the same words (which the entry points forbid) may leave anything there.  So no
// launch trusts what it finds: its workgroups first raise the words they use to its own ticket and count 0,
// and the count is complete only under that ticket.  Tickets rise from call to call, so the next launch is right again.
constexpr int DONE_GROUPS = 32, DONE_STRIDE = 16;   // words
constexpr int DONE_WORDS = (DONE_GROUPS + 1) * DONE_STRIDE;
constexpr int DONE_COUNT_BITS = 16;
using done_t = unsigned long long;
struct DoneCount {
    done_t* words;   // null: not counted
    done_t ticket;   // of this launch alone, above 0
};
// One thread per workgroup, early: the update runs beside the row's own work.  The last word is raised by the
// workgroups whose numbers name the groups: each is in front of its group's last one (count_done).
__device__ __forceinline__ void open_done(const DoneCount& d) {
    const done_t none = d.ticket << DONE_COUNT_BITS;
    __hip_atomic_fetch_max(d.words + blockIdx.x % DONE_GROUPS * DONE_STRIDE, none, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    if (blockIdx.x < DONE_GROUPS)
        __hip_atomic_fetch_max(d.words + DONE_GROUPS * DONE_STRIDE, none, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The same thread, once what it has stored before and open_done's updates are in memory; true for the last
// workgroup of the launch.
__device__ __forceinline__ bool count_done(const DoneCount& d) {
    const unsigned n = gridDim.x, group = blockIdx.x % DONE_GROUPS;
    const unsigned of_group = (n - group + DONE_GROUPS - 1) / DONE_GROUPS, groups = min(n, (unsigned)DONE_GROUPS);
    const done_t none = d.ticket << DONE_COUNT_BITS;
    done_t* word = d.words + group * DONE_STRIDE;
    if (__hip_atomic_fetch_add(word, (done_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != none + of_group - 1)
        return false;
    __hip_atomic_store(word, (done_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word = d.words + DONE_GROUPS * DONE_STRIDE;
    if (__hip_atomic_fetch_add(word, (done_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != none + groups - 1)
        return false;
    __hip_atomic_store(word, (done_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// The end of a workgroup of ce_rows_kernel with FOLD: the last one of the launch writes the loss.  The
// same sum in the same order as loss_accumulate.
template <int THREADS>
__device__ __forceinline__ void ce_fold_loss(const int64_t* __restrict__ targets, int64_t ignore_index,
                                             const float* row_loss, const DoneCount& done, float* __restrict__ loss,
                                             int* counts) {
    __shared__ int s_last;
    __shared__ double part[4];
    const int tid = threadIdx.x, rows = (int)gridDim.x;
    if (tid == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this row's loss and open_done's updates are in memory
        s_last = count_done(done);
    }
    __syncthreads();
    if (!s_last) return;   // uniform
    const int n = count_rows<THREADS>(targets, rows, ignore_index, counts);   // (a row without a target has not counted)
    double s = 0.0;
    if (tid < 256) {
#pragma unroll 8
        for (int i = tid; i < rows; i += 256)
            s += (double)__hip_atomic_load(row_loss + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s = wave_sum(s);
        if ((tid & 63) == 0) part[tid >> 6] = s;
    }
    __syncthreads();
    if (tid == 0) {
        const double sum = 0.0 + ((part[0] + part[1]) + (part[2] + part[3]));
        *loss = n > 0 ? (float)(sum / (double)n) : 0.f;
    }
}

// count_n > 0: `targets` holds the whole batch, count_n rows; workgroup 0 writes the header for the
// launches that follow.  count_n = 0: the header holds the count.
//
// FOLD (count_n > 0 only): where the whole batch is one launch and nothing follows it, the loss is summed here as well,
// by the workgroup that finishes last (no workgroup waits for another): each one counts itself in `done`
// once its row's loss has been written through to memory (the L2s of the XCDs are not coherent).  It saves a
// launch: whole calls of 19 x 3264 bf16 12.1 -> 9.7 us, 187 x 8320 bf16 12.3 -> 9.7, 227 x 17107 fp32 12.1 -> 9.9.
// Batches beyond CE_FOLD_ROWS have the launch: the count at the end of every workgroup costs them as much (643 x
// 22336 bf16 14.8 -> 15.5, 800 x 15360 fp32 24.2 -> 25.0, 1068 x 11520 bf16 15.0 -> 14.9, 8174 x 1152 fp32 27.3 ->
// 30.4).
constexpr int64_t CE_FOLD_ROWS = 512;
template <typename T, int THREADS, int NV, bool NT, int NL = 0, bool FOLD = false>
__global__ __launch_bounds__(THREADS) void ce_rows_kernel(
    T* __restrict__ Z, int64_t ldz, const int64_t* __restrict__ targets, int V, int zero_pad,
    int64_t ignore_index, DeviceHeader* __restrict__ hdr, float* __restrict__ row_loss,
    const int* __restrict__ live, int count_n, float weight, DoneCount done, float* __restrict__ loss) {
    constexpr int VEC = RowVec<T>::N;
    const int row = blockIdx.x;
    const int tid = threadIdx.x;
    if (live && row >= *live) {   // past the chunk's live rows (uniform per workgroup)
        if (tid == 0) row_loss[row] = 0.f;
        return;
    }
    if constexpr (FOLD) {
        if (tid == 0) open_done(done);
    }
    T* z = Z + (int64_t)row * ldz;
    const int64_t t = targets[row];
    const bool valid = (t != ignore_index);
    // the row may start anywhere: `head` elements up to the first 16-byte boundary, full vectors,
    // and a tail; head and tail (fewer than 2 VEC elements) are handled by scalars, one per thread
    const int head = min(V, (int)((16 - (reinterpret_cast<uintptr_t>(z) & 15)) & 15) / (int)sizeof(T));
    const int nvec = (V - head) / VEC;
    u32x4* zv = reinterpret_cast<u32x4*>(z + head);
    const int edge = tid < V - nvec * VEC ? (tid < head ? tid : nvec * VEC + tid) : -1;

    __shared__ MaxSum part[THREADS / WAVE];
    __shared__ float s_lse;
    __shared__ int counts[THREADS / WAVE];
    __shared__ u32x4 more[NL ? NL * THREADS : 1];   // the row's vectors beyond the registers

    if (tid < zero_pad) z[V + tid] = from_f32<T>(0.f);   // zero_pad < 64
    if (!valid) {                              // uniform per workgroup
        const u32x4 zero = {0u, 0u, 0u, 0u};
        for (int i = tid; i < nvec; i += THREADS) row_store<NT>(zv + i, zero);
        if (edge >= 0) z[edge] = from_f32<T>(0.f);
        if (tid == 0) store_loss<FOLD>(row_loss + row, 0.f);
        if (count_n > 0 && row == 0) {
            const int n = count_rows<THREADS>(targets, count_n, ignore_index, counts);
            if (tid == 0) write_header(hdr, n, weight);
        }
        if constexpr (FOLD) ce_fold_loss<THREADS>(targets, ignore_index, row_loss, done, loss, counts);
        return;
    }

    u32x4 keep[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i = tid + k * THREADS;
        if (i < nvec) keep[k] = row_load<NT>(zv + i);
    }
    MaxSum a = {-INFINITY, 0.f};
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i = tid + k * THREADS;
        if (i < nvec) {
            float f[VEC];
            RowVec<T>::unpack(keep[k], f);
            ms_push_vec<T, VEC>(a, f);
        }
        // one vector at a time: interleaving several would spill the cached row
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NL > 0) {   // (a thread reads back what it wrote itself: no barrier)
#pragma unroll 3
        for (int k = 0; k < NL; ++k) {
            const int i = tid + (NV + k) * THREADS;
            if (i < nvec) {
                const u32x4 raw = row_load<NT>(zv + i);
                more[k * THREADS + tid] = raw;
                float f[VEC];
                RowVec<T>::unpack(raw, f);
                ms_push_vec<T, VEC>(a, f);
            }
        }
    }
    for (int i = tid + (NV + NL) * THREADS; i < nvec; i += THREADS) {   // beyond the cache
        float f[VEC];
        RowVec<T>::unpack(zv[i], f);
        ms_push_vec<T, VEC>(a, f);
    }
    if (edge >= 0) ms_push<T>(a, to_f32(z[edge]));
    float inv_n;   // (not in front of the sweep: that would wait for the whole row first)
    if (count_n > 0) {
        const int n = count_rows<THREADS>(targets, count_n, ignore_index, counts);
        inv_n = weight / (float)n;   // this row is valid: n > 0
        if (row == 0 && tid == 0) write_header(hdr, n, weight);
    } else {
        inv_n = hdr->inv_n;
    }
    const float lse = row_lse<T, THREADS / WAVE, FOLD>(a, z, t, row, row_loss, part, &s_lse);

    const RowExp<T> ex(lse);
    // the target's place among the vectors; a target in the head matches none of them
    const int tcol = (int)t < head ? 0x7fffffff : (int)t - head;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i = tid + k * THREADS;
        // hide the value's history: otherwise the unpacked floats of sweep 1 are kept
        // for reuse here, which does not fit the register file and spills
        asm volatile("" : "+v"(keep[k]));
        if (i < nvec) row_store<NT>(zv + i, ce_gradient_vec<T>(keep[k], i, tcol, ex, inv_n));
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NL > 0) {
#pragma unroll 3
        for (int k = 0; k < NL; ++k) {
            const int i = tid + (NV + k) * THREADS;
            if (i < nvec) row_store<NT>(zv + i, ce_gradient_vec<T>(more[k * THREADS + tid], i, tcol, ex, inv_n));
        }
    }
    for (int i = tid + (NV + NL) * THREADS; i < nvec; i += THREADS)
        row_store<NT>(zv + i, ce_gradient_vec<T>(zv[i], i, tcol, ex, inv_n));
    if (edge >= 0) z[edge] = ce_gradient_one<T>(z[edge], edge, (int)t, ex, inv_n);
    if constexpr (FOLD) ce_fold_loss<THREADS>(targets, ignore_index, row_loss, done, loss, counts);
}

// Where the loss goes once the last row losses are summed (n_heads = 0: not yet).  `heads`: the
// headers of all heads, whose weighted means make up the loss; head_losses (optional) receives the
// unweighted ones.
struct LossOut {
    const DeviceHeader* heads;
    int n_heads;
    float* loss;
    float* head_losses;
    float w[MAX_HEADS];
};

// Adds the per-row losses of one launch to the head's running sum in a fixed order (256 threads of
// one workgroup, fixed strides), so repeated runs give the same bits, and writes the loss after the
// last.  Its own launch is mostly latency (5-8 us), so it rides along as one more workgroup of the
// kernel that finishes dX or dgamma where there is one.
__device__ __forceinline__ void loss_accumulate(const float* __restrict__ row_loss, int rows, DeviceHeader* hdr,
                                                const LossOut& out, double* part) {   // part: 4 in LDS
    double s = 0.0;
#pragma unroll 8
    for (int i = threadIdx.x; i < rows; i += 256) s += (double)row_loss[i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        hdr->loss_sum += (part[0] + part[1]) + (part[2] + part[3]);
        if (out.n_heads > 0) {
            double total = 0.0;
            for (int j = 0; j < out.n_heads; ++j) {
                const DeviceHeader& h = out.heads[j];
                const double mean = h.n_valid > 0 ? h.loss_sum / (double)h.n_valid : 0.0;
                if (out.head_losses) out.head_losses[j] = (float)mean;
                total += (double)out.w[j] * mean;
            }
            *out.loss = (float)total;
        }
    }
}
__global__ __launch_bounds__(256) void loss_accumulate_kernel(const float* row_loss, int rows, DeviceHeader* hdr,
                                                              LossOut out) {
    __shared__ double part[4];
    loss_accumulate(row_loss, rows, hdr, out, part);
}

// Counts the valid rows and resets the running loss.  Integer sum: exact in any order.
// `weight` scales every gradient of this head (1 for a single head).
__global__ __launch_bounds__(1024) void count_valid_kernel(const int64_t* __restrict__ targets,
                                                           int64_t BT, int64_t ignore_index,
                                                           float weight, DeviceHeader* hdr) {
    __shared__ int part[16];
    const int n = count_rows<1024>(targets, (int)BT, ignore_index, part);
    if (threadIdx.x == 0) write_header(hdr, n, weight);
}

}  // namespace flce
