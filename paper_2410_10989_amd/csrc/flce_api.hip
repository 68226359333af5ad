// C ABI of the fused linear cross-entropy library for gfx950: argument checks,
// chunk loop, workspace handling, kernel launches.  Declarations and the
// meaning of every argument are in include/flce.h.
#include <hip/hip_runtime.h>
#include <atomic>
#include <mutex>
#include <vector>

#include "../../include/flce.h"
#include "compact.h"
#include "flce_device.h"
#include "gemm_bf16_nt.h"
#include "gemm_generic.h"
#include "mfma_ceiling.h"
#include "misc_kernels.h"
#include "rmsnorm.h"
#include "rowreduce.h"
#include "scheduler.h"

using namespace flce;

// Scratch of flce_cross_entropy_inplace_noalloc: the device header and one loss per
// row, in the image of the code object instead of allocated memory.  Every GPU the
// library runs on holds its own copy at its own address until the process ends.  In
// host code this name is only a handle for hipGetSymbolAddress, never an address.
constexpr size_t CE_NOALLOC_BYTES = 256 + (size_t)FLCE_CE_NOALLOC_MAX_ROWS * sizeof(float);
static __device__ __align__(256) unsigned char scratch[CE_NOALLOC_BYTES];
// Counters of ce_rows_kernel (DoneCount), for calls that must not overlap anyway because they share their
// scratch memory: one set for that entry point, one for the library's own workspace.
static __device__ done_t ce_done[2 * DONE_WORDS];

namespace {

constexpr int MAX_DEVICES = 64;
constexpr int64_t MAX_DIM = (int64_t)1 << 30;      // per-dimension limit, keeps int tile math safe
constexpr int64_t CE_ROWS_PER_LAUNCH = 65536;
constexpr int64_t SEL_IN_LOGITS_ROWS = TileRows<4>::MAX_ROWS, SEL_ROWS_IN_LOGITS = 8;   // 2048
constexpr int RIDE_BLOCKS = 1024;   // finish_dx as workgroups of the dW launch: at most this many
constexpr int64_t ROT_A_BYTES = (int64_t)2 << 20;
constexpr int64_t CE_CACHE_BYTES = (int64_t)256 << 20;   // memory-side cache
constexpr int64_t MAX_GRID_X = 0x7fffffff;        // workgroups along grid x
constexpr size_t AUTO_BUDGET_BYTES = (size_t)1 << 30;
constexpr int64_t AUTO_BUDGET_MIN_ROWS = 4096;

struct DeviceWorkspace {
    void* lent = nullptr;
    size_t lent_bytes = 0;
    void* own = nullptr;
    size_t own_bytes = 0;
    size_t own_failed = 0;   // an allocation of this size found too little memory, 0 if none did
};

std::mutex g_mutex;
DeviceWorkspace g_ws[MAX_DEVICES];
// device addresses of `scratch` and `ce_done` on each device, once looked up
void* g_scratch_ptr[MAX_DEVICES] = {};
void* g_done_ptr[MAX_DEVICES] = {};
// Process-wide settings: read by every call, written by the setters (any thread).
std::atomic<size_t> g_budget{0};   // 0 = the automatic rule of effective_budget()
std::atomic<bool> g_compact{true};
std::atomic<done_t> g_ce_ticket{0};   // the last one given to a launch that counts its workgroups (DoneCount)

// What a call's plan depends on besides the shape: the process-wide settings, or the
// options a caller passes with the call.
struct Settings {
    size_t budget;   // 0 = the automatic rule
    bool compact;
    void* ws = nullptr;   // the call's own workspace (flce_options), null = the device's shared one
    size_t ws_bytes = 0;
};
Settings global_settings() { return {g_budget.load(), g_compact.load()}; }

// The byte budget of the logits chunk: what the caller set, or by default 1 GiB but at
// least 4096 rows of logits.  Every chunk costs one more pass over W and an fp32
// read-modify-write of the dW partial sums (16 V H bytes) whatever its row count, which
// is about 433 / C of the chunk's product time on this chip: 10 % at 4096 rows.
size_t effective_budget(const Settings& st, int64_t V, int dtype) {
    if (st.budget) return st.budget;
    const size_t rows_bytes = (size_t)AUTO_BUDGET_MIN_ROWS * (size_t)round_up(V, 64) * elem_size(dtype);
    return rows_bytes > AUTO_BUDGET_BYTES ? rows_bytes : AUTO_BUDGET_BYTES;
}

// Up to how many bytes of logits a batch runs as ONE chunk.  With an explicit budget:
// the budget.  Automatic rule: the chunk budget plus the fp32 dW partial sums that only
// a chunked run needs (bf16 storage), i.e. one chunk whenever that takes no more memory
// than chunking would; it is also the faster plan.
size_t single_chunk_bytes(const Settings& st, int64_t H, int64_t V, int dtype) {
    const size_t b = effective_budget(st, V, dtype);
    if (st.budget || dtype == FLCE_F32) return b;
    return b + (size_t)V * (size_t)H * sizeof(float);
}

// An explicit budget never takes the full plan: its caller limits memory (see Room).
Plan plan_for(const Settings& st, int64_t BT, int64_t H, int64_t V, int dtype, Room room = Room::full,
              bool worst_case_bt = false, size_t part_bytes = SIZE_MAX) {
    if (st.budget && room == Room::full) room = Room::bounded;
    return make_plan(BT, H, V, dtype, effective_budget(st, V, dtype), worst_case_bt, st.compact,
                     single_chunk_bytes(st, H, V, dtype), room, part_bytes);
}
Plan plan_for(int64_t BT, int64_t H, int64_t V, int dtype) { return plan_for(global_settings(), BT, H, V, dtype); }

// ---- optional per-kernel timing (benchmarks only) ----
struct TimingRecord {
    hipEvent_t start, stop;
    int kind, also;   // also: a second kind of the same launch, which gets half its time, or -1
};
constexpr int MAX_TIMING_RECORDS = 8192;
std::atomic<bool> g_timing_on{false};
std::vector<TimingRecord> g_records;   // guarded by g_mutex

struct ScopedKernelTimer {
    hipStream_t stream;
    bool active = false;
    TimingRecord rec{};
    ScopedKernelTimer(int kind, hipStream_t s, int also = -1) : stream(s) {   // kind < 0: never timed
        if (kind < 0 || !g_timing_on.load()) return;
        {
            std::lock_guard<std::mutex> lock(g_mutex);
            if ((int)g_records.size() >= MAX_TIMING_RECORDS) return;
        }
        if (hipEventCreate(&rec.start) != hipSuccess) return;
        if (hipEventCreate(&rec.stop) != hipSuccess) {
            (void)hipEventDestroy(rec.start);
            return;
        }
        rec.kind = kind;
        rec.also = also;
        active = (hipEventRecord(rec.start, stream) == hipSuccess);
    }
    ~ScopedKernelTimer() {
        if (!active) return;
        (void)hipEventRecord(rec.stop, stream);
        std::lock_guard<std::mutex> lock(g_mutex);
        g_records.push_back(rec);
    }
};

#define HIP_TRY(expr)                          \
    do {                                       \
        if ((expr) != hipSuccess) {            \
            (void)hipGetLastError();           \
            return FLCE_ERR_HIP;               \
        }                                      \
    } while (0)

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// The device's shared workspace: the lent buffer, or memory of the library's own that grows as needed.
// last = false: the caller has a plan that needs less, so an allocation that found too little memory is
// not tried again on every call (but after flce_release_workspace, or once one as large succeeds).
// lent: whether it is the lent buffer.
int acquire_workspace(size_t need, char** out, bool last = true, bool* lent = nullptr) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return FLCE_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceWorkspace& w = g_ws[dev];
    if (lent) *lent = w.lent != nullptr;
    if (w.lent) {
        if (w.lent_bytes < need) return FLCE_ERR_WORKSPACE;
        *out = static_cast<char*>(w.lent);
        return FLCE_OK;
    }
    if (w.own_bytes < need) {
        if (!last && w.own_failed && need >= w.own_failed) return FLCE_ERR_WORKSPACE;
        if (w.own) {
            HIP_TRY(hipDeviceSynchronize());
            HIP_TRY(hipFree(w.own));
            w.own = nullptr;
            w.own_bytes = 0;
        }
        const hipError_t rc = hipMalloc(&w.own, need);
        if (rc != hipSuccess) {
            (void)hipGetLastError();
            w.own = nullptr;
            if (rc == hipErrorOutOfMemory) w.own_failed = need;   // (not where a stream is being captured)
            return FLCE_ERR_WORKSPACE;
        }
        if (need >= w.own_failed) w.own_failed = 0;
        w.own_bytes = need;
    }
    *out = static_cast<char*>(w.own);
    return FLCE_OK;
}

// Bytes of the buffer lent to the current device, 0 if there is none.
int lent_workspace(size_t* bytes) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return FLCE_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_mutex);
    *bytes = g_ws[dev].lent ? g_ws[dev].lent_bytes : 0;
    return FLCE_OK;
}

// What only the device knows about a product launch of a compacted chunk (see FGArgs).
struct FastDyn {
    const int* rows = nullptr;      // live rows: replaces M (is_k = 0) or K (is_k = 1)
    int is_k = 0;
    const int* ksplit = nullptr;    // number of K ranges, at most the launch's ksplit
    const int* first_live = nullptr;
    int launch = 0;
};

// Guarded kernel (see gemm_generic.h): any shape and alignment, both storage types.  Cin is an
// fp32 addend or null, cin_own one of C's type.  With ksplit > 1 range z writes its partial
// result to C + z * split_stride (no addend then).
template <typename T, typename OutT, bool A_KM, bool B_KM>
int launch_gemm_guarded(int kind, const T* A, int64_t lda, const T* B, int64_t ldb, OutT* C, int64_t ldc,
                        const float* Cin, const OutT* cin_own, int64_t M, int64_t N, int64_t K,
                        hipStream_t s, int tile, int ksplit = 1, int64_t split_stride = 0,
                        const FastDyn& d = FastDyn{}, const FinishArgs* fin = nullptr,
                        const SelectArgs<T>* sel = nullptr) {
    if (M <= 0 || N <= 0) return FLCE_OK;
    if (ksplit > 1 && (Cin || cin_own)) return FLCE_ERR_SHAPE;
    ScopedKernelTimer timer(kind, s);
    constexpr int VEC = GGTraits<T>::VEC;
    const void* in = Cin ? static_cast<const void*>(Cin) : static_cast<const void*>(cin_own);
    GGArgs a{A, lda, B, ldb, C, ldc, in, ldc, Cin ? 1 : 0, (int)M, (int)N, (int)K, ksplit, split_stride,
             (lda % VEC == 0 && aligned(A, 16)) ? 1 : 0, (ldb % VEC == 0 && aligned(B, 16)) ? 1 : 0,
             (ldc % 4 == 0 && split_stride % 4 == 0 && aligned(C, 4 * sizeof(OutT))) ? 1 : 0,
             d.rows, d.is_k, d.ksplit, d.first_live, d.launch,
             FG_GROUP_TILES, kind == FLCE_KIND_LOGITS_GEMM ? 1 : 0, 1};
    const int64_t total = ((M + tile - 1) / tile) * ((N + tile - 1) / tile) * ksplit;
    if (total > MAX_GRID_X - FG_XCDS) return FLCE_ERR_SHAPE;   // check_launch_limits refuses such shapes up front
    const dim3 grid((unsigned)((total + FG_XCDS - 1) / FG_XCDS * FG_XCDS + (fin ? fin->blocks : sel ? sel->blocks : 0)));
    const dim3 block((unsigned)gg_threads(tile));
    // finish_dx rides along with the dW product of fp32 storage
    constexpr bool CAN_FIN = A_KM && B_KM && std::is_same<T, float>::value;
    if (fin && (!CAN_FIN || tile == 256)) return FLCE_ERR_SHAPE;   // (ride_along keeps such calls away)
    // the selection of the rows with the logits product of fp32 storage
    constexpr bool CAN_SEL = !A_KM && !B_KM && std::is_same<T, float>::value && std::is_same<OutT, float>::value;
    if (sel && (!CAN_SEL || tile == 256)) return FLCE_ERR_SHAPE;   // (select_in_logits keeps such calls away)
#define GG_LAUNCH(TILE) \
    hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, TILE>), grid, block, 0, s, a, NoFinish{})
    constexpr bool CAN_FEW = std::is_same<T, float>::value && A_KM == B_KM;   // (the dX product comes out the same)
    const bool few = CAN_FEW && tile == 64 && total <= 256;
    if (sel) {
        if constexpr (CAN_SEL) {
            if (few)
                hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, 64, SelectArgs<T>, true>), grid, block, 0, s, a, *sel);
            else if (tile == 64)
                hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, 64, SelectArgs<T>>), grid, block, 0, s, a, *sel);
            else
                hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, 128, SelectArgs<T>>), grid, block, 0, s, a, *sel);
        }
    } else if (fin) {
        if constexpr (CAN_FIN) {
            if (few)
                hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, 64, FinishArgs, true>), grid, block, 0, s, a, *fin);
            else if (tile == 64)
                hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, 64, FinishArgs>), grid, block, 0, s, a, *fin);
            else
                hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, 128, FinishArgs>), grid, block, 0, s, a, *fin);
        }
    } else if (few) {
        if constexpr (CAN_FEW)
            hipLaunchKernelGGL((gemm_guarded<T, OutT, A_KM, B_KM, 64, NoFinish, true>), grid, block, 0, s, a, NoFinish{});
    } else if (tile == 64) GG_LAUNCH(64);
    else if (tile == 128) GG_LAUNCH(128);
    else GG_LAUNCH(256);
#undef GG_LAUNCH
    HIP_TRY(hipGetLastError());
    return FLCE_OK;
}

// Tuned bf16 kernel (see gemm_bf16_nt.h for what A_KM / B_KM / InT mean).  The
// caller has checked the shape limits (Plan::fast_*).  tail_part: tail_bytes of
// room for fp32 partial blocks; when that is enough for the launch's tail_plan (and the
// launch is not cut into K ranges as a whole and its tile count is known here), the tiles
// of a poorly filled last round are cut along K and summed by a second, small launch.
template <typename OutT, typename InT, bool A_KM, bool B_KM>
int launch_gemm_fast(int kind, const bf16_t* A, int64_t lda, const bf16_t* B, int64_t ldb, OutT* C,
                     int64_t ldc, const InT* Cin, int64_t ldcin, int64_t M, int64_t N, int64_t K,
                     hipStream_t s, int tile, int ksplit = 1, int64_t split_stride = 0, const FastDyn& d = FastDyn{},
                     float* tail_part = nullptr, size_t tail_bytes = 0, const FinishArgs* fin = nullptr,
                     const SelectArgs<bf16_t>* sel = nullptr) {
    if (M <= 0 || N <= 0 || K <= 0) return FLCE_OK;
    if (!aligned(A, 16) || !aligned(B, 16)) return FLCE_ERR_ARG;
    ScopedKernelTimer timer(kind, s);
    FGArgs a{A, lda, B, ldb, C, ldc, Cin, ldcin, (int)M, (int)N, (int)K,
             (int)((M + tile - 1) / tile), (int)((N + tile - 1) / tile), ksplit, split_stride,
             d.rows, d.is_k, d.ksplit, d.first_live, d.launch, 0, 0, 1, tail_part,
             FG_GROUP_TILES, kind == FLCE_KIND_LOGITS_GEMM ? 1 : 0, 1};
    const int64_t total = (int64_t)a.tiles_m * a.tiles_n * ksplit;
    if (total >= ((int64_t)1 << 30)) return FLCE_ERR_SHAPE;   // the kernel counts tiles in 32 bits
    int64_t wgs_per_xcd = (total + FG_XCDS - 1) / FG_XCDS;
    const bool m_static = !(d.rows && !d.is_k);   // a dynamic M changes the tile count on the device
    if (tile == 256 && tail_part && ksplit == 1 && !d.ksplit && m_static) {
        const TailPlan t = tail_plan(total, (K + FG_BK - 1) / FG_BK);
        if (t.s > 1 && (size_t)FG_XCDS * t.r * t.s * TAIL_BLOCK_BYTES <= tail_bytes) {
            a.tail_begin = t.begin;
            a.tail_r = t.r;
            a.tail_s = t.s;
            wgs_per_xcd = (int64_t)t.begin + (int64_t)t.r * t.s;
        }
    }
    const dim3 grid((unsigned)(wgs_per_xcd * FG_XCDS + (fin ? fin->blocks : sel ? sel->blocks : 0)));
    constexpr bool CAN_FIN = A_KM && B_KM && std::is_void<InT>::value && std::is_same<OutT, bf16_t>::value;
    if (fin && (!CAN_FIN || tile != 128)) return FLCE_ERR_SHAPE;   // (ride_along keeps such calls away)
    // Row-form operands, one 256-row tile: B is fetched once, and all of A stays in an XCD's L2 (4 MB)
    // at whatever K step its tiles are, so the tile columns can start their K loops at different steps
    // (FG_ROTATED).  Measured, V = 128256, H = 4096: 16 rows 230 -> 175 us, 64 rows 240 -> 190, 200 rows 281 ->
    // 250; a whole call of 8192 x 4096 x 32000 in 256-row chunks 20.3 -> 18.7 ms; launches of 512 rows: no
    // difference, of 4096: 1 % slower.  (The bits of a logit therefore depend on whether its
    // chunk has more than 256 rows.)
    constexpr bool ROWS = !A_KM && !B_KM;
    constexpr int ROT = ROWS ? FG_ROTATED : FG_PLAIN, CUT = ROWS ? FG_K_TAIL : FG_PLAIN;
    const bool tail = ROWS && K % FG_BK != 0;
    const bool rot = ROWS && !tail && M <= FG_BM && M * K * (int64_t)sizeof(bf16_t) <= ROT_A_BYTES;
    constexpr bool CAN_SEL = ROWS && std::is_void<InT>::value && std::is_same<OutT, bf16_t>::value;
    if (sel && (!CAN_SEL || tile != 128)) return FLCE_ERR_SHAPE;   // (select_in_logits keeps such calls away)
#define FG_LAUNCH(TILE, ORDER) \
    hipLaunchKernelGGL((gemm_bf16<OutT, InT, A_KM, B_KM, TILE, ORDER>), grid, dim3(FG_THREADS), 0, s, a, NoFinish{})
#define FG_LAUNCH_SEL(ORDER)                                                                                       \
    hipLaunchKernelGGL((gemm_bf16<OutT, InT, A_KM, B_KM, 128, ORDER, SelectArgs<bf16_t>>), grid, dim3(FG_THREADS), 0, \
                       s, a, *sel)
    if (sel) {
        if constexpr (CAN_SEL) {
            if (rot) FG_LAUNCH_SEL(FG_ROTATED); else if (tail) FG_LAUNCH_SEL(FG_K_TAIL); else FG_LAUNCH_SEL(FG_PLAIN);
        }
    } else if (fin) {
        if constexpr (CAN_FIN)
            hipLaunchKernelGGL((gemm_bf16<OutT, InT, A_KM, B_KM, 128, FG_PLAIN, FinishArgs>), grid, dim3(FG_THREADS), 0, s,
                               a, *fin);
    } else if (tile == 128) {
        if (rot) FG_LAUNCH(128, ROT); else if (tail) FG_LAUNCH(128, CUT); else FG_LAUNCH(128, FG_PLAIN);
    } else {
        if (rot) FG_LAUNCH(256, ROT); else if (tail) FG_LAUNCH(256, CUT); else FG_LAUNCH(256, FG_PLAIN);
    }
#undef FG_LAUNCH
#undef FG_LAUNCH_SEL
    HIP_TRY(hipGetLastError());
    if (a.tail_s > 1) {
        hipLaunchKernelGGL((fg_tail_reduce_kernel<OutT, InT>), dim3((unsigned)(FG_XCDS * a.tail_r * 8)), dim3(256),
                           0, s, a);
        HIP_TRY(hipGetLastError());
    }
    return FLCE_OK;
}

// zero_pad: columns V .. V + zero_pad - 1 of every row are set to zero as well (the
// padding of the workspace's dlogits chunk, which the dX product reads as part of K).
template <typename T>
int launch_ce_rows(T* Z, int64_t ldz, const int64_t* targets, int64_t rows, int64_t V,
                   int zero_pad, int64_t ignore_index, DeviceHeader* hdr, float* row_loss,
                   hipStream_t s, const int* n_rows, bool timed, int count_n, float weight, bool fused,
                   const DoneCount& done = DoneCount{}, float* loss = nullptr) {
    ScopedKernelTimer timer(timed ? FLCE_KIND_CE_ROWS : -1, s);
    // shape by row length, nontemporal accesses by size: see ce_rows_kernel
    const int64_t row_bytes = V * (int64_t)sizeof(T);
    const bool nt = !fused && rows * row_bytes > CE_CACHE_BYTES;
#define CE_LAUNCH(TH, NV, NT, NL, FOLD)                                                                     \
    hipLaunchKernelGGL((ce_rows_kernel<T, TH, NV, NT, NL, FOLD>), dim3((unsigned)rows), dim3(TH), 0, s, Z, ldz,  \
                       targets, (int)V, zero_pad, ignore_index, hdr, row_loss, n_rows, count_n, weight, done, loss)
#define CE_SHAPE(TH, NV, NL) \
    do {                                                                                             \
        if (done.words) CE_LAUNCH(TH, NV, false, NL, true);                                          \
        else if (nt) CE_LAUNCH(TH, NV, true, NL, false);                                             \
        else CE_LAUNCH(TH, NV, false, NL, false);                                                    \
    } while (0)
    if (row_bytes > 400 * 1024) CE_SHAPE(RC_THREADS, RC_NV, RC_NL);
    else if (row_bytes > 112 * 1024) CE_SHAPE(RC_THREADS, RC_NV, 0);
    else if (row_bytes > 48 * 1024) CE_SHAPE(RM_THREADS, RM_NV, 0);
    else CE_SHAPE(RS_THREADS, RS_NV, 0);
#undef CE_SHAPE
#undef CE_LAUNCH
    HIP_TRY(hipGetLastError());
    return FLCE_OK;
}

int launch_loss(const float* row_loss, int64_t rows, DeviceHeader* hdr, const LossOut& out, bool timed, hipStream_t s) {
    ScopedKernelTimer timer(timed ? FLCE_KIND_CE_ROWS : -1, s);
    hipLaunchKernelGGL(loss_accumulate_kernel, dim3(1), dim3(256), 0, s, row_loss, (int)rows, hdr, out);
    HIP_TRY(hipGetLastError());
    return FLCE_OK;
}

#define FLCE_TRY(expr)                 \
    do {                               \
        const int rc_ = (expr);        \
        if (rc_ != FLCE_OK) return rc_; \
    } while (0)

static_assert(MAX_HEADS * sizeof(DeviceHeader) <= 256, "header slot too small");

// RMSNorm in front of the projection: the chunk loop normalises each chunk of the
// raw hidden states just before its logits product (into the chunk buffer that
// otherwise holds gathered rows) and turns the chunk's dX into the gradient of the
// raw hidden states right after.
template <typename T>
struct NormCtx {
    const T* gamma;
    float eps;
    float* rstd;     // [C]
    float* partial;  // [RN_SLOTS x H] fp32 partial sums of dgamma, started by the first chunk
    T* dh;           // [BT x H] out
};

// See finish_dx_kernel: K-range partial results summed, rows put in place, loss summed.
template <typename T>
bool finish_is_vec(const FinishArgs& f) {
    return f.n % 4 == 0 && f.split_stride % 4 == 0 && aligned(f.src, 4 * (f.src_f32 ? sizeof(float) : sizeof(T))) &&
           aligned(f.out, 4 * sizeof(T));
}
template <typename T>
int launch_finish_dx(const FinishArgs& f, hipStream_t s) {
    ScopedKernelTimer timer(FLCE_KIND_DX_GEMM, s);
    const dim3 grid((unsigned)f.blocks), block(256);
    if (!finish_is_vec<T>(f))
        hipLaunchKernelGGL((finish_dx_kernel<T, false, false>), grid, block, 0, s, f);
    else if (f.nsplit > FIN_AHEAD)
        hipLaunchKernelGGL((finish_dx_kernel<T, true, true>), grid, block, 0, s, f);
    else
        hipLaunchKernelGGL((finish_dx_kernel<T, true, false>), grid, block, 0, s, f);
    HIP_TRY(hipGetLastError());
    return FLCE_OK;
}

// Which form of the RMSNorm kernels a row length takes: 1, 2 or 4 16-byte vectors per
// thread (rows of whole vectors, at most 1024 of them, 16-byte aligned operands; the
// workspace buffers always are), or 0 for the scalar form.
template <typename T>
int rmsnorm_vectors_per_thread(int64_t H, const void* x, const void* gamma, const void* dh) {
    constexpr int N = 16 / (int)sizeof(T);
    if (H % N != 0 || !aligned(x, 16) || !aligned(gamma, 16) || !aligned(dh, 16)) return 0;
    const int64_t nvec = H / N;
    return nvec <= RN_THREADS ? 1 : nvec <= 2 * RN_THREADS ? 2 : nvec <= 4 * RN_THREADS ? 4 : 0;
}

// Partial rows of dgamma that a chunk of C rows can reach.
inline unsigned rn_slots(int64_t C) { return (unsigned)std::min<int64_t>(C, RN_SLOTS); }

// dX = G W and dW = G^T X (dW not null) in one launch.
template <typename T>
int launch_grad(const T* Z, int64_t ldz, const T* W, const T* Xc, float* part, T* rows_out, T* dW, int64_t rows, int64_t H,
                int64_t V, const Plan& p, const FastDyn& dm, const FastDyn& dk, GradArgs g, hipStream_t s) {
    ScopedKernelTimer timer(FLCE_KIND_DX_GEMM, s, dW ? FLCE_KIND_DW_GEMM : -1);   // (as many operations each)
    const int tile = p.dx_tile, ranges = p.dx_ranges;
    const bool cut = ranges > 1;
    auto up = [](int64_t n) { return (n + FG_XCDS - 1) / FG_XCDS * FG_XCDS; };
    g.dx_blocks = (int)up(tiles_of(rows, H, tile) * ranges);
    const int64_t dw_blocks = dW ? up(tiles_of(V, H, tile)) : 0;
    g.dw_first = dW && rows > V / ranges ? (int)dw_blocks : 0;
    const dim3 grid((unsigned)((cut ? 0 : FG_XCDS) + g.dx_blocks + dw_blocks)), block(256);
    void* out = cut ? static_cast<void*>(part) : rows_out;
    if constexpr (sizeof(T) == 2) {
        auto tiles = [&](int64_t n) { return (int)((n + tile - 1) / tile); };
        const FGArgs dx{Z, ldz, W, H, out, H, nullptr, 0, (int)rows, (int)H, (int)V, tiles(rows), tiles(H), ranges, p.C * H,
                        dm.rows, 0, nullptr, nullptr, 0, 0, 0, 1, nullptr, FG_GROUP_TILES, 0, 1};
        const FGArgs dw{Z, ldz, Xc, H, dW, H, nullptr, 0, (int)V, (int)H, (int)rows, tiles(V), tiles(H), 1, 0,
                        dk.rows, 1, nullptr, dk.first_live, dk.launch, 0, 0, 1, nullptr, FG_GROUP_TILES, 0, 1};
        if (cut) hipLaunchKernelGGL((grad_bf16<true>), grid, block, 0, s, dx, dw, g);
        else hipLaunchKernelGGL((grad_bf16<false>), grid, block, 0, s, dx, dw, g);
    } else {
        const GGArgs dx{Z, ldz, W, H, out, H, nullptr, H, 0, (int)rows, (int)H, (int)V, ranges, p.C * H, ldz % 4 == 0, 0, 1,
                        dm.rows, 0, nullptr, nullptr, 0, FG_GROUP_TILES, 0, 1};
        const GGArgs dw{Z, ldz, Xc, H, dW, H, nullptr, H, 0, (int)V, (int)H, (int)rows, 1, 0, 0, 0, 1,
                        dk.rows, 1, nullptr, dk.first_live, dk.launch, FG_GROUP_TILES, 0, 1};
#define GRAD_LAUNCH(TILE, CUT) hipLaunchKernelGGL((grad_f32<TILE, CUT>), grid, block, 0, s, dx, dw, g)
        if (tile == 64) {
            if (cut) GRAD_LAUNCH(64, true); else GRAD_LAUNCH(64, false);
        } else {
            if (cut) GRAD_LAUNCH(128, true); else GRAD_LAUNCH(128, false);
        }
#undef GRAD_LAUNCH
    }
    HIP_TRY(hipGetLastError());
    return FLCE_OK;
}

// Whether a batch that is one chunk has its rows selected by workgroups of the logits launch.  That saves a
// launch (4-5 us, on the host as well) and costs every tile its own look at the targets, 1-2 us per
// workgroup: for launches that fit the chip, or of one tile row, where the look is short.  Whole calls with the
// launch of its own / without, us: bf16 24 x 680 x 1026 26.9 / 24.1, 495 x 896 x 3674 36.5 / 33.7, 1572 x 576 x
// 2176 59.6 / 53.5, 1024 x 512 x 8192 60 / 57, 51 x 3328 x 24297 129 / 119, one tile row in 1136 tiles (31 x 576 x
// 144923) 100.3 / 96.9; 2664 tiles in three rows (294 x 128 x 113344) 110.5 / 112.9.  A handful of tiles with long
// K loops waits for its loads alone, and the rows of X are further away than gathered ones: 30 x 2496 x 384 (3
// tiles) 34.1 / 35.1, 53 x 2352 x 2560 (20 tiles) 41.8 / 40.1.  Longer batches gain nothing (3195 x 2560 x 829:
// launches of 10.6 + 25.0 / 36.8).
template <typename T>
bool select_in_logits(const Plan& p, const VocabCut& cut, int64_t BT, int64_t H, int64_t V) {
    const int64_t tiles = tiles_of(BT, V, cut.tile);
    return p.nchunks == 1 && cut.main == V && cut.tile < 256 && BT <= SEL_IN_LOGITS_ROWS &&
           BT * H * (int64_t)sizeof(T) < ((int64_t)1 << 30) && tiles <= (BT <= cut.tile ? 4096 : 512) &&
           (tiles >= 16 || H <= 1024);
}

// One head: count its valid rows, then run the chunk loop.  Gradients are scaled by
// weight / N_valid.  With dx_add the head's dX is added to what dX already holds
// (rounded to the storage type once per head), otherwise dX is overwritten.  loss_out: where the
// loss goes after the last head (n_heads = 0 for the others).
template <typename T>
int run_head(const T* X, const T* W, const int64_t* targets, int64_t BT, int64_t H, int64_t V,
             int64_t ignore_index, float weight, DeviceHeader* hdr, const LossOut& loss_out, bool dx_add, T* dX,
             T* dW, unsigned flags, const Plan& p, char* ws, hipStream_t s,
             const NormCtx<T>* norm = nullptr) {
    constexpr bool BF16 = (sizeof(T) == 2);
    const bool want_dx = !(flags & FLCE_SKIP_DX), want_dw = !(flags & FLCE_SKIP_DW);
    float* row_loss = reinterpret_cast<float*>(ws + p.off_row_loss);
    T* Z = reinterpret_cast<T*>(ws + p.off_z);
    float* dWacc = reinterpret_cast<float*>(ws + p.off_dwacc);
    T* Xg = reinterpret_cast<T*>(ws + p.off_xg);     // gathered (or normalised) rows of the chunk
    T* dXg = reinterpret_cast<T*>(ws + p.off_dxg);   // their gradient
    int* idx = reinterpret_cast<int*>(ws + p.off_idx);
    int64_t* tv = reinterpret_cast<int64_t*>(ws + p.off_tv);
    int* dyn = reinterpret_cast<int*>(ws + p.off_dyn);   // [0] row cursor, [1] live rows of the chunk
    float* tail = reinterpret_cast<float*>(ws + p.off_tail);   // partial blocks of the dW product's last round
    constexpr int VEC = 16 / (int)sizeof(T);

    // A head whose dX is added to the heads before it: the product's epilogue adds its fp32 sums, rounded
    // once, but only when the rows of the chunk are rows of dX; rows that are staged and scattered are
    // rounded to the storage type first, unless K ranges hold them as fp32 sums.  bf16 with H % 64 != 0
    // keeps the single rounding and projects the ignored rows instead (3 heads of 16384 x 200 x 4000, 10 %
    // ignored: 816 us either way, error of dX against 64 bits 2.6e-3 with it, 2.95e-3 staged).
    const bool adds_in_epilogue = BF16 && want_dx && dx_add && !norm && p.dx_ranges == 1 && H % 64 != 0;
    const bool compact = p.compact && !adds_in_epilogue;
    const bool select = compact && one_launch_selects(BT, p.nchunks);   // one launch per chunk finds its rows
    const bool norm_in_select = select && norm && aligned(norm->gamma, 16);
    const bool count_in_rows = !compact && p.nchunks == 1 && BT <= ce_count_rows(V * (int64_t)sizeof(T));
    T* zero_out = (want_dx && !dx_add) ? (norm ? norm->dh : dX) : nullptr;   // rows without a target: zero gradient
    if (!select && !count_in_rows) {
        hipLaunchKernelGGL(count_valid_kernel, dim3(1), dim3(1024), 0, s, targets, BT, ignore_index,
                           weight, hdr);
        HIP_TRY(hipGetLastError());
    }
    if (compact && !select && zero_out) {
        ScopedKernelTimer timer(FLCE_KIND_OTHER, s);
        hipLaunchKernelGGL((zero_ignored_rows_kernel<T>), dim3((unsigned)(BT < 8192 ? BT : 8192)),
                           dim3(256), 0, s, targets, BT, ignore_index, (int)H, zero_out);
        HIP_TRY(hipGetLastError());
    }

    for (int64_t c = 0; c < p.nchunks; ++c) {
        const int64_t r0 = c * p.C;
        const bool last = (c == p.nchunks - 1);
        // Compacted: the chunk is the next rows of the batch that have a target, wherever they
        // are, at most C of them (the valid rows are dealt evenly to the last launches, see
        // compact_chunk_kernel); Xc, Z and dXc hold *n_live rows (a device value), the launches
        // below are sized for C rows, and idx maps the chunk's rows to batch rows.  Otherwise
        // the chunk is rows r0 .. r0 + rows - 1 of the batch.
        const int64_t rows = compact ? p.C : ((BT - r0 < p.C) ? BT - r0 : p.C);
        const int* n_live = compact ? dyn + DYN_LIVE : nullptr;
        const int* row_map = compact ? idx : nullptr;
        const T* Xin = compact ? X : X + r0 * H;   // what the chunk's row indices refer to
        const T* Xc = Xin;
        const int64_t* tc = targets + r0;
        const bool dw_fast = BF16 && (last ? p.fast_dw_last : p.fast_dw_full);
        const VocabCut dw_cut = vocab_cut(dw_fast, V, H, rows, p.tail_bytes > 0);
        const bool one_grad = select && want_dx && grads_in_one(p, dw_cut, BF16, want_dw, dw_fast, !norm, rows, H, V);
        const VocabCut z_cut = vocab_cut(BF16 && p.fast_logits, V, rows, H, false);
        const bool in_logits = select && !norm && select_in_logits<T>(p, z_cut, BT, H, V);
        SelectArgs<T> sel{};
        FastDyn dyn_m, dyn_dx, dyn_dw;   // logits (M = live rows), dX (M and K ranges), dW (K = live rows)
        if (compact) {
            ScopedKernelTimer timer(in_logits ? -1 : FLCE_KIND_OTHER, s);   // (else nothing is launched here)
            const int dx_tiles_n = (int)((H + FG_BN - 1) / FG_BN), dx_ksteps = (int)((V + FG_BK - 1) / FG_BK);
            if (select) {
                // (logits that pick their rows from X leave the gathered ones to the dW product)
                const bool gather = norm ? norm_in_select : want_dw || !in_logits;
                sel = {targets, (int)BT, ignore_index, weight, (int)p.C, (int)c, (int)p.nchunks, dx_tiles_n, dx_ksteps,
                       p.dx_ranges, hdr, gather ? X : static_cast<const T*>(nullptr), (int)H, Xg,
                       c == 0 ? zero_out : static_cast<T*>(nullptr), idx, tv, dyn,
                       norm_in_select ? norm->gamma : static_cast<const T*>(nullptr), norm ? norm->eps : 0.f,
                       norm ? norm->rstd : static_cast<float*>(nullptr), (int)std::min<int64_t>((BT + 3) / 4, SEL_GRID)};
                if (in_logits)
                    sel.blocks = (int)((BT + SEL_ROWS_IN_LOGITS - 1) / SEL_ROWS_IN_LOGITS + FG_XCDS - 1) / FG_XCDS * FG_XCDS;
                else
                    hipLaunchKernelGGL((select_rows_kernel<T>), dim3((unsigned)sel.blocks), dim3(256), 0, s, sel);
            } else {
                hipLaunchKernelGGL(compact_chunk_kernel, dim3(1), dim3(CP_THREADS), 0, s, targets, (int)BT,
                                   ignore_index, (int)p.C, (int)c, (int)p.nchunks, hdr, dx_tiles_n, dx_ksteps,
                                   p.dx_ranges, idx, tv, dyn);
            }
            HIP_TRY(hipGetLastError());
            tc = tv;
            dyn_m.rows = dyn_dx.rows = dyn_dw.rows = n_live;
            dyn_dw.is_k = 1;
            if (p.dx_dyn) dyn_dx.ksplit = dyn + DYN_DX_RANGES;
            dyn_dw.first_live = dyn + DYN_FIRST_LIVE;
            dyn_dw.launch = (int)c;
        }
        if (norm_in_select) {
            Xc = Xg;
        } else if (norm) {   // X holds the raw hidden states: normalise the chunk's rows
            ScopedKernelTimer timer(FLCE_KIND_OTHER, s);
#define RN_FWD(KERNEL)                                                                           \
    hipLaunchKernelGGL((KERNEL), dim3((unsigned)rows), dim3(RN_THREADS), 0, s, Xin, norm->gamma, \
                       norm->eps, (int)H, Xg, norm->rstd, row_map, n_live)
            switch (rmsnorm_vectors_per_thread<T>(H, Xin, norm->gamma, norm->dh)) {
                case 1: RN_FWD((rmsnorm_fwd_vec_kernel<T, 1>)); break;
                case 2: RN_FWD((rmsnorm_fwd_vec_kernel<T, 2>)); break;
                case 4: RN_FWD((rmsnorm_fwd_vec_kernel<T, 4>)); break;
                default: RN_FWD((rmsnorm_fwd_kernel<T>)); break;
            }
#undef RN_FWD
            HIP_TRY(hipGetLastError());
            Xc = Xg;
        } else if (compact) {
            Xc = Xg;
        }
        if (compact && !norm && !select) {
            ScopedKernelTimer timer(FLCE_KIND_OTHER, s);
            hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)rows), dim3(256), 0, s,
                               reinterpret_cast<const u32x4*>(X), idx, n_live, (int)(H / VEC),
                               reinterpret_cast<u32x4*>(Xg));
            HIP_TRY(hipGetLastError());
        }

        // logits of the chunk: Z = X_c W^T
        {
            const bool fast = BF16 && p.fast_logits;
            const VocabCut& cut = z_cut;
            const SelectArgs<T>* with = in_logits ? &sel : nullptr;   // (the rows are picked from X itself then)
            const T* Xz = in_logits ? X : Xc;
            const FastDyn dz = in_logits ? FastDyn{} : dyn_m;
            auto product = [&](int64_t v0, int64_t nv, int tile) -> int {   // columns v0 .. v0 + nv - 1
                if constexpr (BF16) {
                    if (fast)
                        return launch_gemm_fast<bf16_t, void, false, false>(FLCE_KIND_LOGITS_GEMM, Xz, H, W + v0 * H, H,
                                                                            Z + v0, p.ldz, nullptr, 0, rows, nv, H, s,
                                                                            tile, 1, 0, dz, nullptr, 0, nullptr, with);
                }
                return launch_gemm_guarded<T, T, false, false>(FLCE_KIND_LOGITS_GEMM, Xz, H, W + v0 * H, H, Z + v0,
                                                               p.ldz, nullptr, nullptr, rows, nv, H, s, tile, 1, 0,
                                                               dz, nullptr, with);
            };
            FLCE_TRY(product(0, cut.main, cut.tile));
            if (cut.main < V) FLCE_TRY(product(cut.main, V - cut.main, cut.rest_tile));
        }

        // loss and in-place dlogits
        FLCE_TRY(launch_ce_rows<T>(Z, p.ldz, tc, rows, V, (int)(p.ldz - V), ignore_index, hdr,
                                   row_loss, s, n_live, true, count_in_rows ? (int)BT : 0, weight, true));
        const LossOut loss_here = last ? loss_out : LossOut{};

        // dX_c (+)= G W: straight into dX, or into the chunk buffer when the rows still have to be
        // scattered back or to pass through the RMSNorm backward; cut along K into fp32 partial
        // results when there are few output tiles.  `fin` is what is left to do for dX then.
        FinishArgs fin{};
        bool finish = false;
        const bool loss_in_norm = norm && want_dx;   // (see below)
        if (one_grad) {
            float* part = reinterpret_cast<float*>(ws + p.off_dxpart);
            const bool cut = p.dx_ranges > 1;
            fin = {cut ? static_cast<const void*>(part) : dXg, cut ? 1 : 0, p.C * H, p.dx_ranges, nullptr,
                   norm ? nullptr : row_map, n_live, (int)rows, (int)H, norm ? dXg : dX, dx_add,
                   norm ? nullptr : row_loss, hdr, loss_here, finish_segs(H), (int)finish_blocks(rows, H)};
            FLCE_TRY(launch_grad<T>(Z, p.ldz, W, Xc, part, dXg, want_dw ? dW : nullptr, rows, H, V, p, dyn_m, dyn_dw,
                                    GradArgs{fin, 0, 0}, s));
            if (cut) FLCE_TRY(launch_finish_dx<T>(fin, s));
        } else if (want_dx) {
            const bool staged = compact || norm;
            const bool scatter = compact && !norm;
            T* dXc = staged ? dXg : dX + r0 * H;
            const bool add_in_gemm = dx_add && !staged;
            if (p.dx_ranges > 1) {
                float* part = reinterpret_cast<float*>(ws + p.off_dxpart);
                if constexpr (BF16) {
                    if (p.fast_dx)
                        FLCE_TRY((launch_gemm_fast<float, void, false, true>(
                            FLCE_KIND_DX_GEMM, Z, p.ldz, W, H, part, H, nullptr, 0, rows, H, V, s, p.dx_tile, p.dx_ranges,
                            p.C * H, dyn_dx)));
                }
                if (!p.fast_dx)
                    FLCE_TRY((launch_gemm_guarded<T, float, false, true>(
                        FLCE_KIND_DX_GEMM, Z, p.ldz, W, H, part, H, nullptr, nullptr, rows, H, V, s, p.dx_tile, p.dx_ranges,
                        p.C * H, dyn_m)));
                fin = {part, 1, p.C * H, p.dx_ranges, dyn_dx.ksplit, scatter ? row_map : nullptr, n_live, (int)rows, (int)H,
                       scatter ? dX : dXc, dx_add && (scatter || add_in_gemm), nullptr, hdr, LossOut{},
                       finish_segs(H), (int)finish_blocks(rows, H)};
                finish = true;
            } else {
                if constexpr (BF16) {
                    if (p.fast_dx && add_in_gemm)
                        FLCE_TRY((launch_gemm_fast<bf16_t, bf16_t, false, true>(
                            FLCE_KIND_DX_GEMM, Z, p.ldz, W, H, dXc, H, dXc, H, rows, H, V, s, p.dx_tile)));
                    else if (p.fast_dx)
                        FLCE_TRY((launch_gemm_fast<bf16_t, void, false, true>(
                            FLCE_KIND_DX_GEMM, Z, p.ldz, W, H, dXc, H, nullptr, 0, rows, H, V, s, p.dx_tile, 1, 0, dyn_m)));
                }
                if (!p.fast_dx)
                    FLCE_TRY((launch_gemm_guarded<T, T, false, true>(
                        FLCE_KIND_DX_GEMM, Z, p.ldz, W, H, dXc, H, nullptr, add_in_gemm ? dXc : nullptr, rows, H, V, s,
                        p.dx_tile, 1, 0, dyn_m)));
                if (scatter) {
                    fin = {dXg, 0, 0, 1, nullptr, row_map, n_live, (int)rows, (int)H, dX, dx_add, nullptr, hdr, LossOut{},
                           finish_segs(H), (int)finish_blocks(rows, H)};
                    finish = true;
                }
            }
        }
        // The chunk's losses are summed by a workgroup of the RMSNorm backward launch, or of the one
        // that finishes dX, or, with neither, by a launch of their own.
        if (finish && !loss_in_norm) {
            fin.row_loss = row_loss;
            fin.loss = loss_here;
        } else if (!loss_in_norm && !one_grad) {
            FLCE_TRY(launch_loss(row_loss, rows, hdr, loss_here, true, s));
        }
        // dX is finished by workgroups of the dW launch where that is one launch on small tiles
        const bool ride_along = finish && want_dw && p.nchunks == 1 && dw_cut.main == V && dw_cut.tile < 256 &&
                                (dw_fast || !BF16) && fin.blocks <= RIDE_BLOCKS && finish_is_vec<T>(fin);
        if (finish && !ride_along) FLCE_TRY(launch_finish_dx<T>(fin, s));

        // dW (+)= G^T X_c   (K = the chunk's rows; in a compacted chunk K = *n_live)
        if (want_dw && !one_grad) {
            const bool fast = dw_fast;
            const VocabCut& cut = dw_cut;
            const FinishArgs* with = ride_along ? &fin : nullptr;
            // rows v0 .. v0 + nv - 1 of dW: the first chunk writes its sums, the others add to them, the
            // last writes dW; bf16 sums over several chunks are kept in fp32 (dWacc)
            auto product = [&](int64_t v0, int64_t nv, int tile) -> int {
                const T* G = Z + v0;
                T* out = dW + v0 * H;
                float* acc = p.fp32_dw_acc ? dWacc + v0 * H : nullptr;
                if constexpr (BF16) {
                    if (fast) {
                        float* part = nv == V ? tail : nullptr;
                        const int kind = FLCE_KIND_DW_GEMM;
                        if (p.nchunks == 1)
                            return launch_gemm_fast<bf16_t, void, true, true>(kind, G, p.ldz, Xc, H, out, H, nullptr, 0, nv,
                                                                              H, rows, s, tile, 1, 0, dyn_dw, part,
                                                                              p.tail_bytes, with);
                        if (c == 0)
                            return launch_gemm_fast<float, void, true, true>(kind, G, p.ldz, Xc, H, acc, H, nullptr, 0, nv, H,
                                                                             rows, s, tile, 1, 0, dyn_dw, part,
                                                                             p.tail_bytes);
                        if (!last)
                            return launch_gemm_fast<float, float, true, true>(kind, G, p.ldz, Xc, H, acc, H, acc, H, nv, H,
                                                                              rows, s, tile, 1, 0, dyn_dw, part,
                                                                              p.tail_bytes);
                        return launch_gemm_fast<bf16_t, float, true, true>(kind, G, p.ldz, Xc, H, out, H, acc, H, nv, H, rows,
                                                                           s, tile, 1, 0, dyn_dw, part, p.tail_bytes);
                    }
                }
                if (acc && !last)
                    return launch_gemm_guarded<T, float, true, true>(FLCE_KIND_DW_GEMM, G, p.ldz, Xc, H, acc, H,
                                                                     c > 0 ? acc : nullptr, nullptr, nv, H, rows, s, tile,
                                                                     1, 0, dyn_dw);
                return launch_gemm_guarded<T, T, true, true>(FLCE_KIND_DW_GEMM, G, p.ldz, Xc, H, out, H, acc,
                                                             !acc && c > 0 ? out : nullptr, nv, H, rows, s, tile, 1, 0,
                                                             dyn_dw, with);
            };
            FLCE_TRY(product(0, cut.main, cut.tile));
            if (cut.main < V) FLCE_TRY(product(cut.main, V - cut.main, cut.rest_tile));
        }
        if (norm && want_dx) {   // the chunk's dX into dh and the partial sums of dgamma
            ScopedKernelTimer timer(FLCE_KIND_OTHER, s);
            const RnLoss rn_loss{row_loss, (int)rows, hdr, loss_here};
#define RN_BWD(KERNEL)                                                                              \
    hipLaunchKernelGGL((KERNEL), dim3(rn_slots(p.C) + 1), dim3(RN_THREADS), 0, s, Xin, norm->gamma,  \
                       norm->rstd, dXg, (int)rows, (int)H, compact ? norm->dh : norm->dh + r0 * H, \
                       norm->partial, row_map, n_live, c == 0 ? 1 : 0, rn_loss)
            switch (rmsnorm_vectors_per_thread<T>(H, Xin, norm->gamma, norm->dh)) {
                case 1: RN_BWD((rmsnorm_bwd_vec_kernel<T, 1>)); break;
                case 2: RN_BWD((rmsnorm_bwd_vec_kernel<T, 2>)); break;
                case 4: RN_BWD((rmsnorm_bwd_vec_kernel<T, 4>)); break;
                default: RN_BWD((rmsnorm_bwd_kernel<T>)); break;
            }
#undef RN_BWD
            HIP_TRY(hipGetLastError());
        }
    }
    return FLCE_OK;
}

// All heads one after the other on the same stream and the same workspace; the last one's last
// row losses complete loss = sum_j weight_j * mean loss of head j.
template <typename T>
int run_heads(const T* X, const void* const* W, const int64_t* const* targets, const float* weights,
              int n_heads, int64_t BT, int64_t H, int64_t V, int64_t ignore_index, float* loss,
              float* head_losses, T* dX, void* const* dW, unsigned flags, const Plan& p, char* ws,
              hipStream_t s) {
    DeviceHeader* hdr = reinterpret_cast<DeviceHeader*>(ws + p.off_hdr);
    const bool want_dw = !(flags & FLCE_SKIP_DW);
    LossOut out{hdr, n_heads, loss, head_losses, {}};
    for (int j = 0; j < n_heads; ++j) {
        out.w[j] = weights ? weights[j] : 1.0f;
        FLCE_TRY(run_head<T>(X, static_cast<const T*>(W[j]), targets[j], BT, H, V, ignore_index,
                             out.w[j], hdr + j, j == n_heads - 1 ? out : LossOut{}, j > 0, dX, want_dw ? static_cast<T*>(dW[j]) : nullptr,
                             flags, p, ws, s));
    }
    return FLCE_OK;
}

int check_dims(int64_t BT, int64_t H, int64_t V, int dtype) {
    if (dtype != FLCE_F32 && dtype != FLCE_BF16) return FLCE_ERR_DTYPE;
    if (BT <= 0 || H <= 0 || V <= 0 || BT > MAX_DIM || H > MAX_DIM || V > MAX_DIM)
        return FLCE_ERR_SHAPE;
    return FLCE_OK;
}

// Launch-size limits of the kernels a plan uses, checked before anything is launched: the
// guarded product numbers its tiles along grid x, the row kernels and the row copies take one
// workgroup per row of a chunk.
int check_launch_limits(const Plan& p, int64_t H, int64_t V) {
    auto tiles = [](int64_t r, int64_t c, int64_t t) { return ((r + t - 1) / t) * ((c + t - 1) / t); };
    if (p.C > MAX_GRID_X) return FLCE_ERR_SHAPE;
    const bool all_fast = p.fast_logits && p.fast_dx && p.fast_dw_full && p.fast_dw_last;
    if (!all_fast) {
        // (64 x 64 tiles are the most; a launch is rounded up to whole rounds over the XCDs)
        const int64_t worst = std::max(std::max(tiles(V, H, 64), tiles(p.C, V, 64)),
                                       tiles(p.C, H, p.dx_tile) * p.dx_ranges);
        if (worst > MAX_GRID_X - FG_XCDS) return FLCE_ERR_SHAPE;
    }
    return FLCE_OK;
}

// The fastest plan whose workspace (need_of(plan) bytes) there is room for, and that workspace: the
// call's own, the buffer lent to the device or the library's.
template <typename NeedOf>
int plan_and_workspace(const Settings& st, int64_t BT, int64_t H, int64_t V, int dtype, NeedOf need_of, Plan* p,
                       char** ws) {
    for (const Room room : {Room::full, Room::bounded, Room::least}) {
        *p = plan_for(st, BT, H, V, dtype, room);
        if (room == Room::full) {   // (the launches' sizes do not depend on the room)
            FLCE_TRY(check_launch_limits(*p, H, V));
            if (st.ws && !aligned(st.ws, 256)) return FLCE_ERR_ALIGN;
        }
        auto take = [&](size_t need) -> int {
            if (!st.ws) return acquire_workspace(need, ws, room == Room::least);
            *ws = static_cast<char*>(st.ws);
            return st.ws_bytes >= need ? FLCE_OK : FLCE_ERR_WORKSPACE;
        };
        const size_t need = need_of(*p);
        int rc = take(need);
        if (rc == FLCE_ERR_WORKSPACE && room == Room::full) {
            // a buffer between the bounded plan and this one: as many K ranges as there is room for
            size_t have = st.ws_bytes;
            if (!st.ws) FLCE_TRY(lent_workspace(&have));
            if (have < need && need - have < p->dxpart_bytes &&
                have >= need_of(plan_for(st, BT, H, V, dtype, Room::bounded))) {
                *p = plan_for(st, BT, H, V, dtype, room, false, p->dxpart_bytes - (need - have));
                rc = take(need_of(*p));
            }
        }
        if (rc != FLCE_ERR_WORKSPACE) return rc;
    }
    return FLCE_ERR_WORKSPACE;
}

struct NormLayout {
    size_t off_rstd, off_partial, total;
};
NormLayout norm_layout(const Plan& p, int64_t H) {
    NormLayout l{};
    size_t off = p.total;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) / 256 * 256;
        return at;
    };
    l.off_rstd = take((size_t)p.C * sizeof(float));
    l.off_partial = take((size_t)RN_SLOTS * H * sizeof(float));
    l.total = off;
    return l;
}

template <typename T>
int run_rmsnorm_head(const T* h, const T* gamma, float eps, const T* W, const int64_t* targets,
                     int64_t BT, int64_t H, int64_t V, int64_t ignore_index, float* loss, T* dh,
                     T* dgamma, T* dW, unsigned flags, const Plan& p, const NormLayout& l, char* ws,
                     hipStream_t s) {
    const bool want_dx = !(flags & FLCE_SKIP_DX);
    NormCtx<T> n{gamma, eps, reinterpret_cast<float*>(ws + l.off_rstd),
                 reinterpret_cast<float*>(ws + l.off_partial), dh};
    DeviceHeader* hdr = reinterpret_cast<DeviceHeader*>(ws + p.off_hdr);
    FLCE_TRY(run_head<T>(h, W, targets, BT, H, V, ignore_index, 1.0f, hdr, LossOut{hdr, 1, loss, nullptr, {1.0f}},
                         false, nullptr, dW, flags, p, ws, s, &n));
    if (want_dx) {
        hipLaunchKernelGGL((rmsnorm_dgamma_kernel<T>), dim3((unsigned)((H + RN_DG_COLS - 1) / RN_DG_COLS)),
                           dim3(RN_DG_COLS * RN_DG_PARTS), 0, s, n.partial, (int)rn_slots(p.C), (int)H, dgamma);
        HIP_TRY(hipGetLastError());
    }
    return FLCE_OK;
}

// Argument checks shared by the two stand-alone cross-entropy entry points.
int check_ce_args(const void* Z, const int64_t* targets, int64_t BT, int64_t V, int64_t ldz,
                  int64_t ignore_index, int dtype, const float* loss) {
    FLCE_TRY(check_dims(BT, 1, V, dtype));
    if (!Z || !targets || !loss) return FLCE_ERR_NULL;
    if (ldz < V || ldz > MAX_DIM * 4) return FLCE_ERR_SHAPE;
    if (!aligned(Z, elem_size(dtype)) || !aligned(targets, 8) || !aligned(loss, 4))
        return FLCE_ERR_ALIGN;
    if (ignore_index >= 0 && ignore_index < V) return FLCE_ERR_ARG;
    return FLCE_OK;
}

// Stand-alone cross entropy on logits Z, `step` rows per launch, with the device header
// and the per-row losses (`step` floats) in memory the caller of this function provides; done_words:
// the counters that go with that memory, or null.
int run_ce_inplace(void* Z, const int64_t* targets, int64_t BT, int64_t V, int64_t ldz,
                   int64_t ignore_index, int dtype, float* loss, DeviceHeader* hdr, float* row_loss,
                   int64_t step, done_t* done_words, bool timed, hipStream_t s) {
    const int count_n = BT <= ce_count_rows(V * (int64_t)elem_size(dtype)) && BT <= step ? (int)BT : 0;
    // (logits beyond the memory-side cache: milliseconds, and they want the nontemporal variants)
    DoneCount done{};
    if (done_words && count_n && BT * V * (int64_t)elem_size(dtype) <= CE_CACHE_BYTES)
        done = {done_words, g_ce_ticket.fetch_add(1) + 1};
    if (!count_n) {
        hipLaunchKernelGGL(count_valid_kernel, dim3(1), dim3(1024), 0, s, targets, BT, ignore_index,
                           1.0f, hdr);
        HIP_TRY(hipGetLastError());
    }
    for (int64_t r0 = 0; r0 < BT; r0 += step) {
        const int64_t rows = (BT - r0 < step) ? BT - r0 : step;
        if (dtype == FLCE_F32)
            FLCE_TRY(launch_ce_rows<float>(static_cast<float*>(Z) + r0 * ldz, ldz, targets + r0,
                                           rows, V, 0, ignore_index, hdr, row_loss, s, nullptr, timed, count_n, 1.0f, false,
                                           done, loss));
        else
            FLCE_TRY(launch_ce_rows<bf16_t>(static_cast<bf16_t*>(Z) + r0 * ldz, ldz, targets + r0,
                                            rows, V, 0, ignore_index, hdr, row_loss, s, nullptr, timed, count_n, 1.0f, false,
                                            done, loss));
        if (!done.words) FLCE_TRY(launch_loss(row_loss, rows, hdr,
                             r0 + rows == BT ? LossOut{hdr, 1, loss, nullptr, {1.0f}} : LossOut{}, timed, s));
    }
    return FLCE_OK;
}

// The current device's copies of `scratch` and `ce_done` (on the first call on a device the runtime is asked).
int static_addresses(unsigned char** scratch_at, done_t** done_at) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return FLCE_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr, *q = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        HIP_TRY(hipGetSymbolAddress(&q, HIP_SYMBOL(ce_done)));
        if (!p || !q) return FLCE_ERR_HIP;
        g_scratch_ptr[dev] = p;
        g_done_ptr[dev] = q;
    }
    *scratch_at = static_cast<unsigned char*>(g_scratch_ptr[dev]);
    *done_at = static_cast<done_t*>(g_done_ptr[dev]);
    return FLCE_OK;
}

// Whether a stand-alone cross entropy may be the one launch that counts its workgroups.  Not while the
// stream is captured: every replay of the launch would bring the same ticket.
bool folds_loss(int64_t BT, hipStream_t s) {
    if (BT > CE_FOLD_ROWS) return false;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return status == hipStreamCaptureStatusNone;
}

// flce_multihead_fwd_bwd with the settings given (the process-wide ones, or a call's options)
int multihead_fwd_bwd(const Settings& st, const void* X, const void* const* W, const int64_t* const* targets,
                      const float* weights, int n_heads, int64_t BT, int64_t H, int64_t V,
                      int64_t ignore_index, int dtype, float* loss, float* head_losses, void* dX,
                      void* const* dW, unsigned flags, void* stream) {
    FLCE_TRY(check_dims(BT, H, V, dtype));
    if (n_heads < 1 || n_heads > MAX_HEADS) return FLCE_ERR_ARG;
    if (flags & ~(unsigned)(FLCE_SKIP_DX | FLCE_SKIP_DW)) return FLCE_ERR_ARG;
    const bool want_dx = !(flags & FLCE_SKIP_DX), want_dw = !(flags & FLCE_SKIP_DW);
    if (!X || !W || !targets || !loss || (want_dx && !dX) || (want_dw && !dW)) return FLCE_ERR_NULL;
    if (!aligned(X, 16) || (want_dx && !aligned(dX, 16)) || !aligned(loss, 4) ||
        (head_losses && !aligned(head_losses, 4)))
        return FLCE_ERR_ALIGN;
    for (int j = 0; j < n_heads; ++j) {
        if (!W[j] || !targets[j] || (want_dw && !dW[j])) return FLCE_ERR_NULL;
        if (!aligned(W[j], 16) || !aligned(targets[j], 8) || (want_dw && !aligned(dW[j], 16)))
            return FLCE_ERR_ALIGN;
        if (weights && !(weights[j] == weights[j] && weights[j] - weights[j] == 0.0f))
            return FLCE_ERR_ARG;   // NaN or infinite weight
        for (int k = 0; want_dw && k < j; ++k)
            if (dW[k] == dW[j]) return FLCE_ERR_ARG;   // every head needs a dW of its own
    }
    if (ignore_index >= 0 && ignore_index < V) return FLCE_ERR_ARG;   // would shadow a class

    Plan p;
    char* ws = nullptr;
    FLCE_TRY(plan_and_workspace(st, BT, H, V, dtype, [](const Plan& q) { return q.total; }, &p, &ws));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (dtype == FLCE_F32)
        return run_heads<float>(static_cast<const float*>(X), W, targets, weights, n_heads, BT, H, V,
                                ignore_index, loss, head_losses, static_cast<float*>(dX), dW, flags,
                                p, ws, s);
    return run_heads<bf16_t>(static_cast<const bf16_t*>(X), W, targets, weights, n_heads, BT, H, V,
                             ignore_index, loss, head_losses, static_cast<bf16_t*>(dX), dW, flags, p,
                             ws, s);
}

}  // namespace

extern "C" {

int flce_multihead_fwd_bwd(const void* X, const void* const* W, const int64_t* const* targets,
                           const float* weights, int n_heads, int64_t BT, int64_t H, int64_t V,
                           int64_t ignore_index, int dtype, float* loss, float* head_losses, void* dX,
                           void* const* dW, unsigned flags, void* stream) {
    return multihead_fwd_bwd(global_settings(), X, W, targets, weights, n_heads, BT, H, V, ignore_index,
                             dtype, loss, head_losses, dX, dW, flags, stream);
}

void flce_default_options(flce_options* opt) {
    if (!opt) return;
    const Settings st = global_settings();
    opt->size = sizeof(flce_options);
    opt->logits_budget_bytes = st.budget;
    opt->row_compaction = st.compact ? 1 : 0;
    opt->flags = 0u;
    opt->workspace = nullptr;
    opt->workspace_bytes = 0;
}

// The settings a call's options stand for; FLCE_ERR_ARG for a struct this library cannot read.
static int settings_from(const flce_options* opt, Settings* st, unsigned* flags) {
    *st = global_settings();
    *flags = 0u;
    if (!opt) return FLCE_OK;
    if (opt->size != sizeof(flce_options)) return FLCE_ERR_ARG;
    if (opt->row_compaction != 0 && opt->row_compaction != 1) return FLCE_ERR_ARG;
    st->budget = opt->logits_budget_bytes;
    st->compact = opt->row_compaction != 0;
    st->ws = opt->workspace;
    st->ws_bytes = opt->workspace ? opt->workspace_bytes : 0;
    *flags = opt->flags;
    return FLCE_OK;
}

int flce_fwd_bwd_opt(const void* X, const void* W, const int64_t* targets, int64_t BT, int64_t H,
                     int64_t V, int64_t ignore_index, int dtype, float* loss, void* dX, void* dW,
                     const flce_options* opt, void* stream) {
    Settings st;
    unsigned flags;
    FLCE_TRY(settings_from(opt, &st, &flags));
    const void* Ws[1] = {W};
    const int64_t* ts[1] = {targets};
    void* dWs[1] = {dW};
    return multihead_fwd_bwd(st, X, Ws, ts, nullptr, 1, BT, H, V, ignore_index, dtype, loss, nullptr, dX,
                             dWs, flags, stream);
}

size_t flce_workspace_bytes_opt(int64_t BT, int64_t H, int64_t V, int dtype, const flce_options* opt) {
    Settings st;
    unsigned flags;
    if (check_dims(BT, H, V, dtype) != FLCE_OK || settings_from(opt, &st, &flags) != FLCE_OK) return 0;
    return plan_for(st, BT, H, V, dtype).total;
}

int flce_rmsnorm_fwd_bwd(const void* h, const void* gamma, float eps, const void* W,
                         const int64_t* targets, int64_t BT, int64_t H, int64_t V,
                         int64_t ignore_index, int dtype, float* loss, void* dh, void* dgamma,
                         void* dW, unsigned flags, void* stream) {
    FLCE_TRY(check_dims(BT, H, V, dtype));
    if (flags & ~(unsigned)(FLCE_SKIP_DX | FLCE_SKIP_DW)) return FLCE_ERR_ARG;
    const bool want_dx = !(flags & FLCE_SKIP_DX), want_dw = !(flags & FLCE_SKIP_DW);
    if (!h || !gamma || !W || !targets || !loss || (want_dx && (!dh || !dgamma)) || (want_dw && !dW))
        return FLCE_ERR_NULL;
    if (!aligned(h, 16) || !aligned(W, 16) || !aligned(gamma, elem_size(dtype)) ||
        (want_dx && (!aligned(dh, 16) || !aligned(dgamma, elem_size(dtype)))) ||
        (want_dw && !aligned(dW, 16)) || !aligned(targets, 8) || !aligned(loss, 4))
        return FLCE_ERR_ALIGN;
    if (ignore_index >= 0 && ignore_index < V) return FLCE_ERR_ARG;
    if (!(eps >= 0.0f) || eps - eps != 0.0f) return FLCE_ERR_ARG;   // negative, NaN or infinite

    Plan p;
    char* ws = nullptr;
    FLCE_TRY(plan_and_workspace(global_settings(), BT, H, V, dtype,
                                [&](const Plan& q) { return norm_layout(q, H).total; }, &p, &ws));
    const NormLayout l = norm_layout(p, H);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (dtype == FLCE_F32)
        return run_rmsnorm_head<float>(static_cast<const float*>(h), static_cast<const float*>(gamma),
                                       eps, static_cast<const float*>(W), targets, BT, H, V,
                                       ignore_index, loss, static_cast<float*>(dh),
                                       static_cast<float*>(dgamma), static_cast<float*>(dW), flags, p,
                                       l, ws, s);
    return run_rmsnorm_head<bf16_t>(static_cast<const bf16_t*>(h), static_cast<const bf16_t*>(gamma),
                                    eps, static_cast<const bf16_t*>(W), targets, BT, H, V,
                                    ignore_index, loss, static_cast<bf16_t*>(dh),
                                    static_cast<bf16_t*>(dgamma), static_cast<bf16_t*>(dW), flags, p,
                                    l, ws, s);
}

size_t flce_rmsnorm_workspace_bytes(int64_t BT, int64_t H, int64_t V, int dtype) {
    if (check_dims(BT, H, V, dtype) != FLCE_OK) return 0;
    return norm_layout(plan_for(BT, H, V, dtype), H).total;
}

int flce_fwd_bwd_ex(const void* X, const void* W, const int64_t* targets, int64_t BT, int64_t H,
                    int64_t V, int64_t ignore_index, int dtype, float* loss, void* dX, void* dW,
                    unsigned flags, void* stream) {
    const void* Ws[1] = {W};
    const int64_t* ts[1] = {targets};
    void* dWs[1] = {dW};
    return flce_multihead_fwd_bwd(X, Ws, ts, nullptr, 1, BT, H, V, ignore_index, dtype, loss, nullptr,
                                  dX, dWs, flags, stream);
}

int flce_fwd_bwd(const void* X, const void* W, const int64_t* targets, int64_t BT, int64_t H,
                 int64_t V, int64_t ignore_index, int dtype, float* loss, void* dX, void* dW,
                 void* stream) {
    return flce_fwd_bwd_ex(X, W, targets, BT, H, V, ignore_index, dtype, loss, dX, dW, 0u, stream);
}

int flce_cross_entropy_inplace(void* Z, const int64_t* targets, int64_t BT, int64_t V, int64_t ldz,
                               int64_t ignore_index, int dtype, float* loss, void* stream) {
    FLCE_TRY(check_ce_args(Z, targets, BT, V, ldz, ignore_index, dtype, loss));
    const int64_t step = BT < CE_ROWS_PER_LAUNCH ? BT : CE_ROWS_PER_LAUNCH;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = nullptr;
    bool lent = false;
    FLCE_TRY(acquire_workspace(256 + (size_t)step * sizeof(float), &ws, true, &lent));
    // Calls on different lent buffers may overlap, and a buffer's contents are anybody's: no counters for them.
    done_t* done = nullptr;
    unsigned char* unused;
    if (!lent && folds_loss(BT, s) && static_addresses(&unused, &done) == FLCE_OK) done += DONE_WORDS;
    return run_ce_inplace(Z, targets, BT, V, ldz, ignore_index, dtype, loss,
                          reinterpret_cast<DeviceHeader*>(ws), reinterpret_cast<float*>(ws + 256), step,
                          done, true, s);
}

int flce_cross_entropy_inplace_noalloc(void* Z, const int64_t* targets, int64_t BT, int64_t V,
                                       int64_t ldz, int64_t ignore_index, int dtype, float* loss,
                                       void* stream) {
    FLCE_TRY(check_ce_args(Z, targets, BT, V, ldz, ignore_index, dtype, loss));
    if (BT > FLCE_CE_NOALLOC_MAX_ROWS) return FLCE_ERR_TOO_LARGE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    unsigned char* ptr = nullptr;
    done_t* done = nullptr;
    FLCE_TRY(static_addresses(&ptr, &done));
    // The header is reset by the counting kernel or, for small batches, by the row kernel, and every
    // row's loss slot is written by the row kernel before it is summed, so nothing of the previous
    // call's contents is read.
    return run_ce_inplace(Z, targets, BT, V, ldz, ignore_index, dtype, loss,
                          reinterpret_cast<DeviceHeader*>(ptr), reinterpret_cast<float*>(ptr + 256), BT,
                          folds_loss(BT, s) ? done : nullptr, false, s);
}

size_t flce_workspace_bytes(int64_t BT, int64_t H, int64_t V, int dtype) {
    if (check_dims(BT, H, V, dtype) != FLCE_OK) return 0;
    return plan_for(BT, H, V, dtype).total;
}

size_t flce_workspace_bytes_max(int64_t H, int64_t V, int dtype) {
    if (check_dims(1, H, V, dtype) != FLCE_OK) return 0;
    return plan_for(global_settings(), 0, H, V, dtype, Room::full, true).total;
}

int flce_set_workspace(void* ws, size_t bytes) {
    if (ws && !aligned(ws, 256)) return FLCE_ERR_ALIGN;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return FLCE_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_ws[dev].lent = ws;
    g_ws[dev].lent_bytes = ws ? bytes : 0;
    return FLCE_OK;
}

int flce_release_workspace(void) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return FLCE_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceWorkspace& w = g_ws[dev];
    if (w.own) {
        HIP_TRY(hipDeviceSynchronize());
        HIP_TRY(hipFree(w.own));
        w.own = nullptr;
        w.own_bytes = 0;
    }
    w.own_failed = 0;
    return FLCE_OK;
}

int flce_set_logits_budget_bytes(size_t bytes) {
    g_budget.store(bytes);
    return FLCE_OK;
}

size_t flce_get_logits_budget_bytes(void) { return g_budget.load(); }

int flce_set_row_compaction(int on) {
    g_compact.store(on != 0);
    return FLCE_OK;
}

int flce_get_row_compaction(void) { return g_compact.load() ? 1 : 0; }

int64_t flce_chunk_rows(int64_t BT, int64_t H, int64_t V, int dtype) {
    if (check_dims(BT, H, V, dtype) != FLCE_OK) return 0;
    return plan_for(BT, H, V, dtype).C;
}

int64_t flce_num_chunks(int64_t BT, int64_t H, int64_t V, int dtype) {
    if (check_dims(BT, H, V, dtype) != FLCE_OK) return 0;
    return plan_for(BT, H, V, dtype).nchunks;
}

size_t flce_logits_budget_for_workspace(int64_t BT, int64_t H, int64_t V, int dtype, size_t max_workspace_bytes) {
    if (check_dims(BT, H, V, dtype) != FLCE_OK) return 0;
    Settings st = global_settings();
    const size_t row_bytes = (size_t)round_up(V, 64) * elem_size(dtype);
    // the workspace grows with the rows per chunk apart from small steps in the dX partial
    // results, so the first fit from the top is the largest
    for (int64_t c = round_up(BT, CHUNK_ALIGN); c >= CHUNK_ALIGN; c -= CHUNK_ALIGN) {
        st.budget = (size_t)c * row_bytes;
        const Plan p = plan_for(st, BT, H, V, dtype);
        if (p.total <= max_workspace_bytes && check_launch_limits(p, H, V) == FLCE_OK) return st.budget;
    }
    return 0;
}

int flce_dx_k_ranges(int64_t BT, int64_t H, int64_t V, int dtype) {
    if (check_dims(BT, H, V, dtype) != FLCE_OK) return 0;
    return plan_for(BT, H, V, dtype).dx_ranges;
}

int64_t flce_paper_chunk_rows(int64_t BT, int64_t H, int64_t V) {
    if (BT <= 0 || H <= 0 || V <= 0) return 0;
    return paper_chunk_rows(BT, H, V);
}

size_t flce_full_logits_bytes(int64_t BT, int64_t V, int dtype) {
    if (BT <= 0 || V <= 0 || (dtype != FLCE_F32 && dtype != FLCE_BF16)) return 0;
    return (size_t)BT * (size_t)V * elem_size(dtype);
}

int flce_mfma_ceiling_launch(int pattern, int workgroups, int iters, float std_b, float* out,
                             size_t out_floats, void* stream) {
    if (!out) return FLCE_ERR_NULL;
    if (pattern < 0 || pattern > 2 || workgroups <= 0 || workgroups > 65536 || iters <= 0 ||
        (int64_t)workgroups * iters > ((int64_t)1 << 26) || !(std_b >= 0.0f) ||
        out_floats < (size_t)workgroups * 256)
        return FLCE_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const dim3 grid((unsigned)workgroups), block(256);
    if (pattern == 0) hipLaunchKernelGGL((mfma_ceiling_kernel<0>), grid, block, 0, s, out, iters, std_b);
    if (pattern == 1) hipLaunchKernelGGL((mfma_ceiling_kernel<1>), grid, block, 0, s, out, iters, std_b);
    if (pattern == 2) hipLaunchKernelGGL((mfma_ceiling_kernel<2>), grid, block, 0, s, out, iters, std_b);
    HIP_TRY(hipGetLastError());
    return FLCE_OK;
}

int flce_timing_enable(int on) {
    g_timing_on.store(on != 0);
    return FLCE_OK;
}

int flce_timing_collect(double* total_ms, int64_t* launches) {
    if (!total_ms || !launches) return FLCE_ERR_NULL;
    std::lock_guard<std::mutex> lock(g_mutex);
    for (int k = 0; k < FLCE_NUM_KINDS; ++k) {
        total_ms[k] = 0.0;
        launches[k] = 0;
    }
    int rc = FLCE_OK;
    for (TimingRecord& r : g_records) {
        float ms = 0.f;
        if (hipEventSynchronize(r.stop) == hipSuccess &&
            hipEventElapsedTime(&ms, r.start, r.stop) == hipSuccess) {
            for (const int kind : {r.kind, r.also}) {
                if (kind < 0) continue;
                total_ms[kind] += r.also < 0 ? ms : 0.5 * ms;
                launches[kind] += 1;
            }
        } else {
            (void)hipGetLastError();
            rc = FLCE_ERR_HIP;
        }
        (void)hipEventDestroy(r.start);
        (void)hipEventDestroy(r.stop);
    }
    g_records.clear();
    return rc;
}

const char* flce_status_string(int status) {
    switch (status) {
        case FLCE_OK: return "ok";
        case FLCE_ERR_NULL: return "a required pointer is NULL";
        case FLCE_ERR_SHAPE: return "BT, H, V or a stride is out of range";
        case FLCE_ERR_DTYPE: return "unknown dtype";
        case FLCE_ERR_ALIGN: return "a pointer misses its required alignment";
        case FLCE_ERR_WORKSPACE: return "workspace too small or allocation failed";
        case FLCE_ERR_HIP: return "a HIP runtime call or kernel launch failed";
        case FLCE_ERR_ARG: return "invalid argument";
        case FLCE_ERR_TOO_LARGE: return "problem larger than the fixed scratch of the allocation-free entry point";
        default: return "unknown status";
    }
}

}  // extern "C"
