// Guarded matrix product on the matrix cores, any shape, any alignment, fp32 or bf16 storage:
//     C[M x N] = (Cin +) sum_k a(m,k) * b(n,k)
// with each operand K-contiguous ("row" form, KM = false: a(m,k) = A[m*lda + k]) or K-major
// ("column" form, KM = true: a(m,k) = A[k*lda + m]), so no operand is ever transposed in
// memory.  It serves the fp32 storage type and the bf16 shapes the tuned kernel does not take.
//
// fp32 on the bf16 matrix cores.  v_mfma_f32_32x32x2_f32 runs at 1/16 of the bf16 rate, so an
// fp32 operand is split, while it is staged, into three bf16 planes x = hi + mid + lo (each the
// rounded remainder of the planes before: 8 + 8 + 8 bits and the signs hold all 24 bits), and
// the six plane products that matter (lo*hi, mid*mid, hi*lo, mid*hi, hi*mid, hi*hi; the other
// three are below 2^-26 of the product) are accumulated in fp32.  A product of two bf16 is exact
// in fp32, and six 16-wide matrix instructions round the accumulator 6 times per 16 K where the
// fp32 instruction rounds it 8 times.
// An infinite or NaN operand (or one that rounds to infinity in bf16) makes the split remainders
// NaN; a workgroup that finds a NaN among its sums computes its tile again with fp32 matrix
// instructions, so such inputs give what plain fp32 products give.
//
// Shape: 256 threads = 4 wavefronts (2 x 2); macro tile TILE x TILE, TILE = 128 or 64 (each
// wavefront owns 2 x 2 or one 32 x 32 MFMA tile), K step 32.  A thread stages 8 consecutive K
// values of one tile row per slot: row form 32 contiguous bytes, column form 8 loads that are
// contiguous across the wavefront's lanes.  The next K step's loads are in flight while the
// current one is multiplied; one LDS stage, so that several workgroups fit a CU and one splits
// while another multiplies.  LDS rows are 64 bytes whose four 16-byte pieces are XOR swizzled
// with (row / 4) % 4: writes and fragment reads touch all banks evenly.
// What bounds it (fp32): the six products per K, i.e. the bf16 matrix pipe, and the split's lane
// operations (5.5 per staged element).  Measured at 2048 x 1024 x 50257: logits 2.15 -> 1.26 ms,
// dX 4.82 -> 1.19, dW 2.31 -> 1.33 (167-178 TFLOP/s of fp32 products, 1.0-1.07 PFLOP/s on the
// matrix pipe) against the fp32 instruction's 151 TFLOP/s peak in a large library product, and 0.29
// ms of transposed copies are gone; at 256 x 512 x 4096, 64-tiles: 51 -> 19, 29 -> 17, 29 -> 18 us.
#pragma once
#include "flce_device.h"
#include "gemm_bf16_nt.h"

namespace flce {

constexpr int GG_THREADS = 256;
constexpr int GG_BK = 32;   // K elements per step

struct GGArgs {
    const void* A;
    int64_t lda;
    const void* B;
    int64_t ldb;
    void* C;
    int64_t ldc;
    const void* Cin;    // optional addend: fp32, or C's type with cin_f32 = 0
    int64_t ldcin;
    int cin_f32;
    int M, N, K;
    int ksplit;            // K is cut into this many ranges, one workgroup per tile and range
    int64_t split_stride;  // elements between the partial results of consecutive K ranges in C
    int vec_a, vec_b;      // row form: 16-byte loads are aligned (base and leading dimension)
    int vec_c;             // C (and Cin): groups of 4 columns are aligned
    // values only the device knows, as in FGArgs
    const int* dyn_rows;
    int dyn_is_k;
    const int* dyn_ksplit;
    const int* first_live;
    int launch;
    int group_m, group_cols, xcd_interleave;   // tile order, as in FGArgs
};

template <typename T> struct GGTraits;
template <> struct GGTraits<float> {
    static constexpr int PLANES = 3;
    static constexpr int VEC = 4;   // elements per 16 bytes
};
template <> struct GGTraits<bf16_t> {
    static constexpr int PLANES = 1;
    static constexpr int VEC = 8;
};

// One operand's staging: which slots (tile row, 8 K values) this thread fetches.
template <typename T, bool KM, int TILE>
struct GGStage {
    static constexpr int SLOTS = TILE / 64;
    static constexpr int PLANES = GGTraits<T>::PLANES;
    const T* ptr[SLOTS];   // row form: the slot's row; column form: the slot's column
    int64_t ld;
    int row[SLOTS], piece[SLOTS];
    T raw[SLOTS][8];

    __device__ __forceinline__ void init(const void* base, int64_t ld_, int r0, int extent, int tid) {
        ld = ld_;
#pragma unroll
        for (int h = 0; h < SLOTS; ++h) {
            if constexpr (KM) {
                row[h] = tid % TILE;
                piece[h] = __builtin_amdgcn_readfirstlane(tid / TILE + h * (GG_THREADS / TILE));
            } else {
                row[h] = (tid >> 2) + 64 * h;
                piece[h] = tid & 3;
            }
            // rows past the matrix repeat its last row: they only feed outputs that are not stored
            const int r = min(r0 + row[h], extent - 1);
            ptr[h] = static_cast<const T*>(base) + (KM ? (int64_t)r : (int64_t)r * ld);
        }
    }
    // K step starting at k0; K values from `K` on are zero
    __device__ __forceinline__ void load(int k0, int K, bool vec) {
        const bool whole = k0 + GG_BK <= K;   // uniform
#pragma unroll
        for (int h = 0; h < SLOTS; ++h) {
            const int k = k0 + piece[h] * 8;
            if constexpr (KM) {
                if (whole) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) raw[h][e] = ptr[h][(int64_t)(k + e) * ld];
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        raw[h][e] = (k + e < K) ? ptr[h][(int64_t)(k + e) * ld] : from_f32<T>(0.f);
                }
            } else {
                if (whole && vec) {
                    constexpr int V = GGTraits<T>::VEC;
                    struct alignas(16) Vec { T e[V]; };
#pragma unroll
                    for (int q = 0; q < 8 / V; ++q) {
                        const Vec v = *reinterpret_cast<const Vec*>(ptr[h] + k + q * V);
#pragma unroll
                        for (int e = 0; e < V; ++e) raw[h][q * V + e] = v.e[e];
                    }
                } else if (whole) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) raw[h][e] = ptr[h][k + e];
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) raw[h][e] = (k + e < K) ? ptr[h][k + e] : from_f32<T>(0.f);
                }
            }
        }
    }
    // the loaded step, split into bf16 planes, to LDS
    __device__ __forceinline__ void store(unsigned char* lds) const {
#pragma unroll
        for (int h = 0; h < SLOTS; ++h) {
            unsigned char* dst = lds + row[h] * 64 + ((piece[h] ^ ((row[h] >> 2) & 3)) << 4);
            u32x4 out[PLANES];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (PLANES == 1) {
                    const bf16x2 p = {raw[h][2 * q], raw[h][2 * q + 1]};
                    out[0][q] = __builtin_bit_cast(uint32_t, p);
                } else {
                    float a = raw[h][2 * q], b = raw[h][2 * q + 1];
#pragma unroll
                    for (int p = 0; p < PLANES; ++p) {
                        const bf16x2 c = {(bf16_t)a, (bf16_t)b};   // round to nearest even
                        const uint32_t u = __builtin_bit_cast(uint32_t, c);
                        out[p][q] = u;
                        if (p + 1 < PLANES) {   // exact: the remainder of a rounding
                            a -= __uint_as_float(u << 16);
                            b -= __uint_as_float(u & 0xffff0000u);
                        }
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < PLANES; ++p) *reinterpret_cast<u32x4*>(dst + p * TILE * 64) = out[p];
        }
    }
};

// element (r, k) of an operand, zero past K (the fp32 recomputation of a tile)
template <bool KM>
__device__ __forceinline__ float gg_element(const float* base, int64_t ld, int r, int k, int K) {
    return k < K ? (KM ? base[(int64_t)k * ld + r] : base[(int64_t)r * ld + k]) : 0.f;
}

template <typename T, typename OutT, bool A_KM, bool B_KM, int TILE>
__global__ __launch_bounds__(GG_THREADS, 2) void gemm_guarded(GGArgs a) {
    constexpr int PLANES = GGTraits<T>::PLANES;
    constexpr int W = TILE / 64;            // 32 x 32 MFMA tiles per wavefront and direction
    constexpr int SIDE = TILE * 64;         // bytes of one plane of one operand
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * PLANES * SIDE];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    const FgResolved rs = fg_resolve(a, a.Cin != nullptr);
    if (rs.skip) return;
    const int M = rs.M, K = rs.K, N = a.N;
    // workgroup id -> (K range, tile): as in gemm_bf16_256
    const int tiles_m = (M + TILE - 1) / TILE, tiles_n = (N + TILE - 1) / TILE;
    const int tiles = tiles_m * tiles_n;
    const int total = tiles * rs.ksplit;
    const int per_xcd = (total + FG_XCDS - 1) / FG_XCDS;
    const int in_xcd = (int)blockIdx.x / FG_XCDS;
    if (in_xcd >= per_xcd) return;
    const int seq = fg_seq(a, (int)blockIdx.x % FG_XCDS, in_xcd, per_xcd);
    if (seq >= total) return;
    const int split = seq / tiles;
    int m0, n0;
    fg_tile_origin<TILE>(seq - split * tiles, tiles_m, tiles_n, a.group_m, a.group_cols, m0, n0);
    const int steps = (K + GG_BK - 1) / GG_BK;
    const int k_begin = (int)((int64_t)steps * split / rs.ksplit) * GG_BK;
    const int k_end = min(K, (int)((int64_t)steps * (split + 1) / rs.ksplit) * GG_BK);

    f32x16 acc[W][W];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int g = 0; g < 16; ++g) acc[i][j][g] = 0.f;

    GGStage<T, A_KM, TILE> sa;
    GGStage<T, B_KM, TILE> sb;
    sa.init(a.A, a.lda, m0, M, tid);
    sb.init(a.B, a.ldb, n0, N, tid);
    unsigned char* lds_a = lds;
    unsigned char* lds_b = lds + PLANES * SIDE;
    const int frow = lane & 31, fhalf = lane >> 5;

    if (k_begin < k_end) {
        sa.load(k_begin, k_end, a.vec_a);
        sb.load(k_begin, k_end, a.vec_b);
    }
    for (int k0 = k_begin; k0 < k_end; k0 += GG_BK) {
        __syncthreads();   // the previous step's fragments have been read
        sa.store(lds_a);
        sb.store(lds_b);
        __syncthreads();
        if (k0 + GG_BK < k_end) {
            sa.load(k0 + GG_BK, k_end, a.vec_a);
            sb.load(k0 + GG_BK, k_end, a.vec_b);
        }
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int at = frow * 64 + (((2 * kk + fhalf) ^ ((frow >> 2) & 3)) << 4);
            bf16x8 fa[PLANES][W], fb[PLANES][W];
#pragma unroll
            for (int p = 0; p < PLANES; ++p)
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    fa[p][i] = *reinterpret_cast<const bf16x8*>(lds_a + p * SIDE + (wm * W + i) * 2048 + at);
                    fb[p][i] = *reinterpret_cast<const bf16x8*>(lds_b + p * SIDE + (wn * W + i) * 2048 + at);
                }
            // plane pairs (of a, of b), smallest products first
            constexpr int PAIRS = PLANES == 3 ? 6 : 1;
            constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
            for (int q = 0; q < PAIRS; ++q) {
                const int pa = PLANES == 3 ? PA[q] : 0, pb = PLANES == 3 ? PB[q] : 0;
#pragma unroll
                for (int i = 0; i < W; ++i)
#pragma unroll
                    for (int j = 0; j < W; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[pb][j], fa[pa][i], acc[i][j], 0, 0, 0);
            }
        }
    }

    if constexpr (PLANES == 3) {
        bool nan = false;
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int j = 0; j < W; ++j)
#pragma unroll
                for (int g = 0; g < 16; ++g) {
                    const float v = acc[i][j][g];
                    nan |= (v != v);
                }
        if (__syncthreads_or(nan)) {
            int ra[W], rb[W];
#pragma unroll
            for (int i = 0; i < W; ++i) {
                ra[i] = min(m0 + (wm * W + i) * 32 + frow, M - 1);
                rb[i] = min(n0 + (wn * W + i) * 32 + frow, N - 1);
#pragma unroll
                for (int j = 0; j < W; ++j)
#pragma unroll
                    for (int g = 0; g < 16; ++g) acc[i][j][g] = 0.f;
            }
            const float* A = static_cast<const float*>(a.A);
            const float* B = static_cast<const float*>(a.B);
            for (int k0 = k_begin; k0 < k_end; k0 += 8) {
                float va[4][W], vb[4][W];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < W; ++i) {
                        va[u][i] = gg_element<A_KM>(A, a.lda, ra[i], k0 + 2 * u + fhalf, k_end);
                        vb[u][i] = gg_element<B_KM>(B, a.ldb, rb[i], k0 + 2 * u + fhalf, k_end);
                    }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < W; ++i)
#pragma unroll
                        for (int j = 0; j < W; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(vb[u][j], va[u][i], acc[i][j], 0, 0, 0);
            }
        }
    }

    // the B fragment is the MFMA's first operand: accumulator register g of lane l holds row
    // l % 32, column 8*(g/4) + 4*(l/32) + g%4 of its 32 x 32 tile
    OutT* C = static_cast<OutT*>(a.C) + (int64_t)split * a.split_stride;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int row = m0 + (wm * W + i) * 32 + frow;
        if (row >= M) continue;
        OutT* crow = C + (int64_t)row * a.ldc;
        const unsigned char* inrow =
            static_cast<const unsigned char*>(a.Cin) + (int64_t)row * a.ldcin * (a.cin_f32 ? 4 : (int)sizeof(OutT));
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int col = n0 + (wn * W + j) * 32 + 8 * g4 + 4 * fhalf;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * g4 + e];
                if (rs.use_in) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < N)
                            v[e] += a.cin_f32 ? reinterpret_cast<const float*>(inrow)[col + e]
                                              : to_f32(reinterpret_cast<const OutT*>(inrow)[col + e]);
                }
                if (a.vec_c && col + 4 <= N) {
                    struct alignas(4 * sizeof(OutT)) Quad { OutT e[4]; } q;
#pragma unroll
                    for (int e = 0; e < 4; ++e) q.e[e] = from_f32<OutT>(v[e]);
                    *reinterpret_cast<Quad*>(crow + col) = q;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < N) crow[col + e] = from_f32<OutT>(v[e]);
                }
            }
    }
}

}  // namespace flce
