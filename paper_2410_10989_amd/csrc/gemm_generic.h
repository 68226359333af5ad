// Guarded matrix product on the matrix cores, any shape, any alignment, fp32 or bf16 storage:
//     C[M x N] = (Cin +) sum_k a(m,k) * b(n,k)
// with each operand K-contiguous ("row" form, KM = false: a(m,k) = A[m*lda + k]) or K-major
// ("column" form, KM = true: a(m,k) = A[k*lda + m]), so no operand is ever transposed in
// memory.  It serves the fp32 storage type and the bf16 shapes the tuned kernel does not take.
//
// fp32 on the bf16 matrix cores.  v_mfma_f32_32x32x2_f32 runs at 1/16 of the bf16 rate, so an
// fp32 operand is split, while it is staged, into three bf16 planes 2^24 x = hi + mid + lo (each
// the rounded remainder of the planes before: 8 + 8 + 8 bits and the signs hold all 24 bits), and
// the six plane products that matter (lo*hi, mid*mid, hi*lo, mid*hi, hi*mid, hi*hi; the other
// three are below 2^-26 of the product) are accumulated in fp32.  A product of two bf16 is exact
// in fp32, and six 16-wide matrix instructions round the accumulator 6 times per 16 K where the
// fp32 instruction rounds it 8 times.
// The factor 2^24 (taken back as 2^-48 when the sums are written; both exact) is there because
// bf16 has the exponents of fp32: without it lo is subnormal and loses bits below |x| = 2^-103,
// mid below 2^-111, with it every plane of every fp32 value, subnormal ones too, is zero or a
// normal bf16.  It costs 2 lane operations of 13 per pair of elements: 2048 x 1024 x 50257 2854 ->
// 2938 us, 4096 x 4096 x 32000 13.13 -> 13.48 ms, 256 x 512 x 4096 54.7 -> 55.9 (with the factor as a
// literal 1.2 more: such short launches wait for their instructions).
// Where that leaves the range of the type (|x| >= 2^104, infinite or NaN operands, sums of 2^80
// and more) the split remainders or the sums are infinite or NaN; a workgroup that finds one among
// its sums computes them again with fp32 matrix instructions, so such inputs give what plain
// fp32 products give.  A NaN operand alone makes the same sums NaN either way, so the workgroup first
// looks through its operands and computes only the 32 x 32 blocks again in which something else is out of
// range (gg_needs_fp32).  2048 x 1024 x 50257, 2.94 ms: with a NaN in X 3.8 ms (21.7 when every such tile was
// computed again), with an infinite X 4.1, with a weight of -inf 6.2 (19.5 and 17.5; products on the fp32
// instructions alone took 9.6).
//
// Shape: macro tile TILE x TILE.  TILE = 256: 512 threads = 8 wavefronts (2 x 4), each with 4 x 2 MFMA
// tiles of 32 x 32, K step 16; 128: 256 threads = 4 wavefronts (2 x 2) with 2 x 2 MFMA tiles, K step
// 16; 64: 4 wavefronts with one MFMA tile in two accumulators, so that the plane products do not wait
// for one another, K step 32.  A thread stages 8 consecutive K values of one tile row per operand and
// step: row form 32 contiguous bytes, column form 8 loads that are contiguous across the wavefront's
// lanes.  Loads run gg_depth steps ahead in registers; LDS is double buffered with one barrier per step,
// and the split of step t + 1 (lane operations) stands beside the products of step t (matrix pipe) in the
// same instruction stream.  LDS: per plane, [K piece of 8][row] 16-byte entries, the rows of a piece
// permuted by gg_fold: writes and fragment reads touch all banks evenly.
#pragma once
#include "flce_device.h"
#include "gemm_bf16_nt.h"

namespace flce {

constexpr int gg_threads(int tile) { return tile == 256 ? 512 : 256; }
constexpr int gg_bk(int tile) { return tile == 64 ? 32 : 16; }      // K elements per step
constexpr int gg_depth(int tile) { return tile == 64 ? 4 : 2; } // K steps whose loads are in flight

constexpr float GG_SCALE = 16777216.f;                            // 2^24, on both operands of an fp32 product
constexpr float GG_UNSCALE = 1.f / (GG_SCALE * GG_SCALE);         // 2^-48

// LDS holds the rows of K piece p permuted by XOR with this, so that the 8 or 16 neighbouring lanes
// of a row-form write (2 or 4 pieces of 4 consecutive rows) touch all banks once.
__device__ __forceinline__ int gg_fold(int piece) { return (0x6ac0 >> (4 * piece)) & 15; }

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

// One operand's staging: the tile row and the 8 K values of a step this thread fetches.
template <typename T, bool KM, int TILE>
struct GGStage {
    static constexpr int PLANES = GGTraits<T>::PLANES;
    static constexpr int PIECES = gg_bk(TILE) / 8;
    static_assert(TILE * PIECES == gg_threads(TILE), "one slot per thread");
    const T* ptr;   // row form: the slot's row; column form: the slot's column
    int64_t ld;
    int k8;         // first of the slot's K values inside a step
    int lds_at;
    T raw[gg_depth(TILE)][8];

    // rows_at (row form, not null): LDS, the tile's rows are these of the matrix
    __device__ __forceinline__ void init(const void* base, int64_t ld_, int r0, int extent, int tid,
                                         const int* rows_at = nullptr) {
        ld = ld_;
        // column form: a wavefront's lanes are consecutive columns of one piece
        const int row = KM ? tid % TILE : tid / PIECES;
        const int piece = KM ? __builtin_amdgcn_readfirstlane(tid / TILE) : tid % PIECES;
        k8 = piece * 8;
        lds_at = (piece * TILE + (row ^ gg_fold(piece))) * 16;
        // rows past the matrix repeat its last row: they only feed outputs that are not stored
        const int r = rows_at ? rows_at[min(row, extent - 1 - r0)] : min(r0 + row, extent - 1);
        ptr = static_cast<const T*>(base) + (KM ? (int64_t)r : (int64_t)r * ld);
    }
    // the whole K step starting at k0, into ring position D; V: 16-byte loads (row form)
    template <int D, bool V>
    __device__ __forceinline__ void load(int k0) {
        if constexpr (KM) {
            const T* p = ptr + (int64_t)(k0 + k8) * ld;
#pragma unroll
            for (int e = 0; e < 8; ++e) raw[D][e] = p[e * ld];
        } else if constexpr (V) {
            constexpr int N = GGTraits<T>::VEC;
            struct alignas(16) Vec { T e[N]; };
#pragma unroll
            for (int q = 0; q < 8 / N; ++q) {
                const Vec v = *reinterpret_cast<const Vec*>(ptr + k0 + k8 + q * N);
#pragma unroll
                for (int e = 0; e < N; ++e) raw[D][q * N + e] = v.e[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) raw[D][e] = ptr[k0 + k8 + e];
        }
    }
    // a K step that K cuts: zero from K on
    template <int D>
    __device__ __forceinline__ void load_tail(int k0, int K) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + k8 + e;
            raw[D][e] = k < K ? ptr[KM ? (int64_t)k * ld : (int64_t)k] : from_f32<T>(0.f);
        }
    }
    // ring position D, split into bf16 planes, to LDS
    template <int D>
    __device__ __forceinline__ void store(unsigned char* lds) const {
        u32x4 out[PLANES];
        float scale = GG_SCALE;
        asm("" : "+s"(scale));   // in a register: as a literal it doubles the code of 16 operations per step
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (PLANES == 1) {
                const bf16x2 p = {raw[D][2 * q], raw[D][2 * q + 1]};
                out[0][q] = __builtin_bit_cast(uint32_t, p);
            } else {
                float a = raw[D][2 * q] * scale, b = raw[D][2 * q + 1] * scale;
#pragma unroll
                for (int p = 0; p < PLANES; ++p) {
                    uint32_t u;   // both rounded to nearest even
                    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(u) : "v"(a), "v"(b));
                    out[p][q] = u;
                    if (p + 1 < PLANES) {   // exact: the remainder of a rounding
                        a -= __uint_as_float(u << 16);
                        b -= __uint_as_float(u & 0xffff0000u);
                    }
                }
            }
        }
#pragma unroll
        for (int p = 0; p < PLANES; ++p) *reinterpret_cast<u32x4*>(lds + lds_at + p * TILE * gg_bk(TILE) * 2) = out[p];
    }
};

// element (r, k) of an operand, zero past K (the fp32 recomputation of a tile)
template <bool KM>
__device__ __forceinline__ float gg_element(const float* base, int64_t ld, int r, int k, int K) {
    return k < K ? (KM ? base[(int64_t)k * ld + r] : base[(int64_t)r * ld + k]) : 0.f;
}

// Per row of an operand's tile, the largest |x| over K values k0 .. k1 - 1 as the bits of a float (more
// than those of infinity: the row holds a NaN), by all threads of the workgroup; top: LDS, zero before.
template <bool KM, int TILE>
__device__ __forceinline__ void gg_row_tops(const float* base, int64_t ld, int r0, int rows, int k0, int k1, int tid,
                                            unsigned* top, const int* rows_at = nullptr) {
    constexpr int THREADS = gg_threads(TILE);
    if constexpr (KM) {   // lanes along the rows: contiguous
        const int r = tid % TILE;
        unsigned m = 0;
        if (r < rows) {
#pragma unroll 8
            for (int k = k0 + tid / TILE; k < k1; k += THREADS / TILE)
                m = max(m, __float_as_uint(base[(int64_t)k * ld + r0 + r]) & 0x7fffffffu);
            atomicMax(&top[r], m);
        }
    } else {              // lanes along K
        for (int r = tid / WAVE; r < rows; r += THREADS / WAVE) {
            const float* row = base + (int64_t)(rows_at ? rows_at[r] : r0 + r) * ld;
            unsigned m = 0;
#pragma unroll 8
            for (int k = k0 + tid % WAVE; k < k1; k += WAVE) m = max(m, __float_as_uint(row[k]) & 0x7fffffffu);
            atomicMax(&top[r], m);
        }
    }
}
// Which 32 x 32 blocks (bit i WN + j) of a wavefront's part of a tile whose split sums hold infinities or
// NaN need the fp32 instructions: not those where every one of them stems from a NaN operand, which
// makes its whole row or column NaN in any arithmetic while all other sums stayed in range, i.e. where
// among the block's rows without a NaN all |a| and |b| are below 2^103 and K |a| |b| below 2^79.
template <bool A_KM, bool B_KM, int TILE, int WM, int WN>
__device__ __forceinline__ unsigned gg_needs_fp32(const GGArgs& a, int m0, int M, int n0, int N, int k0, int k1, int tid,
                                                  int wm, int wn, unsigned* lds,   // 2 TILE words
                                                  const int* rows_at) {
    for (int i = tid; i < 2 * TILE; i += gg_threads(TILE))   // (rows past the matrix count as NaN)
        lds[i] = (i < TILE ? m0 + i < M : n0 + i - TILE < N) ? 0u : 0xffffffffu;
    __syncthreads();
    gg_row_tops<A_KM, TILE>(static_cast<const float*>(a.A), a.lda, m0, min(TILE, M - m0), k0, k1, tid, lds, rows_at);
    gg_row_tops<B_KM, TILE>(static_cast<const float*>(a.B), a.ldb, n0, min(TILE, N - n0), k0, k1, tid, lds + TILE);
    __syncthreads();
    auto top_of = [&](const unsigned* row) {   // of 32 rows: 1 + the largest that is no NaN, 0 if there is none
        const unsigned u = row[tid & 31];
        unsigned m = u <= 0x7f800000u ? u + 1 : 0u;
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o, WAVE));
        return m;
    };
    unsigned blocks = 0;
#pragma unroll 1
    for (int ij = 0; ij < WM * WN; ++ij) {
        const unsigned ma = top_of(lds + (wm * WM + ij / WN) * 32), mb = top_of(lds + TILE + (wn * WN + ij % WN) * 32);
        const float ta = __uint_as_float(ma - 1), tb = __uint_as_float(mb - 1);
        if (ma && mb && (ta >= 0x1p103f || tb >= 0x1p103f || (double)ta * tb * (k1 - k0) >= 0x1p79)) blocks |= 1u << ij;
    }
    return __builtin_amdgcn_readfirstlane(blocks);
}

// Fin: as in gemm_bf16.
//
// FEW: for at most one workgroup per CU.  The room in LDS keeps a third workgroup off the CU, so that the
// compiler spends 250 registers per lane instead of 168 on loads and fragments in flight (no other way was
// found to make it: waves_per_eu does not).  fp32 64-tiles, whole calls: 29 x 2816 x 1124 74 -> 66 us, 256 x 512 x 4096
// 52.8 -> 51.0; with two and more workgroups per CU 3 % slower (593 x 256 x 13824 102 -> 107).
template <typename T, int TILE, bool FEW = false>
struct GGLds {
    static constexpr int PLANE = TILE * gg_bk(TILE) * 2;             // bytes of one plane of one operand
    static constexpr int SIDE = GGTraits<T>::PLANES * PLANE;
    unsigned char tiles[2][2 * SIDE + (FEW ? 4096 : 0)];
};
template <typename T, typename OutT, bool A_KM, bool B_KM, int TILE, typename Fin, bool FEW>
__device__ __forceinline__ ProductTile gg_product(const GGArgs& a, const Fin& fin, int block, GGLds<T, TILE, FEW>& smem,
                                                  int* row_list) {
    constexpr bool SELECT = IsSelect<Fin>::value;
    static_assert(!SELECT || !A_KM, "rows are picked from a row-form operand");
    constexpr int PLANES = GGTraits<T>::PLANES;
    constexpr int WAVES_N = TILE == 256 ? 4 : 2;              // wavefronts: 2 x WAVES_N
    constexpr int WM = TILE / 64, WN = TILE / 32 / WAVES_N;   // 32 x 32 MFMA tiles per wavefront
    constexpr int BK = gg_bk(TILE), DEPTH = gg_depth(TILE);
    constexpr int PLANE = GGLds<T, TILE, FEW>::PLANE, SIDE = GGLds<T, TILE, FEW>::SIDE;
    constexpr int ACCS = TILE == 64 ? 2 : 1;
    auto& lds = smem.tiles;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    FgResolved rs = fg_resolve(a, a.Cin != nullptr);
    if (rs.skip) return ProductTile{};
    TileRows<gg_threads(TILE) / WAVE> picked;
    if constexpr (SELECT) rs.M = picked.begin(fin.targets, fin.BT, fin.ignore_index, row_list + TILE);
    const int* rows_at = SELECT ? row_list : nullptr;
    const int M = rs.M, K = rs.K, N = a.N;
    // workgroup id -> (K range, tile): as in gemm_bf16
    const int tiles_m = (M + TILE - 1) / TILE, tiles_n = (N + TILE - 1) / TILE;
    const int tiles = tiles_m * tiles_n;
    const int total = tiles * rs.ksplit;
    const int per_xcd = (total + FG_XCDS - 1) / FG_XCDS;
    const int in_xcd = block / FG_XCDS;
    if (in_xcd >= per_xcd) return ProductTile{};
    const int seq = fg_seq(a, block % FG_XCDS, in_xcd, per_xcd);
    if (seq >= total) return ProductTile{};
    const int split = seq / tiles;
    int m0, n0;
    fg_tile_origin<TILE>(seq - split * tiles, tiles_m, tiles_n, a.group_m, a.group_cols, m0, n0);
    const int steps_all = (K + BK - 1) / BK;
    const int k_begin = (int)((int64_t)steps_all * split / rs.ksplit) * BK;
    const int k_end = min(K, (int)((int64_t)steps_all * (split + 1) / rs.ksplit) * BK);
    const int n_whole = max(0, k_end - k_begin) / BK;   // K steps that are whole; at most one more is not

    f32x16 acc[WM][WN], acc2[ACCS];   // acc2[1]: the second accumulator of a 64-tile
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int g = 0; g < 16; ++g) acc[i][j][g] = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) acc2[ACCS - 1][g] = 0.f;

    GGStage<T, A_KM, TILE> sa;
    GGStage<T, B_KM, TILE> sb;
    if constexpr (SELECT) picked.place(m0, min(TILE, M - m0), row_list);
    sa.init(a.A, a.lda, m0, M, tid, rows_at);
    sb.init(a.B, a.ldb, n0, N, tid);
    const int frow = lane & 31, fhalf = lane >> 5;

    // the barrier waits for this wavefront's LDS accesses only, not for the loads in flight
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // plane pairs (of a, of b), smallest products first
    constexpr int PAIRS = PLANES == 3 ? 6 : 1;
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
    auto multiply = [&](int buf) {
        const unsigned char* la = lds[buf] + wm * WM * 512;
        const unsigned char* lb = lds[buf] + SIDE + wn * WN * 512;
        auto fragment = [&](const unsigned char* side, int p, int kk, int i) {   // of plane p, pieces 2 kk and 2 kk + 1
            const int at = ((2 * kk + fhalf) * TILE + (frow ^ gg_fold(2 * kk + fhalf))) * 16;
            return *reinterpret_cast<const bf16x8*>(side + p * PLANE + at + i * 512);
        };
        if constexpr (ACCS == 2) {   // the two halves of the K step alternate: neighbouring products are independent
            bf16x8 fa[2][PLANES], fb[2][PLANES];
#pragma unroll
            for (int p = PLANES - 1; p >= 0; --p)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    fa[kk][p] = fragment(la, p, kk, 0);
                    fb[kk][p] = fragment(lb, p, kk, 0);
                }
#pragma unroll
            for (int q = 0; q < PAIRS; ++q) {
                const int pa = PLANES == 3 ? PA[q] : 0, pb = PLANES == 3 ? PB[q] : 0;
                acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[0][pb], fa[0][pa], acc[0][0], 0, 0, 0);
                acc2[ACCS - 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[1][pb], fa[1][pa], acc2[ACCS - 1], 0, 0, 0);
            }
        } else {
            static_assert(BK == 16 || TILE == 64, "one K piece pair per step");
            bf16x8 fb[PLANES][WN];
#pragma unroll
            for (int p = 0; p < PLANES; ++p)
#pragma unroll
                for (int j = 0; j < WN; ++j) fb[p][j] = fragment(lb, p, 0, j);
            // IB rows of MFMA tiles at a time: few enough fragments of A to leave room for the sums
            constexpr int IB = TILE == 256 ? 2 : WM;
#pragma unroll
            for (int ib = 0; ib < WM; ib += IB) {
                bf16x8 fa[PLANES][IB];
#pragma unroll
                for (int p = 0; p < PLANES; ++p)
#pragma unroll
                    for (int i = 0; i < IB; ++i) fa[p][i] = fragment(la, p, 0, ib + i);
#pragma unroll
                for (int q = 0; q < PAIRS; ++q) {
                    const int pa = PLANES == 3 ? PA[q] : 0, pb = PLANES == 3 ? PB[q] : 0;
#pragma unroll
                    for (int i = 0; i < IB; ++i)
#pragma unroll
                        for (int j = 0; j < WN; ++j)
                            acc[ib + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[pb][j], fa[pa][i], acc[ib + i][j], 0, 0, 0);
                }
            }
        }
    };
    // The whole K steps.  Loads past the last one repeat it and are not used: no branch, so that
    // the waits for a step's loads leave the later ones in flight.
    auto run = [&](auto vec_) {
        constexpr bool V = decltype(vec_)::value;
        const int last = k_begin + (n_whole - 1) * BK;
        auto fetch = [&](auto d_, int t) {
            constexpr int D = decltype(d_)::value;
            const int k0 = min(k_begin + t * BK, last);
            sa.template load<D, V>(k0);
            sb.template load<D, V>(k0);
        };
        auto put = [&](auto d_, int buf) {
            constexpr int D = decltype(d_)::value;
            sa.template store<D>(lds[buf]);
            sb.template store<D>(lds[buf] + SIDE);
        };
        // step t, t % DEPTH = D: request step t + DEPTH, multiply step t, split step t + 1
        auto step = [&](auto d_, int t) {
            constexpr int D = decltype(d_)::value;
            barrier();
            fetch(d_, t + DEPTH);
            multiply(D & 1);
            put(std::integral_constant<int, (D + 1) % DEPTH>{}, (D + 1) & 1);
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2 % DEPTH>;
        using I3 = std::integral_constant<int, 3 % DEPTH>;
        fetch(I0{}, 0);
        fetch(I1{}, 1);
        if constexpr (DEPTH == 4) {
            fetch(I2{}, 2);
            fetch(I3{}, 3);
        }
        put(I0{}, 0);
        int t = 0;
        for (; t + DEPTH <= n_whole; t += DEPTH) {
            step(I0{}, t);
            step(I1{}, t + 1);
            if constexpr (DEPTH == 4) {
                step(I2{}, t + 2);
                step(I3{}, t + 3);
            }
        }
        if (t < n_whole) step(I0{}, t++);
        if constexpr (DEPTH == 4) {
            if (t < n_whole) step(I1{}, t++);
            if (t < n_whole) step(I2{}, t++);
        }
    };
    if (n_whole > 0) {
        if ((A_KM || a.vec_a) && (B_KM || a.vec_b)) run(std::true_type{}); else run(std::false_type{});
    }
    if (k_begin + n_whole * BK < k_end) {   // the cut step
        sa.template load_tail<0>(k_begin + n_whole * BK, k_end);
        sb.template load_tail<0>(k_begin + n_whole * BK, k_end);
        barrier();
        sa.template store<0>(lds[0]);
        sb.template store<0>(lds[0] + SIDE);
        barrier();
        multiply(0);
    }
    if constexpr (ACCS == 2) {
#pragma unroll
        for (int g = 0; g < 16; ++g) acc[0][0][g] += acc2[ACCS - 1][g];
    }

    // the B fragment is the MFMA's first operand: accumulator register g of lane l holds row
    // l % 32, column 8*(g/4) + 4*(l/32) + g%4 of its 32 x 32 tile
    OutT* C = static_cast<OutT*>(a.C) + (int64_t)split * a.split_stride;
    auto write = [&](int i, int j, const f32x16& sum, float scale) {   // MFMA tile (i, j) of the wavefront
        const int row = m0 + (wm * WM + i) * 32 + frow;
        if (row >= M) return;
        OutT* crow = C + (int64_t)row * a.ldc;
        const unsigned char* inrow =
            static_cast<const unsigned char*>(a.Cin) + (int64_t)row * a.ldcin * (a.cin_f32 ? 4 : (int)sizeof(OutT));
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            __builtin_amdgcn_sched_barrier(0);   // one store's addresses at a time
            const int col = n0 + (wn * WN + j) * 32 + 8 * g4 + 4 * fhalf;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = sum[4 * g4 + e] * scale;
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
    };
    unsigned again = 0;   // MFMA tiles to compute on the fp32 instructions
    if constexpr (PLANES == 3) {
        bool out = false;   // of the range: infinite or NaN
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int g = 0; g < 16; ++g) {
                    const float v = acc[i][j][g];
                    out |= !(v - v == 0.f);
                }
        if (__syncthreads_or(out)) {
            again = gg_needs_fp32<A_KM, B_KM, TILE, WM, WN>(a, m0, M, n0, N, k_begin, k_end, tid, wm, wn,
                                                            reinterpret_cast<unsigned*>(lds), rows_at);
            // one MFMA tile at a time: few registers and enough loads in flight (a rare path, off the other's
            // registers and instructions)
            constexpr int U = 16;   // K pairs in flight
            const float* A = static_cast<const float*>(a.A);
            const float* B = static_cast<const float*>(a.B);
#pragma unroll 1
            for (int ij = 0; ij < WM * WN; ++ij) {
                if (!(again >> ij & 1)) continue;
                const int i = ij / WN, j = ij % WN;
                int ra = min(m0 + (wm * WM + i) * 32 + frow, M - 1);
                if constexpr (SELECT) ra = row_list[ra - m0];
                const int rb = min(n0 + (wn * WN + j) * 32 + frow, N - 1);
                f32x16 sum;
#pragma unroll
                for (int g = 0; g < 16; ++g) sum[g] = 0.f;
#pragma unroll 1
                for (int k0 = k_begin; k0 < k_end; k0 += 2 * U) {
                    float va[U], vb[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) va[u] = gg_element<A_KM>(A, a.lda, ra, k0 + 2 * u + fhalf, k_end);
#pragma unroll
                    for (int u = 0; u < U; ++u) vb[u] = gg_element<B_KM>(B, a.ldb, rb, k0 + 2 * u + fhalf, k_end);
#pragma unroll
                    for (int u = 0; u < U; ++u) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(vb[u], va[u], sum, 0, 0, 0);
                }
                write(i, j, sum, 1.f);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
            if (!(again >> (i * WN + j) & 1)) write(i, j, acc[i][j], PLANES == 3 ? GG_UNSCALE : 1.f);
    return ProductTile{m0, n0, min(TILE, M - m0)};
}

template <typename T, typename OutT, bool A_KM, bool B_KM, int TILE, typename Fin = NoFinish, bool FEW = false>
__global__ __launch_bounds__(gg_threads(TILE), 2) void gemm_guarded(GGArgs a, Fin fin) {
    __shared__ __attribute__((aligned(16))) GGLds<T, TILE, FEW> lds;
    // SELECT: the tile's rows of A, and the wavefronts' counts
    __shared__ int row_list[IsSelect<Fin>::value ? TILE + gg_threads(TILE) / WAVE : 1];
    int block = (int)blockIdx.x;
    if constexpr (!std::is_same<Fin, NoFinish>::value) {
        if (block < fin.blocks) {
            if constexpr (IsSelect<Fin>::value) select_rows(fin, block, reinterpret_cast<int (*)[2]>(&lds));
            else finish_dx<OutT, 4>(fin, block, &lds);
            return;
        }
        block -= fin.blocks;
    }
    gg_product<T, OutT, A_KM, B_KM, TILE, Fin, FEW>(a, fin, block, lds, row_list);
}

// As grad_bf16, fp32 storage.
template <int TILE, bool CUT>
__global__ __launch_bounds__(gg_threads(TILE), 2) void grad_f32(GGArgs dx, GGArgs dw, GradArgs g) {
    __shared__ __attribute__((aligned(16))) GGLds<float, TILE> lds;
    int block = (int)blockIdx.x;
    if constexpr (!CUT) {
        if (block == 0 && g.fin.row_loss)
            loss_accumulate(g.fin.row_loss, g.fin.rows, g.fin.hdr, g.fin.loss, reinterpret_cast<double*>(&lds));
        if (block < FG_XCDS) return;
        block -= FG_XCDS;
    }
    block = block < g.dw_first ? block + g.dx_blocks : block - g.dw_first;
    if (block < g.dx_blocks) {
        const ProductTile t = gg_product<float, float, false, true, TILE, NoFinish, false>(dx, NoFinish{}, block, lds, nullptr);
        if (!CUT && t.rows > 0 && g.fin.idx) place_tile<float, TILE>(g.fin, t.m0, t.n0, t.rows);
    } else {
        gg_product<float, float, true, true, TILE, NoFinish, false>(dw, NoFinish{}, block - g.dx_blocks, lds, nullptr);
    }
}

}  // namespace flce
