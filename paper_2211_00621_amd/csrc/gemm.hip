// Dense nested map (map (reduce (+) 0 (map2 (*) row col))): FP32 matrix
// product on the CDNA matrix cores (v_mfma_f32_16x16x4_f32), FP32 accumulate.
//
// Three kernels, chosen by a cost model over tile shapes (gemm_choice below):
//  * pipelined: 128 x 128 tiles of 16 waves, for aligned sizes that are whole
//    tiles;
//  * split: 64 x 32 .. 128 x 128 tiles of any size and alignment, the K slices
//    dealt to groups of waves;
//  * direct: 16 x 16 or 32 x 32 tiles read straight from memory by waves that
//    split K, where latency counts.
// The first two walk K in slices of 32, each operand slice staged in LDS in the
// orientation it has in memory -- [row][k] (32-float rows, 16-byte quads
// swizzled by row) when k is contiguous, [k][row] when rows are contiguous --
// so every global load is a 16-byte vector and every LDS store a 16-byte
// store.
//
// Fragments.  MFMA step s of a slice takes k = 8g + s in lane group
// g = lane / 16 (the reduction over k is associative, so any fixed dealing of
// the 32 k values over steps and lane groups is valid), and every operand is
// read from LDS in vectors:
//  * [row][k] operand: lane (g, l16) needs the 8 consecutive k values 8g..8g+7
//    of one row per 16-row block -- two 16-byte reads per block per slice;
//  * [k][row] operand with R 16-row blocks per wave: at step s the lane reads
//    rows R*l16 .. R*l16 + R-1 of LDS row k = 8g + s in one 8- or 16-byte
//    read, and value c feeds the MFMA of block c.  Block c thus covers the
//    interleaved rows R*rho + c of the wave's tile (rho = 0..15), which the
//    epilogue maps back; for C's columns this makes each lane's R outputs
//    contiguous, so they are stored as one vector.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "mx_internal.h"

namespace mx {
namespace {

constexpr int BK = 32;
// [row][k] slices: rows of BK = 32 floats (eight 16-byte quads) with the quad
// position swizzled by the row, quad q of row r at q ^ ((r >> 1) & 7): the
// 16-byte stores of two consecutive rows and the reads of quads 2g, 2g + 1 by
// 16 consecutive rows then fall on distinct banks.
__device__ __forceinline__ int swz(int row, int quad) { return row * BK + 4 * (quad ^ ((row >> 1) & 7)); }
constexpr int kGroupM = 4;   // tile rows per scheduling group

typedef float v4f __attribute__((ext_vector_type(4)));

template <int ROWS, bool ROWK> struct Operand {
    static constexpr int LD = ROWK ? BK : ROWS;  // LDS stride in floats
    static constexpr int FLOATS = ROWS * BK;
};

// [k][row] slices: k rows of ROWS floats, unpadded, the 16-byte group q of
// row k at q ^ (8 (k >> 3 & 1)), so the k rows 8 apart that lane groups g and
// g + 1 read in one pass land 32 banks apart.  (Rows padded to ROWS + 4
// floats did the same for the reads; with this layout A^T dC, whose operands
// are both [k][row], runs as fast as the other transposes, 134 against 139 us
// at 2048^3.)
template <int ROWS> __device__ __forceinline__ int kswz(int k, int row) {
    static_assert(ROWS >= 64, "the swizzle moves groups by 8 of at least 16 per row");
    return k * ROWS + 4 * ((row >> 2) ^ (((k >> 3) & 1) << 3)) + (row & 3);
}

// One K-slice of an operand (ROWS rows) into registers, NT threads.
template <int ROWS, bool ROWK, int NT>
__device__ __forceinline__ void load_slice(float4 (&r)[ROWS * BK / 4 / NT], const float *__restrict__ p,
                                           int64_t ld, int64_t row0, int64_t k0) {
#pragma unroll
    for (int i = 0; i < ROWS * BK / 4 / NT; ++i) {
        const int idx = threadIdx.x + NT * i;
        if constexpr (ROWK) {
            const int row = idx >> 3, kq = idx & 7;  // rows x 8 quads of k
            r[i] = *reinterpret_cast<const float4 *>(p + (row0 + row) * ld + k0 + 4 * kq);
        } else {
            constexpr int Q = ROWS / 4;  // quads of rows per k
            const int k = idx / Q, rq = idx % Q;
            r[i] = *reinterpret_cast<const float4 *>(p + (k0 + k) * ld + row0 + 4 * rq);
        }
    }
}

template <int ROWS, bool ROWK, int NT>
__device__ __forceinline__ void store_slice(float *__restrict__ s, const float4 (&r)[ROWS * BK / 4 / NT]) {
#pragma unroll
    for (int i = 0; i < ROWS * BK / 4 / NT; ++i) {
        const int idx = threadIdx.x + NT * i;
        if constexpr (ROWK) {
            const int row = idx >> 3, kq = idx & 7;
            *reinterpret_cast<float4 *>(s + swz(row, kq)) = r[i];
        } else {
            constexpr int Q = ROWS / 4;
            const int k = idx / Q, rq = idx % Q;
            *reinterpret_cast<float4 *>(s + kswz<ROWS>(k, 4 * rq)) = r[i];
        }
    }
}

template <int R> struct VecOf;
template <> struct VecOf<1> { using T = float; };
template <> struct VecOf<2> { using T = float2; };
template <> struct VecOf<4> { using T = float4; };

// R consecutive floats from LDS (16-byte aligned for R = 4, 8-byte for R = 2)
template <int R> __device__ __forceinline__ void lds_read(float (&v)[R], const float *p) {
    const typename VecOf<R>::T t = *reinterpret_cast<const typename VecOf<R>::T *>(p);
    __builtin_memcpy(v, &t, sizeof t);
}

// Tile scheduling: consecutive blocks land on different XCDs (round robin over
// 8), so blocks b, b+8, b+16, ... share an L2.  Give each XCD a contiguous
// range of logical tiles, and walk logical tiles in groups of kGroupM tile rows
// so that neighbouring tiles reuse the same A row panels and B column panels.
// Blocks come in rows of 2^20 (a grid's threads in x stay below 2^32); false
// for the surplus ones of the last row.
constexpr int kGridRowBits = 20;
__device__ __forceinline__ bool tile_of(int tiles_m, int tiles_n, int &tm, int &tn) {
    const int nt = tiles_m * tiles_n, b = (int)(blockIdx.y << kGridRowBits | blockIdx.x);
    if (b >= nt) return false;
    // XCD x takes nt / 8 tiles, one more where x < nt % 8
    const int x = b & 7, rem = nt & 7;
    const int L = x * (nt >> 3) + (x < rem ? x : rem) + (b >> 3);
    const int per_group = kGroupM * tiles_n;
    const int gi = L / per_group;
    const int first_m = gi * kGroupM;
    const int gm = min(tiles_m - first_m, kGroupM);
    const int in = L - gi * per_group;
    tm = first_m + in % gm;
    tn = in / gm;
    return true;
}

// The wave's operand fragments of one K slice held in LDS: fa[s][i] is the
// value lane (g, l16) feeds MFMA step s of row block i, fb[s][j] that of column
// block j.
template <int BM, int BN, int WM, int WN, bool RA, bool RB>
__device__ __forceinline__ void read_frags(float (&fa)[8][BM / WM / 16], float (&fb)[8][BN / WN / 16],
                                           const float *__restrict__ as, const float *__restrict__ bs, int wrow0,
                                           int wcol0, int l16, int g) {
    constexpr int MI = BM / WM / 16, NI = BN / WN / 16;
    if constexpr (RA) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int row = wrow0 + 16 * i + l16;
            const float4 lo = *reinterpret_cast<const float4 *>(as + swz(row, 2 * g));
            const float4 hi = *reinterpret_cast<const float4 *>(as + swz(row, 2 * g + 1));
            fa[0][i] = lo.x; fa[1][i] = lo.y; fa[2][i] = lo.z; fa[3][i] = lo.w;
            fa[4][i] = hi.x; fa[5][i] = hi.y; fa[6][i] = hi.z; fa[7][i] = hi.w;
        }
    } else {
#pragma unroll
        for (int s = 0; s < 8; ++s) lds_read<MI>(fa[s], as + kswz<BM>(8 * g + s, wrow0 + MI * l16));
    }
    if constexpr (RB) {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int row = wcol0 + 16 * j + l16;
            const float4 lo = *reinterpret_cast<const float4 *>(bs + swz(row, 2 * g));
            const float4 hi = *reinterpret_cast<const float4 *>(bs + swz(row, 2 * g + 1));
            fb[0][j] = lo.x; fb[1][j] = lo.y; fb[2][j] = lo.z; fb[3][j] = lo.w;
            fb[4][j] = hi.x; fb[5][j] = hi.y; fb[6][j] = hi.z; fb[7][j] = hi.w;
        }
    } else {
#pragma unroll
        for (int s = 0; s < 8; ++s) lds_read<NI>(fb[s], bs + kswz<BN>(8 * g + s, wcol0 + NI * l16));
    }
}

// MFMA work of one K slice from its fragments: the wave's MI x NI blocks of 16 x 16
template <int MI, int NI>
__device__ __forceinline__ void mma_frags(v4f (&acc)[MI][NI], const float (&fa)[8][MI], const float (&fb)[8][NI]) {
#pragma unroll
    for (int step = 0; step < 8; ++step)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[step][i], fb[step][j], acc[i][j], 0, 0, 0);
}

// ---------------------------------------------------------------- pipelined
// Whole tiles only: M and N multiples of the tile, K a multiple of 64 of at
// least 128, A and B on 16-byte boundaries.
template <int BM, int BN, int WM, int WN, int TA, int TB>
__global__ void __launch_bounds__(64 * WM * WN) k_gemm_mfma(const float *__restrict__ A, const float *__restrict__ B,
                                                            float *__restrict__ C, int64_t M, int64_t N, int64_t K,
                                                            int tiles_m, int tiles_n, int cvec) {
    constexpr int NT = 64 * WM * WN;
    static_assert((BM * BK / 4) % NT == 0 && (BN * BK / 4) % NT == 0, "slice loads must split evenly");
    static_assert(BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "wave tiles are whole 16 x 16 blocks");
    constexpr bool RA = !TA, RB = TB;  // [row][k] in memory
    constexpr int MI = BM / WM / 16, NI = BN / WN / 16;
    static_assert(RA || MI == 1 || MI == 2 || MI == 4, "[k][row] A: reads of 1, 2 or 4 rows");
    static_assert(RB || NI == 1 || NI == 2 || NI == 4, "[k][row] B: reads of 1, 2 or 4 columns");
    using OA = Operand<BM, RA>;
    using OB = Operand<BN, RB>;
    __shared__ __attribute__((aligned(16))) float As0[OA::FLOATS], As1[OA::FLOATS];
    __shared__ __attribute__((aligned(16))) float Bs0[OB::FLOATS], Bs1[OB::FLOATS];
    auto As = [&](int i) { return i ? As1 : As0; };
    auto Bs = [&](int i) { return i ? Bs1 : Bs0; };

    int tm, tn;
    if (!tile_of(tiles_m, tiles_n, tm, tn)) return;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t lda = TA ? M : K;
    const int64_t ldb = TB ? K : N;
    const int nk = (int)(K / BK);

    v4f acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    const int wrow0 = wm * (BM / WM), wcol0 = wn * (BN / WN);
    constexpr int NA = BM * BK / 4 / NT, NB = BN * BK / 4 / NT;
    {
        // An even number (at least four) of whole slices.  Iteration kt multiplies slice kt from fragments already in registers
        // while the fragments of slice kt + 1 are read from LDS, then stores
        // slice kt + 2 (loaded two iterations earlier) into the buffer slice kt
        // occupied and issues the global loads of slice kt + 4; one barrier.
        // The fragment reads are in flight across the MFMAs and the barrier,
        // so no wave waits on LDS latency between slices.  The last four
        // iterations are peeled: nothing is loaded past the end of K.
        float4 ga[NA], gb[NB], ha[NA], hb[NB];  // staging of two slices in flight
        float fa0[8][MI], fb0[8][NI], fa1[8][MI], fb1[8][NI];
        load_slice<BM, RA, NT>(ga, A, lda, m0, 0);
        load_slice<BN, RB, NT>(gb, B, ldb, n0, 0);
        load_slice<BM, RA, NT>(ha, A, lda, m0, BK);
        load_slice<BN, RB, NT>(hb, B, ldb, n0, BK);
        store_slice<BM, RA, NT>(As(0), ga);
        store_slice<BN, RB, NT>(Bs(0), gb);
        load_slice<BM, RA, NT>(ga, A, lda, m0, 2 * BK);
        load_slice<BN, RB, NT>(gb, B, ldb, n0, 2 * BK);
        __syncthreads();
        read_frags<BM, BN, WM, WN, RA, RB>(fa0, fb0, As(0), Bs(0), wrow0, wcol0, l16, g);
        store_slice<BM, RA, NT>(As(1), ha);
        store_slice<BN, RB, NT>(Bs(1), hb);
        load_slice<BM, RA, NT>(ha, A, lda, m0, 3 * BK);
        load_slice<BN, RB, NT>(hb, B, ldb, n0, 3 * BK);
        __syncthreads();
        // one iteration; buffer (kt + 1) & 1 holds slice kt + 1, buffer kt & 1
        // is free once slice kt's fragments are in registers
#define MX_GEMM_ITER(KT, FA, FB, NFA, NFB, SA, SB, DO_R, DO_S, DO_L)                                      \
        {                                                                                                 \
            const int b1 = ((KT) + 1) & 1, b0 = (KT) & 1;                                                 \
            if (DO_R) read_frags<BM, BN, WM, WN, RA, RB>(NFA, NFB, As(b1), Bs(b1), wrow0, wcol0, l16, g); \
            __builtin_amdgcn_sched_barrier(0);                                                            \
            mma_frags(acc, FA, FB);                                                                       \
            __builtin_amdgcn_sched_barrier(0);                                                            \
            if (DO_S) {                                                                                   \
                store_slice<BM, RA, NT>(As(b0), SA);                                                      \
                store_slice<BN, RB, NT>(Bs(b0), SB);                                                      \
            }                                                                                             \
            if (DO_L) {                                                                                   \
                const int64_t kl = (int64_t)((KT) + 4) * BK;                                              \
                load_slice<BM, RA, NT>(SA, A, lda, m0, kl);                                   \
                load_slice<BN, RB, NT>(SB, B, ldb, n0, kl);                                   \
            }                                                                                             \
            if (DO_S) __syncthreads();                                                                    \
        }
        int kt = 0;
        for (; kt + 4 < nk; kt += 2) {
            MX_GEMM_ITER(kt, fa0, fb0, fa1, fb1, ga, gb, true, true, true)
            MX_GEMM_ITER(kt + 1, fa1, fb1, fa0, fb0, ha, hb, true, true, true)
        }
        MX_GEMM_ITER(kt, fa0, fb0, fa1, fb1, ga, gb, true, true, false)
        MX_GEMM_ITER(kt + 1, fa1, fb1, fa0, fb0, ha, hb, true, true, false)
        MX_GEMM_ITER(kt + 2, fa0, fb0, fa1, fb1, ga, gb, true, false, false)
        MX_GEMM_ITER(kt + 3, fa1, fb1, fa0, fb0, ha, hb, false, false, false)
#undef MX_GEMM_ITER
    }

    // D block (i, j): lane holds block rows rho = 4g .. 4g+3 of block column
    // l16; blocked or interleaved as the operand layout dealt them
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rho = 4 * g + r;
            const int64_t row = m0 + wrow0 + (RA ? 16 * i + rho : MI * rho + i);
            if constexpr (!RB) {
                // the lane's NI columns NI*l16 .. NI*l16 + NI-1 are contiguous
                const int64_t col = n0 + wcol0 + NI * l16;
                if (cvec) {
                    float v[NI];
#pragma unroll
                    for (int j = 0; j < NI; ++j) v[j] = acc[i][j][r];
                    typename VecOf<NI>::T t;
                    __builtin_memcpy(&t, v, sizeof t);
                    *reinterpret_cast<typename VecOf<NI>::T *>(C + row * N + col) = t;
                } else {
#pragma unroll
                    for (int j = 0; j < NI; ++j) C[row * N + col + j] = acc[i][j][r];
                }
            } else {
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const int64_t col = n0 + wcol0 + 16 * j + l16;
                    C[row * N + col] = acc[i][j][r];
                }
            }
        }
    }
}

// ---------------------------------------------------------------- direct
// Small products, where latency counts: no LDS staging.  A block owns a
// (16 MI) x (16 NI) tile; its KS waves each take every KS-th slice of K, read
// their fragments straight from memory, one slice ahead, and their sums are
// added in wave order through LDS.
//
// Every size and alignment takes the same loads, vectors at 4-byte alignment:
// the last slice, and only it, is read element by element with clamped indices
// and zeros past K; before it a vector of consecutive rows may run past the
// matrix's edge into the next k (never past its end: with fewer than four rows
// MI, NI are 1), where it only reaches elements of C that are not stored.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));

template <int R, bool ROWK> struct Frag {
    // lane (g, l16) at slice k0: f[s][i] feeds MFMA step s (k = k0 + 8 g + s) of
    // block i: row 16 i + l16 (ROWK) or R l16 + i of the tile
    float f[8][R];
    const float *p[ROWK ? R : 1];  // ROWK: row starts; else column start
    int64_t ld;
    int rows_left;  // !ROWK: rows of the matrix from this lane's first on
    __device__ __forceinline__ void init(const float *base, int64_t ld_, int64_t row0, int64_t rows, int l16) {
        ld = ld_;
        if constexpr (ROWK) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int64_t r = row0 + 16 * i + l16;
                p[i] = base + (r < rows ? r : rows - 1) * ld_;
            }
        } else {
            int64_t r = row0 + R * l16;
            if (r >= rows) r = 0;  // a lane past the edge: any rows do
            p[0] = base + r;
            rows_left = rows - r < R ? (int)(rows - r) : R;
        }
    }
    __device__ __forceinline__ void load(int64_t k0, int g) {
        if constexpr (ROWK) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const f4u *q = reinterpret_cast<const f4u *>(p[i] + k0 + 8 * g);
                const f4u lo = q[0], hi = q[1];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    f[e][i] = lo[e];
                    f[4 + e][i] = hi[e];
                }
            }
        } else {
            const float *q = p[0] + (k0 + 8 * g) * ld;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if constexpr (R == 4) {
                    const f4u v = *reinterpret_cast<const f4u *>(q + s * ld);
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[s][e] = v[e];
                } else if constexpr (R == 2) {
                    const f2u v = *reinterpret_cast<const f2u *>(q + s * ld);
                    f[s][0] = v[0];
                    f[s][1] = v[1];
                } else {
                    f[s][0] = q[s * ld];
                }
            }
        }
    }
    __device__ __forceinline__ void load_last(int64_t k0, int64_t K, int g) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int64_t k = k0 + 8 * g + s, kc = k < K ? k : K - 1;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                float v;
                if constexpr (ROWK) v = p[i][kc];
                else v = p[0][kc * ld + (i < rows_left ? i : rows_left - 1)];
                f[s][i] = k < K ? v : 0.f;
            }
        }
    }
};

template <int MI, int NI, int KS, int TA, int TB>
__global__ void __launch_bounds__(64 * KS) k_gemm_direct(const float *__restrict__ A, const float *__restrict__ B,
                                                         float *__restrict__ C, int64_t M, int64_t N, int64_t K,
                                                         int tiles_m, int tiles_n) {
    constexpr bool RA = !TA, RB = TB;
    __shared__ float4 red[KS * MI * NI * 64];
    int tm, tn;
    if (!tile_of(tiles_m, tiles_n, tm, tn)) return;
    const int lane = threadIdx.x & 63;
    const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t m0 = (int64_t)tm * (16 * MI), n0 = (int64_t)tn * (16 * NI);
    v4f acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    if (K > 0) {
        Frag<MI, RA> fa, na;
        Frag<NI, RB> fb, nb;
        fa.init(A, TA ? M : K, m0, M, l16);
        fb.init(B, TB ? K : N, n0, N, l16);
        const int last = (int)((K - 1) / BK);  // the last slice's index; `last` whole ones before it
        na = fa;
        nb = fb;
        int t = ks;
        if (t < last) {
            fa.load((int64_t)t * BK, g);
            fb.load((int64_t)t * BK, g);
            for (; t + KS < last; t += KS) {
                na.load((int64_t)(t + KS) * BK, g);
                nb.load((int64_t)(t + KS) * BK, g);
                __builtin_amdgcn_sched_barrier(0);
                mma_frags(acc, fa.f, fb.f);
                __builtin_memcpy(fa.f, na.f, sizeof fa.f);
                __builtin_memcpy(fb.f, nb.f, sizeof fb.f);
            }
            mma_frags(acc, fa.f, fb.f);
            t += KS;
        }
        if (t == last) {
            fa.load_last((int64_t)t * BK, K, g);
            fb.load_last((int64_t)t * BK, K, g);
            mma_frags(acc, fa.f, fb.f);
        }
    }
    // the waves' sums, added in wave order; each wave adds and stores its share
    // of the blocks
#pragma unroll
    for (int b = 0; b < MI * NI; ++b) {
        const v4f v = acc[b / NI][b % NI];
        red[(ks * MI * NI + b) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
    }
    __syncthreads();
    for (int b = ks; b < MI * NI; b += KS) {
        const int i = b / NI, j = b % NI;
        const float4 f = red[b * 64 + lane];
        v4f v = v4f{f.x, f.y, f.z, f.w};
#pragma unroll
        for (int o = 1; o < KS; ++o) {
            const float4 q = red[(o * MI * NI + b) * 64 + lane];
            v += v4f{q.x, q.y, q.z, q.w};
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rho = 4 * g + r;
            const int64_t row = m0 + (RA ? 16 * i + rho : MI * rho + i);
            const int64_t col = n0 + (RB ? 16 * j + l16 : NI * l16 + j);
            if (row < M && col < N) C[row * N + col] = v[r];
        }
    }
}

// ---------------------------------------------------------------- split tiles
// Products whose 128 x 128 tiles leave CUs idle: a smaller tile per block,
// chosen so that the tiles come out just below a multiple of the CUs, and its
// K slices dealt to KG groups of WM x WN waves (group q takes slices q, q + KG,
// ...), each group with LDS buffers of its own, so that a CU has four waves per
// SIMD on one tile and a group's next slice has a whole round of all groups to
// arrive.  The groups' sums are added in group order through LDS.
//
// Every size and alignment takes the same loads: 16-byte vectors at 4-byte
// alignment, rows past the edge clamped; the last round alone reads element by
// element with clamped indices and zeros past K (before it, a vector of
// consecutive rows may run past the matrix's edge into the next k, where it
// only reaches elements of C that are not stored).
template <int ROWS, bool ROWK> struct Slice {
    static constexpr int LD = ROWK ? BK : ROWS + 4;  // [k][row]: lane groups 8 k rows apart read other banks
    static constexpr int FLOATS = ROWK ? ROWS * BK : LD * BK;
    static constexpr int QUADS = ROWS * BK / 4;
    static __device__ __forceinline__ int at(int row, int k) {
        if constexpr (ROWK) return swz(row, k >> 2) + (k & 3);
        else return k * LD + row;
    }
};

// A group's staging of one operand: NT threads, quads idx = t + NT i.
template <int ROWS, bool ROWK, int NT> struct Stage {
    using S = Slice<ROWS, ROWK>;
    static constexpr int N = (S::QUADS + NT - 1) / NT;
    float4 r[N];
    static __device__ __forceinline__ int quad(int t, int i) {
        const int q = t + NT * i;
        return S::QUADS % NT == 0 || q < S::QUADS ? q : S::QUADS - 1;  // surplus threads repeat the last quad
    }
    __device__ __forceinline__ void load(const float *__restrict__ p, int64_t ld, int64_t row0, int64_t rows,
                                         int64_t k0, int t) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int q = quad(t, i);
            const float *a;
            if constexpr (ROWK) {
                const int64_t row = row0 + (q >> 3);
                a = p + (row < rows ? row : rows - 1) * ld + k0 + 4 * (q & 7);
            } else {
                const int64_t row = row0 + 4 * (q % (ROWS / 4));
                a = p + (k0 + q / (ROWS / 4)) * ld + (row < rows ? row : 0);
            }
            const f4u v = *reinterpret_cast<const f4u *>(a);
            r[i] = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
    __device__ __forceinline__ void load_last(const float *__restrict__ p, int64_t ld, int64_t row0, int64_t rows,
                                              int64_t k0, int64_t K, int t) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int q = quad(t, i);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int64_t row, k;
                if constexpr (ROWK) {
                    row = row0 + (q >> 3);
                    k = k0 + 4 * (q & 7) + e;
                } else {
                    row = row0 + 4 * (q % (ROWS / 4)) + e;
                    k = k0 + q / (ROWS / 4);
                }
                const int64_t rc = row < rows ? row : rows - 1, kc = k < K ? k : K - 1;
                const float x = ROWK ? p[rc * ld + kc] : p[kc * ld + rc];
                v[e] = k < K ? x : 0.f;
            }
            r[i] = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
    __device__ __forceinline__ void store(float *s, int t) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int q = quad(t, i);
            float *d = ROWK ? s + S::at(q >> 3, 4 * (q & 7)) : s + S::at(4 * (q % (ROWS / 4)), q / (ROWS / 4));
            *reinterpret_cast<float4 *>(d) = r[i];
        }
    }
};

// rows of block i of a wave's R blocks: interleaved (R rho + i) where a lane
// reads its R rows as one vector, else 16 i + rho
template <bool ROWK, int R> constexpr bool kDealt = !ROWK && (R == 1 || R == 2 || R == 4);

template <int ROWS, bool ROWK, int R>
__device__ __forceinline__ void slice_frags(float (&f)[8][R], const float *__restrict__ s, int row0, int l16, int g) {
    using S = Slice<ROWS, ROWK>;
    if constexpr (ROWK) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int row = row0 + 16 * i + l16;
            const float4 lo = *reinterpret_cast<const float4 *>(s + S::at(row, 8 * g));
            const float4 hi = *reinterpret_cast<const float4 *>(s + S::at(row, 8 * g + 4));
            f[0][i] = lo.x; f[1][i] = lo.y; f[2][i] = lo.z; f[3][i] = lo.w;
            f[4][i] = hi.x; f[5][i] = hi.y; f[6][i] = hi.z; f[7][i] = hi.w;
        }
    } else if constexpr (kDealt<ROWK, R>) {
#pragma unroll
        for (int e = 0; e < 8; ++e) lds_read<R>(f[e], s + S::at(row0 + R * l16, 8 * g + e));
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < R; ++i) f[e][i] = s[S::at(row0 + 16 * i + l16, 8 * g + e)];
    }
}

template <int MI, int NI, int WM, int WN, int KG, int TA, int TB>
__global__ void __launch_bounds__(64 * WM * WN * KG) k_gemm_split(const float *__restrict__ A,
                                                                  const float *__restrict__ B,
                                                                  float *__restrict__ C, int64_t M, int64_t N,
                                                                  int64_t K, int tiles_m, int tiles_n) {
    constexpr bool RA = !TA, RB = TB;
    constexpr int BM = 16 * MI * WM, BN = 16 * NI * WN, NW = WM * WN, NT = 64 * NW;
    using SA = Slice<BM, RA>;
    using SB = Slice<BN, RB>;
    constexpr int BUF = SA::FLOATS + SB::FLOATS;
    constexpr int SUM = KG > 1 ? KG * NW * MI * NI * 256 : 0;  // floats of the groups' sums
    constexpr int LDSF = 2 * KG * BUF > SUM ? 2 * KG * BUF : SUM;
    __shared__ __attribute__((aligned(16))) float lds[LDSF];
    int tm, tn;
    if (!tile_of(tiles_m, tiles_n, tm, tn)) return;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave / NW, wt = wave % NW, wm = wt / WN, wn = wt % WN;
    const int t = threadIdx.x - grp * NT;
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t lda = TA ? M : K, ldb = TB ? K : N;
    float *const buf = lds + grp * 2 * BUF;
    v4f acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    const int last = (int)((K - 1) / BK);  // the last slice; whole, safe ones before it
    const int rounds = last / KG;          // rounds in which every group has a safe slice; one more follows
    Stage<BM, RA, NT> sa;
    Stage<BN, RB, NT> sb;
    auto fetch = [&](int r) {
        const int64_t k0 = (int64_t)(r * KG + grp) * BK;
        sa.load(A, lda, m0, M, k0, t);
        sb.load(B, ldb, n0, N, k0, t);
    };
    auto fetch_last = [&]() {
        const int sl = rounds * KG + grp;
        if (sl > last) return;
        const int64_t k0 = (int64_t)sl * BK;
        if (sl < last) {
            sa.load(A, lda, m0, M, k0, t);
            sb.load(B, ldb, n0, N, k0, t);
        } else {
            sa.load_last(A, lda, m0, M, k0, K, t);
            sb.load_last(B, ldb, n0, N, k0, K, t);
        }
    };
    auto put = [&](int b) {
        sa.store(buf + b * BUF, t);
        sb.store(buf + b * BUF + SA::FLOATS, t);
    };
    auto multiply = [&](int b) {
        float fa[8][MI], fb[8][NI];
        slice_frags<BM, RA, MI>(fa, buf + b * BUF, wm * 16 * MI, l16, g);
        slice_frags<BN, RB, NI>(fb, buf + b * BUF + SA::FLOATS, wn * 16 * NI, l16, g);
        mma_frags(acc, fa, fb);
    };
    if (rounds > 0) {
        fetch(0);
        put(0);
        __syncthreads();
        for (int r = 0; r + 1 < rounds; ++r) {
            fetch(r + 1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(r & 1);
            put((r + 1) & 1);
            __syncthreads();
        }
        fetch_last();
        multiply((rounds - 1) & 1);
    } else {
        fetch_last();
    }
    put(rounds & 1);
    __syncthreads();
    if (rounds * KG + grp <= last) multiply(rounds & 1);

    int b_lo = 0, b_hi = MI * NI;  // the blocks of the wave's tile this group stores
    if constexpr (KG > 1) {
        __syncthreads();  // the buffers are read no more
        float4 *red = reinterpret_cast<float4 *>(lds);
#pragma unroll
        for (int b = 0; b < MI * NI; ++b) {
            const v4f v = acc[b / NI][b % NI];
            red[(wave * MI * NI + b) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
        }
        __syncthreads();
        b_lo = grp * MI * NI / KG;
        b_hi = (grp + 1) * MI * NI / KG;
    }
#pragma unroll
    for (int b = 0; b < MI * NI; ++b) {
        if (KG > 1 && (b < b_lo || b >= b_hi)) continue;
        const int i = b / NI, j = b % NI;
        v4f v = acc[i][j];
        if constexpr (KG > 1) {
            const float4 *red = reinterpret_cast<const float4 *>(lds) + (wt * MI * NI + b) * 64 + lane;
#pragma unroll
            for (int o = 0; o < KG; ++o) {
                const float4 q = red[o * NW * MI * NI * 64];
                if (o == 0) v = v4f{q.x, q.y, q.z, q.w};
                else v += v4f{q.x, q.y, q.z, q.w};
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rho = 4 * g + r;
            const int64_t row = m0 + wm * 16 * MI + (kDealt<RA, MI> ? MI * rho + i : 16 * i + rho);
            const int64_t col = n0 + wn * 16 * NI + (kDealt<RB, NI> ? NI * l16 + j : 16 * j + l16);
            if (row < M && col < N) C[row * N + col] = v[r];
        }
    }
}

// Plain form: one thread per output element, k loop over global memory.
template <int TA, int TB>
__global__ void __launch_bounds__(256) k_gemm_plain(const float *__restrict__ A,
                                                    const float *__restrict__ B,
                                                    float *__restrict__ C, int64_t M, int64_t N,
                                                    int64_t K) {
    const int64_t j = (int64_t)blockIdx.x * 16 + (threadIdx.x & 15);
    const int64_t i = (int64_t)blockIdx.y * 16 + (threadIdx.x >> 4);
    if (i >= M || j >= N) return;
    float acc = 0.f;
    for (int64_t k = 0; k < K; ++k) {
        const float a = TA ? A[k * M + i] : A[i * K + k];
        const float b = TB ? B[j * K + k] : B[k * N + j];
        acc += a * b;
    }
    C[i * N + j] = acc;
}

mx_status check(const char *who, int ta, int tb, int64_t M, int64_t N, int64_t K, const float *A,
                const float *B, float *C) {
    MX_REQUIRE((ta == 0 || ta == 1) && (tb == 0 || tb == 1), MX_ERR_INVALID, "%s: ta, tb must be 0 or 1", who);
    MX_REQUIRE(M >= 0 && N >= 0 && K >= 0, MX_ERR_SHAPE, "%s: negative size", who);
    MX_REQUIRE(M == 0 || N == 0 || C, MX_ERR_INVALID, "%s: null C", who);
    MX_REQUIRE(M == 0 || N == 0 || K == 0 || (A && B), MX_ERR_INVALID, "%s: null A or B", who);
    MX_REQUIRE(M < (1LL << 31) && N < (1LL << 31), MX_ERR_SHAPE, "%s: M, N must be below 2^31", who);
    return MX_OK;
}

// ---------------------------------------------------------------- dispatch
struct GemmArgs {
    int ta, tb;
    int64_t M, N, K;
    const float *A, *B;
    float *C;
    hipStream_t s;
    int64_t num_cus;
};

#define MX_GEMM_LAUNCH(BM, BN, THREADS, KERNEL, ...)                                                              \
    const int64_t tiles_m = ceil_div(a.M, BM), tiles_n = ceil_div(a.N, BN);                                       \
    MX_REQUIRE(tiles_m * tiles_n < (1LL << 31), MX_ERR_SHAPE, "mx_map_map_reduce_f32: too many tiles");           \
    const int64_t tiles = tiles_m * tiles_n, per_row = 1 << kGridRowBits;                                         \
    const dim3 grid((unsigned)std::min(tiles, per_row), (unsigned)ceil_div(tiles, per_row)), block(THREADS);      \
    auto go = [&](auto kernel) {                                                                                  \
        hipLaunchKernelGGL(kernel, grid, block, 0, a.s, a.A, a.B, a.C, a.M, a.N, a.K, (int)tiles_m, (int)tiles_n __VA_ARGS__); \
    };                                                                                                            \
    if (!a.ta && !a.tb) go(KERNEL<SHAPE, 0, 0>);                                                                  \
    else if (!a.ta) go(KERNEL<SHAPE, 0, 1>);                                                                      \
    else if (!a.tb) go(KERNEL<SHAPE, 1, 0>);                                                                      \
    else go(KERNEL<SHAPE, 1, 1>);                                                                                 \
    return last_launch("mx_map_map_reduce_f32")

mx_status launch_pipelined(const GemmArgs &a) {
#define SHAPE 128, 128, 4, 4
    const int cvec = ((uintptr_t)a.C % 16 == 0) && (a.N % 4 == 0);
    MX_GEMM_LAUNCH(128, 128, 1024, k_gemm_mfma, , cvec);
#undef SHAPE
}
template <int MI, int NI, int WM, int WN, int KG> mx_status launch_split(const GemmArgs &a) {
#define SHAPE MI, NI, WM, WN, KG
    MX_GEMM_LAUNCH(16 * MI * WM, 16 * NI * WN, 64 * WM * WN * KG, k_gemm_split);
#undef SHAPE
}
// Past three rounds of blocks no wave without a slice of K: 10^6 x 1 x 32 took
// 167 us with eight waves a tile, 63 us with one.  Of more than two slices that holds
// where both operands' rows run along K (787 343 x 1 x 93, B transposed, 94 us with
// eight waves, 64 us with four); elsewhere a tile's rows lie far apart, and the idle
// waves keep fewer tiles open at once (A transposed 105 us with eight, 175 us with
// four).  In fewer rounds the idle waves cost nothing, and their instruction fetches
// serve the one that works (1000 x 8 x 64 2.6 us with eight, 3.3 us with two).
template <int MI, int NI, int KS> mx_status launch_direct(const GemmArgs &a) {
    if constexpr (KS > 1)
        if (a.K <= (!a.ta && a.tb ? KS / 2 : std::min(KS / 2, 2)) * BK &&
            ceil_div(a.M, 16 * MI) * ceil_div(a.N, 16 * NI) > 3 * a.num_cus)
            return launch_direct<MI, NI, KS / 2>(a);
#define SHAPE MI, NI, KS
    MX_GEMM_LAUNCH(16 * MI, 16 * NI, 64 * KS, k_gemm_direct);
#undef SHAPE
}
#undef MX_GEMM_LAUNCH

// The tile shapes and what they cost, in us: a product takes about
//   2 + rounds (fixed + per_k K / 1000),  rounds = tiles / CUs rounded up
// (fitted to products of 64 .. 2048 a side, all transposes; 157.3 TFLOP/s are
// 3.3 us per 32 x 32 tile, 13 per 64 x 64 and 53 per 128 x 128 at K = 1000).
// A larger tile reuses more, a smaller one wastes less of the last round: at
// 1024 x 1056 x 992 the 221 tiles of 80 x 64 take 28 us, the 272 of 64 x 64
// 39 us, the 136 of 128 x 64 38 us (and 60 us before, 128 x 64 tiles one slice
// ahead).  The 16 x 16 tiles share a CU by several, so their rounds need not be
// whole; the direct 32 x 32 tiles read too much memory past one round.
//
// Products of K <= 256, where no wave of a direct tile has two slices and the
// groups of a split tile's waves have one or none: past the first rounds the fixed
// part becomes `more` a round.  The direct tiles share a CU by up to 32; the blocks
// of twelve and sixteen waves mostly wait, and hardly overlap, which up to K = 128
// the larger feel from their first round on (10^6 x 8 by 16 x 16, 32 x 32, 64 x 32 and
// 64 x 64 tiles, us: K = 8 74, 76, 157 and 103; K = 32 84, 79, 184 and 127; K = 256
// 237, 315, 349 and 366; 2853 x 3201 x 12, A transposed, by 32 x 32, 64 x 64, 96 x 64
// and 128 x 128 20, 25, 32 and 23, of which `fixed` alone picked the third).
struct GemmShape {
    const char *name;  // MX_GEMM_TILE in the environment forces a shape, for tuning and tests
    int bm, bn;
    double fixed, per_k;
    mx_status (*launch)(const GemmArgs &);
    double first = 0., more = 0.;  // rounds at `fixed`, and the fixed part of those after them
};
const GemmShape kShapes[] = {
    {"16x16", 16, 16, 0.95, 2.3, launch_direct<1, 1, 8>, 3., .1},
    {"32x32", 32, 32, 1.4, 5.5, launch_direct<2, 2, 4>, 3., .2},
    {"32x64", 32, 64, 1.5, 10.5, launch_split<2, 2, 1, 2, 6>, 1., 2.4},
    {"64x32", 64, 32, 1.5, 10.5, launch_split<2, 2, 2, 1, 6>, 1., 2.4},
    {"64x64", 64, 64, 1.8, 19., launch_split<2, 2, 2, 2, 2>, 1., 1.4},
    {"80x64", 80, 64, 2.2, 23.5, launch_split<5, 1, 1, 4, 4>, 0., 3.6},
    {"64x80", 64, 80, 2.2, 24., launch_split<1, 5, 4, 1, 4>, 0., 3.6},
    {"96x64", 96, 64, 2.5, 27.5, launch_split<3, 2, 2, 2, 3>, 0., 3.6},
    {"64x96", 64, 96, 2.5, 27.5, launch_split<2, 3, 2, 2, 3>, 0., 3.6},
    {"128x64", 128, 64, 3., 34., launch_split<2, 2, 4, 2, 2>, 0., 4.},
    {"64x128", 64, 128, 3., 34., launch_split<2, 2, 2, 4, 2>, 0., 4.},
    {"128x96", 128, 96, 4., 49.5, launch_split<2, 3, 4, 2, 2>, 0., 4.},
    {"128x128", 128, 128, 5., 65.5, launch_split<2, 2, 4, 4, 1>, 1., 3.},
    {"128x128w16", 128, 128, 5., 62., launch_pipelined, 1., 2.9},
};
constexpr int kNumShapes = sizeof kShapes / sizeof kShapes[0], kPipelined = kNumShapes - 1;

const GemmShape &gemm_choice(const GemmArgs &a) {
    const int64_t lda = a.ta ? a.M : a.K, ldb = a.tb ? a.K : a.N;
    // the pipelined kernel takes whole tiles of aligned rows
    const bool whole = a.M % 128 == 0 && a.N % 128 == 0 && a.K % 64 == 0 && a.K >= 128 && lda % 4 == 0 &&
                       ldb % 4 == 0 && (uintptr_t)a.A % 16 == 0 && (uintptr_t)a.B % 16 == 0;
    // nothing to read, or rows so few that a vector of them could pass the end
    if (a.K == 0 || (a.ta && a.M < 4) || (!a.tb && a.N < 4)) return kShapes[0];
    // read on every call (a getenv is cheap next to a launch), so one process
    // can run every shape; a number of waves ("128x64w8") that no kernel has for
    // this product leaves the sides
    if (const char *e = getenv("MX_GEMM_TILE")) {
        if (!strcmp(e, kShapes[kPipelined].name) && whole) return kShapes[kPipelined];
        const std::string sides(e, strcspn(e, "w"));
        for (int i = 0; i < kPipelined; ++i)
            if (sides == kShapes[i].name) return kShapes[i];
    }
    int best = 0;
    double best_us = 1e300;
    for (int i = 0; i < kNumShapes; ++i) {
        const GemmShape &s = kShapes[i];
        if (i == kPipelined && !whole) continue;
        const double tiles = (double)ceil_div(a.M, s.bm) * (double)ceil_div(a.N, s.bn);
        double rounds = tiles / (double)a.num_cus;
        if (rounds < 1.) rounds = 1.;
        else if (i > 0) rounds = ceil(rounds);
        const double per_k = i == 1 && rounds > 1. ? 9. : s.per_k;
        double fixed = s.fixed * rounds;
        if (a.K <= (s.first > 0. ? 256 : 128) && s.more > 0. && rounds > s.first) fixed = s.fixed * s.first + s.more * (rounds - s.first);
        const double us = fixed + rounds * per_k * (double)a.K * 1e-3;
        if (us < best_us) {
            best_us = us;
            best = i;
        }
    }
    return kShapes[best];
}

}  // namespace
}  // namespace mx

using namespace mx;

extern "C" {

mx_status mx_map_map_reduce_f32(int ta, int tb, int64_t M, int64_t N, int64_t K, const float *A_dev,
                                const float *B_dev, float *C_dev, hipStream_t stream) {
    if (mx_status st = check("mx_map_map_reduce_f32", ta, tb, M, N, K, A_dev, B_dev, C_dev)) return st;
    if (M == 0 || N == 0) return MX_OK;
    const DeviceInfo *d;
    if (mx_status st = device_info(&d)) return st;
    const GemmArgs a{ta, tb, M, N, K, A_dev, B_dev, C_dev, stream, d->num_cus};
    return gemm_choice(a).launch(a);
}

mx_status mx_map_map_reduce_plain_f32(int ta, int tb, int64_t M, int64_t N, int64_t K,
                                      const float *A_dev, const float *B_dev, float *C_dev,
                                      hipStream_t stream) {
    if (mx_status st = check("mx_map_map_reduce_plain_f32", ta, tb, M, N, K, A_dev, B_dev, C_dev)) return st;
    if (M == 0 || N == 0) return MX_OK;
    MX_REQUIRE(ceil_div(M, 16) < 65536, MX_ERR_SHAPE, "mx_map_map_reduce_plain_f32: M too large");
    const dim3 grid((unsigned)ceil_div(N, 16), (unsigned)ceil_div(M, 16));
#define MX_GEMMP(TA, TB) \
    hipLaunchKernelGGL((k_gemm_plain<TA, TB>), grid, dim3(256), 0, stream, A_dev, B_dev, C_dev, M, N, K)
    if (!ta && !tb) MX_GEMMP(0, 0);
    else if (!ta && tb) MX_GEMMP(0, 1);
    else if (ta && !tb) MX_GEMMP(1, 0);
    else MX_GEMMP(1, 1);
#undef MX_GEMMP
    return last_launch("mx_map_map_reduce_plain_f32");
}

}  // extern "C"
