// Many uneven accelerated expressions in one launch.
//
// The paper notes that expression acceleration pays off when work is
// concentrated in few `accelerate` uses and that small problems leave the GPU
// idle (Section 5.2).  A batch runs thousands of independent small
// expressions -- dot products reduce (+) 0 (map2 (*) a b) and matrix-vector
// products map (reduce (+) 0 . map2 (*) x) over rows -- as one launch.
//
// Plan (host, once): every task is cut into tiles of equal bytes -- element
// ranges of `tile_elems` for a dot (two streamed operands), whole-row ranges
// of about 2 * `tile_elems` elements for a matvec (one); backward a tile is at
// most what a block takes at once -- and the tiles are ordered longest first.  Forward: a block per tile;
// a single-tile task writes its result, a multi-tile dot
// writes one partial per tile.  A combine launch adds each task's partials in
// tile order (deterministic for a given plan).  Backward
// (dot: ga = g b, gb = g a; matvec y = A x: gA = g x^T, gx = A^T g) has the same
// structure, with per-tile partial column sums for gx and long rows in several tiles.  No float atomics, no
// cross-block fences.  The autotuner times candidate (tile_elems,
// blocks_per_cu) pairs on the caller's buffers and caches the choice per task
// table and device in a JSON file.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <sstream>
#include <string>
#include <vector>

#include "mx_internal.h"

namespace mx {
namespace {

constexpr int NT = 256;
constexpr int kDot = 0, kMatvec = 1;
constexpr int kMinTile = 4096;
constexpr int kXLds = 2048;  // matvec x staged in LDS up to this many columns
constexpr int NB = 512;      // threads of a backward block
constexpr int kBwdVec = 2;   // 16-byte vectors per operand and thread of a dot's backward tile
constexpr int64_t kDotChunk = 4 * kBwdVec * NB;  // elements of a dot's backward tile
constexpr int kAdjRows = 8;  // rows of a matvec's backward that a thread has in flight
constexpr int kWidthShift = 8;
constexpr unsigned kAdjParts = 16;  // sums that a column's phases are added in
constexpr int64_t kLongRow = 1 << 22;  // matvec rows past this length are walked one at a time backward

struct TaskDev {
    int32_t kind, pad;
    int64_t rows, cols, a_off, b_off, out_off;
    int64_t fwd_part, fwd_ntiles, bwd_part, bwd_ntiles;
};

// One tile, carrying the task fields its kernels need, the offsets those of its
// first element or row, so that taking a tile costs one descriptor load.
struct TileDev {
    uint32_t kind;         // the kind, and from kWidthShift on the columns of a matvec's tile backward
    uint32_t count;        // dot: elements; matvec: rows
    int64_t part;          // partial slot (float offset) or -1 to write the result directly
    int64_t cols, a_off, b_off, out_off;
};

// sum over the 16 lanes of a DPP row, result in every lane of the row
__device__ __forceinline__ float row16_sum(float v) {
    using R = Red<MX_ADD, float>;
    v = R::ap(v, dpp_move<0xB1, 0xF>(v, 0.f));
    v = R::ap(v, dpp_move<0x4E, 0xF>(v, 0.f));
    v = R::ap(v, dpp_move<0x141, 0xF>(v, 0.f));
    v = R::ap(v, dpp_move<0x140, 0xF>(v, 0.f));
    return v;
}

// Four floats at any float address: element alignment is all a 16-byte access
// needs, so tasks and rows of every offset and length take the same path.  The
// address is a base that is the same in all lanes plus a 32-bit element offset
// of the lane, which costs one register where a pointer per access costs two.
using f4u = uvec<float>;
template <bool PAST> __device__ __forceinline__ f4u ld4(const float *base, unsigned off) {
    const f4u *q = reinterpret_cast<const f4u *>(reinterpret_cast<const char *>(base) + 4u * off);
    if constexpr (PAST) return __builtin_nontemporal_load(q);
    else return *q;
}
__device__ __forceinline__ void st4(f4u v, float *base, unsigned off) {
    __builtin_nontemporal_store(v, reinterpret_cast<f4u *>(reinterpret_cast<char *>(base) + 4u * off));
}
__device__ __forceinline__ float dot4(f4u a, f4u b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }

// This thread's part of the dot product of n elements: contiguous chunks of
// 4 NT vectors per operand, all in flight, the last chunk predicated.
__device__ __forceinline__ float block_dot(const float *__restrict__ a, const float *__restrict__ b, int64_t n) {
    const int64_t nv = n >> 2;
    float ac[4] = {0.f, 0.f, 0.f, 0.f};
    for (int64_t c = 0; c < nv; c += 4 * NT) {
        const float *ac4 = a + 4 * c, *bc4 = b + 4 * c;
        f4u x[4], y[4];
        if (c + 4 * NT <= nv) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = ld4<false>(ac4, 4 * (threadIdx.x + u * NT));
                y[u] = ld4<false>(bc4, 4 * (threadIdx.x + u * NT));
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = y[u] = f4u{0.f, 0.f, 0.f, 0.f};
                if (threadIdx.x + u * NT < (unsigned)(nv - c)) {
                    x[u] = ld4<false>(ac4, 4 * (threadIdx.x + u * NT));
                    y[u] = ld4<false>(bc4, 4 * (threadIdx.x + u * NT));
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) ac[u] += dot4(x[u], y[u]);
    }
    if (threadIdx.x < (unsigned)(n & 3)) {
        ac[1] += a[4 * nv + threadIdx.x] * b[4 * nv + threadIdx.x];
    }
    return (ac[0] + ac[1]) + (ac[2] + ac[3]);
}

// The rows of a matvec tile of c <= kXLds columns: 16 lanes per row, R rows
// per group of lanes and 8 / R vectors per row and lane in flight (R: as many
// rows as eight vectors per lane cover).  x in LDS: its whole vectors, zeros for
// the lanes past them (up to 16 (K - 1) vectors, whose elements of A read as zeros,
// so an infinite element of x must not meet them), then the last c % 4 elements.
constexpr int kXPad = 64 * 7;  // at K = 8
template <int R>
__device__ __forceinline__ void matvec_rows(const float *__restrict__ A, const float *__restrict__ b, float *x,
                                            float *__restrict__ out, unsigned c, int64_t n) {
    constexpr int K = 8 / R, G = NT / 16;
    constexpr unsigned PAD = 64 * (K - 1);
    const unsigned grp = threadIdx.x >> 4, l = threadIdx.x & 15, nv = c >> 2;
    for (unsigned v = threadIdx.x; v < nv + PAD / 4; v += NT)
        *reinterpret_cast<f4u *>(x + 4 * v) = v < nv ? ld4<false>(b, 4 * v) : f4u{0.f, 0.f, 0.f, 0.f};
    if (threadIdx.x < (c & 3)) x[4 * nv + PAD + threadIdx.x] = b[4 * nv + threadIdx.x];
    __syncthreads();
    const unsigned row = 4u * grp * c;  // byte offset of this group's first row
    for (int64_t r0 = 0; r0 < n; r0 += G * R) {
        const unsigned rows = (unsigned)(n - r0 < G * R ? n - r0 : G * R);
        const buf a = make_buf(A + r0 * c, 4u * rows * c);
        float ac[R][2];
#pragma unroll
        for (int q = 0; q < R; ++q) ac[q][0] = ac[q][1] = 0.f;
        for (unsigned v = l; v < nv; v += 16 * K) {
            f4u av[R][K];
#pragma unroll
            for (int u = 0; u < K; ++u) {
                const unsigned at = v + 16 * u < nv ? row + 16 * (v + 16 * u) : kOutside;
#pragma unroll
                for (int q = 0; q < R; ++q) av[q][u] = bld4<false>(a, at + 4u * q * G * c);
            }
#pragma unroll
            for (int u = 0; u < K; ++u) {
                const float4 xv = *reinterpret_cast<const float4 *>(x + 4 * (v + 16 * u));
#pragma unroll
                for (int q = 0; q < R; ++q) ac[q][u & 1] += dot4(av[q][u], f4u{xv.x, xv.y, xv.z, xv.w});
            }
        }
        if (4 * nv + l < c) {
            const float xv = x[4 * nv + PAD + l];
#pragma unroll
            for (int q = 0; q < R; ++q) ac[q][1] += bld1(a, row + 4 * (4 * nv + l) + 4u * q * G * c) * xv;
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const float acc = row16_sum(ac[q][0] + ac[q][1]);
            if (l == 0 && grp + q * G < rows) out[r0 + grp + q * G] = acc;
        }
    }
}

// A block per tile, dispatched by the hardware in tile order.  Bound by HBM: of
// 2048 uneven expressions (1.29 GB) 222 us, 5.8 TB/s.  Persistent blocks that
// took tiles by ticket waited for a round trip to memory before each tile's
// first load, 260 us; 512 expressions of 49 MB 31 us, now 14.6 us.
__global__ void __launch_bounds__(NT, 8) k_batch_fwd(const TileDev *__restrict__ tiles, int64_t ntiles,
                                                  const float *__restrict__ A, const float *__restrict__ B,
                                                  float *__restrict__ out, float *__restrict__ part) {
    __shared__ float red[NT / kWave];
    __shared__ __attribute__((aligned(16))) float xs[kXLds + kXPad];
    using R = Red<MX_ADD, float>;
    const int64_t t = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (t >= ntiles) return;
    const TileDev tk = tiles[t];
    const float *a = A + tk.a_off, *b = B + tk.b_off;
    float *o = out + tk.out_off;
    if (tk.kind == kDot) {
        const float acc = block_reduce<R, NT>(block_dot(a, b, tk.count), red);
        if (threadIdx.x == 0) *(tk.part >= 0 ? part + tk.part : o) = acc;
    } else if (tk.cols <= kXLds) {
        const unsigned c = (unsigned)tk.cols;
        if (c > 256) matvec_rows<1>(a, b, xs, o, c, tk.count);
        else if (c > 128) matvec_rows<2>(a, b, xs, o, c, tk.count);
        else if (c > 64) matvec_rows<4>(a, b, xs, o, c, tk.count);
        else matvec_rows<8>(a, b, xs, o, c, tk.count);
    } else {
        for (int64_t r = 0; r < tk.count; ++r) {  // a long row is a dot product
            const float acc = block_reduce<R, NT>(block_dot(a + r * tk.cols, b, tk.cols), red);
            if (threadIdx.x == 0) o[r] = acc;
            __syncthreads();
        }
    }
}

// One matvec tile's backward, w columns of rows c apart: gA rows get g[r] x, and dst
// (the tile's partial column sums, or gB) the sums over its rows of g[r] A[r].  A
// thread takes four columns and, when there are fewer groups of four than
// threads, one of P phases of the rows (rows ph, ph + P, ...), whose partials are
// added in phase order through LDS, of many phases sixteen strided parts first.
// The tile has no more rows than the block takes at once (adj_round), U to a
// thread, and no more columns (adj_cols).  The last group of a width that is not
// a multiple of four overlaps the one before it and leaves its first `skip`
// columns to that, so rows of any length take 16-byte accesses.
//
// Bound by HBM: 447 MB of matrices in 198 us (4.5 TB/s of matrix and gradient,
// 4.8 with the partial sums), 190 us if all rows are multiples of four; with
// blocks of 256 threads that walked four rounds of rows 214 us, in interleaved
// rounds 226 us, four rows per thread in flight 199 us.
template <bool PAST>
__device__ __forceinline__ void matvec_adj_tile(const float *__restrict__ a, const float *__restrict__ x,
                                                const float *__restrict__ g, float *__restrict__ ga, int64_t c,
                                                unsigned w, unsigned rows, float *__restrict__ dst, float4 *red) {
    constexpr int U = kAdjRows;
    if (rows == 0) {  // no range to describe: the sums over no rows
        for (unsigned j = threadIdx.x; j < w; j += NB) dst[j] = 0.f;
        return;
    }
    if (w < 4) {  // whole rows, one thread each, element by element
        constexpr int U = 4;
        float s[3] = {0.f, 0.f, 0.f}, xe[3];
#pragma unroll
        for (unsigned e = 0; e < 3; ++e) xe[e] = e < w ? x[e] : 0.f;
        for (unsigned r0 = threadIdx.x; r0 < rows; r0 += U * NB) {
            float gv[U], av[U][3];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned r = r0 + u * NB;
                gv[u] = r < rows ? g[r] : 0.f;
#pragma unroll
                for (unsigned e = 0; e < 3; ++e) av[u][e] = r < rows && e < w ? a[r * w + e] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (unsigned e = 0; e < 3; ++e) {
                    s[e] += av[u][e] * gv[u];
                    if (r0 + u * NB < rows && e < w) ga[(r0 + u * NB) * w + e] = xe[e] * gv[u];
                }
        }
        float *ws = reinterpret_cast<float *>(red);  // [wave][3]
#pragma unroll
        for (unsigned e = 0; e < 3; ++e) {
            const float v = wave_reduce<Red<MX_ADD, float>>(s[e]);
            if (threadIdx.x % kWave == 0) ws[threadIdx.x / kWave * 3 + e] = v;
        }
        __syncthreads();
        if (threadIdx.x < w) {
            float t = ws[threadIdx.x];
#pragma unroll
            for (int k = 1; k < NB / kWave; ++k) t += ws[3 * k + threadIdx.x];
            dst[threadIdx.x] = t;
        }
        return;
    }
    const unsigned cv = (w + 3) >> 2;  // groups of four columns, at most NB
    const unsigned P = __builtin_amdgcn_readfirstlane(NB / cv < rows ? NB / cv : rows), j = threadIdx.x % cv,
                   ph = threadIdx.x / cv;
    // the byte stride from a thread's row to its next; rows too long for a
    // 32-bit offset to reach it come one to a tile
    const unsigned step = c <= kLongRow ? 4u * P * (unsigned)c : 0x10000000u;
    const bool mine = ph < P;
    const unsigned first = 4 * j + 4 <= w ? 4 * j : w - 4;  // this group's first column
    const int skip = (int)(4 * j - first);
    const int64_t bytes = 4 * ((rows - 1) * (c <= kLongRow ? c : 0) + w);
    const buf ab = make_buf(a, bytes), ob = make_buf(ga, bytes), gb = make_buf(g, 4u * rows);
    const unsigned off = (P > 1 ? 4u * ph * (unsigned)c : 0u) + 4u * first;
    unsigned ld_at = mine ? off : kOutside, st_at = mine && skip == 0 ? off : kOutside, g_at = 4u * ph;
    f4u av[U], s = {0.f, 0.f, 0.f, 0.f}, xj = s;
    float gv[U];
    if (mine) xj = ld4<false>(x, first);
#pragma unroll
    for (int u = 0; u < U; ++u, ld_at += step, g_at += 4 * P) {
        av[u] = bld4<PAST>(ab, ld_at);
        gv[u] = bld1(gb, g_at);
    }
#pragma unroll
    for (int u = 0; u < U; ++u, st_at += step) {
        s += av[u] * gv[u];
        bst4(xj * gv[u], ob, st_at);
    }
    if (mine && skip != 0)  // the last one to three columns of gA
        for (unsigned r = ph; r < rows; r += P) {
            const float gr = g[r];
            float *o = ga + r * c + first;
            o[3] = xj[3] * gr;
            if (skip < 3) o[2] = xj[2] * gr;
            if (skip < 2) o[1] = xj[1] * gr;
        }
    if (P > 1) {
        red[threadIdx.x] = make_float4(s.x, s.y, s.z, s.w);
        __syncthreads();
        unsigned parts = P;
        if (P > kAdjParts) {  // part k: phases k, k + kAdjParts, ...
            f4u t = {0.f, 0.f, 0.f, 0.f};
            if (ph < kAdjParts)
#pragma unroll 4
                for (unsigned q = ph; q < P; q += kAdjParts) {
                    const float4 v = red[q * cv + j];
                    t += f4u{v.x, v.y, v.z, v.w};
                }
            __syncthreads();
            if (ph < kAdjParts) red[threadIdx.x] = make_float4(t.x, t.y, t.z, t.w);
            s = t;
            parts = kAdjParts;
            __syncthreads();
        }
        if (ph == 0)
#pragma unroll 8
            for (unsigned q = 1; q < parts; ++q) {
                const float4 v = red[q * cv + j];
                s += f4u{v.x, v.y, v.z, v.w};
            }
    }
    if (ph == 0)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e >= skip) dst[first + e] = s[e];
}

// Bound by HBM.  A dot's tile is one round of the block's accesses, so that the
// blocks which run together walk the four arrays as one front: 843 MB of
// operands and as much of gradients took 345 us with tiles of 64 KB walked in
// four rounds (their starts a power of two apart), now 310 us.  Loads past the
// caches in passes larger than the memory-side cache leave what the forward
// pass put there: forward and backward of 1.29 GB 704 us, 731 us without.
template <bool PAST>
__global__ void __launch_bounds__(NB) k_batch_bwd(const TileDev *__restrict__ tiles, int64_t ntiles,
                                                  const float *__restrict__ A, const float *__restrict__ B,
                                                  const float *__restrict__ gout, float *__restrict__ gA,
                                                  float *__restrict__ gB, float *__restrict__ part) {
    __shared__ float4 red[NB];
    const int64_t t = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (t >= ntiles) return;
    const TileDev tk = tiles[t];
    if (tk.kind == kDot) {
        const float g = gout[tk.out_off];
        const float *a = A + tk.a_off, *b = B + tk.b_off;
        float *ga = gA + tk.a_off, *gb = gB + tk.b_off;
        const int64_t n = tk.count, nv = n >> 2;
        for (int64_t c = 0; c < nv; c += kBwdVec * NB) {
            const int64_t at = 4 * c;
            f4u x[kBwdVec], y[kBwdVec];
            if (c + kBwdVec * NB <= nv) {
#pragma unroll
                for (int u = 0; u < kBwdVec; ++u) {
                    x[u] = ld4<PAST>(a + at, 4 * (threadIdx.x + u * NB));
                    y[u] = ld4<PAST>(b + at, 4 * (threadIdx.x + u * NB));
                }
#pragma unroll
                for (int u = 0; u < kBwdVec; ++u) {
                    st4(y[u] * g, ga + at, 4 * (threadIdx.x + u * NB));
                    st4(x[u] * g, gb + at, 4 * (threadIdx.x + u * NB));
                }
            } else {
                const unsigned left = (unsigned)(nv - c);
#pragma unroll
                for (int u = 0; u < kBwdVec; ++u)
                    if (threadIdx.x + u * NB < left) {
                        x[u] = ld4<PAST>(a + at, 4 * (threadIdx.x + u * NB));
                        y[u] = ld4<PAST>(b + at, 4 * (threadIdx.x + u * NB));
                    }
#pragma unroll
                for (int u = 0; u < kBwdVec; ++u)
                    if (threadIdx.x + u * NB < left) {
                        st4(y[u] * g, ga + at, 4 * (threadIdx.x + u * NB));
                        st4(x[u] * g, gb + at, 4 * (threadIdx.x + u * NB));
                    }
            }
        }
        const int64_t e = 4 * nv + threadIdx.x;
        if (e < n) {
            ga[e] = g * b[e];
            gb[e] = g * a[e];
        }
    } else {
        float *dst = tk.part >= 0 ? part + tk.part : gB + tk.b_off;
        matvec_adj_tile<PAST>(A + tk.a_off, B + tk.b_off, gout + tk.out_off, gA + tk.a_off, tk.cols, tk.kind >> kWidthShift, tk.count,
                              dst, red);
    }
}

// sum of q = 0 .. nq-1 of p[q * stride], in q order, eight loads in flight
__device__ __forceinline__ float sum_strided(const float *__restrict__ p, int64_t nq, int64_t stride) {
    float s = 0.f;
    int64_t q = 0;
    for (; q + 8 <= nq; q += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(q + u) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; q < nq; ++q) s += p[q * stride];
    return s;
}

// Adds the tile partials of each multi-tile task in tile order.
__global__ void __launch_bounds__(NT) k_batch_combine_fwd(const TaskDev *__restrict__ tasks,
                                                          const int32_t *__restrict__ list, int64_t nlist,
                                                          const float *__restrict__ part, float *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= nlist) return;
    const TaskDev tk = tasks[list[i]];
    out[tk.out_off] = sum_strided(part + tk.fwd_part, tk.fwd_ntiles, 1);
}

// grid (tasks in the list, column chunks): column j of a task gets the sum of
// its per-tile partial column sums, PARTS runs of tiles each in tile order, then
// the runs in order.  One run up to kRunTiles tiles; past them a thread per column
// would wait for eight loads at a time (2000 x 2000, 250 tiles: backward 18.1 us
// with one run).
constexpr int kRunTiles = 16;
template <int PARTS>
__global__ void __launch_bounds__(NT) k_batch_combine_bwd(const TaskDev *__restrict__ tasks,
                                                          const int32_t *__restrict__ list, int64_t nlist,
                                                          const float *__restrict__ part, float *__restrict__ gB) {
    constexpr int COLS = NT / PARTS;
    __shared__ float red[PARTS][COLS];
    if ((int64_t)blockIdx.x >= nlist) return;
    const TaskDev tk = tasks[list[blockIdx.x]];
    const int64_t c = tk.cols, per = (tk.bwd_ntiles + PARTS - 1) / PARTS;
    const int q = threadIdx.x / COLS, l = threadIdx.x % COLS;
    const int64_t q0 = q * per, n = q0 + per < tk.bwd_ntiles ? per : tk.bwd_ntiles - q0;
    for (int64_t j0 = (int64_t)blockIdx.y * COLS; j0 < c; j0 += (int64_t)gridDim.y * COLS) {
        const int64_t j = j0 + l;
        float s = j < c ? sum_strided(part + tk.bwd_part + q0 * c + j, n, c) : 0.f;
        if constexpr (PARTS > 1) {
            red[q][l] = s;
            __syncthreads();
            if (q == 0)
#pragma unroll
                for (int k = 1; k < PARTS; ++k) s += red[k][l];
            __syncthreads();
        }
        if (q == 0 && j < c) gB[tk.b_off + j] = s;
    }
}

// ---------------------------------------------------------------- plain: one launch per task
__global__ void __launch_bounds__(NT) k_dot_plain(const float *__restrict__ a, const float *__restrict__ b, int64_t n,
                                                  float *__restrict__ out) {
    __shared__ float red[NT / kWave];
    float acc = 0.f;
    for (int64_t e = threadIdx.x; e < n; e += NT) acc += a[e] * b[e];
    acc = block_reduce<Red<MX_ADD, float>, NT>(acc, red);
    if (threadIdx.x == 0) out[0] = acc;
}

__global__ void __launch_bounds__(NT) k_matvec_plain(const float *__restrict__ A, const float *__restrict__ x,
                                                     int64_t rows, int64_t cols, float *__restrict__ y) {
    const int64_t r = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (r >= rows) return;
    float acc = 0.f;
    for (int64_t j = 0; j < cols; ++j) acc += A[r * cols + j] * x[j];
    y[r] = acc;
}

__global__ void __launch_bounds__(NT) k_dot_adj_plain(const float *__restrict__ a, const float *__restrict__ b,
                                                      int64_t n, const float *__restrict__ g, float *__restrict__ ga,
                                                      float *__restrict__ gb) {
    const int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (e >= n) return;
    ga[e] = g[0] * b[e];
    gb[e] = g[0] * a[e];
}

__global__ void __launch_bounds__(NT) k_matvec_adj_plain(const float *__restrict__ A, const float *__restrict__ x,
                                                         int64_t rows, int64_t cols, const float *__restrict__ g,
                                                         float *__restrict__ gA, float *__restrict__ gx) {
    const int64_t j = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (j >= cols) return;
    float acc = 0.f;
    for (int64_t r = 0; r < rows; ++r) {
        acc += A[r * cols + j] * g[r];
        gA[r * cols + j] = g[r] * x[j];
    }
    gx[j] = acc;
}

}  // namespace
}  // namespace mx

using namespace mx;

struct mx_batch_plan {
    int device = 0;
    std::vector<int64_t> table;  // [ntasks][6]
    int64_t ntasks = 0;
    int64_t a_len = 0, b_len = 0, out_len = 0;
    mx_batch_config cfg{};
    TaskDev *d_tasks = nullptr;
    TileDev *d_fwd = nullptr, *d_bwd = nullptr;
    int32_t *d_fwd_list = nullptr, *d_bwd_list = nullptr;
    int64_t n_fwd = 0, n_bwd = 0, n_fwd_list = 0, n_bwd_list = 0;
    int64_t bwd_list_max_cols = 1, bwd_list_max_tiles = 1;
    int64_t fwd_part_floats = 0, bwd_part_floats = 0;
    size_t ws_need = 0;
};

namespace {

void free_device(mx_batch_plan *p) {
    (void)hipFree(p->d_tasks);
    (void)hipFree(p->d_fwd);
    (void)hipFree(p->d_bwd);
    (void)hipFree(p->d_fwd_list);
    (void)hipFree(p->d_bwd_list);
    p->d_tasks = nullptr;
    p->d_fwd = p->d_bwd = nullptr;
    p->d_fwd_list = p->d_bwd_list = nullptr;
}

// rows that a block takes at once in a matvec's backward
int64_t adj_round(int64_t c) {
    if (c < 4) return 2 * kMinTile / std::max<int64_t>(c, 1);  // one to two rounds
    if (c > kLongRow) return 1;
    return kAdjRows * (NB / std::min<int64_t>(ceil_div(c, 4), NB));
}
// columns of a matvec's tile backward with `left` more to go: a row's parts share
// no sum, and 1 x 2^23 takes 6.0 ms by one block that walks it; never one to three
// columns, which would be no group of four
int64_t adj_cols(int64_t left) {
    const int64_t most = 4 * NB;
    return left <= most ? left : left < most + 4 ? most - 4 : most;
}
// rows of a matvec's tile backward (at most what a block takes at once) and forward
int64_t fwd_rows(int64_t cols, int64_t tile) { return std::max<int64_t>(1, 2 * tile / std::max<int64_t>(cols, 1)); }
int64_t bwd_rows(int64_t cols, int64_t tile) { return std::min(adj_round(cols), fwd_rows(cols, tile)); }

// Partial-storage requirement at the smallest tile size (covers every candidate).
void partial_floats(const std::vector<int64_t> &tb, int64_t ntasks, int64_t tile, int64_t *fwd, int64_t *bwd) {
    *fwd = 0;
    *bwd = 0;
    for (int64_t t = 0; t < ntasks; ++t) {
        const int64_t kind = tb[6 * t], rows = tb[6 * t + 1], cols = tb[6 * t + 2];
        if (kind == kDot) {
            const int64_t nt = ceil_div(cols > 0 ? cols : 1, tile);
            if (nt > 1) *fwd += nt;
        } else {
            const int64_t nt = ceil_div(rows > 0 ? rows : 1, bwd_rows(cols, tile));
            if (nt > 1) *bwd += nt * cols;
        }
    }
}

// elements (dot) or rows (matvec) [begin, end) of a task
TileDev make_tile(const TaskDev &tk, int64_t begin, int64_t end, int64_t part) {
    const bool dot = tk.kind == kDot;
    return TileDev{(uint32_t)tk.kind, (uint32_t)(end - begin), part, tk.cols, tk.a_off + begin * (dot ? 1 : tk.cols),
                   tk.b_off + (dot ? begin : 0), tk.out_off + (dot ? 0 : begin)};
}

// Longest first by operand bytes in classes of an eighth of an octave, in task
// order within a class (so plans are reproducible): one counting pass.
void order_tiles(std::vector<TileDev> &v) {
    auto cls = [](const TileDev &t) {
        const uint64_t w = t.kind >> kWidthShift;
        const uint64_t c = t.kind == kDot ? 2 * (uint64_t)t.count : t.count * (w ? w : (uint64_t)t.cols);
        if (c < 8) return 511 - (int)c;
        const int e = 63 - __builtin_clzll(c);
        return 511 - (8 * (e - 2) + (int)((c >> (e - 3)) & 7));
    };
    std::vector<size_t> at(513, 0);
    for (const TileDev &t : v) ++at[(size_t)cls(t) + 1];
    for (size_t i = 1; i < at.size(); ++i) at[i] += at[i - 1];
    std::vector<TileDev> o(v.size());
    for (const TileDev &t : v) o[at[(size_t)cls(t)]++] = t;
    v.swap(o);
}

mx_status build_tiles(mx_batch_plan *p) {
    const int64_t T = p->cfg.tile_elems;
    std::vector<TaskDev> tasks((size_t)p->ntasks);
    std::vector<TileDev> fwd, bwd;
    std::vector<int32_t> fwd_list, bwd_list;
    int64_t fpart = 0, bpart = 0, max_cols = 1, max_tiles = 1;
    for (int64_t t = 0; t < p->ntasks; ++t) {
        const int64_t *r = &p->table[(size_t)(6 * t)];
        TaskDev &tk = tasks[(size_t)t];
        tk.kind = (int32_t)r[0];
        tk.rows = r[1];
        tk.cols = r[2];
        tk.a_off = r[3];
        tk.b_off = r[4];
        tk.out_off = r[5];
        if (tk.kind == kDot) {
            const int64_t n = tk.cols;
            const int64_t nt = std::max<int64_t>(1, ceil_div(n, T));
            tk.fwd_ntiles = nt;
            tk.fwd_part = nt > 1 ? fpart : -1;
            for (int64_t q = 0; q < nt; ++q)
                fwd.push_back(make_tile(tk, q * T, std::min(n, (q + 1) * T), nt > 1 ? fpart + q : -1));
            if (nt > 1) {
                fwd_list.push_back((int32_t)t);
                fpart += nt;
            }
            // nothing to add up backward: a chunk of the block's loads each
            for (int64_t e = 0; e == 0 || e < n; e += kDotChunk)
                bwd.push_back(make_tile(tk, e, std::min(n, e + kDotChunk), -1));
            tk.bwd_ntiles = nt;
            tk.bwd_part = -1;
        } else {
            // a matvec streams one operand (4 bytes per element) where a dot
            // streams two: twice the elements give tiles of equal bytes
            const int64_t rpt = fwd_rows(tk.cols, T);
            const int64_t nt = std::max<int64_t>(1, ceil_div(tk.rows, rpt));
            tk.fwd_ntiles = nt;
            tk.fwd_part = -1;
            for (int64_t q = 0; q < nt; ++q)
                fwd.push_back(make_tile(tk, q * rpt, std::min(tk.rows, (q + 1) * rpt), -1));
            // backward a tile is what a block takes at once
            const int64_t rows = bwd_rows(tk.cols, T);
            const int64_t nb = std::max<int64_t>(1, ceil_div(tk.rows, rows));
            tk.bwd_ntiles = nb;
            tk.bwd_part = nb > 1 ? bpart : -1;
            for (int64_t q = 0; q < nb; ++q)
                for (int64_t c0 = 0, w; c0 == 0 || c0 < tk.cols; c0 += std::max<int64_t>(w, 1)) {
                    w = adj_cols(tk.cols - c0);
                    TileDev t = make_tile(tk, q * rows, std::min(tk.rows, (q + 1) * rows), nb > 1 ? bpart + q * tk.cols + c0 : -1);
                    t.kind |= (uint32_t)w << kWidthShift;
                    t.a_off += c0;
                    t.b_off += c0;
                    bwd.push_back(t);
                }
            if (nb > 1) {
                bwd_list.push_back((int32_t)t);
                bpart += nb * tk.cols;
                max_cols = std::max(max_cols, tk.cols);
                max_tiles = std::max(max_tiles, nb);
            }
        }
    }
    order_tiles(fwd);
    order_tiles(bwd);
    MX_REQUIRE((int64_t)fwd.size() < (1LL << 31) && (int64_t)bwd.size() < (1LL << 31), MX_ERR_SHAPE,
               "mx_batch_plan: too many tiles");
    free_device(p);
    auto up = [](auto **dst, const auto &v) -> mx_status {
        using E = typename std::decay_t<decltype(v)>::value_type;
        const size_t bytes = std::max<size_t>(v.size() * sizeof(E), 16);
        MX_TRY_HIP(hipMalloc((void **)dst, bytes));
        if (!v.empty()) MX_TRY_HIP(hipMemcpy(*dst, v.data(), v.size() * sizeof(E), hipMemcpyHostToDevice));
        return MX_OK;
    };
    if (mx_status st = up(&p->d_tasks, tasks)) return st;
    if (mx_status st = up(&p->d_fwd, fwd)) return st;
    if (mx_status st = up(&p->d_bwd, bwd)) return st;
    if (mx_status st = up(&p->d_fwd_list, fwd_list)) return st;
    if (mx_status st = up(&p->d_bwd_list, bwd_list)) return st;
    p->n_fwd = (int64_t)fwd.size();
    p->n_bwd = (int64_t)bwd.size();
    p->n_fwd_list = (int64_t)fwd_list.size();
    p->n_bwd_list = (int64_t)bwd_list.size();
    p->bwd_list_max_cols = max_cols;
    p->bwd_list_max_tiles = max_tiles;
    p->fwd_part_floats = fpart;
    p->bwd_part_floats = bpart;
    return MX_OK;
}

size_t plan_ws_bytes(const mx_batch_plan *p) {
    int64_t f, b;
    partial_floats(p->table, p->ntasks, kMinTile, &f, &b);
    return kCounterBytes + align256((size_t)f * 4) + align256((size_t)b * 4);
}

mx_status check_ws(const char *who, const mx_batch_plan *p, void *ws, size_t ws_bytes) {
    MX_REQUIRE(p, MX_ERR_INVALID, "%s: null plan", who);
    MX_REQUIRE(ws && ws_bytes >= p->ws_need && ((uintptr_t)ws & 255) == 0, MX_ERR_WORKSPACE,
               "%s: workspace needs %zu bytes, 256-byte aligned", who, p->ws_need);
    return MX_OK;
}

float *fwd_part_ptr(const mx_batch_plan *p, void *ws) { return (float *)((char *)ws + kCounterBytes); }
float *bwd_part_ptr(const mx_batch_plan *p, void *ws) {
    int64_t f, b;
    partial_floats(p->table, p->ntasks, kMinTile, &f, &b);
    return (float *)((char *)ws + kCounterBytes + align256((size_t)f * 4));
}

// a block per tile, in rows of at most 2^20 blocks
dim3 grid_of(int64_t ntiles) {
    constexpr int64_t kRow = 1 << 20;
    return ntiles <= kRow ? dim3((unsigned)std::max<int64_t>(ntiles, 1)) : dim3((unsigned)kRow, (unsigned)ceil_div(ntiles, kRow));
}
// LDS that a launch asks for so that no more than blocks_per_cu blocks are
// resident on a CU (the kernels' own arrays are `own`; eight blocks forward and
// four backward are what its waves allow).  A backward pass past the caches
// keeps to two: more rows open at once cost more than they hide (forward and
// backward of 889 MB of matrices 767 us with four, 744 us with three, 716 us with
// two), where a small one is all latency (20 000 dots of 0 .. 50 elements 37 us
// with two, 23 us with four).
constexpr unsigned kPastBlocks = 2;
constexpr unsigned kCuLds = 163840, kWaveBlocks = 8;
constexpr unsigned lds_for_blocks(unsigned b) { return b >= kWaveBlocks ? 0u : kCuLds / (b + 1) + 1024u; }
constexpr bool lds_holds_blocks() {
    for (unsigned b = 1; b < kWaveBlocks; ++b)
        if (kCuLds / lds_for_blocks(b) != b) return false;
    return true;
}
static_assert(lds_holds_blocks(), "as many blocks as asked for fit a CU, and no more");
unsigned lds_of(const mx_batch_plan *p, unsigned own, unsigned most = kWaveBlocks) {
    const unsigned per = lds_for_blocks(std::min((unsigned)p->cfg.blocks_per_cu, most));
    return per > own ? per - own : 0u;
}

mx_status fwd_impl(const mx_batch_plan *p, const float *A, const float *B, float *out, void *ws, hipStream_t s) {
    float *part = fwd_part_ptr(p, ws);
    hipLaunchKernelGGL(k_batch_fwd, grid_of(p->n_fwd), dim3(NT), lds_of(p, 4 * (kXLds + kXPad + 16)), s, p->d_fwd, p->n_fwd, A, B, out, part);
    if (p->n_fwd_list > 0)
        hipLaunchKernelGGL(k_batch_combine_fwd, dim3((unsigned)ceil_div(p->n_fwd_list, NT)), dim3(NT), 0, s,
                           p->d_tasks, p->d_fwd_list, p->n_fwd_list, part, out);
    return last_launch("mx_batch_forward");
}

mx_status bwd_impl(const mx_batch_plan *p, const float *A, const float *B, const float *gout, float *gA, float *gB,
                   void *ws, hipStream_t s) {
    float *part = bwd_part_ptr(p, ws);
    const bool past = (p->a_len + p->b_len) * 2 * (int64_t)sizeof(float) > kCacheBytes;
    hipLaunchKernelGGL(past ? k_batch_bwd<true> : k_batch_bwd<false>, grid_of(p->n_bwd), dim3(NB),
                       lds_of(p, 16 * NB, past ? kPastBlocks : kWaveBlocks), s, p->d_bwd, p->n_bwd, A, B, gout, gA, gB, part);
    if (p->n_bwd_list > 0) {
        constexpr int PARTS = 8;
        const bool runs = p->bwd_list_max_tiles > kRunTiles;
        const dim3 cgrid((unsigned)p->n_bwd_list,
                         (unsigned)std::min<int64_t>(1024, ceil_div(p->bwd_list_max_cols, runs ? NT / PARTS : NT)));
        hipLaunchKernelGGL(runs ? k_batch_combine_bwd<PARTS> : k_batch_combine_bwd<1>, cgrid, dim3(NT), 0, s, p->d_tasks,
                           p->d_bwd_list, p->n_bwd_list, part, gB);
    }
    return last_launch("mx_batch_backward");
}

uint64_t fnv1a(const void *data, size_t n, uint64_t h = 1469598103934665603ull) {
    const unsigned char *c = (const unsigned char *)data;
    for (size_t i = 0; i < n; ++i) {
        h ^= c[i];
        h *= 1099511628211ull;
    }
    return h;
}

std::string cache_key(const mx_batch_plan *p) {
    // sizes and kinds only: offsets do not change the work
    std::vector<int64_t> shape;
    shape.reserve((size_t)p->ntasks * 3);
    for (int64_t t = 0; t < p->ntasks; ++t)
        for (int c = 0; c < 3; ++c) shape.push_back(p->table[(size_t)(6 * t + c)]);
    hipDeviceProp_t prop;
    char name[300] = "unknown";
    if (hipGetDeviceProperties(&prop, p->device) == hipSuccess) snprintf(name, sizeof name, "%s", prop.gcnArchName);
    char buf[128];
    snprintf(buf, sizeof buf, "%016llx-%s", (unsigned long long)fnv1a(shape.data(), shape.size() * 8), name);
    return buf;
}

bool cache_lookup(const char *path, const std::string &key, mx_batch_config *cfg) {
    std::ifstream f(path);
    if (!f) return false;
    std::string line;
    bool found = false;
    while (std::getline(f, line)) {
        // one JSON object per line: {"key": "...", "tile_elems": N, "blocks_per_cu": M, "us": X}
        if (line.find("\"" + key + "\"") == std::string::npos) continue;
        int te = 0, bpc = 0;
        const size_t a = line.find("\"tile_elems\":"), b = line.find("\"blocks_per_cu\":");
        if (a == std::string::npos || b == std::string::npos) continue;
        te = std::atoi(line.c_str() + a + 13);
        bpc = std::atoi(line.c_str() + b + 16);
        if (te >= kMinTile && bpc >= 1 && bpc <= 32) {
            cfg->tile_elems = te;
            cfg->blocks_per_cu = bpc;
            found = true;  // the last matching line wins
        }
    }
    return found;
}

}  // namespace

extern "C" {

mx_status mx_batch_plan_create(const int64_t *table_host, int64_t ntasks, const mx_batch_config *cfg,
                               mx_batch_plan **plan) {
    MX_REQUIRE(plan, MX_ERR_INVALID, "mx_batch_plan_create: null output");
    *plan = nullptr;
    MX_REQUIRE(ntasks >= 0 && ntasks < (1LL << 31), MX_ERR_SHAPE, "mx_batch_plan_create: bad ntasks");
    MX_REQUIRE(ntasks == 0 || table_host, MX_ERR_INVALID, "mx_batch_plan_create: null table");
    const DeviceInfo *d;
    if (mx_status st = device_info(&d)) return st;
    auto *p = new mx_batch_plan();
    p->device = d->device;
    p->ntasks = ntasks;
    p->table.assign(table_host, table_host + 6 * ntasks);
    for (int64_t t = 0; t < ntasks; ++t) {
        const int64_t *r = table_host + 6 * t;
        if (!((r[0] == kDot && r[1] == 1) || r[0] == kMatvec) || r[1] < 0 || r[2] < 0 || r[3] < 0 || r[4] < 0 ||
            r[5] < 0) {
            delete p;
            return set_error(MX_ERR_SHAPE, "mx_batch_plan_create: bad task %lld", (long long)t);
        }
        p->a_len = std::max(p->a_len, r[3] + r[1] * r[2]);
        p->b_len = std::max(p->b_len, r[4] + r[2]);
        p->out_len = std::max(p->out_len, r[5] + (r[0] == kDot ? 1 : r[1]));
    }
    p->cfg.tile_elems = cfg ? cfg->tile_elems : 16384;
    p->cfg.blocks_per_cu = cfg ? cfg->blocks_per_cu : 8;
    if (p->cfg.tile_elems < kMinTile || p->cfg.blocks_per_cu < 1 || p->cfg.blocks_per_cu > 32) {
        delete p;
        return set_error(MX_ERR_INVALID, "mx_batch_plan_create: need tile_elems >= %d and 1 <= blocks_per_cu <= 32",
                         kMinTile);
    }
    p->ws_need = plan_ws_bytes(p);
    if (mx_status st = build_tiles(p)) {
        free_device(p);
        delete p;
        return st;
    }
    *plan = p;
    return MX_OK;
}

mx_status mx_batch_plan_destroy(mx_batch_plan *plan) {
    if (!plan) return MX_OK;
    free_device(plan);
    delete plan;
    return MX_OK;
}

size_t mx_batch_workspace_bytes(const mx_batch_plan *plan) { return plan ? plan->ws_need : 0; }

mx_status mx_batch_get_config(const mx_batch_plan *plan, mx_batch_config *cfg) {
    MX_REQUIRE(plan && cfg, MX_ERR_INVALID, "mx_batch_get_config: null pointer");
    *cfg = plan->cfg;
    return MX_OK;
}

mx_status mx_batch_set_config(mx_batch_plan *plan, const mx_batch_config *cfg) {
    MX_REQUIRE(plan && cfg, MX_ERR_INVALID, "mx_batch_set_config: null pointer");
    MX_REQUIRE(cfg->tile_elems >= kMinTile && cfg->blocks_per_cu >= 1 && cfg->blocks_per_cu <= 32, MX_ERR_INVALID,
               "mx_batch_set_config: need tile_elems >= %d and 1 <= blocks_per_cu <= 32", kMinTile);
    plan->cfg.tile_elems = cfg->tile_elems;
    plan->cfg.blocks_per_cu = cfg->blocks_per_cu;
    return build_tiles(plan);
}

mx_status mx_batch_forward(const mx_batch_plan *plan, const float *A_dev, const float *B_dev, float *out_dev,
                           void *ws, size_t ws_bytes, hipStream_t stream) {
    if (mx_status st = check_ws("mx_batch_forward", plan, ws, ws_bytes)) return st;
    if (plan->ntasks == 0) return MX_OK;
    MX_REQUIRE(A_dev && B_dev && out_dev, MX_ERR_INVALID, "mx_batch_forward: null pointer");
    return fwd_impl(plan, A_dev, B_dev, out_dev, ws, stream);
}

mx_status mx_batch_backward(const mx_batch_plan *plan, const float *A_dev, const float *B_dev, const float *gout_dev,
                            float *gA_dev, float *gB_dev, void *ws, size_t ws_bytes, hipStream_t stream) {
    if (mx_status st = check_ws("mx_batch_backward", plan, ws, ws_bytes)) return st;
    if (plan->ntasks == 0) return MX_OK;
    MX_REQUIRE(A_dev && B_dev && gout_dev && gA_dev && gB_dev, MX_ERR_INVALID, "mx_batch_backward: null pointer");
    return bwd_impl(plan, A_dev, B_dev, gout_dev, gA_dev, gB_dev, ws, stream);
}

mx_status mx_batch_forward_plain(const mx_batch_plan *plan, const float *A_dev, const float *B_dev, float *out_dev,
                                 hipStream_t stream) {
    MX_REQUIRE(plan, MX_ERR_INVALID, "mx_batch_forward_plain: null plan");
    if (plan->ntasks == 0) return MX_OK;
    MX_REQUIRE(A_dev && B_dev && out_dev, MX_ERR_INVALID, "mx_batch_forward_plain: null pointer");
    for (int64_t t = 0; t < plan->ntasks; ++t) {
        const int64_t *r = &plan->table[(size_t)(6 * t)];
        if (r[0] == kDot)
            hipLaunchKernelGGL(k_dot_plain, dim3(1), dim3(NT), 0, stream, A_dev + r[3], B_dev + r[4], r[2],
                               out_dev + r[5]);
        else if (r[1] > 0)
            hipLaunchKernelGGL(k_matvec_plain, dim3((unsigned)ceil_div(r[1], NT)), dim3(NT), 0, stream, A_dev + r[3],
                               B_dev + r[4], r[1], r[2], out_dev + r[5]);
    }
    return last_launch("mx_batch_forward_plain");
}

mx_status mx_batch_backward_plain(const mx_batch_plan *plan, const float *A_dev, const float *B_dev,
                                  const float *gout_dev, float *gA_dev, float *gB_dev, hipStream_t stream) {
    MX_REQUIRE(plan, MX_ERR_INVALID, "mx_batch_backward_plain: null plan");
    if (plan->ntasks == 0) return MX_OK;
    MX_REQUIRE(A_dev && B_dev && gout_dev && gA_dev && gB_dev, MX_ERR_INVALID, "mx_batch_backward_plain: null pointer");
    for (int64_t t = 0; t < plan->ntasks; ++t) {
        const int64_t *r = &plan->table[(size_t)(6 * t)];
        if (r[0] == kDot) {
            if (r[2] > 0)
                hipLaunchKernelGGL(k_dot_adj_plain, dim3((unsigned)ceil_div(r[2], NT)), dim3(NT), 0, stream,
                                   A_dev + r[3], B_dev + r[4], r[2], gout_dev + r[5], gA_dev + r[3], gB_dev + r[4]);
        } else if (r[2] > 0) {
            hipLaunchKernelGGL(k_matvec_adj_plain, dim3((unsigned)ceil_div(r[2], NT)), dim3(NT), 0, stream,
                               A_dev + r[3], B_dev + r[4], r[1], r[2], gout_dev + r[5], gA_dev + r[3], gB_dev + r[4]);
        }
    }
    return last_launch("mx_batch_backward_plain");
}

mx_status mx_batch_autotune(mx_batch_plan *plan, const float *A_dev, const float *B_dev, float *out_dev,
                            const float *gout_dev, float *gA_dev, float *gB_dev, void *ws, size_t ws_bytes,
                            const char *cache_path, hipStream_t stream, mx_batch_config *chosen) {
    const char *who = "mx_batch_autotune";
    if (mx_status st = check_ws(who, plan, ws, ws_bytes)) return st;
    MX_REQUIRE(A_dev && B_dev && out_dev && gout_dev && gA_dev && gB_dev, MX_ERR_INVALID, "%s: null pointer", who);
    const std::string key = cache_key(plan);
    mx_batch_config best = plan->cfg;
    if (cache_path && cache_lookup(cache_path, key, &best)) {
        if (mx_status st = mx_batch_set_config(plan, &best)) return st;
        if (chosen) *chosen = plan->cfg;
        return MX_OK;
    }
    static const int tiles[] = {4096, 8192, 16384, 32768, 65536};
    static const int bpcs[] = {2, 4, 8};  // more than eight are the same launches
    hipEvent_t e0, e1;
    MX_TRY_HIP(hipEventCreate(&e0));
    MX_TRY_HIP(hipEventCreate(&e1));
    float best_us = 1e30f;
    mx_status rc = MX_OK;
    for (int te : tiles) {
        for (int bpc : bpcs) {
            mx_batch_config c{te, bpc, {0, 0}};
            if ((rc = mx_batch_set_config(plan, &c))) goto done;
            // one warm pass, then the minimum of three timed passes of forward + backward
            if ((rc = fwd_impl(plan, A_dev, B_dev, out_dev, ws, stream))) goto done;
            if ((rc = bwd_impl(plan, A_dev, B_dev, gout_dev, gA_dev, gB_dev, ws, stream))) goto done;
            float tmin = 1e30f;
            for (int rep = 0; rep < 3; ++rep) {
                if (hipEventRecord(e0, stream) != hipSuccess) { rc = hip_error(hipGetLastError(), "hipEventRecord"); goto done; }
                if ((rc = fwd_impl(plan, A_dev, B_dev, out_dev, ws, stream))) goto done;
                if ((rc = bwd_impl(plan, A_dev, B_dev, gout_dev, gA_dev, gB_dev, ws, stream))) goto done;
                if (hipEventRecord(e1, stream) != hipSuccess) { rc = hip_error(hipGetLastError(), "hipEventRecord"); goto done; }
                if (hipEventSynchronize(e1) != hipSuccess) { rc = hip_error(hipGetLastError(), "hipEventSynchronize"); goto done; }
                float ms = 0.f;
                (void)hipEventElapsedTime(&ms, e0, e1);
                tmin = std::min(tmin, ms * 1000.f);
            }
            if (tmin < best_us) {
                best_us = tmin;
                best = c;
            }
        }
    }
    if ((rc = mx_batch_set_config(plan, &best))) goto done;
    if (cache_path) {
        FILE *f = fopen(cache_path, "a");
        if (f) {
            fprintf(f, "{\"key\": \"%s\", \"tile_elems\": %d, \"blocks_per_cu\": %d, \"us\": %.1f}\n", key.c_str(),
                    best.tile_elems, best.blocks_per_cu, best_us);
            fclose(f);
        }
    }
    if (chosen) *chosen = plan->cfg;
done:
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}

}  // extern "C"
