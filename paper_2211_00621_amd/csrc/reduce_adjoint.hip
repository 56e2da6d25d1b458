// Reverse of reduce min / max, flat and per ragged row (derived; the paper
// has no reverse mode).  reduce op ne s is the left fold of op from ne, and
// min / max replace the accumulator only when an element is strictly below
// (above) it, so the result is the element at the lowest index attaining the
// extreme, or ne itself when no element improves on ne.  That element
// receives the upstream gradient; every other element receives 0.
//
// The index is found as the lexicographic best of (value, index) pairs --
// smallest (largest) value first, then lowest index -- with ne standing at
// index -1: an associative and commutative operation, so the tree order of
// the reduction does not change the result: the arg is exact and
// deterministic.  A NaN element never compares below or equal to anything,
// so it is never chosen, as in the fold.
#include "mx_internal.h"

namespace mx {
namespace {

constexpr int NT = 256;
constexpr int kMaxArgBlocks = 2048;  // partial pairs fit MX_WS_REDUCE's 32 KiB
constexpr int64_t kNone = INT64_MAX;

// (v, i) improves on (bv, bi): strictly better value, or the same value at a
// lower index
template <int OP>
__device__ __forceinline__ bool better(float v, int64_t i, float bv, int64_t bi) {
    if (OP == MX_MIN) return v < bv || (v == bv && i < bi);
    return v > bv || (v == bv && i < bi);
}

template <int OP> __device__ __forceinline__ float ident() {
    return OP == MX_MIN ? __builtin_huge_valf() : -__builtin_huge_valf();
}

template <int OP> __device__ __forceinline__ void take(float v, int64_t i, float &bv, int64_t &bi) {
    if (better<OP>(v, i, bv, bi)) {
        bv = v;
        bi = i;
    }
}

template <int OP> __device__ __forceinline__ void wave_argreduce(float &bv, int64_t &bi) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const float ov = __shfl_xor(bv, off, kWave);
        const int64_t oi = __shfl_xor(bi, off, kWave);
        take<OP>(ov, oi, bv, bi);
    }
}

// all threads of the block; the block's pair in every thread
template <int OP> __device__ __forceinline__ void block_argreduce(float &bv, int64_t &bi) {
    __shared__ float sv[NT / kWave];
    __shared__ int64_t si[NT / kWave];
    wave_argreduce<OP>(bv, bi);
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        sv[w] = bv;
        si[w] = bi;
    }
    __syncthreads();
    bv = sv[0];
    bi = si[0];
#pragma unroll
    for (int k = 1; k < NT / kWave; ++k) take<OP>(sv[k], si[k], bv, bi);
    __syncthreads();
}

// Partial pass: a block scans contiguous chunks of C x 256 16-byte vectors of any
// alignment, all loads of a chunk in flight, for its threads' best pairs and
// writes zeros to gx on the way; one pair per block.  Bound by HBM: 2^26 elements
// (537 MB in and out) 99 us with the finish (5.4 TB/s), 111 us with one vector
// in flight and a grid-wide stride; 2^22 9.5 us, 11.3 us.  A small pass goes by the
// chunks of the others, and its zeros stay near.
constexpr int C = 4;
__host__ __device__ constexpr int64_t chunk_of(int64_t nv) { return nv <= kSmallPass ? NT : C * NT; }
template <int OP>
__global__ void __launch_bounds__(NT) k_arg_partial(const float *__restrict__ x, int64_t n, float *__restrict__ gx,
                                                    float *__restrict__ pv, int64_t *__restrict__ pi) {
    float bv = ident<OP>();
    int64_t bi = kNone;
    const uvec<float> zero = {0.f, 0.f, 0.f, 0.f};
    const int64_t nv = n / 4, chunk = chunk_of(nv);
    auto scan = [&](const uvec<float> &q, int64_t j) {
#pragma unroll
        for (int e = 0; e < 4; ++e) take<OP>(q[e], 4 * j + e, bv, bi);
    };
    for (int64_t c = (int64_t)blockIdx.x * chunk; c < nv; c += (int64_t)gridDim.x * chunk) {
        const int64_t j = c + threadIdx.x, end = c + chunk < nv ? c + chunk : nv;
        if (end - c == C * NT) {
            uvec<float> q[C];
#pragma unroll
            for (int u = 0; u < C; ++u) q[u] = load16<false>(x + 4 * (j + u * NT));
#pragma unroll
            for (int u = 0; u < C; ++u) {
                scan(q[u], j + u * NT);
                store16(zero, gx + 4 * (j + u * NT));
            }
        } else {
            for (int64_t i = j; i < end; i += NT) {
                scan(load16<false>(x + 4 * i), i);
                store16_near(zero, gx + 4 * i);
            }
        }
    }
    const int64_t i = 4 * nv + threadIdx.x;  // the last n % 4 elements
    if (blockIdx.x == gridDim.x - 1 && i < n) {
        take<OP>(x[i], i, bv, bi);
        gx[i] = 0.f;
    }
    block_argreduce<OP>(bv, bi);
    if (threadIdx.x == 0) {
        pv[blockIdx.x] = bv;
        pi[blockIdx.x] = bi;
    }
}

// Finish (one block): the best of the partials and of (ne, -1); its element
// receives *gout.  Ordered after the partial pass by the kernel boundary, so
// the store lands on the zeros written there.
template <int OP>
__global__ void __launch_bounds__(NT) k_arg_finish(const float *__restrict__ pv, const int64_t *__restrict__ pi,
                                                   int np, float ne, const float *__restrict__ gout,
                                                   float *__restrict__ gx) {
    float bv = ident<OP>();
    int64_t bi = kNone;
    for (int k = threadIdx.x; k < np; k += NT) take<OP>(pv[k], pi[k], bv, bi);
    block_argreduce<OP>(bv, bi);
    if (threadIdx.x == 0) {
        take<OP>(ne, -1, bv, bi);
        // a NaN ne is never improved on by the fold (no comparison with it holds)
        if (bi >= 0 && bi != kNone && ne == ne) gx[bi] = gout[0];
    }
}

// A group of G lanes per ragged row, a wave, or a 16-lane DPP row where rows are
// short (rows grid-strided over the waves): the row's best pair, then the row
// written as g at the arg and 0 elsewhere.  Reads and writes go in 16-byte vectors
// at 4-byte alignment, four per lane in flight; the best value by the DPP tree,
// then the lowest index among the lanes that hold it.  HBM bound at 65 536 rows of
// mean length 490 (32 M values, 256 MB in and out): 40 us (6.4 TB/s, the last-level
// cache serving part); 89 us with one element per lane and pass and 64-bit pairs
// shuffled.
//
// A row past kRounds rounds of 16 lanes' loads is taken by its whole wave (in a
// vector per lane, since registers for more would cost the others a wave per SIMD): 262 144
// rows of mean length 45, twenty of them of 524 288, took 2.7 ms with a wave and one
// element per lane for every row, 7.4 ms with 16 lanes.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// v at index i improves on bv.  A thread's indices rise, so of equal values the
// lowest index stays; an element equal to the identity never improves on ne, so
// it needs no index.
template <int OP> __device__ __forceinline__ void scan(float v, int64_t i, float &bv, int64_t &bi) {
    if (OP == MX_MIN ? v < bv : v > bv) {
        bv = v;
        bi = i;
    }
}

// row x[0 .. n) with its gradient y, by lane `lane` of L, U vectors in flight (all
// lanes of the wave active)
template <int OP, int L, int U>
__device__ __forceinline__ void arg_row(const float *__restrict__ x, float *__restrict__ y, int64_t n, int lane, float ne,
                                        float g) {
    const int64_t nv = n / 4;
    float bv = ident<OP>();
    int64_t bi = kNone;
    for (int64_t i = lane; i < nv; i += U * L) {
        f4u q[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * L < nv) q[u] = *reinterpret_cast<const f4u *>(x + 4 * (i + u * L));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * L < nv) {
#pragma unroll
                for (int c = 0; c < 4; ++c) scan<OP>(q[u][c], 4 * (i + u * L) + c, bv, bi);
            }
    }
    if (4 * nv + lane < n) scan<OP>(x[4 * nv + lane], 4 * nv + lane, bv, bi);
    using B = Red<OP, float>;
    using I = Red<MX_MIN, int64_t>;
    const float best = group_reduce<B, L>(bv);
    int64_t at = group_reduce<I, L>(bv == best ? bi : kNone);
    // ne stands at index -1; a NaN ne is never improved on by the fold
    if (!better<OP>(best, 0, ne, -1)) at = kNone;
    for (int64_t i = lane; i < nv; i += L) {
        f4u z = f4u{0.f, 0.f, 0.f, 0.f};
        const int64_t c = at - 4 * i;
        if (c >= 0 && c < 4) {
            z.x = c == 0 ? g : 0.f;
            z.y = c == 1 ? g : 0.f;
            z.z = c == 2 ? g : 0.f;
            z.w = c == 3 ? g : 0.f;
        }
        *reinterpret_cast<f4u *>(y + 4 * i) = z;
    }
    if (4 * nv + lane < n) y[4 * nv + lane] = 4 * nv + lane == at ? g : 0.f;
}

template <int OP, int G>
__global__ void __launch_bounds__(NT) k_seg_arg(const float *__restrict__ values, const int64_t *__restrict__ offsets,
                                                int64_t nseg, float ne, const float *__restrict__ gout,
                                                float *__restrict__ gvalues) {
    constexpr int kRounds = 4;
    const int lane = threadIdx.x % G;
    const int64_t ng = (int64_t)gridDim.x * (NT / G);
    // the groups of a wave stay together (their rows may differ): all lanes
    // take part in the reductions
    for (int64_t r0 = (int64_t)blockIdx.x * (NT / G) + threadIdx.x / kWave * (kWave / G); r0 < nseg; r0 += ng) {
        const int64_t r = r0 + threadIdx.x % kWave / G;
        const bool has = r < nseg;
        const int64_t s = has ? offsets[r] : 0, e = has ? offsets[r + 1] : 0;
        const float g = has ? gout[r] : 0.f;
        const bool far = G < kWave && e - s > (int64_t)kRounds * 16 * G;
        arg_row<OP, G, 4>(values + s, gvalues + s, far ? 0 : e - s, lane, ne, g);
        if constexpr (G < kWave)
            for (uint64_t m = __ballot(far && lane == 0); m; m &= m - 1) {
                const int o = __builtin_ctzll(m);
                const int64_t fs = read_lane(s, o), fe = read_lane(e, o);
                arg_row<OP, kWave, 1>(values + fs, gvalues + fs, fe - fs, threadIdx.x % kWave, ne, read_lane(g, o));
            }
    }
}

__global__ void __launch_bounds__(NT) k_fill_from(const float *__restrict__ g, int64_t n, float *__restrict__ out) {
    const float v = g[0];
    const int64_t nt = (int64_t)gridDim.x * NT;
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += nt) out[i] = v;
}

}  // namespace
}  // namespace mx

using namespace mx;

extern "C" {

mx_status mx_reduce_adjoint_f32(mx_redop op, const float *x_dev, int64_t n, const float *ne_host,
                                const float *gout_dev, float *gx_dev, void *ws, size_t ws_bytes, hipStream_t stream) {
    const char *who = "mx_reduce_adjoint_f32";
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "%s: n < 0", who);
    MX_REQUIRE(op == MX_ADD || op == MX_MIN || op == MX_MAX,
               op == MX_MUL ? MX_ERR_UNSUPPORTED : MX_ERR_INVALID, "%s: operator %d has no reverse here", who,
               (int)op);
    MX_REQUIRE(ne_host && gout_dev, MX_ERR_INVALID, "%s: null ne or gout", who);
    if (n == 0) return MX_OK;
    MX_REQUIRE(x_dev && gx_dev, MX_ERR_INVALID, "%s: null x or gx", who);
    MX_REQUIRE(gx_dev != x_dev, MX_ERR_INVALID, "%s: gx must not alias x", who);
    const DeviceInfo *d;
    if (mx_status st = device_info(&d)) return st;
    if (op == MX_ADD) {
        int64_t grid = ceil_div(n, NT);
        if (grid > (int64_t)d->num_cus * 8) grid = (int64_t)d->num_cus * 8;
        hipLaunchKernelGGL(k_fill_from, dim3((unsigned)grid), dim3(NT), 0, stream, gout_dev, n, gx_dev);
        return last_launch(who);
    }
    const size_t need = mx_workspace_bytes(MX_WS_REDUCE, n, 0);
    MX_REQUIRE(ws && ws_bytes >= need && ((uintptr_t)ws & 255) == 0, MX_ERR_WORKSPACE,
               "%s: workspace needs %zu bytes, 256-byte aligned", who, need);
    int64_t grid = ceil_div(n, 4 * chunk_of(n / 4));
    int64_t cap = (int64_t)d->num_cus * 8;
    if (cap > kMaxArgBlocks) cap = kMaxArgBlocks;
    if (grid > cap) grid = cap;
    float *pv = (float *)((char *)ws + kCounterBytes);
    int64_t *pi = (int64_t *)((char *)ws + kCounterBytes + kMaxArgBlocks * sizeof(float));
    const float ne = *ne_host;
    if (op == MX_MIN) {
        hipLaunchKernelGGL(k_arg_partial<MX_MIN>, dim3((unsigned)grid), dim3(NT), 0, stream, x_dev, n, gx_dev, pv, pi);
        hipLaunchKernelGGL(k_arg_finish<MX_MIN>, dim3(1), dim3(NT), 0, stream, pv, pi, (int)grid, ne, gout_dev, gx_dev);
    } else {
        hipLaunchKernelGGL(k_arg_partial<MX_MAX>, dim3((unsigned)grid), dim3(NT), 0, stream, x_dev, n, gx_dev, pv, pi);
        hipLaunchKernelGGL(k_arg_finish<MX_MAX>, dim3(1), dim3(NT), 0, stream, pv, pi, (int)grid, ne, gout_dev, gx_dev);
    }
    return last_launch(who);
}

mx_status mx_segmented_reduce_adjoint_f32(mx_redop op, const float *values_dev, int64_t nvalues,
                                          const int64_t *offsets_dev, int64_t nseg, const float *ne_host,
                                          const float *gout_dev, float *gvalues_dev, hipStream_t stream) {
    const char *who = "mx_segmented_reduce_adjoint_f32";
    MX_REQUIRE(nseg >= 0 && nvalues >= 0, MX_ERR_SHAPE, "%s: nseg < 0 or nvalues < 0", who);
    MX_REQUIRE(op == MX_ADD || op == MX_MIN || op == MX_MAX,
               op == MX_MUL ? MX_ERR_UNSUPPORTED : MX_ERR_INVALID, "%s: operator %d has no reverse here", who,
               (int)op);
    MX_REQUIRE(ne_host, MX_ERR_INVALID, "%s: null ne", who);
    if (nseg == 0) return MX_OK;
    MX_REQUIRE(offsets_dev && gout_dev && (gvalues_dev || nvalues == 0), MX_ERR_INVALID, "%s: null pointer", who);
    if (op == MX_ADD) return mx_segmented_sum_adjoint_f32(gout_dev, offsets_dev, nseg, gvalues_dev, nvalues, stream);
    MX_REQUIRE(values_dev, MX_ERR_INVALID, "%s: null values", who);
    MX_REQUIRE(gvalues_dev != values_dev, MX_ERR_INVALID, "%s: gvalues must not alias values", who);
    if (mx_status st = check_offsets_debug(who, offsets_dev, nseg, stream)) return st;
    const DeviceInfo *d;
    if (mx_status st = device_info(&d)) return st;
    // lanes per row by mean length; with few rows a wave each costs nothing (4000
    // rows of mean 143: 3.9 us against 5.7 us with 16 lanes; 65 536 of mean 79:
    // 20.4 us against 10; 300 of mean 7 2.3 against 2.6, 3000 2.8 against 2.2)
    const int group = (nvalues <= 64 * nseg && nseg >= 1024) || (nvalues <= 160 * nseg && nseg >= 16384) ? 16 : kWave;
    int64_t grid = ceil_div(nseg, NT / group);
    if (grid > (int64_t)d->num_cus * 16) grid = (int64_t)d->num_cus * 16;
    const float ne = *ne_host;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NT), 0, stream, values_dev, offsets_dev, nseg, ne, gout_dev,
                           gvalues_dev);
    };
    if (op == MX_MIN) group == 16 ? go(k_seg_arg<MX_MIN, 16>) : go(k_seg_arg<MX_MIN, kWave>);
    else group == 16 ? go(k_seg_arg<MX_MAX, 16>) : go(k_seg_arg<MX_MAX, kWave>);
    return last_launch(who);
}

}  // extern "C"
