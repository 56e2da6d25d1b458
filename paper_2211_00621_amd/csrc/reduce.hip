// reduce op ne s and the fused reduce op ne (map2 f a b) (Appendix A).
//
// Two launches.  Partial pass: a block folds contiguous chunks of U x 256 16-byte
// vectors per operand (of 256 where the input is small), all of a chunk in flight,
// into one accumulator per vector lane, and each chunk's into one of all its
// chunks; it combines them with the wave64 DPP tree and writes one partial.  Finish
// pass (one block): folds the partials in block order and applies ne.  The kernel
// boundary orders the two passes, so no block pays for a device-wide fence.  An
// input of a few chunks is one block's work, and one launch.  The bracketing
// depends only on n and the device, so results are bit-identical from run to run,
// whatever the alignment.
//
// Bound by HBM; plain loads, which leave the last part of the inputs in the
// memory-side cache for a reverse pass.  The dot of 2^26 pairs of float32
// (537 MB) 97.5 us -> 92.8 us with the finish launch (5.8 TB/s), of 2^24
// 26.7 us -> 23.5 us, against grid-wide strides; the dot and its adjoint at 2^26
// 338 us -> 242 us.
#include <algorithm>

#include "mx_internal.h"

namespace mx {
namespace {

constexpr int NT = 256;
constexpr int U = 4;
constexpr int kMaxBlocks = 4096;
constexpr int NT1 = 1024;  // threads of a block that folds a small input alone
__host__ __device__ constexpr int64_t chunk_of(int64_t nv) { return nv <= kSmallPass ? NT : U * NT; }

// F < 0: plain reduce of a; otherwise element = Bin<F>(a[i], b[i]).
template <mx_dtype D, int OP, int F> struct Elem {
    using Acc = typename DT<D>::Acc;
    using In = typename DT<D>::In;
    static __device__ __forceinline__ Acc at(In x, In y) {
        if constexpr (F < 0) return Acc(x);
        else return Bin<F, Acc>::ap(Acc(x), Acc(y));
    }
};

// A small input by one block, in one launch (the host side of a second is 3 us):
// up to U vectors per thread and operand, all in flight, since an input that the
// call before has written past the caches takes a round trip to memory (2^14
// floats, map then sum: four rounds of a block of 256 threads 5.9 us, now 4.1 us, two
// launches 5.4 us).
template <mx_dtype D, int OP, int F, int T>
__global__ void __launch_bounds__(T) k_reduce_one(const typename DT<D>::In *__restrict__ a,
                                                  const typename DT<D>::In *__restrict__ b, int n,
                                                  typename DT<D>::Acc ne, typename DT<D>::Acc *__restrict__ out) {
    using In = typename DT<D>::In;
    using Acc = typename DT<D>::Acc;
    using R = Red<OP, Acc>;
    using E = Elem<D, OP, F>;
    constexpr int V = DT<D>::kVec;
    constexpr bool TWO = F >= 0;
    __shared__ Acc smem[T / kWave];
    const int nv = n / V, t = threadIdx.x;
    uvec<In> va[U], vb[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (t + u * T < nv) {
            va[u] = load16<false>(a + V * (t + u * T));
            if constexpr (TWO) vb[u] = load16<false>(b + V * (t + u * T));
        }
    const int i = nv * V + t;  // the last n % V elements
    const In ta = i < n ? a[i] : In(0), tb = TWO && i < n ? b[i] : In(0);
    Acc acc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = R::id();
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (t + u * T < nv)
#pragma unroll
            for (int j = 0; j < V; ++j) acc[j] = R::ap(acc[j], E::at(va[u][j], TWO ? vb[u][j] : In(0)));
    if (i < n) acc[0] = R::ap(acc[0], E::at(ta, tb));
    Acc r = acc[0];
#pragma unroll
    for (int j = 1; j < V; ++j) r = R::ap(r, acc[j]);
    r = block_reduce<R, T>(r, smem);
    if (t == 0) out[0] = R::ap(ne, r);
}

template <mx_dtype D, int OP, int F>
__global__ void __launch_bounds__(NT) k_reduce(const typename DT<D>::In *__restrict__ a,
                                               const typename DT<D>::In *__restrict__ b, int64_t n,
                                               typename DT<D>::Acc *__restrict__ partials) {
    using In = typename DT<D>::In;
    using Acc = typename DT<D>::Acc;
    using R = Red<OP, Acc>;
    using E = Elem<D, OP, F>;
    constexpr int V = DT<D>::kVec;
    constexpr bool TWO = F >= 0;
    __shared__ Acc smem[NT / kWave];

    Acc acc[V], sum[V];
#pragma unroll
    for (int j = 0; j < V; ++j) sum[j] = R::id();
    auto fold = [&](const uvec<In> &va, const uvec<In> &vb) {
#pragma unroll
        for (int j = 0; j < V; ++j) acc[j] = R::ap(acc[j], E::at(va[j], TWO ? vb[j] : In(0)));
    };
    const int64_t nv = n / V, chunk = chunk_of(nv), tail = nv * V + threadIdx.x;
    const bool last = blockIdx.x == gridDim.x - 1 && tail < n;  // one of the last n % V elements
    const In ta = last ? a[tail] : In(0), tb = TWO && last ? b[tail] : In(0);
    for (int64_t c = (int64_t)blockIdx.x * chunk; c < nv; c += (int64_t)gridDim.x * chunk) {
        const int64_t i = c + threadIdx.x, end = c + chunk < nv ? c + chunk : nv;
#pragma unroll
        for (int j = 0; j < V; ++j) acc[j] = R::id();
        if (end - c == U * NT) {
            uvec<In> va[U], vb[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                va[u] = load16<false>(a + V * (i + u * NT));
                if constexpr (TWO) vb[u] = load16<false>(b + V * (i + u * NT));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) fold(va[u], vb[u]);
        } else {
            for (int64_t j = i; j < end; j += NT) {
                const uvec<In> va = load16<false>(a + V * j);
                fold(va, TWO ? load16<false>(b + V * j) : va);
            }
        }
#pragma unroll
        for (int j = 0; j < V; ++j) sum[j] = R::ap(sum[j], acc[j]);
    }
    if (last) sum[0] = R::ap(sum[0], E::at(ta, tb));
    Acc t = sum[0];
#pragma unroll
    for (int j = 1; j < V; ++j) t = R::ap(t, sum[j]);
    t = block_reduce<R, NT>(t, smem);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// one block: out = ne (op) (partial_0 (op) ... (op) partial_{nb-1}), strided
// per thread (eight loads in flight), then the DPP tree
template <mx_dtype D, int OP>
__global__ void __launch_bounds__(NT) k_reduce_finish(const typename DT<D>::Acc *__restrict__ partials, int nb,
                                                      typename DT<D>::Acc ne, typename DT<D>::Acc *out) {
    using Acc = typename DT<D>::Acc;
    using R = Red<OP, Acc>;
    __shared__ Acc smem[NT / kWave];
    Acc v = R::id();
    for (int i = threadIdx.x; i < nb; i += 8 * NT) {
        Acc p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = i + u * NT < nb ? partials[i + u * NT] : R::id();
#pragma unroll
        for (int u = 0; u < 8; ++u) v = R::ap(v, p[u]);
    }
    v = block_reduce<R, NT>(v, smem);
    if (threadIdx.x == 0) out[0] = R::ap(ne, v);
}

template <mx_dtype D, int OP, int F>
mx_status launch(const void *a, const void *b, int64_t n, const void *ne_host, void *out, void *ws,
                 hipStream_t s, const DeviceInfo *dev) {
    using In = typename DT<D>::In;
    using Acc = typename DT<D>::Acc;
    Acc ne;
    __builtin_memcpy(&ne, ne_host, sizeof(Acc));
    const In *x = (const In *)a, *y = (const In *)b;
    const int64_t nv = n / DT<D>::kVec;
    auto one = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(threads), 0, s, x, y, (int)n, ne, (Acc *)out);
        return last_launch("reduce");
    };
    if (nv <= U * NT) return one(k_reduce_one<D, OP, F, NT>, NT);
    if (nv <= U * NT1) return one(k_reduce_one<D, OP, F, NT1>, NT1);
    const int64_t grid = std::min<int64_t>(ceil_div(nv, chunk_of(nv)), std::min<int64_t>((int64_t)dev->num_cus * 8, kMaxBlocks));
    Acc *partials = (Acc *)((char *)ws + kCounterBytes);
    hipLaunchKernelGGL((k_reduce<D, OP, F>), dim3((unsigned)grid), dim3(NT), 0, s, x, y, n, partials);
    if (mx_status st = last_launch("reduce")) return st;
    hipLaunchKernelGGL((k_reduce_finish<D, OP>), dim3(1), dim3(NT), 0, s, (const Acc *)partials, (int)grid, ne,
                       (Acc *)out);
    return last_launch("reduce finish");
}

template <mx_dtype D, int F>
mx_status by_op(int op, const void *a, const void *b, int64_t n, const void *ne, void *out, void *ws,
                hipStream_t s, const DeviceInfo *dev) {
    switch (op) {
    case MX_ADD: return launch<D, MX_ADD, F>(a, b, n, ne, out, ws, s, dev);
    case MX_MUL: return launch<D, MX_MUL, F>(a, b, n, ne, out, ws, s, dev);
    case MX_MIN: return launch<D, MX_MIN, F>(a, b, n, ne, out, ws, s, dev);
    case MX_MAX: return launch<D, MX_MAX, F>(a, b, n, ne, out, ws, s, dev);
    }
    return set_error(MX_ERR_INVALID, "unknown reduce operator %d", op);
}

template <mx_dtype D>
mx_status by_f(int f, int op, const void *a, const void *b, int64_t n, const void *ne, void *out,
               void *ws, hipStream_t s, const DeviceInfo *dev) {
    switch (f) {
    case -1: return by_op<D, -1>(op, a, b, n, ne, out, ws, s, dev);
    case MX_B_ADD: return by_op<D, MX_B_ADD>(op, a, b, n, ne, out, ws, s, dev);
    case MX_B_SUB: return by_op<D, MX_B_SUB>(op, a, b, n, ne, out, ws, s, dev);
    case MX_B_MUL: return by_op<D, MX_B_MUL>(op, a, b, n, ne, out, ws, s, dev);
    case MX_B_MIN: return by_op<D, MX_B_MIN>(op, a, b, n, ne, out, ws, s, dev);
    case MX_B_MAX: return by_op<D, MX_B_MAX>(op, a, b, n, ne, out, ws, s, dev);
    case MX_B_DIV:
        if constexpr (D == MX_F32 || D == MX_F64) return by_op<D, MX_B_DIV>(op, a, b, n, ne, out, ws, s, dev);
        else return set_error(MX_ERR_DTYPE, "division needs a floating-point type");
    }
    return set_error(MX_ERR_INVALID, "unknown map2 body %d", f);
}

mx_status run(const char *who, int f, int op, mx_dtype dtype, const void *a, const void *b,
              int64_t n, const void *ne, void *out, void *ws, size_t ws_bytes, hipStream_t s) {
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "%s: n < 0", who);
    MX_REQUIRE(dtype_valid(dtype), MX_ERR_DTYPE, "%s: bad dtype %d", who, (int)dtype);
    MX_REQUIRE(op >= MX_ADD && op <= MX_MAX, MX_ERR_INVALID, "%s: unknown operator %d", who, op);
    MX_REQUIRE(f >= -1 && f <= MX_B_MAX, MX_ERR_INVALID, "%s: unknown map2 body %d", who, f);
    MX_REQUIRE(ne && out, MX_ERR_INVALID, "%s: null ne or out", who);
    MX_REQUIRE(n == 0 || (a && (f < 0 || b)), MX_ERR_INVALID, "%s: null input", who);
    MX_REQUIRE(ws && ws_bytes >= mx_workspace_bytes(MX_WS_REDUCE, n, 0), MX_ERR_WORKSPACE,
               "%s: workspace needs %zu bytes", who, mx_workspace_bytes(MX_WS_REDUCE, n, 0));
    MX_REQUIRE(((uintptr_t)ws & 255) == 0, MX_ERR_INVALID, "%s: workspace must be 256-byte aligned", who);
    const DeviceInfo *d;
    if (mx_status st = device_info(&d)) return st;
    switch (dtype) {
    case MX_F32: return by_f<MX_F32>(f, op, a, b, n, ne, out, ws, s, d);
    case MX_F64: return by_f<MX_F64>(f, op, a, b, n, ne, out, ws, s, d);
    case MX_I32: return by_f<MX_I32>(f, op, a, b, n, ne, out, ws, s, d);
    case MX_I64: return by_f<MX_I64>(f, op, a, b, n, ne, out, ws, s, d);
    }
    return MX_ERR_DTYPE;
}

}  // namespace
}  // namespace mx

using namespace mx;

extern "C" {

mx_status mx_reduce(mx_redop op, mx_dtype dtype, const void *x_dev, int64_t n, const void *ne_host,
                    void *out_dev, void *ws, size_t ws_bytes, hipStream_t stream) {
    return run("mx_reduce", -1, op, dtype, x_dev, nullptr, n, ne_host, out_dev, ws, ws_bytes, stream);
}

mx_status mx_map2_reduce(mx_binop f, mx_redop op, mx_dtype dtype, const void *a_dev,
                         const void *b_dev, int64_t n, const void *ne_host, void *out_dev, void *ws,
                         size_t ws_bytes, hipStream_t stream) {
    MX_REQUIRE((int)f >= 0, MX_ERR_INVALID, "mx_map2_reduce: unknown map2 body %d", (int)f);
    return run("mx_map2_reduce", (int)f, op, dtype, a_dev, b_dev, n, ne_host, out_dev, ws, ws_bytes,
               stream);
}

}  // extern "C"
