// map / map2 (Appendix A) and the elementwise adjoint of the fused dot product.
// Streaming kernels, bound by HBM.  A block takes a contiguous chunk of C x 256
// 16-byte vectors of every array, all its loads in flight together, and up to
// 65536 blocks a chunk is all it does, so that the blocks which run together
// walk each array as one front.  A slice of any element alignment takes the same
// path.  2^26 pairs of float32: map2 (805 MB) 160 us -> 126 us (6.4 TB/s), the
// dot's adjoint (1.07 GB) 211 us -> 174 us (6.2 TB/s), against a vector per thread
// in a grid-wide stride; 2^20 3.3 us -> 3.0 us.  Which caches the accesses pass:
// pass_mode below.
#include "mx_internal.h"

namespace mx {
namespace {

constexpr int NT = 256;
constexpr int C = 4;
constexpr int64_t kMaxBlocks = 65536;

// Elements of a vector: 16 bytes of the result (int32 arrays, whose results
// are int64, are read in 8-byte vectors: whole vectors of the result per lane
// kept two lanes apart wrote half lines, 2^24 map2 53.7 us, now 39.2 us).
template <mx_dtype D> constexpr int kElems = 16 / sizeof(typename DT<D>::Acc);
template <mx_dtype D> struct InVec {
    typedef typename DT<D>::In T;
    typedef T type __attribute__((ext_vector_type(16 / sizeof(typename DT<D>::Acc)), aligned(sizeof(T))));
};
template <mx_dtype D, bool PAST> __device__ __forceinline__ typename InVec<D>::type load_in(const typename DT<D>::In *p) {
    const auto *q = reinterpret_cast<const typename InVec<D>::type *>(p);
    if constexpr (PAST) return __builtin_nontemporal_load(q);
    else return *q;
}

// Vectors of a block's chunk (2^18 elements of the dot's adjoint 2.4 us with four
// per thread, 2.3 us with one).
__host__ __device__ constexpr int64_t chunk_of(int64_t nv) { return nv <= kSmallPass ? NT : C * NT; }

// How a pass goes by the caches.  us, plain stores, through, past the caches, of the
// map2 alone and of map, map, map2 on one another's results (float32):
//   2^20  2.6, 2.3, 2.5;  7.0, 7.1, 6.8       2^21  4.5, 3.4, 4.0;  12.0, 10.9, 12.4
//   2^22  8.4, 8.5, 8.5;  18.7, 17.8, 20.2    2^24  36, 35, 29;  71.5, 69.6, 77.1
// and of the dot's adjoint alone: 2^20 3.6, 3.3, 3.1; 2^21 7.2, 4.9, 5.4; 2^23 20.5,
// 20.5, 20.1; 2^24 49, 48, 39.5.  A map of 2^14, read back by a sum of one block: 4.2,
// 4.0, 4.7; of 2^15, by many: 5.3, 5.5, 5.25.  So the stores of the smallest passes are
// plain, those of small ones go past the caches, those of larger ones into the memory-side cache alone, where the next call finds
// them; past its size, and for gradients, whose reader is seldom the next call,
// past half of it, past all caches; and so do the loads of a pass larger than it.
enum Mode { STORES_NEAR, STORES_PAST, STORES_THROUGH, ALL_PAST };
constexpr int64_t kNearMax = 1 << 20;
constexpr int64_t kThroughMin = 16 << 20;
Mode pass_mode(int64_t bytes, bool gradient) {
    if (bytes > kCacheBytes) return ALL_PAST;
    if (bytes <= kNearMax) return STORES_NEAR;
    return bytes > kThroughMin && bytes < (gradient ? kCacheBytes / 2 : kCacheBytes) ? STORES_THROUGH : STORES_PAST;
}
template <Mode M> constexpr bool kPast = M == ALL_PAST;
template <Mode M, class T> __device__ __forceinline__ void put(uvec<T> v, T *p) {
    if constexpr (M == STORES_THROUGH) store16_through(v, p);
    else if constexpr (M == STORES_NEAR) store16_near(v, p);
    else store16(v, p);
}

int grid_for(int64_t n, int64_t elems) {
    const int64_t nv = n / elems, g = ceil_div(nv, chunk_of(nv));
    return (int)(g < 1 ? 1 : g < kMaxBlocks ? g : kMaxBlocks);
}

// Calls full(j) for this thread's first vector of a whole chunk, part(j) for
// its vectors of other chunks, and rest(i) for the n % V elements at the end.
template <int V, class Full, class Part, class Rest>
__device__ __forceinline__ void walk_chunks(int64_t n, Full full, Part part, Rest rest) {
    const int64_t nv = n / V, chunk = chunk_of(nv);
    for (int64_t c = (int64_t)blockIdx.x * chunk; c < nv; c += (int64_t)gridDim.x * chunk) {
        const int64_t end = c + chunk < nv ? c + chunk : nv;
        if (end - c == C * NT) full(c + threadIdx.x);
        else
            for (int64_t j = c + threadIdx.x; j < end; j += NT) part(j);
    }
    const int64_t i = nv * V + threadIdx.x;
    if (blockIdx.x == gridDim.x - 1 && i < n) rest(i);
}

// ---------------------------------------------------------------- map
template <mx_dtype D, int F, Mode M>
__global__ void __launch_bounds__(NT) k_map(const typename DT<D>::In *__restrict__ x,
                                            typename DT<D>::Acc *__restrict__ out, int64_t n,
                                            typename DT<D>::Acc p0, typename DT<D>::Acc p1) {
    using Acc = typename DT<D>::Acc;
    constexpr int V = kElems<D>;
    using Vec = typename InVec<D>::type;
    auto one = [&](const Vec &v, int64_t j) {
        uvec<Acc> r;
#pragma unroll
        for (int e = 0; e < V; ++e) r[e] = Un<F, Acc>::ap(Acc(v[e]), p0, p1);
        put<M>(r, out + V * j);
    };
    walk_chunks<V>(
        n,
        [&](int64_t j) {
            Vec v[C];
#pragma unroll
            for (int u = 0; u < C; ++u) v[u] = load_in<D, kPast<M>>(x + V * (j + u * NT));
#pragma unroll
            for (int u = 0; u < C; ++u) one(v[u], j + u * NT);
        },
        [&](int64_t j) { one(load_in<D, false>(x + V * j), j); },
        [&](int64_t i) { out[i] = Un<F, Acc>::ap(Acc(x[i]), p0, p1); });
}

// ---------------------------------------------------------------- map2
template <mx_dtype D, int F, Mode M>
__global__ void __launch_bounds__(NT) k_map2(const typename DT<D>::In *__restrict__ a,
                                             const typename DT<D>::In *__restrict__ b,
                                             typename DT<D>::Acc *out, int64_t n) {
    using Acc = typename DT<D>::Acc;
    constexpr int V = kElems<D>;
    using Vec = typename InVec<D>::type;
    auto one = [&](const Vec &va, const Vec &vb, int64_t j) {
        uvec<Acc> r;
#pragma unroll
        for (int e = 0; e < V; ++e) r[e] = Bin<F, Acc>::ap(Acc(va[e]), Acc(vb[e]));
        put<M>(r, out + V * j);
    };
    walk_chunks<V>(
        n,
        [&](int64_t j) {
            Vec va[C], vb[C];
#pragma unroll
            for (int u = 0; u < C; ++u) {
                va[u] = load_in<D, kPast<M>>(a + V * (j + u * NT));
                vb[u] = load_in<D, kPast<M>>(b + V * (j + u * NT));
            }
#pragma unroll
            for (int u = 0; u < C; ++u) one(va[u], vb[u], j + u * NT);
        },
        [&](int64_t j) { one(load_in<D, false>(a + V * j), load_in<D, false>(b + V * j), j); },
        [&](int64_t i) { out[i] = Bin<F, Acc>::ap(Acc(a[i]), Acc(b[i])); });
}

// ---------------------------------------------------------------- dot adjoint
template <Mode M>
__global__ void __launch_bounds__(NT) k_dot_adjoint(const float *__restrict__ a,
                                                    const float *__restrict__ b, int64_t n,
                                                    const float *__restrict__ gout,
                                                    float *__restrict__ ga,
                                                    float *__restrict__ gb) {
    const float g = gout[0];
    walk_chunks<4>(
        n,
        [&](int64_t j) {
            uvec<float> va[C], vb[C];
#pragma unroll
            for (int u = 0; u < C; ++u) {
                if (ga) vb[u] = load16<kPast<M>>(b + 4 * (j + u * NT));
                if (gb) va[u] = load16<kPast<M>>(a + 4 * (j + u * NT));
            }
#pragma unroll
            for (int u = 0; u < C; ++u) {
                if (ga) put<M>(vb[u] * g, ga + 4 * (j + u * NT));
                if (gb) put<M>(va[u] * g, gb + 4 * (j + u * NT));
            }
        },
        [&](int64_t j) {
            if (ga) put<M>(load16<false>(b + 4 * j) * g, ga + 4 * j);
            if (gb) put<M>(load16<false>(a + 4 * j) * g, gb + 4 * j);
        },
        [&](int64_t i) {
            if (ga) ga[i] = g * b[i];
            if (gb) gb[i] = g * a[i];
        });
}

// ---------------------------------------------------------------- dispatch
template <class Go> void by_mode(Mode m, Go go) {
    switch (m) {
    case STORES_NEAR: return go(std::integral_constant<Mode, STORES_NEAR>{});
    case STORES_PAST: return go(std::integral_constant<Mode, STORES_PAST>{});
    case STORES_THROUGH: return go(std::integral_constant<Mode, STORES_THROUGH>{});
    case ALL_PAST: return go(std::integral_constant<Mode, ALL_PAST>{});
    }
}

template <mx_dtype D>
mx_status launch_map(int f, const void *x, int64_t n, const void *params, void *out, hipStream_t s) {
    using In = typename DT<D>::In;
    using Acc = typename DT<D>::Acc;
    Acc p0 = Acc(0), p1 = Acc(0);
    if (params) {
        __builtin_memcpy(&p0, params, sizeof(Acc));
        __builtin_memcpy(&p1, (const char *)params + sizeof(Acc), sizeof(Acc));
    }
    const Mode mode = pass_mode(n * (int64_t)(sizeof(In) + sizeof(Acc)), false);
    const int grid = grid_for(n, kElems<D>);
    const In *xi = (const In *)x;
    Acc *o = (Acc *)out;
#define MX_MAPCASE(F)                                                                       \
    case F:                                                                                 \
        by_mode(mode, [&](auto m) {                                                         \
            hipLaunchKernelGGL((k_map<D, F, decltype(m)::value>), dim3(grid), dim3(NT), 0, s, xi, o, n, p0, p1); \
        });                                                                                 \
        break;
    switch (f) {
        MX_MAPCASE(MX_U_ID)
        MX_MAPCASE(MX_U_NEG)
        MX_MAPCASE(MX_U_ABS)
        MX_MAPCASE(MX_U_SQ)
        MX_MAPCASE(MX_U_AFFINE)
    default:
        if constexpr (D == MX_F32 || D == MX_F64) {
            switch (f) {
                MX_MAPCASE(MX_U_EXP)
                MX_MAPCASE(MX_U_LOG)
                MX_MAPCASE(MX_U_SQRT)
                MX_MAPCASE(MX_U_RSQRT)
            default:
                return set_error(MX_ERR_INVALID, "mx_map: unknown map body %d", f);
            }
        } else {
            return set_error(MX_ERR_DTYPE, "mx_map: body %d needs a floating-point type", f);
        }
    }
#undef MX_MAPCASE
    return last_launch("mx_map");
}

template <mx_dtype D>
mx_status launch_map2(int f, const void *a, const void *b, int64_t n, void *out, hipStream_t s) {
    using In = typename DT<D>::In;
    using Acc = typename DT<D>::Acc;
    const Mode mode = pass_mode(n * (int64_t)(2 * sizeof(In) + sizeof(Acc)), false);
    const int grid = grid_for(n, kElems<D>);
    const In *ai = (const In *)a, *bi = (const In *)b;
    Acc *o = (Acc *)out;
    auto go = [&](auto body) {
        by_mode(mode, [&](auto m) {
            hipLaunchKernelGGL((k_map2<D, decltype(body)::value, decltype(m)::value>), dim3(grid), dim3(NT), 0, s, ai, bi, o, n);
        });
    };
#define MX_MAP2CASE(F)                             \
    case F:                                        \
        go(std::integral_constant<int, F>{});      \
        break;
    switch (f) {
        MX_MAP2CASE(MX_B_ADD)
        MX_MAP2CASE(MX_B_SUB)
        MX_MAP2CASE(MX_B_MUL)
        MX_MAP2CASE(MX_B_MIN)
        MX_MAP2CASE(MX_B_MAX)
    case MX_B_DIV:
        if constexpr (D == MX_F32 || D == MX_F64) {
            go(std::integral_constant<int, MX_B_DIV>{});
            break;
        } else {
            return set_error(MX_ERR_DTYPE, "mx_map2: division needs a floating-point type");
        }
    default:
        return set_error(MX_ERR_INVALID, "mx_map2: unknown map2 body %d", f);
    }
#undef MX_MAP2CASE
    return last_launch("mx_map2");
}

}  // namespace
}  // namespace mx

using namespace mx;

extern "C" {

mx_status mx_map(mx_unop f, mx_dtype dtype, const void *x_dev, int64_t n, const void *params_host,
                 void *out_dev, hipStream_t stream) {
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "mx_map: n < 0");
    MX_REQUIRE(dtype_valid(dtype), MX_ERR_DTYPE, "mx_map: bad dtype %d", (int)dtype);
    MX_REQUIRE((int)f >= 0 && (int)f <= MX_U_RSQRT, MX_ERR_INVALID, "mx_map: unknown body %d", (int)f);
    MX_REQUIRE(f != MX_U_AFFINE || params_host, MX_ERR_INVALID, "mx_map: AFFINE needs params");
    if (!is_float(dtype) && f >= MX_U_EXP)
        return set_error(MX_ERR_DTYPE, "mx_map: body %d needs a floating-point type", (int)f);
    if (n == 0) return MX_OK;
    MX_REQUIRE(x_dev && out_dev, MX_ERR_INVALID, "mx_map: null pointer");
    switch (dtype) {
    case MX_F32: return launch_map<MX_F32>(f, x_dev, n, params_host, out_dev, stream);
    case MX_F64: return launch_map<MX_F64>(f, x_dev, n, params_host, out_dev, stream);
    case MX_I32: return launch_map<MX_I32>(f, x_dev, n, params_host, out_dev, stream);
    case MX_I64: return launch_map<MX_I64>(f, x_dev, n, params_host, out_dev, stream);
    }
    return MX_ERR_DTYPE;
}

mx_status mx_map2(mx_binop f, mx_dtype dtype, const void *a_dev, const void *b_dev, int64_t n,
                  void *out_dev, hipStream_t stream) {
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "mx_map2: n < 0");
    MX_REQUIRE(dtype_valid(dtype), MX_ERR_DTYPE, "mx_map2: bad dtype %d", (int)dtype);
    MX_REQUIRE((int)f >= 0 && (int)f <= MX_B_MAX, MX_ERR_INVALID, "mx_map2: unknown body %d", (int)f);
    if (!is_float(dtype) && f == MX_B_DIV)
        return set_error(MX_ERR_DTYPE, "mx_map2: division needs a floating-point type");
    if (n == 0) return MX_OK;
    MX_REQUIRE(a_dev && b_dev && out_dev, MX_ERR_INVALID, "mx_map2: null pointer");
    switch (dtype) {
    case MX_F32: return launch_map2<MX_F32>(f, a_dev, b_dev, n, out_dev, stream);
    case MX_F64: return launch_map2<MX_F64>(f, a_dev, b_dev, n, out_dev, stream);
    case MX_I32: return launch_map2<MX_I32>(f, a_dev, b_dev, n, out_dev, stream);
    case MX_I64: return launch_map2<MX_I64>(f, a_dev, b_dev, n, out_dev, stream);
    }
    return MX_ERR_DTYPE;
}

mx_status mx_dot_adjoint_f32(const float *a_dev, const float *b_dev, int64_t n,
                             const float *gout_dev, float *ga_dev, float *gb_dev,
                             hipStream_t stream) {
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "mx_dot_adjoint_f32: n < 0");
    if (n == 0) return MX_OK;
    MX_REQUIRE(gout_dev, MX_ERR_INVALID, "mx_dot_adjoint_f32: null gout");
    MX_REQUIRE(!ga_dev || b_dev, MX_ERR_INVALID, "mx_dot_adjoint_f32: ga needs b");
    MX_REQUIRE(!gb_dev || a_dev, MX_ERR_INVALID, "mx_dot_adjoint_f32: gb needs a");
    if (!ga_dev && !gb_dev) return MX_OK;
    by_mode(pass_mode(n * (int64_t)sizeof(float) * 2 * ((ga_dev != nullptr) + (gb_dev != nullptr)), true), [&](auto m) {
        hipLaunchKernelGGL(k_dot_adjoint<decltype(m)::value>, dim3(grid_for(n, 4)), dim3(NT), 0, stream, a_dev, b_dev, n,
                           gout_dev, ga_dev, gb_dev);
    });
    return last_launch("mx_dot_adjoint_f32");
}

}  // extern "C"
