// Sequential loop around a pairwise map (reduce): gravitational N-body with
// Plummer softening and explicit Euler steps (the ODE-solver pattern of the
// CUDA-backend evaluation, Table 2), its adjoint, and the checkpointed reverse
// sweep of the loop.
//
//   a_i = G sum_j m_j d_ij (|d_ij|^2 + eps2)^(-3/2),   d_ij = x_j - x_i
//   x_{t+1} = x_t + dt v_t,   v_{t+1} = v_t + dt a(x_t)
//   (J_a^T abar)_k = G sum_j [phi I - 3 phi/s d d^T] (m_k abar_j - m_j abar_k),
//     d = x_j - x_k, s = |d|^2 + eps2, phi = s^(-3/2)
//
// Layout: bodies as float4 records (x, y, z, m); velocities and adjoints as
// float4 (x, y, z, 0).
//
// Three schedules of the pair sum, chosen from n alone (pair_path below), all
// with fixed bracketings, so a recomputation reproduces the forward bit for
// bit whatever the block scheduling:
//  * direct (few bodies): one wave per few bodies i, the bodies j across its
//    lanes; one launch, no partials.
//  * symmetric: every unordered pair is evaluated once and added to both its
//    bodies; partial sums and a second, elementwise kernel that adds them in a
//    fixed order and applies the update.
//  * sliced (many bodies, where the symmetric partials would take too much
//    memory): a block owns a tile of 256 bodies i and one of S slices of the
//    bodies j, staged through LDS.
#include <algorithm>

#include "mx_internal.h"

namespace mx {
namespace {

constexpr int NT = 256;
constexpr int kMaxSlices = 64;

enum Mode { ACCEL = 0, STEP = 1, VJP = 2, ADJSTEP = 3 };
template <int MODE> constexpr bool kAdj = MODE == VJP || MODE == ADJSTEP;

struct PairArgs {
    const float4 *pos;   // x_t (with masses)
    const float4 *aux;   // STEP: v_t; VJP/ADJSTEP: abar (= vbar_{t+1})
    const float4 *aux2;  // ADJSTEP: xbar_{t+1}
    float4 *out0;        // ACCEL: a; STEP: x_{t+1}; VJP: J^T abar; ADJSTEP: xbar_t
    float4 *out1;        // STEP: v_{t+1}; ADJSTEP: vbar_t
    float4 *partial;     // sliced: [S][N]; symmetric: the i sides, then the j sides
    int64_t n;
    int slices;
    int64_t slice_len;   // multiple of NT
    int sets, blocks;    // symmetric: sets of 256 bodies, blocks of the pair kernel
    float eps2, G, dt;
};

__device__ __forceinline__ void pair_accel(const float4 xi, const float4 xj, float eps2, float &ax,
                                           float &ay, float &az) {
    const float dx = xj.x - xi.x, dy = xj.y - xi.y, dz = xj.z - xi.z;
    const float s = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, eps2)));  // eps2 folded into the first FMA
    const float inv = __frsqrt_rn(s);
    const float w = xj.w * (inv * inv * inv);
    ax += w * dx;
    ay += w * dy;
    az += w * dz;
}

// v_rsq_f32 of K values.  The SIMD issues FP32 instructions of two waves in the
// same four cycles, but a transcendental instruction knocks the waves out of
// step for dozens of instructions after it; raised priority for the wave that
// issues them keeps the pairing (one such group per 68 instructions: 47 cycles
// a wave against 65, and 41 with no v_rsq_f32 at all).
template <int K> __device__ __forceinline__ void rsqrt_group(float (&v)[K]) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = __frsqrt_rn(v[k]);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
}

// body i with K bodies j: the i sides into oi (SIDES & 1), the j sides into oj
// (SIDES & 2)
template <bool ADJ, int SIDES, int K>
__device__ __forceinline__ void pairs(const float4 xi, const float4 ai, const float4 (&xj)[K], const float4 (&aj)[K],
                                      float eps2, float (&oi)[3], float (&oj)[K][3]) {
    float dx[K], dy[K], dz[K], inv[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        dx[q] = xj[q].x - xi.x;
        dy[q] = xj[q].y - xi.y;
        dz[q] = xj[q].z - xi.z;
        inv[q] = fmaf(dz[q], dz[q], fmaf(dy[q], dy[q], fmaf(dx[q], dx[q], eps2)));
    }
    rsqrt_group(inv);
    const float mi = -xi.w;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const float inv2 = inv[q] * inv[q];
        const float phi = inv2 * inv[q];
        if constexpr (ADJ) {
            const float psi = 3.0f * phi * inv2;
            // both products rounded before the subtraction (never fused into
            // an FMA), so the self term j = i, where phi = eps^-3 is huge, is
            // exactly zero
            const float wx = sub_rn(mul_rn(xi.w, aj[q].x), mul_rn(xj[q].w, ai.x));
            const float wy = sub_rn(mul_rn(xi.w, aj[q].y), mul_rn(xj[q].w, ai.y));
            const float wz = sub_rn(mul_rn(xi.w, aj[q].z), mul_rn(xj[q].w, ai.z));
            const float t = psi * (dx[q] * wx + dy[q] * wy + dz[q] * wz);
            if constexpr (SIDES == 1) {
                oi[0] += phi * wx - t * dx[q];
                oi[1] += phi * wy - t * dy[q];
                oi[2] += phi * wz - t * dz[q];
            } else {
                const float cx = phi * wx - t * dx[q], cy = phi * wy - t * dy[q], cz = phi * wz - t * dz[q];
                if constexpr (SIDES & 1) {
                    oi[0] += cx;
                    oi[1] += cy;
                    oi[2] += cz;
                }
                oj[q][0] -= cx;
                oj[q][1] -= cy;
                oj[q][2] -= cz;
            }
        } else {
            if constexpr (SIDES & 1) {
                const float wi = xj[q].w * phi;
                oi[0] += wi * dx[q];
                oi[1] += wi * dy[q];
                oi[2] += wi * dz[q];
            }
            if constexpr (SIDES & 2) {
                const float wj = mi * phi;
                oj[q][0] += wj * dx[q];
                oj[q][1] += wj * dy[q];
                oj[q][2] += wj * dz[q];
            }
        }
    }
}

// a zero the compiler takes for each lane's own value, so that loads indexed
// with it go to vector registers (a scalar operand halves the FP32 issue rate)
__device__ __forceinline__ unsigned vector_zero() {
    unsigned z;
    asm("v_mov_b32 %0, 0" : "=v"(z));
    return z;
}

template <int MODE>
__device__ __forceinline__ void finish(const PairArgs &p, int64_t i, float4 xi, float4 ai, float ox, float oy,
                                       float oz) {
    const float G = p.G, dt = p.dt;
    if constexpr (MODE == ACCEL || MODE == VJP) {
        p.out0[i] = make_float4(G * ox, G * oy, G * oz, 0.f);
    } else if constexpr (MODE == STEP) {
        const float4 v = p.aux[i];
        p.out0[i] = make_float4(xi.x + dt * v.x, xi.y + dt * v.y, xi.z + dt * v.z, xi.w);
        p.out1[i] = make_float4(v.x + dt * (G * ox), v.y + dt * (G * oy), v.z + dt * (G * oz), 0.f);
    } else {  // ADJSTEP: xbar_t = xbar + dt G J^T vbar;  vbar_t = vbar + dt xbar
        const float4 xb = p.aux2[i];
        p.out0[i] = make_float4(xb.x + dt * (G * ox), xb.y + dt * (G * oy), xb.z + dt * (G * oz), 0.f);
        p.out1[i] = make_float4(ai.x + dt * xb.x, ai.y + dt * xb.y, ai.z + dt * xb.z, 0.f);
    }
}

template <int MODE>
__global__ void __launch_bounds__(NT) k_pairs(PairArgs p) {
    constexpr bool ADJ = kAdj<MODE>;
    __shared__ float4 sx[NT];
    __shared__ float4 sa[ADJ ? NT : 1];
    const int64_t n = p.n;
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 xi = i < n ? p.pos[i] : zero;
    float4 ai = zero;
    if constexpr (ADJ) ai = i < n ? p.aux[i] : zero;
    float o[3] = {0.f, 0.f, 0.f};
    const int64_t js = (int64_t)blockIdx.y * p.slice_len;
    int64_t je = js + p.slice_len;
    if (je > n) je = n;
    for (int64_t j0 = js; j0 < je; j0 += NT) {
        const int64_t j = j0 + threadIdx.x;
        sx[threadIdx.x] = j < je ? p.pos[j] : zero;  // zero mass: no contribution
        if constexpr (ADJ) sa[threadIdx.x] = j < je ? p.aux[j] : zero;
        __syncthreads();
#pragma unroll 2
        for (int jj = 0; jj < NT; jj += 4) {
            const float4 xj[4] = {sx[jj], sx[jj + 1], sx[jj + 2], sx[jj + 3]};
            float4 aj[4] = {zero, zero, zero, zero};
            if constexpr (ADJ) {
#pragma unroll
                for (int q = 0; q < 4; ++q) aj[q] = sa[jj + q];
            }
            float none[4][3];
            pairs<ADJ, 1>(xi, ai, xj, aj, p.eps2, o, none);
        }
        __syncthreads();
    }
    if (i >= n) return;
    if (p.slices > 1) {
        p.partial[(int64_t)blockIdx.y * n + i] = make_float4(o[0], o[1], o[2], 0.f);
        return;
    }
    finish<MODE>(p, i, xi, ai, o[0], o[1], o[2]);
}

// Adds the S slice partials of body i in slice order and applies the update.
template <int MODE>
__global__ void __launch_bounds__(NT) k_pairs_finish(PairArgs p) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= p.n) return;
    float ox = 0.f, oy = 0.f, oz = 0.f;
    for (int s = 0; s < p.slices; ++s) {
        const float4 q = p.partial[(int64_t)s * p.n + i];
        ox += q.x;
        oy += q.y;
        oz += q.z;
    }
    const float4 xi = p.pos[i];
    float4 ai = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (kAdj<MODE>) ai = p.aux[i];
    finish<MODE>(p, i, xi, ai, ox, oy, oz);
}

// ---------------------------------------------------------------- lane sums
// lanes 32..63 of a trade places with lanes 0..31 of b, then the odd 16-lane
// rows of a with the even rows of b
__device__ __forceinline__ float add_halves(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_rows(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// the sums over the wave of four values: value 0 in row 0, 2 in row 1, 1 in
// row 2, 3 in row 3
__device__ __forceinline__ float wave_sum4(float v0, float v1, float v2, float v3) {
    float v = add_rows(add_halves(v0, v1), add_halves(v2, v3));
    v += dpp_move<0xB1, 0xF>(v, 0.f);
    v += dpp_move<0x4E, 0xF>(v, 0.f);
    v += dpp_move<0x141, 0xF>(v, 0.f);
    v += dpp_move<0x140, 0xF>(v, 0.f);
    return v;
}

// ---------------------------------------------------------------- direct
// A block takes R bodies i, held alike by all its lanes, and its four waves a
// quarter of the bodies j each, across the lanes, U loads per lane in flight;
// the lanes are added by swaps and DPP, the waves through LDS in wave order,
// and thread r applies body r's update.  No partials and no second launch: up
// to kDirectMax bodies a step is bound by its launch and the latency of these
// loads, not by its arithmetic (times: pair_path).
template <int MODE, int R>
__global__ void __launch_bounds__(NT) k_pairs_direct(PairArgs p) {
    constexpr bool ADJ = kAdj<MODE>;
    constexpr int U = 4, NW = NT / kWave;
    static_assert(R % 4 == 0, "sums of four bodies at a time");
    __shared__ float red[NW][3][R];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = (int)p.n;
    const int i0 = blockIdx.x * R;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 xi[R], ai[R];
    float o[R][3];
    const unsigned vz = vector_zero();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = i0 + r < n ? i0 + r : n - 1;
        xi[r] = (p.pos + i)[vz];
        ai[r] = zero;
        if constexpr (ADJ) ai[r] = (p.aux + i)[vz];
        o[r][0] = o[r][1] = o[r][2] = 0.f;
    }
    for (int j0 = w * U * kWave; j0 < n; j0 += NW * U * kWave) {
        float4 xj[U], aj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * kWave + lane;
            xj[u] = j < n ? p.pos[j] : zero;  // zero mass: no contribution
            aj[u] = zero;
            if constexpr (ADJ) aj[u] = j < n ? p.aux[j] : zero;
        }
        float none[U][3];
#pragma unroll
        for (int r = 0; r < R; ++r) pairs<ADJ, 1>(xi[r], ai[r], xj, aj, p.eps2, o[r], none);
    }
    const int g = lane >> 4;
#pragma unroll
    for (int r = 0; r < R; r += 4)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float v = wave_sum4(o[r][c], o[r + 1][c], o[r + 2][c], o[r + 3][c]);
            if ((lane & 15) == 0) red[w][c][r + ((g & 1) << 1 | g >> 1)] = v;
        }
    __syncthreads();
    const int r = threadIdx.x;
    if (r >= R || i0 + r >= n) return;
    float v[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v[c] = red[0][c][r];
#pragma unroll
        for (int k = 1; k < NW; ++k) v[c] += red[k][c][r];
    }
    float4 a = zero;
    if constexpr (ADJ) a = p.aux[i0 + r];
    finish<MODE>(p, i0 + r, p.pos[i0 + r], a, v[0], v[1], v[2]);
}

// ---------------------------------------------------------------- symmetric
// Every unordered pair once.  The two bodies of a pair share the distance, its
// inverse square root and, in the adjoint, the whole term (d and m_k abar_j -
// m_j abar_k both change sign with the roles, so body j receives exactly the
// negative of body k's): 15 VALU instructions and one v_rsq_f32 for the two
// sides of the forward, 35 for the adjoint, against 2 x 12 and 2 x 29.
// What a pair saves is the dear part: v_rsq_f32 issues in 8 cycles per wave,
// and an FMA whose three source registers are all even or all odd (two banks)
// in 4, against 2 for other FMAs, multiplies and adds of VGPRs (measured, two
// waves per SIMD or more; any scalar operand makes it 4, so bodies i are read
// into vector registers).
//
// The bodies are cut into sets of 256.  A wave holds the 256 bodies j of one
// set, four per lane, with their sums; the bodies i of the sets before it come
// one at a time (a load of one address by all lanes), four per round, and
// their sums over the lanes are added by lane swaps and DPP four at a time
// (7 % of the instructions) and stored, one partial per (set, body i).  Inside
// a set every ordered pair is taken, into body j's sums alone.
// The work (set, 16 bodies i) is one list, cut into kSymBlocks shares equal to
// within one unit, so the blocks, four per CU, end together; a block's waves
// take the 16 bodies four each, and where a share leaves a set the waves' sums
// are added in wave order into one partial per (block, set).
// Times: pair_path.
constexpr int kSetBodies = 256;
constexpr int kJ = kSetBodies / kWave;
constexpr int kUnit = 16;  // bodies i per unit, four per wave
constexpr int kSymBlocks = 1024;
constexpr int kUnitsPerBlock = 8;  // at least, while fewer than kSymBlocks blocks run

// units of the sets before set s: 16 (k + 1) units for set k
__host__ __device__ __forceinline__ int sym_first(int s) { return 8 * s * (s + 1); }
__host__ __device__ __forceinline__ int sym_cut(int b, int units, int blocks) {
    return (int)((int64_t)units * b / blocks);
}
__device__ __forceinline__ int sym_set_of(int u) {
    int s = (int)((sqrtf(1.f + 0.5f * (float)u) - 1.f) * 0.5f);
    while (s > 0 && sym_first(s) > u) --s;
    while (sym_first(s + 1) <= u) ++s;
    return s;
}
// i side of set s (bodies before the set): row s of a triangle
__host__ __device__ __forceinline__ int64_t sym_row(int s) { return (int64_t)kSetBodies / 2 * s * (s - 1); }

template <int MODE>
__global__ void __launch_bounds__(NT, 4) k_pairs_sym(PairArgs p) {
    constexpr bool ADJ = kAdj<MODE>;
    constexpr int NW = NT / kWave;
    static_assert(kUnit == 4 * NW && kSetBodies == NT, "a unit is four bodies per wave, a set one body per thread");
    __shared__ float red[NW][3][kSetBodies];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = (int)p.n;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const int units = sym_first(p.sets);
    int u = sym_cut(blockIdx.x, units, p.blocks);
    const int u_end = sym_cut(blockIdx.x + 1, units, p.blocks);
    float4 *jside = p.partial + sym_row(p.sets);
    const unsigned vz = vector_zero();
    for (int s = sym_set_of(u); u < u_end; ++s) {
        float4 xj[kJ], aj[kJ];
        float oj[kJ][3];
#pragma unroll
        for (int q = 0; q < kJ; ++q) {
            const int j = s * kSetBodies + q * kWave + lane;
            xj[q] = j < n ? p.pos[j] : zero;
            aj[q] = zero;
            if constexpr (ADJ) aj[q] = j < n ? p.aux[j] : zero;
            oj[q][0] = oj[q][1] = oj[q][2] = 0.f;
        }
        const int seg_end = sym_first(s + 1) < u_end ? sym_first(s + 1) : u_end;
        const int diag = sym_first(s) + s * (kSetBodies / kUnit);  // first unit inside the set
        int i = (u - sym_first(s)) * kUnit + 4 * w;
        float4 *row = p.partial + sym_row(s);
        const int off_end = seg_end < diag ? seg_end : diag;
        float4 xn = zero, an = zero;
        auto fetch = [&](int k) {
            const int kc = k < n ? k : n - 1;
            xn = (p.pos + kc)[vz];
            if constexpr (ADJ) an = (p.aux + kc)[vz];
        };
        fetch(i);
        for (; u < off_end; ++u, i += kUnit) {
            float oi[4][3];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float4 xi = xn, ai = an;
                fetch(r < 3 ? i + r + 1 : i + kUnit);
                oi[r][0] = oi[r][1] = oi[r][2] = 0.f;
                pairs<ADJ, 3>(xi, ai, xj, aj, p.eps2, oi[r], oj);
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(3);  // lane swaps disturb the pairing as v_rsq_f32 does
            const float sx = wave_sum4(oi[0][0], oi[1][0], oi[2][0], oi[3][0]);
            const float sy = wave_sum4(oi[0][1], oi[1][1], oi[2][1], oi[3][1]);
            const float sz = wave_sum4(oi[0][2], oi[1][2], oi[2][2], oi[3][2]);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            const int g = lane >> 4;
            if ((lane & 15) == 0) row[i + ((g & 1) << 1 | g >> 1)] = make_float4(sx, sy, sz, 0.f);
        }
        for (; u < seg_end; ++u, i += kUnit) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float4 xi = xn, ai = an;
                if (i + r >= n) xi = ai = zero;
                fetch(r < 3 ? i + r + 1 : i + kUnit);
                float none[3];
                pairs<ADJ, 2>(xi, ai, xj, aj, p.eps2, none, oj);
            }
        }
        // the waves' sums of the set's bodies, in wave order
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kJ; ++q)
#pragma unroll
            for (int c = 0; c < 3; ++c) red[w][c][q * kWave + lane] = oj[q][c];
        __syncthreads();
        float v[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] = red[0][c][threadIdx.x];
#pragma unroll
            for (int k = 1; k < NW; ++k) v[c] += red[k][c][threadIdx.x];
        }
        jside[(int64_t)(blockIdx.x + s) * kSetBodies + threadIdx.x] = make_float4(v[0], v[1], v[2], 0.f);
    }
}

// Adds the partials of 64 bodies: the j sides of their set's blocks in block
// order, then the i sides of the sets after it in set order; each of the
// block's waves an equal part of them, the parts in order; then the update.
// Bound by the latency of its partials: with sixteen waves instead of four a
// step of 5000 bodies takes 16.6 us instead of 17.1 us, of 8192 27.7 us instead
// of 28.7 us, of 16 384 69.4 us instead of 70.1 us.
constexpr int kSymFinish = 1024;
template <int MODE>
__global__ void __launch_bounds__(kSymFinish) k_pairs_sym_finish(PairArgs p) {
    constexpr int NW = kSymFinish / kWave;
    __shared__ float red[NW][3][kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t i = (int64_t)blockIdx.x * kWave + lane;
    const int s = (int)(blockIdx.x * kWave / kSetBodies);
    const int units = sym_first(p.sets);
    // blocks whose share meets the set's units
    const int64_t f = sym_first(s), l = sym_first(s + 1) - 1;
    int b0 = (int)(f * p.blocks / units), b1 = (int)(l * p.blocks / units);
    while (sym_cut(b0 + 1, units, p.blocks) <= f) ++b0;
    while (b1 + 1 < p.blocks && sym_cut(b1 + 1, units, p.blocks) <= l) ++b1;
    const int nj = b1 - b0 + 1, total = nj + p.sets - 1 - s;
    const int per = (total + NW - 1) / NW;
    const int q0 = w * per, q1 = q0 + per < total ? q0 + per : total;
    const float4 *js = p.partial + sym_row(p.sets) + (int64_t)(b0 + s) * kSetBodies + (i - (int64_t)s * kSetBodies);
    float ox = 0.f, oy = 0.f, oz = 0.f;
    if (i < p.n) {
#pragma unroll 8
        for (int q = q0; q < q1; ++q) {
            const float4 v = q < nj ? js[(int64_t)q * kSetBodies] : p.partial[sym_row(s + 1 + q - nj) + i];
            ox += v.x;
            oy += v.y;
            oz += v.z;
        }
    }
    red[w][0][lane] = ox;
    red[w][1][lane] = oy;
    red[w][2][lane] = oz;
    __syncthreads();
    if (w != 0 || i >= p.n) return;
#pragma unroll
    for (int k = 1; k < NW; ++k) {
        ox += red[k][0][lane];
        oy += red[k][1][lane];
        oz += red[k][2][lane];
    }
    float4 ai = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (kAdj<MODE>) ai = p.aux[i];
    finish<MODE>(p, i, p.pos[i], ai, ox, oy, oz);
}

// ---------------------------------------------------------------- plain forms
__global__ void __launch_bounds__(NT) k_accel_plain(const float4 *__restrict__ pos, int64_t n, float eps2,
                                                    float G, float4 *__restrict__ acc) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= n) return;
    const float4 xi = pos[i];
    float ax = 0.f, ay = 0.f, az = 0.f;
    for (int64_t j = 0; j < n; ++j) pair_accel(xi, pos[j], eps2, ax, ay, az);
    acc[i] = make_float4(G * ax, G * ay, G * az, 0.f);
}

__global__ void __launch_bounds__(NT) k_euler(const float4 *__restrict__ pos, const float4 *__restrict__ vel,
                                              const float4 *__restrict__ acc, int64_t n, float dt,
                                              float4 *__restrict__ pos_out, float4 *__restrict__ vel_out) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= n) return;
    const float4 x = pos[i], v = vel[i], a = acc[i];
    pos_out[i] = make_float4(x.x + dt * v.x, x.y + dt * v.y, x.z + dt * v.z, x.w);
    vel_out[i] = make_float4(v.x + dt * a.x, v.y + dt * a.y, v.z + dt * a.z, 0.f);
}

// ---------------------------------------------------------------- kinetic energy
// KE = 1/2 sum_i m_i |v_i|^2 folded by one block (fixed bracketing), and the
// start of the reverse sweep: vbar = m v, xbar = 0 (either may be null).
// 1024 threads, four bodies in flight each: one block's latency is all it costs
// (16 384 bodies: 20 us with 256 threads and one body at a time).
constexpr int NTK = 1024;
__global__ void __launch_bounds__(NTK) k_kinetic(const float4 *__restrict__ pos, const float4 *__restrict__ vel,
                                                int64_t n, float *__restrict__ ke, float4 *vbar, float4 *xbar) {
    __shared__ float smem[NTK / kWave];
    using R = Red<MX_ADD, float>;
    float acc = 0.f;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < n; i += NTK) {
        const float4 v = vel[i];
        const float m = pos[i].w;
        acc += 0.5f * m * (v.x * v.x + v.y * v.y + v.z * v.z);
        if (vbar) vbar[i] = make_float4(m * v.x, m * v.y, m * v.z, 0.f);
        if (xbar) xbar[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    acc = block_reduce<R, NTK>(acc, smem);
    if (threadIdx.x == 0) ke[0] = acc;
}

// Start of the reverse sweep for an upstream gradient g of KE (a device
// scalar; null means 1): vbar = g m v, xbar = 0.  With g = 1 the products
// equal k_kinetic's m v bit for bit.
__global__ void __launch_bounds__(NT) k_adjoint_seed(const float4 *__restrict__ pos, const float4 *__restrict__ vel,
                                                     int64_t n, const float *__restrict__ gscale,
                                                     float4 *__restrict__ vbar, float4 *__restrict__ xbar) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= n) return;
    const float g = gscale ? gscale[0] : 1.f;
    const float4 v = vel[i];
    const float m = pos[i].w;
    vbar[i] = make_float4(m * v.x * g, m * v.y * g, m * v.z * g, 0.f);
    xbar[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// ---------------------------------------------------------------- launch helpers
// The j range is cut into S slices so that about kTargetBlocks blocks run
// (8 per CU on 256 CUs); S depends only on n, so results are the same on
// every device.
constexpr int64_t kTargetBlocks = 2048;

int slices_for(int64_t n) {
    if (n <= 0) return 1;  // no bodies: one (empty) slice
    const int64_t tiles = ceil_div(n, NT);
    int64_t s = ceil_div(kTargetBlocks, tiles > 0 ? tiles : 1);
    if (s > tiles) s = tiles;
    if (s > kMaxSlices) s = kMaxSlices;
    if (s < 1) s = 1;
    // snap to whole LDS tiles per slice
    const int64_t len = ceil_div(ceil_div(n, s), NT) * NT;
    return (int)ceil_div(n, len);
}

// Which schedule takes n bodies.  us per step, forward / adjoint, launches
// replayed from a graph:
//     n        direct        symmetric     sliced
//   1 000     3.5 /  4.6    8.5 /  9.7   13.4 /  22.6  (12.3 / 28.3 before)
//   4 096    10.6 / 18.5   16.2 / 21.8   15.0 /  23.9  (13.5 / 36.3 before)
//   6 000    21.2 / 37.5   21.3 / 29.9   22.4 /  39.5  (23.8 / 43.8 before)
//  16 384                  68.6 / 109    79.5 / 169    (87.3 / 178 before)
// ("before": the sliced schedule without the v_rsq_f32 groups).  Past 65 536
// bodies the symmetric partials (n^2 / 32 bytes) would pass 134 MB.
constexpr int64_t kDirectMax = 4096, kSymMax = 65536;
enum PairPath { DIRECT, SYMMETRIC, SLICED };
PairPath pair_path(int64_t n, bool alias) {
    if (n <= kDirectMax && !alias) return DIRECT;
    return n <= kSymMax ? SYMMETRIC : SLICED;
}

int sym_sets(int64_t n) { return (int)ceil_div(n, kSetBodies); }
int sym_blocks(int64_t n) { return std::min(kSymBlocks, sym_first(sym_sets(n)) / kUnitsPerBlock); }

size_t pair_ws_bytes(int64_t n) {
    if (n <= 0) return kCounterBytes;
    if (n <= kSymMax) {
        // the triangle of i sides, then one set of j sides per (block, set) met
        const int64_t rows = sym_row(sym_sets(n)) + (int64_t)(sym_blocks(n) + sym_sets(n)) * kSetBodies;
        return kCounterBytes + align256((size_t)rows * 16);
    }
    const int sl = slices_for(n);
    return kCounterBytes + (sl > 1 ? align256((size_t)sl * (size_t)n * 16) : 0);
}

// An output written over the positions or what the pair sums read of the
// adjoint: the direct schedule, whose waves still read what others write, leaves
// such a call to the symmetric one, which writes when every sum is done.
bool overlaps(const float4 *out, const float4 *in, int64_t n) { return out && in && out < in + n && in < out + n; }
bool in_place(const PairArgs &p) {
    return overlaps(p.out0, p.pos, p.n) || overlaps(p.out0, p.aux, p.n) || overlaps(p.out1, p.pos, p.n) ||
           overlaps(p.out1, p.aux, p.n);
}

template <int MODE>
mx_status launch_pairs(PairArgs p, void *ws, hipStream_t s) {
    const int64_t tiles = ceil_div(p.n, NT);
    MX_REQUIRE(tiles < (1LL << 31), MX_ERR_SHAPE, "nbody: too many bodies");
    p.partial = (float4 *)((char *)ws + kCounterBytes);
    switch (pair_path(p.n, in_place(p))) {
    case DIRECT:
        if (p.n <= 1024)
            hipLaunchKernelGGL((k_pairs_direct<MODE, 4>), dim3((unsigned)ceil_div(p.n, 4)), dim3(NT), 0, s, p);
        else
            hipLaunchKernelGGL((k_pairs_direct<MODE, 8>), dim3((unsigned)ceil_div(p.n, 8)), dim3(NT), 0, s, p);
        return last_launch("nbody pair kernel");
    case SYMMETRIC:
        p.sets = sym_sets(p.n);
        p.blocks = sym_blocks(p.n);
        hipLaunchKernelGGL((k_pairs_sym<MODE>), dim3((unsigned)p.blocks), dim3(NT), 0, s, p);
        hipLaunchKernelGGL((k_pairs_sym_finish<MODE>), dim3((unsigned)ceil_div(p.n, kWave)), dim3(kSymFinish), 0, s, p);
        return last_launch("nbody pair kernel");
    case SLICED: break;
    }
    p.slices = slices_for(p.n);
    p.slice_len = ceil_div(ceil_div(p.n, p.slices), NT) * NT;
    hipLaunchKernelGGL((k_pairs<MODE>), dim3((unsigned)tiles, (unsigned)p.slices), dim3(NT), 0, s, p);
    if (p.slices > 1) hipLaunchKernelGGL((k_pairs_finish<MODE>), dim3((unsigned)tiles), dim3(NT), 0, s, p);
    return last_launch("nbody pair kernel");
}

inline bool a16(const void *p) { return ((uintptr_t)p & 15) == 0; }

mx_status check_common(const char *who, int64_t n, float eps2, void *ws, size_t ws_bytes, size_t need) {
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "%s: n < 0", who);
    MX_REQUIRE(eps2 > 0.f, MX_ERR_INVALID, "%s: eps2 must be positive", who);
    if (n > 0)
        MX_REQUIRE(ws && ws_bytes >= need && ((uintptr_t)ws & 255) == 0, MX_ERR_WORKSPACE,
                   "%s: workspace needs %zu bytes, 256-byte aligned", who, need);
    return MX_OK;
}

mx_status step_impl(const float4 *x, const float4 *v, int64_t n, float eps2, float G, float dt, float4 *xo,
                    float4 *vo, void *pws, hipStream_t s) {
    PairArgs p{};
    p.pos = x; p.aux = v; p.out0 = xo; p.out1 = vo; p.n = n; p.eps2 = eps2; p.G = G; p.dt = dt;
    return launch_pairs<STEP>(p, pws, s);
}

mx_status adjstep_impl(const float4 *x, const float4 *xb, const float4 *vb, int64_t n, float eps2, float G,
                       float dt, float4 *xbo, float4 *vbo, void *pws, hipStream_t s) {
    PairArgs p{};
    p.pos = x; p.aux = vb; p.aux2 = xb; p.out0 = xbo; p.out1 = vbo; p.n = n; p.eps2 = eps2; p.G = G; p.dt = dt;
    return launch_pairs<ADJSTEP>(p, pws, s);
}

mx_status kinetic_impl(const float4 *x, const float4 *v, int64_t n, float *ke, float4 *vbar, float4 *xbar,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_kinetic, dim3(1), dim3(NTK), 0, s, x, v, n, ke, vbar, xbar);
    return last_launch("nbody kinetic");
}

// Workspace of mx_nbody_ke_grad_f32: pair partials, then float4 states of n
// bodies -- final state (x, v), two ping-pong states, nck checkpoints (slot 0
// unused: the input is checkpoint 0), the positions of the last segment's k
// states, a tape of k states, and two adjoint ping-pong pairs (xbar, vbar).
struct NbodyWs {
    void *pair;
    float4 *fin_x, *fin_v, *tmp_x[2], *tmp_v[2], *ck_x, *ck_v, *last_x, *tape_x, *tape_v, *xb[2], *vb[2];
    size_t bytes;
};

NbodyWs nbody_ws_layout(char *base, int64_t n, int nsteps, int k) {
    NbodyWs w{};
    const size_t st = align256((size_t)n * 16);
    const int nck = (nsteps + k - 1) / k;
    size_t off = 0;
    auto take = [&](size_t b) { char *q = base ? base + off : nullptr; off += b; return q; };
    w.pair = take(align256(pair_ws_bytes(n)));
    w.fin_x = (float4 *)take(st);
    w.fin_v = (float4 *)take(st);
    for (int i = 0; i < 2; ++i) { w.tmp_x[i] = (float4 *)take(st); w.tmp_v[i] = (float4 *)take(st); }
    w.ck_x = (float4 *)take(st * (size_t)(nck > 0 ? nck : 1));
    w.ck_v = (float4 *)take(st * (size_t)(nck > 0 ? nck : 1));
    w.last_x = (float4 *)take(st * (size_t)k);
    w.tape_x = (float4 *)take(st * (size_t)k);
    w.tape_v = (float4 *)take(st * (size_t)k);
    for (int i = 0; i < 2; ++i) { w.xb[i] = (float4 *)take(st); w.vb[i] = (float4 *)take(st); }
    w.bytes = off;
    return w;
}

constexpr int kMaxCkptEvery = 64;

}  // namespace
}  // namespace mx

using namespace mx;

extern "C" {

size_t mx_nbody_pair_workspace_bytes(int64_t n) { return n < 0 ? 0 : pair_ws_bytes(n); }

size_t mx_nbody_workspace_bytes(int64_t n, int nsteps, int ckpt_every) {
    if (n < 0 || nsteps < 1 || ckpt_every < 1) return 0;
    const int k = ckpt_every < nsteps ? ckpt_every : nsteps;
    return align256(nbody_ws_layout(nullptr, n, nsteps, k).bytes);
}

mx_status mx_nbody_accel_f32(const float *pos4_dev, int64_t n, float eps2, float G, float *acc4_dev, void *ws,
                             size_t ws_bytes, hipStream_t stream) {
    if (mx_status st = check_common("mx_nbody_accel_f32", n, eps2, ws, ws_bytes, pair_ws_bytes(n))) return st;
    if (n == 0) return MX_OK;
    MX_REQUIRE(pos4_dev && acc4_dev && a16(pos4_dev) && a16(acc4_dev), MX_ERR_INVALID,
               "mx_nbody_accel_f32: null or unaligned pointer");
    PairArgs p{};
    p.pos = (const float4 *)pos4_dev; p.out0 = (float4 *)acc4_dev; p.n = n; p.eps2 = eps2; p.G = G;
    return launch_pairs<ACCEL>(p, ws, stream);
}

mx_status mx_nbody_step_f32(const float *pos4_dev, const float *vel4_dev, int64_t n, float eps2, float G,
                            float dt, float *pos4_out_dev, float *vel4_out_dev, void *ws, size_t ws_bytes,
                            hipStream_t stream) {
    if (mx_status st = check_common("mx_nbody_step_f32", n, eps2, ws, ws_bytes, pair_ws_bytes(n))) return st;
    if (n == 0) return MX_OK;
    MX_REQUIRE(pos4_dev && vel4_dev && pos4_out_dev && vel4_out_dev, MX_ERR_INVALID, "mx_nbody_step_f32: null pointer");
    MX_REQUIRE(a16(pos4_dev) && a16(vel4_dev) && a16(pos4_out_dev) && a16(vel4_out_dev), MX_ERR_INVALID,
               "mx_nbody_step_f32: pointers must be 16-byte aligned");
    MX_REQUIRE(pos4_out_dev != pos4_dev && vel4_out_dev != vel4_dev && pos4_out_dev != vel4_dev &&
                   vel4_out_dev != pos4_dev,
               MX_ERR_INVALID, "mx_nbody_step_f32: outputs must not alias inputs");
    return step_impl((const float4 *)pos4_dev, (const float4 *)vel4_dev, n, eps2, G, dt, (float4 *)pos4_out_dev,
                     (float4 *)vel4_out_dev, ws, stream);
}

mx_status mx_nbody_step_plain_f32(const float *pos4_dev, const float *vel4_dev, int64_t n, float eps2,
                                  float G, float dt, float *acc4_dev, float *pos4_out_dev,
                                  float *vel4_out_dev, hipStream_t stream) {
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "mx_nbody_step_plain_f32: n < 0");
    MX_REQUIRE(eps2 > 0.f, MX_ERR_INVALID, "mx_nbody_step_plain_f32: eps2 must be positive");
    if (n == 0) return MX_OK;
    MX_REQUIRE(pos4_dev && vel4_dev && acc4_dev && pos4_out_dev && vel4_out_dev, MX_ERR_INVALID,
               "mx_nbody_step_plain_f32: null pointer");
    MX_REQUIRE(a16(pos4_dev) && a16(vel4_dev) && a16(acc4_dev) && a16(pos4_out_dev) && a16(vel4_out_dev),
               MX_ERR_INVALID, "mx_nbody_step_plain_f32: pointers must be 16-byte aligned");
    const int64_t grid = ceil_div(n, NT);
    MX_REQUIRE(grid < (1LL << 31), MX_ERR_SHAPE, "mx_nbody_step_plain_f32: too many bodies");
    hipLaunchKernelGGL(k_accel_plain, dim3((unsigned)grid), dim3(NT), 0, stream, (const float4 *)pos4_dev, n, eps2,
                       G, (float4 *)acc4_dev);
    hipLaunchKernelGGL(k_euler, dim3((unsigned)grid), dim3(NT), 0, stream, (const float4 *)pos4_dev,
                       (const float4 *)vel4_dev, (const float4 *)acc4_dev, n, dt, (float4 *)pos4_out_dev,
                       (float4 *)vel4_out_dev);
    return last_launch("mx_nbody_step_plain_f32");
}

mx_status mx_nbody_accel_vjp_f32(const float *pos4_dev, const float *abar4_dev, int64_t n, float eps2,
                                 float G, float *out4_dev, void *ws, size_t ws_bytes, hipStream_t stream) {
    if (mx_status st = check_common("mx_nbody_accel_vjp_f32", n, eps2, ws, ws_bytes, pair_ws_bytes(n))) return st;
    if (n == 0) return MX_OK;
    MX_REQUIRE(pos4_dev && abar4_dev && out4_dev && a16(pos4_dev) && a16(abar4_dev) && a16(out4_dev),
               MX_ERR_INVALID, "mx_nbody_accel_vjp_f32: null or unaligned pointer");
    PairArgs p{};
    p.pos = (const float4 *)pos4_dev; p.aux = (const float4 *)abar4_dev; p.out0 = (float4 *)out4_dev;
    p.n = n; p.eps2 = eps2; p.G = G;
    return launch_pairs<VJP>(p, ws, stream);
}

mx_status mx_nbody_adjoint_step_f32(const float *pos4_dev, const float *xbar4_dev, const float *vbar4_dev,
                                    int64_t n, float eps2, float G, float dt, float *xbar4_out_dev,
                                    float *vbar4_out_dev, void *ws, size_t ws_bytes, hipStream_t stream) {
    const char *who = "mx_nbody_adjoint_step_f32";
    if (mx_status st = check_common(who, n, eps2, ws, ws_bytes, pair_ws_bytes(n))) return st;
    if (n == 0) return MX_OK;
    MX_REQUIRE(pos4_dev && xbar4_dev && vbar4_dev && xbar4_out_dev && vbar4_out_dev, MX_ERR_INVALID,
               "%s: null pointer", who);
    MX_REQUIRE(a16(pos4_dev) && a16(xbar4_dev) && a16(vbar4_dev) && a16(xbar4_out_dev) && a16(vbar4_out_dev),
               MX_ERR_INVALID, "%s: pointers must be 16-byte aligned", who);
    MX_REQUIRE(xbar4_out_dev != xbar4_dev && vbar4_out_dev != vbar4_dev && vbar4_out_dev != xbar4_dev &&
                   xbar4_out_dev != vbar4_dev,
               MX_ERR_INVALID, "%s: outputs must not alias inputs", who);
    return adjstep_impl((const float4 *)pos4_dev, (const float4 *)xbar4_dev, (const float4 *)vbar4_dev, n, eps2, G,
                        dt, (float4 *)xbar4_out_dev, (float4 *)vbar4_out_dev, ws, stream);
}

mx_status mx_nbody_kinetic_f32(const float *pos4_dev, const float *vel4_dev, int64_t n, float *ke_dev,
                               hipStream_t stream) {
    MX_REQUIRE(n >= 0, MX_ERR_SHAPE, "mx_nbody_kinetic_f32: n < 0");
    MX_REQUIRE(ke_dev && (n == 0 || (pos4_dev && vel4_dev)), MX_ERR_INVALID, "mx_nbody_kinetic_f32: null pointer");
    return kinetic_impl((const float4 *)pos4_dev, (const float4 *)vel4_dev, n, ke_dev, nullptr, nullptr, stream);
}

namespace {
mx_status ke_check(const char *who, const float *pos4_dev, const float *vel4_dev, int64_t n, float eps2,
                   int nsteps, int ckpt_every, void *ws, size_t ws_bytes) {
    MX_REQUIRE(nsteps >= 1 && ckpt_every >= 1 && ckpt_every <= kMaxCkptEvery, MX_ERR_INVALID,
               "%s: need nsteps >= 1 and 1 <= ckpt_every <= %d", who, kMaxCkptEvery);
    if (mx_status st = check_common(who, n, eps2, ws, ws_bytes, mx_nbody_workspace_bytes(n, nsteps, ckpt_every)))
        return st;
    if (n > 0)
        MX_REQUIRE(pos4_dev && vel4_dev && a16(pos4_dev) && a16(vel4_dev), MX_ERR_INVALID,
                   "%s: null or unaligned state pointer", who);
    return MX_OK;
}

// Forward loop: checkpoint c (c >= 1) holds the state at t = c k in the
// workspace (checkpoint 0 is the input itself), the final state goes to
// fin_x / fin_v, and the positions of the last segment, which the reverse
// sweep needs first, to entries of their own (so it recomputes nothing of that
// segment, however often it is called); then KE of the final state.
mx_status ke_forward(const float4 *x0, const float4 *v0, int64_t n, float eps2, float G, float dt, int nsteps,
                     int k, float *ke_dev, const NbodyWs &w, hipStream_t stream) {
    const int64_t st4 = (int64_t)(align256((size_t)n * 16) / 16);  // float4 stride between states
    const int t_last = (nsteps - 1) / k * k;  // start of the last segment
    const float4 *x = x0, *v = v0;
    for (int t = 0; t < nsteps; ++t) {
        float4 *xo, *vo;
        if (t >= t_last && t < nsteps - 1) {
            xo = w.last_x + (int64_t)(t + 1 - t_last) * st4; vo = w.tmp_v[t & 1];
        } else if (t == nsteps - 1) {
            xo = w.fin_x; vo = w.fin_v;
        } else if ((t + 1) % k == 0) {
            xo = w.ck_x + (int64_t)((t + 1) / k) * st4; vo = w.ck_v + (int64_t)((t + 1) / k) * st4;
        } else {
            xo = w.tmp_x[t & 1]; vo = w.tmp_v[t & 1];
        }
        if (mx_status st = step_impl(x, v, n, eps2, G, dt, xo, vo, w.pair, stream)) return st;
        x = xo;
        v = vo;
    }
    return kinetic_impl(w.fin_x, w.fin_v, n, ke_dev, nullptr, nullptr, stream);
}

// Reverse sweep from the checkpoints ke_forward left: vbar = g m v_T,
// xbar = 0, then segment by segment (last first) the adjoint steps walked back
// over the segment's positions: the last segment's as ke_forward left them,
// the others' recomputed forward from the segment's checkpoint onto the tape.
mx_status ke_reverse(const float4 *x0, const float4 *v0, int64_t n, float eps2, float G, float dt, int nsteps,
                     int k, const float *gscale, float4 *gx, float4 *gv, const NbodyWs &w, hipStream_t stream) {
    const int64_t st4 = (int64_t)(align256((size_t)n * 16) / 16);
    const int nck = (nsteps + k - 1) / k;
    int cur = 0;
    hipLaunchKernelGGL(k_adjoint_seed, dim3((unsigned)ceil_div(n, NT)), dim3(NT), 0, stream, w.fin_x, w.fin_v, n,
                       gscale, w.vb[0], w.xb[0]);
    if (mx_status st = last_launch("nbody adjoint seed")) return st;
    for (int c = nck - 1; c >= 0; --c) {
        const int t0 = c * k, t1 = (t0 + k < nsteps) ? t0 + k : nsteps;
        // recompute x_t for t0 <= t < t1 from the checkpoint (tape entry 0 is the checkpoint itself)
        const float4 *tape[kMaxCkptEvery];
        const float4 *rx = c == 0 ? x0 : w.ck_x + (int64_t)c * st4;
        const float4 *rv = c == 0 ? v0 : w.ck_v + (int64_t)c * st4;
        tape[0] = rx;
        if (c == nck - 1)
            for (int t = t0 + 1; t < t1; ++t) tape[t - t0] = w.last_x + (int64_t)(t - t0) * st4;
        for (int t = t0; c < nck - 1 && t < t1 - 1; ++t) {
            float4 *xo = w.tape_x + (int64_t)(t - t0 + 1) * st4, *vo = w.tape_v + (int64_t)(t - t0 + 1) * st4;
            if (mx_status st = step_impl(rx, rv, n, eps2, G, dt, xo, vo, w.pair, stream)) return st;
            rx = xo;
            rv = vo;
            tape[t - t0 + 1] = xo;
        }
        for (int t = t1 - 1; t >= t0; --t) {
            float4 *xbo = (t == 0) ? gx : w.xb[cur ^ 1];
            float4 *vbo = (t == 0) ? gv : w.vb[cur ^ 1];
            if (mx_status st = adjstep_impl(tape[t - t0], w.xb[cur], w.vb[cur], n, eps2, G, dt, xbo, vbo, w.pair,
                                            stream))
                return st;
            cur ^= 1;
        }
    }
    return MX_OK;
}
}  // namespace

mx_status mx_nbody_ke_f32(const float *pos4_dev, const float *vel4_dev, int64_t n, float eps2, float G, float dt,
                          int nsteps, int ckpt_every, float *ke_dev, void *ws, size_t ws_bytes,
                          hipStream_t stream) {
    const char *who = "mx_nbody_ke_f32";
    if (mx_status st = ke_check(who, pos4_dev, vel4_dev, n, eps2, nsteps, ckpt_every, ws, ws_bytes)) return st;
    MX_REQUIRE(ke_dev, MX_ERR_INVALID, "%s: null ke pointer", who);
    if (n == 0) return kinetic_impl(nullptr, nullptr, 0, ke_dev, nullptr, nullptr, stream);
    const int k = ckpt_every < nsteps ? ckpt_every : nsteps;
    NbodyWs w = nbody_ws_layout((char *)ws, n, nsteps, k);
    return ke_forward((const float4 *)pos4_dev, (const float4 *)vel4_dev, n, eps2, G, dt, nsteps, k, ke_dev, w,
                      stream);
}

mx_status mx_nbody_ke_vjp_f32(const float *pos4_dev, const float *vel4_dev, int64_t n, float eps2, float G,
                              float dt, int nsteps, int ckpt_every, const float *gscale_dev, float *gx4_dev,
                              float *gv4_dev, void *ws, size_t ws_bytes, hipStream_t stream) {
    const char *who = "mx_nbody_ke_vjp_f32";
    if (mx_status st = ke_check(who, pos4_dev, vel4_dev, n, eps2, nsteps, ckpt_every, ws, ws_bytes)) return st;
    if (n == 0) return MX_OK;
    MX_REQUIRE(gx4_dev && gv4_dev && a16(gx4_dev) && a16(gv4_dev), MX_ERR_INVALID,
               "%s: null or unaligned gradient pointer", who);
    const int k = ckpt_every < nsteps ? ckpt_every : nsteps;
    NbodyWs w = nbody_ws_layout((char *)ws, n, nsteps, k);
    return ke_reverse((const float4 *)pos4_dev, (const float4 *)vel4_dev, n, eps2, G, dt, nsteps, k, gscale_dev,
                      (float4 *)gx4_dev, (float4 *)gv4_dev, w, stream);
}

mx_status mx_nbody_ke_grad_f32(const float *pos4_dev, const float *vel4_dev, int64_t n, float eps2, float G,
                               float dt, int nsteps, int ckpt_every, float *ke_dev, float *gx4_dev,
                               float *gv4_dev, void *ws, size_t ws_bytes, hipStream_t stream) {
    const char *who = "mx_nbody_ke_grad_f32";
    if (mx_status st = ke_check(who, pos4_dev, vel4_dev, n, eps2, nsteps, ckpt_every, ws, ws_bytes)) return st;
    if (n == 0) return MX_OK;
    MX_REQUIRE(ke_dev && gx4_dev && gv4_dev && a16(gx4_dev) && a16(gv4_dev), MX_ERR_INVALID,
               "%s: null or unaligned pointer", who);
    const int k = ckpt_every < nsteps ? ckpt_every : nsteps;
    NbodyWs w = nbody_ws_layout((char *)ws, n, nsteps, k);
    const float4 *x0 = (const float4 *)pos4_dev, *v0 = (const float4 *)vel4_dev;
    if (mx_status st = ke_forward(x0, v0, n, eps2, G, dt, nsteps, k, ke_dev, w, stream)) return st;
    return ke_reverse(x0, v0, n, eps2, G, dt, nsteps, k, nullptr, (float4 *)gx4_dev, (float4 *)gv4_dev, w, stream);
}

}  // extern "C"
