// adjoint.hip -- gradient of the relaxed cut at the last step with respect to
// the per-step schedules K_t, Ks_t and sigma_t of a fixed-noise
// Euler-Maruyama trajectory (Sec. II-E Eq. 5 integrated as in Algorithm 1;
// the schedules are the annealing knobs of Sec. II-D / Fig. 3b).
//
// Loss (sum over replicas and instances), w = -J:
//     L = sum_{i<j} w_ij (1 - cos(th_T,i - th_T,j)) / 2
// Adjoint of th_{t+1} = th_t + dt f(th_t) + sigma_t sqrt(dt) xi_t with
// f_i = -K_t sum_j J_ij sin(th_i - th_j) - Ks_t sin(q th_i), J symmetric:
//     lam_T,i  = 1/2 sum_j w_ij sin(th_i - th_j)
//     lam_t,k  = lam_{t+1,k} + dt [ K_t sum_j J_kj cos(th_k - th_j) (lam_j - lam_k)
//                                   - q Ks_t cos(q th_k) lam_k ]      (lam at t+1)
//     dL/dK_t  = -dt sum_i lam_{t+1,i} sum_j J_ij sin(th_t,i - th_t,j)
//     dL/dKs_t = -dt sum_i lam_{t+1,i} sin(q th_t,i)
//     dL/dsig_t = sqrt(dt) sum_i lam_{t+1,i} xi_t,i
// The wrap of the phase has derivative 1 almost everywhere.  With the
// identities cos(a-b) = ca cb + sa sb and sin(a-b) = sa cb - ca sb every sum
// above is a CSR gather of four per-node values (s, c, s lam, c lam).
//
// One workgroup per (instance, replica).  The rows of an instance are dealt to
// the lanes by length, longest first (AdjRows in internal.hpp): the 64 rows a
// wave walks together have nearly the same length, where consecutive rows are
// padded to twice the mean (G(2000, 10/1999): mean 10, longest of 256 about
// 20).  A group of 64 rows is walked two entries per 32-bit word; groups go to
// the waves back and forth, so every wave has about the same work.  The
// oscillator at sorted position p of its instance is "slot" p: tables and the
// buffers between kernels are in slot order, caller arrays in oscillator
// order.  128 x G(2000, 10/1999), us per step and workgroup, with consecutive
// rows on eight waves and now: forward 3.9 -> 2.05, adjoint 6.7 -> 2.8; bound by
// the LDS reads of the neighbours (8 bytes each at random slots), then by the
// vector instructions beside them.
//
// Forward kernel: phases and own (sin, cos) in registers, neighbour (s, c) in
// an LDS ping-pong table, one barrier per step; the phase words are
// checkpointed every C steps into caller memory.  The Philox normals of a quad
// are drawn by one lane a step ahead and handed to the four rows' owners
// through LDS.  Backward: per segment of C steps (last first) the states are
// recomputed from the checkpoint (the noise is a pure function of (seed,
// oscillator, step, instance), so the recomputation is exact) into device
// scratch, and the adjoint recurrence runs back through them.  Per-step
// gradient partials are reduced over each wave in FP32 and over waves and
// workgroups in FP64 in a fixed order.
#include <float.h>

#include <cmath>

#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "internal.hpp"
#include "noise.hpp"
#include "phase.hpp"

// The forward kernel and the backward kernel's recomputation must round every
// step identically, so no multiply-add is fused unless written as fmaf.
#pragma clang fp contract(off)

namespace oim {

namespace {

constexpr int kMaxTB = 1024;
constexpr int kMaxWaves = kMaxTB / 64;
constexpr int kMaxRounds = kAdjMaxN / kMaxTB;  // rows per lane at the size limit

struct AdjArgs {
    AdjRows rows;          // device arrays of the sorted rows (internal.hpp)
    const int4* inst;      // per instance: first slice, slices, first oscillator, size
    int tabN;              // slots of the largest instance (its rows rounded up to 64)
    int quads;             // quads of the largest instance
    int noise2;            // 1: two noise buffers (0: one, wide segment kernel)
    int img_words;         // LDS words of the largest instance's image (LDSI)
    int I, n_total, P;     // instances, oscillators, padded words per replica
    int R, q, steps, C, nseg;
    int64_t step0;
    float dt;
    const float* K;
    const float* Ks;
    const float* sigma;
    const uint64_t* seeds;
    const float* theta0;   // [R][n_total] radians
    uint32_t* ckpt;        // [nseg][R][P] phase words, oscillator order
    float* thetaT;         // [R][n_total] or null
    double* loss;          // [R * I] or null
    uint32_t* seg;         // [C + 1][R][P] states of one segment, slot order (backward)
    float2* sums;          // [C][R][P] (csin, ccos0) of one segment's steps, or null (backward)
    double* gpart;         // [steps][3][R * I] (backward)
    float* lam;            // [R][P] adjoint state between segments, slot order (backward)
    int cur_seg;           // segment of this launch (backward)
    int wg0;               // the launch's first workgroup
};

template <int QM>
__device__ __forceinline__ float cos_q(float s, float c, uint32_t u, int q) {
    if constexpr (QM == 2) {
        return __builtin_fmaf(-2.0f * s, s, 1.0f);
    } else if constexpr (QM == 3) {
        return c * __builtin_fmaf(4.0f * c, c, -3.0f);
    } else {
        return cos_turn((uint32_t)q * u);
    }
}

// Per-workgroup view of its instance and replica, and the rows of a lane:
// round k holds slot slot[k] (group slot / 64), oscillator osc[k] of the
// instance (nb: no row).
struct Ctx {
    int wg, b, r, off, nb, nq, base, ng, rounds;
    uint32_t k0, k1;
    int grp[kMaxRounds];   // wave-uniform; ng: none
    int slot[kMaxRounds], osc[kMaxRounds];
    int pairs[kMaxRounds]; // wave-uniform: 32-bit words per row of the group
    int first[kMaxRounds]; // wave-uniform: the group's first word (in rows of 64) in the image
};

__device__ __forceinline__ Ctx make_ctx(const AdjArgs& a) {
    Ctx x;
    x.wg = a.wg0 + (int)blockIdx.x;
    x.b = x.wg % a.I;
    x.r = x.wg / a.I;
    const int4 in = a.inst[x.b];
    x.off = in.z;
    x.nb = in.w;
    x.nq = (in.w + 3) / 4;
    x.base = in.x * (4 * kSliceQuads);
    x.ng = (in.w + 63) / 64;
    const uint64_t seed = a.seeds[x.r];
    x.k0 = (uint32_t)seed;
    x.k1 = (uint32_t)(seed >> 32);
    const int lane = threadIdx.x & 63, W = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g0 = a.rows.group0[x.b];
#pragma unroll
    for (int k = 0; k < kMaxRounds; ++k) {
        const int g = k * W + ((k & 1) ? W - 1 - wave : wave);
        x.grp[k] = g < x.ng ? g : x.ng;
        x.slot[k] = g * 64 + lane;
        x.osc[k] = x.nb;
        x.pairs[k] = x.first[k] = 0;
        if (g < x.ng) {
            const int2 gd = a.rows.group[g0 + g];
            x.first[k] = __builtin_amdgcn_readfirstlane(gd.x);
            x.pairs[k] = __builtin_amdgcn_readfirstlane(gd.y);
            const int i = a.rows.osc[(g0 + g) * 64 + lane];
            x.osc[k] = i >= 0 ? i : x.nb;
        }
    }
    return x;
}

// Offset of (step slot, replica, local position) in a [steps][R][P] array.
__device__ __forceinline__ size_t at(const AdjArgs& a, const Ctx& x, int step, int i) {
    return ((size_t)step * a.R + x.r) * a.P + x.base + i;
}

// Where the rows' entries are read.  An entry is 16 bits: the neighbour's slot
// and, for unit weights, the sign of the weight in the top bit; two per word,
// [pair][lane] within a group, padding pointing at the zero entry (slot tabN).
//   UNIT  weights are +-1 (else FP32 weights are streamed from global memory,
//         two per lane and pair)
//   LDSI  the image sits in LDS, else it is streamed through L2
//   WIDE  the table's entries are 16 bytes (s, c, s lam, c lam), else 8
// In LDS the entries of an 8-byte table are byte offsets into it, and with
// unit weights the table has a negated copy that the entries of negative ones
// point into (NEG), so a term is an address, a read and two adds.
template <bool UNIT, bool LDSI, bool WIDE>
struct Image {
    static constexpr bool NEG = UNIT && LDSI && !WIDE;
    static constexpr bool BYTES = LDSI && !WIDE;
    using T = std::conditional_t<WIDE, float4, float2>;
    const uint32_t* idx;  // LDS or global
    const float2* w;      // global, !UNIT
    __device__ __forceinline__ uint32_t pair(int e) const { return idx[e * 64]; }
    __device__ __forceinline__ float2 weight(int e) const { return w[e * 64]; }
    // entry `half` of a word
    __device__ __forceinline__ static T read(const T* tab, uint32_t v, int half) {
        const uint32_t x = half ? v >> 16 : v & 0xffffu;
        if constexpr (BYTES)
            return *reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(tab) + x);
        else
            return tab[UNIT ? x & 0x7fffu : x];
    }
};

__device__ __forceinline__ float sign_weight(uint32_t sign_bit) {
    return __uint_as_float((sign_bit & 0x80000000u) | 0x3f800000u);
}

// Row sums over the table entries, `pairs` words of two entries: even entries
// into one partial sum, odd ones into the other, in order (a padding entry
// adds +-0 to a partial sum that is never -0), so every placement and
// grouping gives the same bits.  S[0] = sum J y_j, S[1] = sum J x_j of the
// table's (x, y); WIDE: S[2] = sum J w_j, S[3] = sum J z_j too.
template <bool UNIT, bool LDSI, bool WIDE>
__device__ __forceinline__ void row_sums(const Image<UNIT, LDSI, WIDE>& im,
                                         const typename Image<UNIT, LDSI, WIDE>::T* tab, int first,
                                         int pairs, float (&S)[4]) {
    using Im = Image<UNIT, LDSI, WIDE>;
    float s0[4] = {0.f, 0.f, 0.f, 0.f}, s1[4] = {0.f, 0.f, 0.f, 0.f};
    auto batch = [&](int e, auto count) __attribute__((always_inline)) {
        constexpr int N = decltype(count)::value;
        uint32_t v[N];
        float2 w[N];
        typename Im::T p[2 * N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            v[k] = im.pair(first + e + k);
            if constexpr (!UNIT) w[k] = im.weight(first + e + k);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            p[2 * k] = Im::read(tab, v[k], 0);
            p[2 * k + 1] = Im::read(tab, v[k], 1);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if constexpr (Im::NEG) {
                s0[0] = s0[0] + p[2 * k].y;
                s0[1] = s0[1] + p[2 * k].x;
                s1[0] = s1[0] + p[2 * k + 1].y;
                s1[1] = s1[1] + p[2 * k + 1].x;
            } else {
                const float w0 = UNIT ? sign_weight(v[k] << 16) : w[k].x;
                const float w1 = UNIT ? sign_weight(v[k]) : w[k].y;
                s0[0] = __builtin_fmaf(w0, p[2 * k].y, s0[0]);
                s0[1] = __builtin_fmaf(w0, p[2 * k].x, s0[1]);
                s1[0] = __builtin_fmaf(w1, p[2 * k + 1].y, s1[0]);
                s1[1] = __builtin_fmaf(w1, p[2 * k + 1].x, s1[1]);
                if constexpr (WIDE) {
                    s0[2] = __builtin_fmaf(w0, p[2 * k].w, s0[2]);
                    s0[3] = __builtin_fmaf(w0, p[2 * k].z, s0[3]);
                    s1[2] = __builtin_fmaf(w1, p[2 * k + 1].w, s1[2]);
                    s1[3] = __builtin_fmaf(w1, p[2 * k + 1].z, s1[3]);
                }
            }
        }
    };
    int e = 0;
    for (; e + 4 <= pairs; e += 4) batch(e, std::integral_constant<int, 4>{});
    if (e + 2 <= pairs) {
        batch(e, std::integral_constant<int, 2>{});
        e += 2;
    }
    if (e < pairs) batch(e, std::integral_constant<int, 1>{});
#pragma unroll
    for (int t = 0; t < 4; ++t) S[t] = s0[t] + s1[t];
}

// Dynamic LDS of a kernel: two tables of tabN + 1 entries (NEG: each followed
// by its negated copy), the noise buffers [2 or 1][quads], the image (LDSI).
// The constructor zeroes the zero entries and copies the instance's image;
// the caller's first barrier publishes them.
template <bool UNIT, bool LDSI, bool WIDE>
struct Lds {
    using Im = Image<UNIT, LDSI, WIDE>;
    using T = typename Im::T;
    T* tabs;
    int stride, neg;   // entries per table, and to the negated copy
    float4* noise;
    Im im;
    __device__ __forceinline__ Lds(const AdjArgs& a, const Ctx& x, unsigned char* smem) {
        neg = a.tabN + 1;
        stride = neg * (Im::NEG ? 2 : 1);
        tabs = reinterpret_cast<T*>(smem);
        noise = reinterpret_cast<float4*>(smem + (((size_t)2 * stride * sizeof(T) + 15) & ~(size_t)15));
        uint32_t* img = reinterpret_cast<uint32_t*>(noise + (a.noise2 ? 2 : 1) * a.quads);
        if (threadIdx.x < (Im::NEG ? 4 : 2))
            tabs[(threadIdx.x & 1) * stride + (threadIdx.x >> 1) * neg + a.tabN] = T{};
        const int lane = threadIdx.x & 63;
        const int2 span = a.rows.span[x.b];  // first row of 64 words, rows
        const uint32_t* src = a.rows.idx + (size_t)span.x * 64;
        if constexpr (LDSI) {
            for (int e = threadIdx.x; e < span.y * 64; e += blockDim.x) {
                uint32_t v = src[e];
                if constexpr (Im::BYTES) {
                    uint32_t lo = v & 0xffffu, hi = v >> 16;
                    if constexpr (Im::NEG) {
                        lo = (lo & 0x7fffu) + (lo >> 15) * neg;
                        hi = (hi & 0x7fffu) + (hi >> 15) * neg;
                    }
                    v = lo * 8 | (hi * 8) << 16;
                }
                img[e] = v;
            }
            im.idx = img + lane;
        } else {
            im.idx = src + lane;
        }
        im.w = UNIT ? nullptr : a.rows.w + (size_t)span.x * 64 + lane;
    }
    __device__ __forceinline__ T* tab(int p) const { return tabs + p * stride; }
    __device__ __forceinline__ void put(int p, int slot, float2 v) const {
        tab(p)[slot] = v;
        if constexpr (Im::NEG) tab(p)[slot + neg] = make_float2(-v.x, -v.y);
    }
};

// The normals of step t of every quad, four per quad in oscillator order.
__device__ __forceinline__ void draw_noise(const AdjArgs& a, const Ctx& x, uint32_t t, float4* noise) {
    for (int m = threadIdx.x; m < x.nq; m += blockDim.x) {
        float z[4];
        normals4((uint32_t)m, t, (uint32_t)x.b, x.k0, x.k1, z);
        noise[m] = make_float4(z[0], z[1], z[2], z[3]);
    }
}

// The schedules, 64 steps at a time in the lanes of every wave (backwards:
// chunks of the same alignment), so that no step waits on a scalar load.
struct Sched {
    float K, Ks, sg;
    int chunk;
    __device__ __forceinline__ void load(const AdjArgs& a, int c) {
        const int i = c * 64 + (int)(threadIdx.x & 63);
        const bool in = i < a.steps;
        K = in ? a.K[i] : 0.f;
        Ks = in ? a.Ks[i] : 0.f;
        sg = in ? a.sigma[i] : 0.f;
        chunk = c;
    }
    __device__ __forceinline__ static float pick(float v, int s) {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), s & 63));
    }
};

// The forward steps t0 .. t1 - 1 from the words u: before(s) sees the state
// before step s in u and sc, sums(s, k, S) the row sums S of round k at it.
// Leaves the state at t1 in u, sc and the table of the returned parity.
template <int QM, bool UNIT, bool LDSI, class Before, class Sums>
__device__ __forceinline__ int forward_steps(const AdjArgs& a, const Ctx& x,
                                             const Lds<UNIT, LDSI, false>& l, int t0, int t1,
                                             uint32_t (&u)[kMaxRounds], float2 (&sc)[kMaxRounds],
                                             Before before, Sums sums) {
    const int q = QM ? QM : a.q;
    const float sqrt_dt = __builtin_sqrtf(a.dt);
#pragma unroll
    for (int k = 0; k < kMaxRounds; ++k)
        if (x.grp[k] < x.ng) {
            sc[k] = make_float2(sin_turn(u[k]), cos_turn(u[k]));
            l.put(0, x.slot[k], sc[k]);
        }
    if (t0 < t1) draw_noise(a, x, (uint32_t)(a.step0 + t0), l.noise);
    Sched sch;
    sch.load(a, t0 >> 6);
    __syncthreads();
    int p = 0;
    for (int s = t0; s < t1; ++s) {
        if ((s >> 6) != sch.chunk) sch.load(a, s >> 6);
        before(s);
        const float kc = -a.dt * Sched::pick(sch.K, s) * kTurnScale;
        const float ks = -a.dt * Sched::pick(sch.Ks, s) * kTurnScale;
        const float ns = Sched::pick(sch.sg, s) * sqrt_dt * kTurnScale;
        const float* z = reinterpret_cast<const float*>(l.noise + p * a.quads);
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k) {
            if (x.grp[k] >= x.ng) break;
            const float zk = z[x.osc[k] < x.nb ? x.osc[k] : 0];
            float S[4];
            row_sums(l.im, l.tab(p), x.first[k], x.pairs[k], S);
            sums(s, k, S);
            const float si = sc[k].x, ci = sc[k].y;
            const float coup = __builtin_fmaf(si, S[0], -(ci * S[1]));
            const float drift = __builtin_fmaf(kc, coup, ks * sin_q<QM>(si, ci, u[k], q));
            u[k] = advance(u[k], __builtin_fmaf(ns, zk, drift));
            sc[k] = make_float2(sin_turn(u[k]), cos_turn(u[k]));
            l.put(p ^ 1, x.slot[k], sc[k]);
        }
        if (s + 1 < t1) draw_noise(a, x, (uint32_t)(a.step0 + s + 1), l.noise + (p ^ 1) * a.quads);
        p ^= 1;
        __syncthreads();
    }
    return p;
}

template <int QM, bool UNIT, bool LDSI>
__global__ __launch_bounds__(kMaxTB) void adjoint_forward_kernel(AdjArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kMaxWaves];
    const Ctx x = make_ctx(a);
    const Lds<UNIT, LDSI, false> l(a, x, smem);
    uint32_t u[kMaxRounds];
    float2 sc[kMaxRounds];
#pragma unroll
    for (int k = 0; k < kMaxRounds; ++k)
        u[k] = x.osc[k] < x.nb
                   ? phase_from_theta(a.theta0[(size_t)x.r * a.n_total + x.off + x.osc[k]])
                   : 0u;
    const int p = forward_steps<QM>(
        a, x, l, 0, a.steps, u, sc,
        [&](int s) {
            if (s % a.C) return;
#pragma unroll
            for (int k = 0; k < kMaxRounds; ++k)
                if (x.osc[k] < x.nb) a.ckpt[at(a, x, s / a.C, x.osc[k])] = u[k];
        },
        [](int, int, const float (&)[4]) {});
    // relaxed cut of the final phases: sum_i (c_i A_i + s_i B_i - sum_j J_ij) / 4
    double part = 0.0;
#pragma unroll
    for (int k = 0; k < kMaxRounds; ++k) {
        if (x.grp[k] >= x.ng) break;
        float S[4];
        row_sums(l.im, l.tab(p), x.first[k], x.pairs[k], S);
        if (x.osc[k] < x.nb) {
            const double rs = a.rows.row_sum[x.off + x.osc[k]];
            part += 0.25 * ((double)sc[k].y * S[0] + (double)sc[k].x * S[1] - rs);
            if (a.thetaT)
                a.thetaT[(size_t)x.r * a.n_total + x.off + x.osc[k]] = theta_from_phase(u[k]);
        }
    }
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
    __syncthreads();
    if (threadIdx.x == 0 && a.loss) {
        double tot = 0.0;
        for (int w = 0; w < (int)blockDim.x / 64; ++w) tot += red[w];
        a.loss[x.wg] = tot;
    }
}

// Backward pass, segment a.cur_seg (steps t0 .. t1 - 1), in two kernels that
// run on two streams so that the recomputation of one segment overlaps the
// adjoint of the next (later) one, each kernel on its own half of the CUs.
//
// Recompute: the segment's states from its checkpoint, written to a.seg
// (step slot s - t0 holds the state at step s; the last segment also computes
// its final step and stores the state at t1 in step slot t1 - t0).  The
// Philox noise is a pure function of (seed, oscillator, step, instance) and
// every placement of the rows gives the same bits, so these are the forward
// pass's states.  With a.sums it also hands over what the adjoint needs of
// the row sums it has formed anyway: csin = s A - c B and ccos0 = c A + s B
// per step, so that the adjoint gathers two values per neighbour instead of
// four.
template <int QM, bool UNIT, bool LDSI>
__global__ __launch_bounds__(kMaxTB) void adjoint_recompute_kernel(AdjArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Ctx x = make_ctx(a);
    const Lds<UNIT, LDSI, false> l(a, x, smem);
    const int sg = a.cur_seg;
    const int t0 = sg * a.C;
    const int t1 = t0 + a.C < a.steps ? t0 + a.C : a.steps;
    const int tend = sg == a.nseg - 1 ? t1 : t1 - 1;  // the last state stored
    uint32_t u[kMaxRounds];
    float2 sc[kMaxRounds];
#pragma unroll
    for (int k = 0; k < kMaxRounds; ++k)
        u[k] = x.osc[k] < x.nb ? a.ckpt[at(a, x, sg, x.osc[k])] : 0u;
    auto store = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k)
            if (x.grp[k] < x.ng) a.seg[at(a, x, s - t0, x.slot[k])] = u[k];
    };
    auto store_sums = [&](int s, int k, const float (&S)[4]) __attribute__((always_inline)) {
        const float si = sc[k].x, ci = sc[k].y;
        if (a.sums)
            a.sums[at(a, x, s - t0, x.slot[k])] =
                make_float2(si * S[0] - ci * S[1], ci * S[0] + si * S[1]);
    };
    const int p = forward_steps<QM>(a, x, l, t0, tend, u, sc, store, store_sums);
    store(tend);
    if (a.sums && tend < t1) {
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k) {
            if (x.grp[k] >= x.ng) break;
            float S[4];
            row_sums(l.im, l.tab(p), x.first[k], x.pairs[k], S);
            store_sums(tend, k, S);
        }
    }
}

// v plus the value a DPP move brings (0 where it brings none).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float add_dpp(float v) {
    return v + __int_as_float(
                   __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

// Sum over the wave by DPP adds (no LDS traffic); valid in lane 63.
__device__ __forceinline__ float wave_sum63(float v) {
    v = add_dpp<0x111, 0xf>(v);  // row_shr:1
    v = add_dpp<0x112, 0xf>(v);  // row_shr:2
    v = add_dpp<0x114, 0xf>(v);  // row_shr:4
    v = add_dpp<0x118, 0xf>(v);  // row_shr:8
    v = add_dpp<0x142, 0xa>(v);  // row_bcast:15
    return add_dpp<0x143, 0xc>(v);  // row_bcast:31
}

// Adjoint: the recurrence back through the segment's stored states, from the
// adjoint state left by the later segment in a.lam (or, for the last
// segment, lam_T from the final phases); the adjoint state at t0 goes back
// to a.lam.  Per-step gradient partials of the workgroup go to a.gpart.
// WIDE: the sums over (s, c) are formed here, from a table of (s, c, s lam,
// c lam); else they come from a.sums and the table holds (s lam, c lam).
template <int QM, bool UNIT, bool LDSI, bool WIDE>
__global__ __launch_bounds__(kMaxTB) void adjoint_segment_kernel(AdjArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float red[2][3][kMaxWaves];
    const Ctx x = make_ctx(a);
    const Lds<UNIT, LDSI, WIDE> lds(a, x, smem);
    const int q = QM ? QM : a.q;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = blockDim.x >> 6;
    const int nwg = a.R * a.I;
    const float sqrt_dt = __builtin_sqrtf(a.dt);
    const int sg = a.cur_seg;
    const int t0 = sg * a.C;
    const int t1 = t0 + a.C < a.steps ? t0 + a.C : a.steps;
    uint32_t u[kMaxRounds], un[kMaxRounds];
    float2 cs[kMaxRounds], csn[kMaxRounds];  // (csin, ccos0) of the step, !WIDE
    float lam[kMaxRounds];
    auto load = [&](int step, bool sums) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k) {
            un[k] = 0u;
            csn[k] = make_float2(0.f, 0.f);
            if (x.grp[k] >= x.ng) continue;
            un[k] = a.seg[at(a, x, step, x.slot[k])];
            if (!WIDE && sums) csn[k] = a.sums[at(a, x, step, x.slot[k])];
        }
    };
    int p = 0;  // table written next
    if (sg == a.nseg - 1) {
        // lam_T from the final phases
        load(t1 - t0, false);
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k) {
            if (x.grp[k] >= x.ng) continue;
            const float si = sin_turn(un[k]), ci = cos_turn(un[k]);
            if constexpr (WIDE) lds.tab(0)[x.slot[k]] = make_float4(si, ci, 0.f, 0.f);
            else lds.put(0, x.slot[k], make_float2(si, ci));
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k) {
            lam[k] = 0.f;
            if (x.grp[k] >= x.ng) continue;
            float S[4];
            row_sums(lds.im, lds.tab(0), x.first[k], x.pairs[k], S);
            const float si = sin_turn(un[k]), ci = cos_turn(un[k]);
            if (x.osc[k] < x.nb) lam[k] = -0.5f * (si * S[0] - ci * S[1]);
        }
        p = 1;
    } else {
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k)
            lam[k] = x.grp[k] < x.ng ? a.lam[at(a, x, 0, x.slot[k])] : 0.f;
    }
    load(t1 - 1 - t0, true);
    Sched sch;
    sch.load(a, (t1 - 1) >> 6);
    // a step's wave partials, after the barrier that follows it: FP64, waves in order
    auto flush = [&](int step, int buf) __attribute__((always_inline)) {
        if (threadIdx.x < 3) {
            double g = 0.0;
            for (int w = 0; w < W; ++w) g += (double)red[buf][threadIdx.x][w];
            a.gpart[((size_t)step * 3 + threadIdx.x) * nwg + x.wg] = g;
        }
    };
    for (int s = t1 - 1; s >= t0; --s) {
        if ((s >> 6) != sch.chunk) sch.load(a, s >> 6);
        float2 sc[kMaxRounds];
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k) {
            u[k] = un[k];
            cs[k] = csn[k];
            if (x.grp[k] >= x.ng) continue;
            sc[k] = make_float2(sin_turn(u[k]), cos_turn(u[k]));
            const float sl = sc[k].x * lam[k], cl = sc[k].y * lam[k];
            if constexpr (WIDE) lds.tab(p)[x.slot[k]] = make_float4(sc[k].x, sc[k].y, sl, cl);
            else lds.put(p, x.slot[k], make_float2(sl, cl));
        }
        if (s > t0) load(s - 1 - t0, true);  // their latency under this step
        float4* nz = lds.noise + (a.noise2 ? p * a.quads : 0);
        draw_noise(a, x, (uint32_t)(a.step0 + s), nz);
        __syncthreads();
        if (s + 1 < t1) flush(s + 1, p ^ 1);
        const float Kt = Sched::pick(sch.K, s), Kst = Sched::pick(sch.Ks, s);
        float gk = 0.f, gks = 0.f, gs = 0.f;
        const float* z = reinterpret_cast<const float*>(nz);
#pragma unroll
        for (int k = 0; k < kMaxRounds; ++k) {
            if (x.grp[k] >= x.ng) break;
            const float zk = z[x.osc[k] < x.nb ? x.osc[k] : 0];
            float S[4];
            row_sums(lds.im, lds.tab(p), x.first[k], x.pairs[k], S);
            const float si = sc[k].x, ci = sc[k].y;
            const float l = lam[k];  // 0 past the instance's rows, and stays 0
            const float Cl = WIDE ? S[2] : S[0], Dl = WIDE ? S[3] : S[1];
            const float csin = WIDE ? si * S[0] - ci * S[1] : cs[k].x;
            const float ccos0 = WIDE ? ci * S[0] + si * S[1] : cs[k].y;
            const float ccos = ci * Cl + si * Dl - l * ccos0;
            gk = __builtin_fmaf(l, csin, gk);
            gks = __builtin_fmaf(l, sin_q<QM>(si, ci, u[k], q), gks);
            gs = __builtin_fmaf(l, zk, gs);
            lam[k] = l + a.dt * (Kt * ccos - (float)q * Kst * cos_q<QM>(si, ci, u[k], q) * l);
        }
        gk = wave_sum63(gk);
        gks = wave_sum63(gks);
        gs = wave_sum63(gs);
        if (lane == 63) {
            red[p][0][wave] = -a.dt * gk;
            red[p][1][wave] = -a.dt * gks;
            red[p][2][wave] = sqrt_dt * gs;
        }
        if (!a.noise2) __syncthreads();  // the one noise buffer is rewritten next
        if (s == t0) {
            __syncthreads();
            flush(s, p);
        }
        p ^= 1;
    }
#pragma unroll
    for (int k = 0; k < kMaxRounds; ++k)
        if (x.grp[k] < x.ng) a.lam[at(a, x, 0, x.slot[k])] = lam[k];
}

// gK[s] etc. = sum over the workgroups' partials, FP64, in a fixed order: one
// workgroup per step, thread t takes partials t, t + 256, ..., then a tree.
__global__ __launch_bounds__(256) void adjoint_reduce_kernel(const double* gpart, int nparts,
                                                             double* gK, double* gKs, double* gS) {
    __shared__ double red[3][4];
    const int s = blockIdx.x;
    for (int v = 0; v < 3; ++v) {
        const double* p = gpart + ((size_t)s * 3 + v) * nparts;
        double t = 0.0;
        for (int k = threadIdx.x; k < nparts; k += 256) t += p[k];
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        if ((threadIdx.x & 63) == 0) red[v][threadIdx.x >> 6] = t;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const double t = (red[threadIdx.x][0] + red[threadIdx.x][1]) +
                         (red[threadIdx.x][2] + red[threadIdx.x][3]);
        (threadIdx.x == 0 ? gK : threadIdx.x == 1 ? gKs : gS)[s] = t;
    }
}

// ---- the sorted rows, made with the problem ----

// Words and weights of one group of 64 rows, a lane per row; row_sum[i] = sum
// of the row's weights in entry order (the loss's constant).
__global__ __launch_bounds__(64) void adjoint_rows_kernel(AdjRows rows, const int64_t* row_ptr,
                                                          const int32_t* col, const float* J,
                                                          const int4* inst, const int32_t* inst_of,
                                                          const uint16_t* slot_of, uint32_t* idx,
                                                          float2* w, double* row_sum, int tabN,
                                                          int unit) {
    const int g = blockIdx.x, lane = threadIdx.x;
    const int b = inst_of[g];
    const int off = inst[b].z;
    const int2 gd = rows.group[g];
    const int i = rows.osc[g * 64 + lane];
    const int64_t r0 = i >= 0 ? row_ptr[off + i] : 0;
    const int len = i >= 0 ? (int)(row_ptr[off + i + 1] - r0) : 0;
    const size_t base = (size_t)(rows.span[b].x + gd.x) * 64 + lane;
    double sum = 0.0;
    for (int e = 0; e < gd.y; ++e) {
        uint32_t v[2];
        float wt[2];
        for (int h = 0; h < 2; ++h) {
            const int x = 2 * e + h;
            v[h] = (uint32_t)tabN;
            wt[h] = 0.f;
            if (x < len) {
                wt[h] = J[r0 + x];
                v[h] = slot_of[col[r0 + x]] | (unit && wt[h] < 0.f ? 0x8000u : 0u);
                sum += (double)wt[h];
            }
        }
        idx[base + (size_t)e * 64] = v[0] | (v[1] << 16);
        if (w) w[base + (size_t)e * 64] = make_float2(wt[0], wt[1]);
    }
    if (i >= 0) row_sum[off + i] = sum;
}

using AdjFn = void (*)(AdjArgs);

constexpr size_t kAdjLdsLimit = 160 * 1024 - 1024;  // dynamic LDS next to the static reduction slots

// Placement of the rows' words and the LDS a kernel needs with it: in LDS
// when they fit next to the tables and noise buffers (which byte offsets of 16
// bits then reach), else streamed from global memory (OIM_ADJ_ROWS=global
// streams them at any size; any other value leaves the choice).  The wide
// segment kernel of instances near 4096 oscillators has room for one noise
// buffer only, at one more barrier per step.
struct Placement {
    bool ldsi;
    int noise2;
    size_t lds;
};

Placement place(const Problem* p, const AdjArgs& a, bool wide) {
    const char* env = getenv("OIM_ADJ_ROWS");
    const bool stream = env && !strcmp(env, "global");
    const size_t noise = (size_t)a.quads * 16, img = (size_t)a.img_words * 4;
    auto tables = [&](bool ldsi) -> size_t {
        if (wide) return (size_t)2 * (a.tabN + 1) * 16;
        return ((size_t)2 * (a.tabN + 1) * 8 * (p->unit_weights && ldsi ? 2 : 1) + 15) & ~(size_t)15;
    };
    if (!stream && tables(true) + 2 * noise + img <= kAdjLdsLimit && (wide || tables(true) <= 131072))
        return {true, 1, tables(true) + 2 * noise + img};
    if (tables(false) + 2 * noise <= kAdjLdsLimit) return {false, 1, tables(false) + 2 * noise};
    return {false, 0, tables(false) + noise};
}

#define OIM_ADJ_FNS(NAME, ...)                                                               \
    {{{adjoint_##NAME##_kernel<0, false, false __VA_ARGS__>,                                 \
       adjoint_##NAME##_kernel<0, false, true __VA_ARGS__>},                                 \
      {adjoint_##NAME##_kernel<0, true, false __VA_ARGS__>,                                  \
       adjoint_##NAME##_kernel<0, true, true __VA_ARGS__>}},                                 \
     {{adjoint_##NAME##_kernel<2, false, false __VA_ARGS__>,                                 \
       adjoint_##NAME##_kernel<2, false, true __VA_ARGS__>},                                 \
      {adjoint_##NAME##_kernel<2, true, false __VA_ARGS__>,                                  \
       adjoint_##NAME##_kernel<2, true, true __VA_ARGS__>}},                                 \
     {{adjoint_##NAME##_kernel<3, false, false __VA_ARGS__>,                                 \
       adjoint_##NAME##_kernel<3, false, true __VA_ARGS__>},                                 \
      {adjoint_##NAME##_kernel<3, true, false __VA_ARGS__>,                                  \
       adjoint_##NAME##_kernel<3, true, true __VA_ARGS__>}}}
const AdjFn kForward[3][2][2] = OIM_ADJ_FNS(forward);
const AdjFn kRecompute[3][2][2] = OIM_ADJ_FNS(recompute);
const AdjFn kSegment[3][2][2] = OIM_ADJ_FNS(segment, , false);
const AdjFn kSegmentWide[3][2][2] = OIM_ADJ_FNS(segment, , true);
#undef OIM_ADJ_FNS

AdjFn pick_fn(const AdjFn (&f)[3][2][2], const Problem* p, int q, bool ldsi) {
    return f[q == 2 ? 1 : q == 3 ? 2 : 0][p->unit_weights][ldsi];
}

// A grid dimension ends at 2^32 threads, past which a launch wraps without an
// error, so more than 2^31 go in several launches.
int launch_adj(AdjFn fn, size_t lds, int grid, int threads, hipStream_t stream, AdjArgs a,
               const char* what) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_error(e, what);
    const int most = (int)(((int64_t)1 << 31) / threads);
    for (int64_t g = 0; g < grid; g += most) {
        a.wg0 = (int)g;
        hipLaunchKernelGGL(fn, dim3((unsigned)(grid - g < most ? grid - g : most)), dim3(threads), lds,
                           stream, a);
    }
    e = hipGetLastError();
    return e == hipSuccess ? OIM_OK : hip_error(e, what);
}

int check_launch(const char* what) {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? OIM_OK : hip_error(e, what);
}

AdjArgs base_args(const Problem* p, const oim_adjoint_cfg* cfg, const float* K, const float* Ks,
                  const float* sigma, const uint64_t* seeds, int64_t step0) {
    AdjArgs a{};
    a.rows = p->adj_rows;
    a.inst = p->d_inst;
    a.I = p->n_inst;
    a.n_total = p->n;
    a.P = p->sell_slices * 4 * kSliceQuads;
    a.R = cfg->R;
    a.q = cfg->q;
    a.steps = cfg->steps;
    a.C = cfg->checkpoint_every;
    a.nseg = (cfg->steps + cfg->checkpoint_every - 1) / cfg->checkpoint_every;
    a.step0 = step0;
    a.dt = cfg->dt;
    a.tabN = (p->max_inst_n + 63) & ~63;
    a.quads = (p->max_inst_n + 3) / 4;
    a.img_words = p->adj_max_words;
    a.K = K;
    a.Ks = Ks;
    a.sigma = sigma;
    a.seeds = seeds;
    return a;
}

// A wave per group of 64 rows of the largest instance, sixteen at most.
int block_threads(const AdjArgs& a) { return a.tabN < kMaxTB ? a.tabN : kMaxTB; }

}  // namespace

void adjoint_layout(const Problem* p, const AdjRowsHost& h, AdjLayout& out) {
    // group spans, groups, first groups, oscillators, slots, instances of groups
    const size_t I = h.span.size(), G = h.group.size(), n = h.slot_of.size();
    auto append = [&](const void* src, size_t bytes) {
        const size_t o = out.blob.size();
        out.blob.resize(o + (bytes + 15) / 16 * 16);
        if (bytes) std::memcpy(out.blob.data() + o, src, bytes);
        return o;
    };
    out.span = append(h.span.data(), I * sizeof(int2));
    out.group = append(h.group.data(), G * sizeof(int2));
    out.group0 = append(h.group0.data(), I * sizeof(int32_t));
    out.osc = append(h.osc.data(), G * 64 * sizeof(int16_t));
    out.slot = append(h.slot_of.data(), n * sizeof(uint16_t));
    out.inst = append(h.inst_of.data(), G * sizeof(int32_t));
    const size_t words = (size_t)h.rows64 * 64;
    out.idx_bytes = (words * 4 + 255) / 256 * 256;
    out.w_bytes = p->unit_weights ? 0 : (words * 8 + 255) / 256 * 256;
    out.image_bytes = out.idx_bytes + out.w_bytes + n * 8 + 16;
}

int adjoint_build(Problem* p, const AdjRowsHost& h, const AdjLayout& l) {
    const unsigned char* d = static_cast<const unsigned char*>(p->d_adj_rows);
    unsigned char* img = static_cast<unsigned char*>(p->d_adj_img);
    uint32_t* idx = reinterpret_cast<uint32_t*>(img);
    float2* w = l.w_bytes ? reinterpret_cast<float2*>(img + l.idx_bytes) : nullptr;
    double* row_sum = reinterpret_cast<double*>(img + l.idx_bytes + l.w_bytes);
    AdjRows& r = p->adj_rows;
    r.span = reinterpret_cast<const int2*>(d + l.span);
    r.group = reinterpret_cast<const int2*>(d + l.group);
    r.group0 = reinterpret_cast<const int32_t*>(d + l.group0);
    r.osc = reinterpret_cast<const int16_t*>(d + l.osc);
    r.idx = idx;
    r.w = w;
    r.row_sum = row_sum;
    p->adj_max_words = h.max_words;
    hipLaunchKernelGGL(adjoint_rows_kernel, dim3((unsigned)h.group.size()), dim3(64), 0, 0, r, p->d_row_ptr, p->d_col,
                       p->d_J, p->d_inst, reinterpret_cast<const int32_t*>(d + l.inst),
                       reinterpret_cast<const uint16_t*>(d + l.slot), idx, w, row_sum,
                       (p->max_inst_n + 63) & ~63, p->unit_weights ? 1 : 0);
    return check_launch("adjoint_rows_kernel");
}

namespace {

int make_rows(Problem* p) {
    std::vector<int64_t> row_ptr((size_t)p->n + 1);
    std::vector<int4> inst((size_t)p->n_inst);
    hipError_t e = hipMemcpy(row_ptr.data(), p->d_row_ptr, row_ptr.size() * 8, hipMemcpyDeviceToHost);
    if (e == hipSuccess)
        e = hipMemcpy(inst.data(), p->d_inst, inst.size() * sizeof(int4), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_error(e, "adjoint rows");
    std::vector<int32_t> off;
    for (const int4& in : inst) off.push_back(in.z);
    off.push_back(p->n);
    AdjRowsHost rows;
    build_adj_rows(p->n, row_ptr.data(), p->n_inst, off.data(), rows);
    AdjLayout layout;
    adjoint_layout(p, rows, layout);
    const size_t blob = (layout.blob.size() + 255) / 256 * 256;
    if (!p->d_adj_own) {
        e = hipMalloc(&p->d_adj_own, blob + layout.image_bytes);
        if (e != hipSuccess) {
            p->d_adj_own = nullptr;
            (void)hipGetLastError();
            return e == hipErrorOutOfMemory ? set_error(OIM_E_NOMEM, "adjoint rows: out of device memory")
                                            : hip_error(e, "adjoint rows");
        }
    }
    p->d_adj_rows = p->d_adj_own;
    p->d_adj_img = static_cast<unsigned char*>(p->d_adj_own) + blob;
    e = hipMemcpy(p->d_adj_rows, layout.blob.data(), layout.blob.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_error(e, "adjoint rows");
    int st = adjoint_build(p, rows, layout);
    // the caller's stream runs next
    if (!st && (e = hipStreamSynchronize(0)) != hipSuccess) st = hip_error(e, "adjoint rows");
    if (st) p->adj_rows = AdjRows{};
    return st;
}

// The adjoint's rows of a problem whose creation found no room for them.
int adjoint_make_rows(Problem* p) {
    static std::mutex mu;
    std::lock_guard<std::mutex> lock(mu);
    if (p->adj_rows.row_sum) return OIM_OK;
    try {
        return make_rows(p);
    } catch (const std::bad_alloc&) {
        return set_error(OIM_E_NOMEM, "adjoint rows: host allocation failed");
    }
}

}  // namespace

int64_t adjoint_checkpoint_words(const Problem* p, const oim_adjoint_cfg* cfg) {
    const int64_t nseg = (cfg->steps + cfg->checkpoint_every - 1) / cfg->checkpoint_every;
    return nseg * cfg->R * (int64_t)p->sell_slices * 4 * kSliceQuads;
}

int launch_adjoint_forward(Problem* p, const oim_adjoint_cfg* cfg, const float* K, const float* Ks,
                           const float* sigma, const uint64_t* seeds, int64_t step0,
                           const float* theta0, uint32_t* ckpt, float* thetaT, double* loss,
                           hipStream_t stream) {
    if (int st = adjoint_make_rows(p)) return st;
    AdjArgs a = base_args(p, cfg, K, Ks, sigma, seeds, step0);
    a.theta0 = theta0;
    a.ckpt = ckpt;
    a.thetaT = thetaT;
    a.loss = loss;
    const Placement pl = place(p, a, false);
    a.noise2 = 1;
    return launch_adj(pick_fn(kForward, p, cfg->q, pl.ldsi), pl.lds, cfg->R * p->n_inst,
                      block_threads(a), stream, a, "adjoint_forward_kernel");
}

namespace {

// The second stream and the events of the overlapped backward pass, made on
// a problem's first backward call (default priority, non-blocking).
int adjoint_streams(Problem* p) {
    if (p->adj_stream) return OIM_OK;
    hipError_t e = hipStreamCreateWithFlags(&p->adj_stream, hipStreamNonBlocking);
    if (e != hipSuccess) {
        p->adj_stream = nullptr;
        return hip_error(e, "adjoint stream");
    }
    for (int k = 0; k < kAdjEvents; ++k) {
        e = hipEventCreateWithFlags(&p->adj_ev[k], hipEventDisableTiming);
        if (e != hipSuccess) {
            p->adj_ev[k] = nullptr;
            return hip_error(e, "adjoint events");
        }
    }
    return OIM_OK;
}

}  // namespace

void adjoint_release(Problem* p) {
    if (p->adj_stream) {
        (void)hipStreamSynchronize(p->adj_stream);
        (void)hipStreamDestroy(p->adj_stream);
        p->adj_stream = nullptr;
    }
    for (int k = 0; k < kAdjEvents; ++k) {
        if (p->adj_ev[k]) (void)hipEventDestroy(p->adj_ev[k]);
        p->adj_ev[k] = nullptr;
    }
}

// Segments last first; segment sg's states live in buffer sg % 2.  The
// recomputation runs on the problem's second stream, the adjoint on the
// caller's: adjoint(sg) waits for recompute(sg), recompute(sg - 2) waits for
// adjoint(sg) (the buffer it overwrites), so recompute(sg - 1) overlaps
// adjoint(sg).  The caller's stream ends after every kernel of the pass.
int launch_adjoint_backward(Problem* p, const oim_adjoint_cfg* cfg, const float* K, const float* Ks,
                            const float* sigma, const uint64_t* seeds, int64_t step0,
                            const uint32_t* ckpt, double* gK, double* gKs, double* gS,
                            hipStream_t stream) {
    if (cfg->steps == 0) return OIM_OK;
    if (int st = adjoint_make_rows(p)) return st;
    AdjArgs a = base_args(p, cfg, K, Ks, sigma, seeds, step0);
    const int nwg = cfg->R * p->n_inst;
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t seg_bytes = up((size_t)(cfg->checkpoint_every + 1) * cfg->R * a.P * sizeof(uint32_t));
    const size_t lam_bytes = up((size_t)cfg->R * a.P * sizeof(float));
    const size_t part_bytes = (size_t)cfg->steps * nwg * 3 * sizeof(double);
    const size_t sums_bytes = up((size_t)cfg->checkpoint_every * cfg->R * a.P * sizeof(float2));
    // The recomputation's row sums are kept where they take a small part of
    // the card, else (or when they cannot be had) the adjoint forms them
    // again: 128 x G(2000, 10/1999), C = 64 (0.27 GB): a segment of the adjoint
    // 182 us with them, 221 without; its recomputation 158 and 150.
    // (OIM_ADJ_SUMS=0 forms them again at any size.)
    const size_t base = 2 * seg_bytes + lam_bytes + part_bytes + 256;
    const char* env = getenv("OIM_ADJ_SUMS");
    const bool hand_over = !(env && !strcmp(env, "0")) && 2 * sums_bytes <= ((size_t)8 << 30);
    const size_t extra = hand_over ? 2 * sums_bytes : 0;
    bool keep = false;
    hipError_t e = hipSuccess;
    int st = grow_workspace(
        p->adj_work, base, extra, keep,
        [&](size_t bytes, void** ptr) {
            e = hipMalloc(ptr, bytes);
            if (e == hipErrorOutOfMemory) (void)hipGetLastError();  // not the next launch's error
            return e == hipSuccess ? 0 : e == hipErrorOutOfMemory ? kRefused : -1;
        },
        [](void* ptr) { (void)hipFree(ptr); });
    if (st == kRefused) return set_error(OIM_E_NOMEM, "adjoint workspace: out of device memory");
    if (st) return hip_error(e, "adjoint workspace");
    st = adjoint_streams(p);
    if (st) return st;
    unsigned char* w = static_cast<unsigned char*>(p->adj_work.ptr);
    uint32_t* segbuf[2] = {reinterpret_cast<uint32_t*>(w), reinterpret_cast<uint32_t*>(w + seg_bytes)};
    a.ckpt = const_cast<uint32_t*>(ckpt);
    a.lam = reinterpret_cast<float*>(w + 2 * seg_bytes);
    a.gpart = reinterpret_cast<double*>(w + 2 * seg_bytes + lam_bytes);
    unsigned char* sums = w + base;
    const Placement prec = place(p, a, false), padj = place(p, a, !keep);
    const AdjFn frec = pick_fn(kRecompute, p, cfg->q, prec.ldsi);
    const AdjFn fadj = pick_fn(keep ? kSegment : kSegmentWide, p, cfg->q, padj.ldsi);
    const int tb = block_threads(a);
    hipStream_t side = p->adj_stream;
    hipEvent_t* start = &p->adj_ev[0];
    hipEvent_t* rec = &p->adj_ev[1];   // [2]
    hipEvent_t* adj = &p->adj_ev[3];   // [2]
    e = hipEventRecord(*start, stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(side, *start, 0);
    if (e != hipSuccess) return hip_error(e, "adjoint stream fork");
    for (int sg = a.nseg - 1; sg >= 0 && !st; --sg) {
        const int buf = sg & 1;
        a.cur_seg = sg;
        a.seg = segbuf[buf];
        a.sums = keep ? reinterpret_cast<float2*>(sums + buf * sums_bytes) : nullptr;
        a.noise2 = 1;
        if (sg + 2 <= a.nseg - 1 && (e = hipStreamWaitEvent(side, adj[buf], 0)) != hipSuccess)
            return hip_error(e, "adjoint buffer wait");
        if ((st = launch_adj(frec, prec.lds, nwg, tb, side, a, "adjoint_recompute_kernel"))) break;
        if ((e = hipEventRecord(rec[buf], side)) != hipSuccess ||
            (e = hipStreamWaitEvent(stream, rec[buf], 0)) != hipSuccess)
            return hip_error(e, "adjoint segment order");
        a.noise2 = padj.noise2;
        if ((st = launch_adj(fadj, padj.lds, nwg, tb, stream, a, "adjoint_segment_kernel"))) break;
        if ((e = hipEventRecord(adj[buf], stream)) != hipSuccess)
            return hip_error(e, "adjoint segment order");
    }
    if (st) return st;
    constexpr int64_t kSteps = (int64_t)1 << 23;  // of one launch, as in launch_adj
    for (int64_t s = 0; s < cfg->steps; s += kSteps)
        hipLaunchKernelGGL(adjoint_reduce_kernel,
                           dim3((unsigned)(cfg->steps - s < kSteps ? cfg->steps - s : kSteps)), dim3(256), 0,
                           stream, a.gpart + 3 * s * nwg, nwg, gK + s, gKs + s, gS + s);
    return check_launch("adjoint_reduce_kernel");
}

}  // namespace oim
