// stepwise.hip -- Algorithm 1 with the replica state in device memory, one
// kernel per Euler-Maruyama step, for replicas too large for the
// LDS-resident kernel.
//
// Layout: replica index fastest, [n][Rp] (Rp = R rounded up to 64; below 33
// replicas, where the packed kernel runs, to a power of two, 4 at least), two buffers of phase words (ping-pong: step s
// reads buffer s % 2 and writes buffer (s + 1) % 2, which keeps the
// synchronous update of Algorithm 1).
// The state is the phase word alone (4 bytes per oscillator and replica):
// the (sin, cos) of a neighbour is recomputed from its word where it is
// gathered, the same function of the same word as anywhere else, so the
// results equal the LDS-resident loop's bit for bit.  A wave owns one quad
// (4 consecutive oscillators) and 64 replicas: CSR entries are wave-uniform
// (scalar loads) and each neighbour gather is one coalesced 256-byte load.
// Lane r draws the quad's four normals with one Philox call keyed by replica
// r's seed.  With fewer than 33 replicas a wave can take 64 / Rp quads, the lanes
// of a quad reading the same entries (stepwise_packed_kernel).
//
// The step loop is a hipGraph of `chunk` step kernels plus a node that
// advances a device-resident step base; the executable graph is replayed
// ceil(steps / chunk) times (step kernels past the last step return at
// once).  In-run readouts are graph nodes too (chunk is a multiple of the
// readout period), with the final partial readout launched after the
// replays.  Everything a call changes (schedule, seed and readout pointers,
// first step, step count) lives in a small device block that the captured
// kernels read, written by a one-thread kernel at the start of each call, so
// a graph is captured once per problem and launch shape (q, R, readout
// period, chunk) and kept in the problem's plan cache; a call enqueues work
// and returns without waiting for it.
#include <float.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <new>
#include <type_traits>

#include "internal.hpp"
#include "noise.hpp"
#include "phase.hpp"
#include "tree.hpp"

namespace oim {

namespace {

constexpr int kQuadsPerBlock = 4;  // one per wave, 256 threads

// Per-call arguments, in device memory (see the header comment).
struct CallArgs {
    const float* K;
    const float* Ks;
    const float* sigma;
    const uint64_t* seeds;
    double* trace;        // [ceil(steps/M)][R] or null
    int8_t* best_colour;  // [R][n] or null
    int64_t step0;        // global index of local step 0
    int32_t steps;
    int32_t sched_stride; // 0: one schedule for all replicas; steps: [R][steps]
    float dt;
    int32_t base;         // local index of node 0 of the current chunk
};

struct StepArgs {
    const int64_t* row_ptr;  // n + 1 entries and 4 copies of nnz
    const int32_t* col;   // nnz entries and 4 zero entries of padding, or the padded image
    const float* J;       // the same
    int64_t nnz;
    int ell_D;            // entries per row of the padded image (ELL kernels)
    uint32_t state_bytes; // bytes of one [np][Rp] buffer of phase words (BUF kernels: < 2^32)
    const uint32_t* Uin;  // [np][Rp] phase words of step s
    uint32_t* Uout;       // [np][Rp] phase words of step s + 1
    const CallArgs* call;
    int k;                // position of this node in the chunk
    int n, R, Rp, q;
    int lr_shift;         // Rp = 1 << lr_shift (packed kernel)
    int gx;               // quad blocks (workgroups per replica block)
};

// Workgroup id -> (quad block, replica block).  Consecutive workgroup ids go
// to the 8 XCDs in turn; each XCD is given a contiguous range of quad
// blocks (all of one replica block before the next), so the neighbour rows
// a workgroup gathers (the quads around its own) were mostly fetched into
// the same XCD's L2 by its neighbours.  A bijection on [0, nb): the blocks
// past the last multiple of 8 keep their index.
__device__ __forceinline__ void step_block(int b, int nb, int gx, int& qb, int& rb) {
    constexpr int kXcds = 8;
    const int full = nb / kXcds * kXcds;
    int t = b;
    if (b < full) t = (b % kXcds) * (full / kXcds) + b / kXcds;
    rb = t / gx;
    qb = t - rb * gx;
}

// A pointer read from the per-call block, as a global-memory pointer (such a
// pointer is generic to the compiler, which would otherwise load through it
// with flat instructions).
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* global_ptr(const T* p) {
    return (const __attribute__((address_space(1))) T*)p;
}

// The new phase word of one oscillator from its own word u, its sums A = sum J
// c_j and B = sum J s_j, the step's coefficients and its normal z.  The
// multiply-adds are written out, so both step kernels round alike.
template <int QM>
__device__ __forceinline__ uint32_t step_word(uint32_t u, float A, float B, float kc, float ks,
                                              float ns, float z, int q) {
#pragma clang fp contract(off)
    const float os = sin_turn(u), oc = cos_turn(u);
    const float coup = __builtin_fmaf(os, A, -(oc * B));
    const float sq = QM == 3 ? os * __builtin_fmaf(-4.0f * os, os, 3.0f) : sin_q<QM>(os, oc, u, q);
    const float drift = __builtin_fmaf(ks, sq, kc * coup);
    return advance(u, __builtin_fmaf(ns, z, drift));
}

// One Euler-Maruyama step of one quad for 64 replicas per wave.  ELL: the
// entries come from the padded row image (every row ell_D entries, padding
// of weight 0), so their positions follow from the quad index and their
// loads go out with the per-call block's: two batches of dependent loads per
// step instead of three.  BUF: the state words are addressed as buffer
// offsets (state buffers below 4 GiB), else at 64-bit global addresses.
template <int QM, bool ELL, bool BUF>
__global__ __launch_bounds__(256) void stepwise_step_kernel(StepArgs a) {
    const int lane = threadIdx.x & 63;
    int qb, rb;
    step_block(blockIdx.x, gridDim.x, a.gx, qb, rb);
    const int m = qb * kQuadsPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (4 * m >= a.n) return;
    const int r = rb * 64 + lane;
    const int Rp = a.Rp, q = QM ? QM : a.q;
    const int rs = r < a.R ? r : a.R - 1;  // padding lanes borrow a replica's entries
    // Lane r's word of a row of the [np][Rp] state.  BUF: a buffer access
    // with the row's byte offset in a scalar register (scalar arithmetic on
    // the wave-uniform row) and the lane's in a vector register shared by
    // every load and store of the step, so no 64-bit address arithmetic per
    // lane and access; this needs a state buffer below 4 GiB.  Otherwise a
    // global access at a 64-bit address.
    const int roff = r * 4;
    const uint32_t row_bytes = (uint32_t)Rp * 4u;
    const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.Uin, (short)0, (int)a.state_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.Uout, (short)0, (int)a.state_bytes, 0x00020000);
    auto lane_word = [&](int row) -> uint32_t {
        if constexpr (BUF)
            return __builtin_amdgcn_raw_buffer_load_b32(rin, roff, (int)((uint32_t)row * row_bytes), 0);
        else
            return a.Uin[(size_t)row * Rp + r];
    };
    auto store_word = [&](int row, uint32_t v) {
        if constexpr (BUF)
            __builtin_amdgcn_raw_buffer_store_b32(v, rout, roff, (int)((uint32_t)row * row_bytes), 0);
        else
            a.Uout[(size_t)row * Rp + r] = v;
    };
    // Every load of a step is issued up front, in batches with one wait
    // each: the per-call block, the quad's row bounds and its own words;
    // then the schedule entries, the seed and the first group of each row's
    // entries; then the neighbours' words (with the padded image the first
    // two batches are one).  Nothing before the store depends on whether
    // this node's step is still part of the run (a node past the last step
    // computes on local step 0's entries and writes nothing), and no select
    // or branch depends on a loaded value, so the compiler keeps the loads
    // together.
    const CallArgs& c = *a.call;
    int base = c.base, steps = c.steps, stride = c.sched_stride;
    int64_t step0 = c.step0;
    float dt = c.dt;
    const float* Kp = c.K;
    const float* Ksp = c.Ks;
    const float* sgp = c.sigma;
    const uint64_t* seedp = c.seeds;
    int64_t eb[4];
    int len[4];
    int lmax = 0;
    if constexpr (ELL) {
        // group g / 4 of row j of the quad at m * 4D + 4g + 4j (in steps
        // of 4 entries: g advances the base by 16)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            eb[j] = (int64_t)m * 4 * a.ell_D + 4 * j;
            len[j] = a.ell_D;
        }
        lmax = a.ell_D;
    } else {
        int64_t rp[5];  // row_ptr carries 4 entries of padding (empty rows)
#pragma unroll
        for (int j = 0; j < 5; ++j) rp[j] = a.row_ptr[4 * m + j];
        // one wait for the per-call block and the row bounds together: every
        // use of them goes through this statement
        asm(""
            : "+s"(base), "+s"(steps), "+s"(stride), "+s"(step0), "+s"(dt), "+s"(Kp),
                       "+s"(Ksp), "+s"(sgp), "+s"(seedp), "+s"(rp[0]), "+s"(rp[1]), "+s"(rp[2]),
                       "+s"(rp[3]), "+s"(rp[4]));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            eb[j] = rp[j];
            len[j] = (int)(rp[j + 1] - rp[j]);
            lmax = len[j] > lmax ? len[j] : lmax;
        }
    }
    // The quad's four rows are walked in lock-step, four entries of each
    // per group, so sixteen neighbour loads are in flight together.  Row
    // lengths are wave-uniform (every lane is a replica of the same quad), so
    // a row shorter than the longest costs only its idle slots.  Group t of
    // row j is the 4 entries from eb + t, clamped to nnz (the arrays carry 4
    // zero entries past the end, so a group is always in bounds and its
    // column indexes valid); a slot past the row's end gets weight 0 by
    // masking its bits, which leaves the sums unchanged (the words are
    // finite).  The padded image needs neither: its groups are in bounds
    // and its padding weighs 0.  Each row keeps its order: entries at even
    // offsets into one partial sum, odd ones into the other.
    int ci[4][4];
    uint32_t wb[4][4];
    auto load_cols = [&](int g) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int64_t base = eb[j] + (ELL ? 4 * g : g);
            if constexpr (!ELL) base = base < a.nnz ? base : a.nnz;
#pragma unroll
            for (int h = 0; h < 4; ++h) ci[j][h] = a.col[base + h];
        }
    };
    auto load_weights = [&](int g) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int64_t base = eb[j] + (ELL ? 4 * g : g);
            if constexpr (!ELL) base = base < a.nnz ? base : a.nnz;
#pragma unroll
            for (int h = 0; h < 4; ++h) wb[j][h] = __float_as_uint(a.J[base + h]);
        }
    };
    auto load_entries = [&](int g) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int64_t base = eb[j] + (ELL ? 4 * g : g);
            if constexpr (!ELL) base = base < a.nnz ? base : a.nnz;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                wb[j][h] = __float_as_uint(a.J[base + h]);
                ci[j][h] = a.col[base + h];
            }
        }
    };
    // The first group's four rows' entry loads (scalar loads) are all issued
    // before the first use: the loaded values pass through empty asm
    // statements that no load may cross, so nothing that uses them is
    // scheduled between the loads (each use of a scalar load waits for all
    // of them).  Later groups are read with vector loads, which complete in
    // order, and need no such help.
    auto pin_entries = [&]() {
        asm(""
            : "+s"(ci[0][0]), "+s"(ci[0][1]), "+s"(ci[0][2]), "+s"(ci[0][3]),
              "+s"(ci[1][0]), "+s"(ci[1][1]), "+s"(ci[1][2]), "+s"(ci[1][3]),
              "+s"(ci[2][0]), "+s"(ci[2][1]), "+s"(ci[2][2]), "+s"(ci[2][3]),
              "+s"(ci[3][0]), "+s"(ci[3][1]), "+s"(ci[3][2]), "+s"(ci[3][3]),
              "+s"(wb[0][0]), "+s"(wb[0][1]), "+s"(wb[0][2]), "+s"(wb[0][3]),
              "+s"(wb[1][0]), "+s"(wb[1][1]), "+s"(wb[1][2]), "+s"(wb[1][3]),
              "+s"(wb[2][0]), "+s"(wb[2][1]), "+s"(wb[2][2]), "+s"(wb[2][3]),
              "+s"(wb[3][0]), "+s"(wb[3][1]), "+s"(wb[3][2]), "+s"(wb[3][3]));
    };
    uint32_t p[4][4];
    float w[4][4];
    auto load_words = [&](int g) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                // the column is wave-uniform (every lane is a replica of the
                // same quad); later groups' columns arrive in vector
                // registers, so say so
                p[j][h] = lane_word(__builtin_amdgcn_readfirstlane(ci[j][h]));
                if constexpr (ELL) {
                    w[j][h] = __uint_as_float(wb[j][h]);
                } else {
                    const uint32_t keep = 0u - (uint32_t)(g + h < len[j]);
                    w[j][h] = __uint_as_float(wb[j][h] & keep);
                }
            }
    };
    uint32_t u0[4];
    if constexpr (ELL) {
        // the first group's columns (the weights are not needed before the
        // neighbours' words arrive: they go out with them)
        load_cols(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) u0[j] = lane_word(4 * m + j);
        // one wait for the per-call block and the columns together
        asm(""
            : "+s"(base), "+s"(steps), "+s"(stride), "+s"(step0), "+s"(dt), "+s"(Kp),
              "+s"(Ksp), "+s"(sgp), "+s"(seedp),
              "+s"(ci[0][0]), "+s"(ci[0][1]), "+s"(ci[0][2]), "+s"(ci[0][3]),
              "+s"(ci[1][0]), "+s"(ci[1][1]), "+s"(ci[1][2]), "+s"(ci[1][3]),
              "+s"(ci[2][0]), "+s"(ci[2][1]), "+s"(ci[2][2]), "+s"(ci[2][3]),
              "+s"(ci[3][0]), "+s"(ci[3][1]), "+s"(ci[3][2]), "+s"(ci[3][3]));
        load_weights(0);
    }
    const int s_node = base + a.k;
    const bool live = s_node < steps;
    const int s = live ? s_node : 0;
    const uint32_t t = (uint32_t)(step0 + s);
    const int64_t so = (int64_t)rs * stride + s;
    const float Kv = global_ptr(Kp)[so];
    const float Ksv = global_ptr(Ksp)[so];
    const float sgv = global_ptr(sgp)[so];
    const uint64_t seed = global_ptr(seedp)[rs];
    if constexpr (!ELL) {
#pragma unroll
        for (int j = 0; j < 4; ++j) u0[j] = lane_word(4 * m + j);
        load_entries(0);
        pin_entries();
    }
    auto gather = [&](int g) {
        load_entries(g);
        load_words(g);
    };
    float A0[4], B0[4], A1[4], B1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) A0[j] = B0[j] = A1[j] = B1[j] = 0.f;
    auto accumulate = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 4; h += 2) {
                const float s0 = sin_turn(p[j][h]), c0 = cos_turn(p[j][h]);
                const float s1 = sin_turn(p[j][h + 1]), c1 = cos_turn(p[j][h + 1]);
                A0[j] = __builtin_fmaf(w[j][h], c0, A0[j]);
                B0[j] = __builtin_fmaf(w[j][h], s0, B0[j]);
                A1[j] = __builtin_fmaf(w[j][h + 1], c1, A1[j]);
                B1[j] = __builtin_fmaf(w[j][h + 1], s1, B1[j]);
            }
    };
    load_words(0);
    // the quad's normals while the neighbour loads are in flight
    float z[4];
    normals4((uint32_t)m, t, 0u, (uint32_t)seed, (uint32_t)(seed >> 32), z);
    // pin the normals here (left alone, the compiler sinks them to the
    // update, after the last neighbour load has returned)
    asm volatile("" ::"v"(z[0]), "v"(z[1]), "v"(z[2]), "v"(z[3]) : "memory");
    accumulate();
    for (int g = 4; g < lmax; g += 4) {
        gather(g);
        accumulate();
    }
    if (!live) return;
    const float kc = -dt * Kv * kTurnScale;
    const float ks = -dt * Ksv * kTurnScale;
    const float ns = sgv * __builtin_sqrtf(dt) * kTurnScale;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i = 4 * m + j;
        if (i >= a.n) break;
        store_word(i, step_word<QM>(u0[j], A0[j] + A1[j], B0[j] + B1[j], kc, ks, ns, z[j], q));
    }
}

// Four consecutive entries from any entry on, one 16-byte load.
template <typename T>
struct __attribute__((packed, aligned(4))) Four {
    T v[4];
};

// The same step with fewer than 33 replicas: a wave holds 64 / Rp quads (Rp a
// power of two), lane l replica l % Rp of quad l / Rp, so that no lane is left
// without a replica (at 64 lanes per quad one replica used one lane in 64).
// The lanes of a quad load the same entries; the sums and the update are
// those of the kernel above, operation for operation.  A quad gets four lanes
// at least: with one, a wave's 64 quads scatter its entry loads (n = 50000 of
// degree 6, real weights, one replica: 64 steps 934 us, with four 757).  Whole
// solves of 100 steps with two readouts on a 200 x 300 torus, 64 lanes per
// quad before and now: 1936 -> 474 us (one replica), 1979 -> 632 (8), 1970 ->
// 854 (16), 1976 -> 1101 (32); n = 50000 of degree 6, 64 steps, 2377 -> 757 (4
// replicas), 2346 -> 1239 (32).  Bound by the latency of two dependent batches
// of loads (words and entries, then neighbours' words) and by the launches.
template <int QM, bool ELL>
__global__ __launch_bounds__(256) void stepwise_packed_kernel(StepArgs a) {
    const int Rp = a.Rp, shift = a.lr_shift, q = QM ? QM : a.q;
    const int t0 = blockIdx.x * 256 + threadIdx.x;
    const int m = t0 >> shift, r = t0 & (Rp - 1);
    if (4 * (int64_t)m >= a.n) return;
    const int rs = r < a.R ? r : a.R - 1;  // padding lanes borrow a replica's entries
    const CallArgs& c = *a.call;
    const int s_node = c.base + a.k;
    if (s_node >= c.steps) return;
    auto word = [&](int row) -> uint32_t { return a.Uin[((uint32_t)row << shift) + r]; };
    uint32_t u0[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) u0[j] = word(4 * m + j);
    int64_t eb[4];
    int len[4], lmax = a.ell_D;
    if constexpr (!ELL) {
        int64_t rp[5];  // row_ptr carries 4 entries of padding (empty rows)
        lmax = 0;
#pragma unroll
        for (int j = 0; j < 5; ++j) rp[j] = a.row_ptr[4 * m + j];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            eb[j] = rp[j];
            len[j] = (int)(rp[j + 1] - rp[j]);
            lmax = len[j] > lmax ? len[j] : lmax;
        }
    }
    const uint32_t t = (uint32_t)(c.step0 + s_node);
    const int64_t so = (int64_t)rs * c.sched_stride + s_node;
    const float Kv = global_ptr(c.K)[so], Ksv = global_ptr(c.Ks)[so], sgv = global_ptr(c.sigma)[so];
    const uint64_t seed = global_ptr(c.seeds)[rs];
    float A0[4], B0[4], A1[4], B1[4], z[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) A0[j] = B0[j] = A1[j] = B1[j] = 0.f;
    for (int g = 0; g < lmax || g == 0; g += 4) {
        // group g of the quad's four rows (past a row's end: weight 0)
        int ci[4][4];
        float w[4][4];
        if constexpr (ELL) {
            const size_t at = (size_t)m * a.ell_D + g;  // 16-byte units
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int4 cv = reinterpret_cast<const int4*>(a.col)[at + j];
                const float4 wv = reinterpret_cast<const float4*>(a.J)[at + j];
                ci[j][0] = cv.x; ci[j][1] = cv.y; ci[j][2] = cv.z; ci[j][3] = cv.w;
                w[j][0] = wv.x; w[j][1] = wv.y; w[j][2] = wv.z; w[j][3] = wv.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t base = eb[j] + g < a.nnz ? eb[j] + g : a.nnz;
                const Four<int32_t> cv = *reinterpret_cast<const Four<int32_t>*>(a.col + base);
                const Four<float> wv = *reinterpret_cast<const Four<float>*>(a.J + base);
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    ci[j][h] = cv.v[h];
                    w[j][h] = g + h < len[j] ? wv.v[h] : 0.f;
                }
            }
        }
        uint32_t p[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 4; ++h) p[j][h] = word(ci[j][h]);
        if (g == 0) {
            // the quad's normals while the neighbours' words are in flight
            normals4((uint32_t)m, t, 0u, (uint32_t)seed, (uint32_t)(seed >> 32), z);
            asm volatile("" ::"v"(z[0]), "v"(z[1]), "v"(z[2]), "v"(z[3]) : "memory");
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 4; h += 2) {
                A0[j] = __builtin_fmaf(w[j][h], cos_turn(p[j][h]), A0[j]);
                B0[j] = __builtin_fmaf(w[j][h], sin_turn(p[j][h]), B0[j]);
                A1[j] = __builtin_fmaf(w[j][h + 1], cos_turn(p[j][h + 1]), A1[j]);
                B1[j] = __builtin_fmaf(w[j][h + 1], sin_turn(p[j][h + 1]), B1[j]);
            }
    }
    const float kc = -c.dt * Kv * kTurnScale;
    const float ks = -c.dt * Ksv * kTurnScale;
    const float ns = sgv * __builtin_sqrtf(c.dt) * kTurnScale;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i = 4 * m + j;
        if (i >= a.n) break;
        a.Uout[((uint32_t)i << shift) + r] =
            step_word<QM>(u0[j], A0[j] + A1[j], B0[j] + B1[j], kc, ks, ns, z[j], q);
    }
}

__global__ void advance_base_kernel(CallArgs* call, int chunk) { call->base += chunk; }

__global__ void set_call_kernel(CallArgs* call, CallArgs v) { *call = v; }

// [R][n] theta or phase words <-> [np][Rp] phase words, through LDS in tiles of
// 64 rows x 64 (or Rp) replicas so that both sides are read and written in
// runs (a thread per element, with one side at a stride, took 25 us in and 53
// out for 60000 x 64).
constexpr int kTile = 64;

// Tile of a workgroup: first row and first replica (a one-dimensional grid,
// row tiles first; the other grid dimensions are too short for many replicas).
__device__ __forceinline__ void tile_of(int np, int& i0, int& r0) {
    const int tiles = (np + kTile - 1) / kTile;
    i0 = (int)(blockIdx.x % tiles) * kTile;
    r0 = (int)(blockIdx.x / tiles) * kTile;
}

// Fills buffer 0 and, in buffer 1, the padding rows alone: the first step
// writes the others.  Padding rows and replicas hold 0.
__global__ __launch_bounds__(1024) void stepwise_init_kernel(const float* theta, const uint32_t* phase,
                                                            uint32_t* U0, uint32_t* U1,
                                                            int n, int R, int np, int Rp) {
    __shared__ uint32_t tile[kTile][kTile + 1];
    int i0, r0;
    tile_of(np, i0, r0);
    const int lr = Rp < kTile ? Rp : kTile;
    const int lane = threadIdx.x & 63;
    for (int r = threadIdx.x >> 6; r < lr; r += blockDim.x >> 6) {
        const int i = i0 + lane;
        uint32_t u = 0;
        if (i < n && r0 + r < R) {
            const size_t src = (size_t)(r0 + r) * n + i;
            u = phase ? phase[src] : phase_from_theta(theta[src]);
        }
        tile[lane][r] = u;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kTile * lr; e += blockDim.x) {
        const int row = e / lr, r = e % lr, i = i0 + row;
        if (i >= np) break;
        const size_t o = (size_t)i * Rp + r0 + r;
        U0[o] = tile[row][r];
        if (i >= n) U1[o] = 0;
    }
}

__global__ __launch_bounds__(1024) void stepwise_final_kernel(const uint32_t* U, float* theta,
                                                             uint32_t* phase, int n, int R, int Rp) {
    __shared__ uint32_t tile[kTile][kTile + 1];
    int i0, r0;
    tile_of(n, i0, r0);
    const int lr = Rp < kTile ? Rp : kTile;
    const int lane = threadIdx.x & 63;
    for (int e = threadIdx.x; e < kTile * lr; e += blockDim.x) {
        const int row = e / lr, r = e % lr;
        if (i0 + row < n) tile[row][r] = U[(size_t)(i0 + row) * Rp + r0 + r];
    }
    __syncthreads();
    const int i = i0 + lane;
    if (i >= n) return;
    for (int r = threadIdx.x >> 6; r < lr && r0 + r < R; r += blockDim.x >> 6) {
        const size_t dst = (size_t)(r0 + r) * n + i;
        theta[dst] = theta_from_phase(tile[lane][r]);
        if (phase) phase[dst] = tile[lane][r];
    }
}

struct ReadArgs {
    const int64_t* row_ptr;
    const int32_t* col;
    const float* J;
    const uint32_t* U;
    double* part;  // [gridDim.x][Rp] sums of a block of rows
    const CallArgs* call;
    int k;         // node position in the chunk, or -1: after the last step
    int n, Rp, q;
};

// Partial sums of sum_{i<j} J_ij term(k_i, k_j) per block of rows and replica
// (term = s_i s_j for q = 2, delta(k_i, k_j) for q >= 3), in the library's
// fixed FP64 order: each row over j > i in column order, a quad's rows as (r0
// + r1) + (r2 + r3), then the block's threads pairwise -- the pairwise tree over
// the block's rows.  A thread is one replica of its quad: 64 replicas make
// blocks of 16 rows, four of 256.  (Four quads per thread, for fewer partials,
// were a longer chain: 64 steps with 8 readouts of n = 3000 of degree 20, 64
// replicas 1210 us, 830 so; of a 200 x 300 torus, 64 replicas 1060 and 1050.)

// Blocks of rows of a readout.
int read_blocks(int quads, int Rp) {
    const int per = 256 / (Rp < 64 ? Rp : 64);
    return (quads + per - 1) / per;
}

__global__ __launch_bounds__(256) void stepwise_readout_kernel(ReadArgs a) {
    __shared__ double red[256];
    const int steps = a.call->steps;
    const int s = a.k < 0 ? steps - 1 : a.call->base + a.k;
    if (s >= steps) return;
    const int lr = a.Rp < 64 ? a.Rp : 64, slots = 256 / lr;
    const int slot = threadIdx.x / lr, r = blockIdx.y * 64 + threadIdx.x % lr;
    auto state = [&](int row) { return nearest_state(a.U[(size_t)row * a.Rp + r], a.q); };
    const int m = blockIdx.x * slots + slot;
    double rs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i = 4 * m + j;
        if (i >= a.n) continue;
        const int ci = state(i);
        const int64_t e1 = a.row_ptr[i + 1];
        double acc = 0.0;
        // four entries at a time, their words in flight together
        for (int64_t e = a.row_ptr[i]; e < e1; e += 4) {
            int c[4], k[4];
            float w[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const int64_t ee = e + h < e1 ? e + h : e1 - 1;
                c[h] = a.col[ee];
                w[h] = a.J[ee];
            }
#pragma unroll
            for (int h = 0; h < 4; ++h) k[h] = state(c[h]);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const double wd = (double)w[h];
                const double term = a.q == 2 ? (ci == k[h] ? wd : -wd) : (ci == k[h] ? wd : 0.0);
                acc += e + h < e1 && c[h] > i ? term : 0.0;
            }
        }
        rs[j] = acc;
    }
    red[threadIdx.x] = (rs[0] + rs[1]) + (rs[2] + rs[3]);
    __syncthreads();
    for (int d = 1; d < slots; d <<= 1) {
        if ((slot & (2 * d - 1)) == 0) red[threadIdx.x] = red[threadIdx.x] + red[threadIdx.x + d * lr];
        __syncthreads();
    }
    if (slot == 0) a.part[(size_t)blockIdx.x * a.Rp + r] = red[threadIdx.x];
}

struct BestArgs {
    const double* part;
    int nblocks;
    const uint32_t* U;
    double* best;     // running best (workspace)
    int32_t* best_at; // running best step (workspace)
    const CallArgs* call;
    int k;            // node position in the chunk, or -1: after the last step
    int M, n, R, Rp, q;
    int colours;      // 1: the best kernel writes the colours of a new best
};

// One workgroup per replica: H = -(the pairwise tree over the blocks'
// partials), trace entry, best-so-far and (a.colours) the colours of a new best.  The
// partials, zero-padded to a power of two P, are taken in rounds of
// CH = min(P, 4096) values; in a round each of the 256 threads folds an
// aligned chunk of CH / 256 (at most 16) values by the pairwise tree in
// registers, the 256 chunk sums are folded pairwise in LDS, and thread 0
// pushes the round's sum into a tree over rounds.  This is the pairwise tree
// over the padded sequence (padding zeros add exactly).
__global__ __launch_bounds__(256) void stepwise_best_kernel(BestArgs a) {
    __shared__ int improved;
    __shared__ double sums[256];
    __shared__ double stack[TreeAcc::kLevels];
    const CallArgs& c = *a.call;
    const int s = a.k < 0 ? c.steps - 1 : c.base + a.k;
    if (s >= c.steps) return;
    const int r = blockIdx.x;
    int64_t P = 1;
    while (P < a.nblocks) P <<= 1;
    const int CH = P < 4096 ? (int)P : 4096;
    const int B = CH >= 256 ? CH / 256 : 1;
    const int64_t rounds = P / CH;
    TreeAcc outer(stack);
    for (int64_t rd = 0; rd < rounds; ++rd) {
        const int64_t first = rd * CH + (int64_t)threadIdx.x * B;
        double v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            v[i] = (i < B && first + i < a.nblocks) ? a.part[(size_t)(first + i) * a.Rp + r] : 0.0;
        // the tree over 16 slots; slots past B hold +0, so the result is the
        // tree over the chunk's B values
#pragma unroll
        for (int len = 16; len > 1; len >>= 1)
#pragma unroll
            for (int i = 0; i < len / 2; ++i) v[i] = v[2 * i] + v[2 * i + 1];
        sums[threadIdx.x] = v[0];
        __syncthreads();
        for (int d = 1; d < 256; d <<= 1) {
            if ((threadIdx.x & (2 * d - 1)) == 0) sums[threadIdx.x] = sums[threadIdx.x] + sums[threadIdx.x + d];
            __syncthreads();
        }
        if (threadIdx.x == 0) outer.push(sums[0]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double H = -outer.finish();
        const int kread = (s + a.M) / a.M - 1;
        if (c.trace) c.trace[(size_t)kread * a.R + r] = H;
        improved = kread == 0 || H < a.best[r] ? 1 : 0;
        if (improved) {
            a.best[r] = H;
            a.best_at[r] = (int32_t)(c.step0 + s + 1);
        }
    }
    if (!a.colours || !c.best_colour) return;
    __syncthreads();
    if (improved)
        for (int i = threadIdx.x; i < a.n; i += blockDim.x)
            c.best_colour[(size_t)r * a.n + i] = (int8_t)nearest_state(a.U[(size_t)i * a.Rp + r], a.q);
}

// The colours of the replicas whose best is this readout's (best_at names its
// step), in tiles through LDS as the kernels above; tiles without one end at
// once.  (One workgroup per replica reading its words at a stride of Rp took
// most of a 98 us readout of 60000 x 64.)
__global__ __launch_bounds__(256) void stepwise_colour_kernel(BestArgs a) {
    __shared__ int8_t tile[kTile][kTile + 1];
    __shared__ int any;
    const CallArgs& c = *a.call;
    const int s = a.k < 0 ? c.steps - 1 : c.base + a.k;
    if (s >= c.steps || !c.best_colour) return;
    const int32_t now = (int32_t)(c.step0 + s + 1);
    int i0, r0;
    tile_of(a.n, i0, r0);
    const int lr = a.Rp < kTile ? a.Rp : kTile;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    if (threadIdx.x < lr && r0 + threadIdx.x < a.R && a.best_at[r0 + threadIdx.x] == now) any = 1;
    __syncthreads();
    if (!any) return;
    for (int e = threadIdx.x; e < kTile * lr; e += blockDim.x) {
        const int row = e / lr, r = e % lr;
        if (i0 + row < a.n)
            tile[row][r] = (int8_t)nearest_state(a.U[(size_t)(i0 + row) * a.Rp + r0 + r], a.q);
    }
    __syncthreads();
    const int i = i0 + lane;
    if (i >= a.n) return;
    for (int r = threadIdx.x >> 6; r < lr && r0 + r < a.R; r += blockDim.x >> 6)
        if (a.best_at[r0 + r] == now) c.best_colour[(size_t)(r0 + r) * a.n + i] = tile[lane][r];
}

int check_launch(const char* what) {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? OIM_OK : hip_error(e, what);
}

// One captured step loop: the executable graphs of a chunk (two when the
// chunk is odd: the table parity then flips from replay to replay), the
// workspace they were captured on, and an event recorded after their last
// use so they can be destroyed safely.
struct Plan {
    int q = 0, R = 0, M = 0, chunk = 0, global_addr = 0;
    const void* work = nullptr;
    hipGraph_t g[2] = {nullptr, nullptr};
    hipGraphExec_t x[2] = {nullptr, nullptr};
    hipEvent_t done = nullptr;
    uint64_t last_use = 0;
};

struct PlanCache {
    static constexpr int kMax = 4;
    Plan plans[kMax];
    int count = 0;
    uint64_t clock = 0;
};

void destroy_plan(Plan& pl) {
    if (pl.done) {
        (void)hipEventSynchronize(pl.done);
        (void)hipEventDestroy(pl.done);
    }
    for (int i = 0; i < 2; ++i) {
        if (pl.x[i]) (void)hipGraphExecDestroy(pl.x[i]);
        if (pl.g[i]) (void)hipGraphDestroy(pl.g[i]);
    }
    pl = Plan{};
}

void clear_plans(Problem* p) {
    PlanCache* c = static_cast<PlanCache*>(p->step_plans);
    if (!c) return;
    for (int i = 0; i < c->count; ++i) destroy_plan(c->plans[i]);
    c->count = 0;
}

}  // namespace

void stepwise_release(Problem* p) {
    clear_plans(p);
    delete static_cast<PlanCache*>(p->step_plans);
    p->step_plans = nullptr;
}

namespace {

struct Shape {
    int n, R, steps, M, Rp, quads, np, gx, rblocks, chunk;
    int global_addr;  // 64-bit global addressing asked for
    int packed;       // several quads per wave
    size_t cells, args_off, bytes;
};

// Whether a run with fewer than 33 replicas (a power of two, Rp) takes the
// packed kernel: where the waves of 64 lanes per quad would be many, where the
// entries come from the padded image and few lanes need them, or where rows are
// longer than the image's first group.  Its entry loads are vector loads with
// a longer latency, which a small graph pays on every step: 64 steps with 64
// lanes per quad and packed (us): n = 2000 of degree 6, CSR, one replica 374
// and 416, n = 5000, 8 replicas 455 and 454, n = 10000 569 and 472; 50 x 20 and
// 300 x 20 tori, 16 replicas 198 and 217, 242 and 223; n = 60 of degree 4, one
// replica 196 and 161; n = 300 of degree 6 (image rows of 8) 309 and 244.
bool packs(const Problem* p, int quads, int Rp) {
    if (Rp >= 64) return false;
    if (!p->d_ell_col) return quads >= (Rp <= 4 ? 2000 : 1250) || quads * Rp <= 128;
    return p->ell_D > 4 || Rp <= 8 || quads >= 1024;
}

Shape shape_of(const Problem* p, const oim_run_cfg* cfg) {
    Shape sh{};
    sh.n = p->n;
    sh.R = cfg->R;
    sh.steps = cfg->steps;
    sh.M = cfg->readout_every;
    // OIM_STEPWISE_GLOBAL_ADDR=1 takes the 64-lane kernel and the 64-bit global
    // addressing of states of 4 GiB and more for any size
    const char* env = getenv("OIM_STEPWISE_GLOBAL_ADDR");
    sh.global_addr = env && atoi(env) != 0;
    sh.Rp = (sh.R + 63) / 64 * 64;
    int pow2 = 4;
    while (pow2 < sh.R && pow2 < 64) pow2 *= 2;
    sh.packed = !sh.global_addr && packs(p, (sh.n + 3) / 4, pow2);
    if (sh.packed) sh.Rp = pow2;
    sh.quads = (sh.n + 3) / 4;
    sh.np = sh.quads * 4;
    sh.gx = (sh.quads + kQuadsPerBlock - 1) / kQuadsPerBlock;
    sh.rblocks = read_blocks(sh.quads, sh.Rp);
    sh.cells = (size_t)sh.np * sh.Rp;
    // chunk: a multiple of the readout period, about 64 steps
    int chunk = std::min(sh.steps, 64);
    if (sh.M > 0) chunk = std::max(1, (std::min(sh.steps, std::max(64, sh.M)) / sh.M)) * sh.M;
    sh.chunk = std::max(1, std::min(chunk, sh.steps));
    sh.args_off = (sh.cells * (4 + 4) + (size_t)sh.rblocks * sh.Rp * 8 + (size_t)sh.R * 12 + 255) &
                  ~(size_t)255;
    // the workspace is sized for whole waves of replicas at any R, as the
    // allocation-free entry point's limit is stated
    const size_t rp64 = (size_t)(sh.R + 63) / 64 * 64;
    sh.bytes = (((size_t)sh.np * rp64 * (4 + 4) + (size_t)sh.gx * rp64 * 8 + (size_t)sh.R * 12 + 255) &
                ~(size_t)255) + 256;
    return sh;
}

// The stepwise loop on a workspace of at least stepwise_workspace_bytes:
// with `graph`, the chunk of steps comes from the problem's plan cache
// (captured on first use) and is replayed; without, the same kernels are
// launched one by one on the stream (no capture, no allocation).
int run_stepwise(Problem* p, const oim_run_cfg* cfg, const float* K, const float* Ks,
                 const float* sigma, const uint64_t* seeds, int64_t step0, float* theta,
                 uint32_t* phase, const oim_readout* ro, hipStream_t stream, void* work,
                 bool graph) {
    const Shape sh = shape_of(p, cfg);
    const int n = sh.n, R = sh.R, steps = sh.steps, M = sh.M, Rp = sh.Rp, np = sh.np, gx = sh.gx;
    const int chunk = sh.chunk, rblocks = sh.rblocks;
    const size_t cells = sh.cells, args_off = sh.args_off;
    if (graph && !p->step_plans) {
        p->step_plans = new (std::nothrow) PlanCache();
        if (!p->step_plans) return set_error(OIM_E_NOMEM, "plan cache");
    }
    unsigned char* w = static_cast<unsigned char*>(work);
    uint32_t* U0 = reinterpret_cast<uint32_t*>(w);
    uint32_t* U1 = U0 + cells;
    double* part = reinterpret_cast<double*>(U1 + cells);
    double* best = part + (size_t)rblocks * Rp;
    int32_t* best_at = reinterpret_cast<int32_t*>(best + R);
    CallArgs* call = reinterpret_cast<CallArgs*>(w + args_off);

    // this call's arguments, for every kernel below (stream order)
    CallArgs ca{};
    ca.K = K;
    ca.Ks = Ks;
    ca.sigma = sigma;
    ca.seeds = seeds;
    ca.trace = ro ? ro->trace : nullptr;
    ca.best_colour = ro ? ro->best_colour : nullptr;
    ca.step0 = step0;
    ca.steps = steps;
    ca.sched_stride = (cfg->flags & OIM_SCHED_PER_REPLICA) ? cfg->steps : 0;
    ca.dt = cfg->dt;
    ca.base = 0;
    hipLaunchKernelGGL(set_call_kernel, dim3(1), dim3(1), 0, stream, call, ca);
    int st = check_launch("set_call_kernel");
    if (st) return st;
    const dim3 tiles((unsigned)(((np + kTile - 1) / kTile) * ((Rp + kTile - 1) / kTile)));
    // a tile of few replicas is small work
    const dim3 tile_tb(Rp >= 64 ? 1024 : Rp >= 32 ? 512 : 256);
    hipLaunchKernelGGL(stepwise_init_kernel, tiles, tile_tb, 0, stream, theta, phase, U0, U1, n, R,
                       np, Rp);
    if ((st = check_launch("stepwise_init_kernel"))) return st;

    using StepFn = void (*)(StepArgs);
    const bool ell = p->d_ell_col != nullptr;
    // buffer addressing for states below 4 GiB
    const bool buf = cells * 4 < ((size_t)1 << 32) && !sh.global_addr;
    static const StepFn kStep[2][2][3] = {
        {{stepwise_step_kernel<0, false, false>, stepwise_step_kernel<2, false, false>,
          stepwise_step_kernel<3, false, false>},
         {stepwise_step_kernel<0, false, true>, stepwise_step_kernel<2, false, true>,
          stepwise_step_kernel<3, false, true>}},
        {{stepwise_step_kernel<0, true, false>, stepwise_step_kernel<2, true, false>,
          stepwise_step_kernel<3, true, false>},
         {stepwise_step_kernel<0, true, true>, stepwise_step_kernel<2, true, true>,
          stepwise_step_kernel<3, true, true>}}};
    static const StepFn kPacked[2][3] = {
        {stepwise_packed_kernel<0, false>, stepwise_packed_kernel<2, false>,
         stepwise_packed_kernel<3, false>},
        {stepwise_packed_kernel<0, true>, stepwise_packed_kernel<2, true>,
         stepwise_packed_kernel<3, true>}};
    const int qi = cfg->q == 2 ? 1 : cfg->q == 3 ? 2 : 0;
    const bool packed = sh.packed;
    StepFn fn = packed ? kPacked[ell][qi] : kStep[ell][buf][qi];
    const int64_t lanes = (int64_t)sh.quads * Rp;  // packed: a lane per quad and replica
    const dim3 step_grid(packed ? (unsigned)((lanes + 255) / 256) : (unsigned)(gx * (Rp / 64)));
    const dim3 read_grid(rblocks, (Rp + 63) / 64);
    StepArgs sa{};
    sa.row_ptr = p->d_row_ptr;
    sa.col = ell ? p->d_ell_col : p->d_col;
    sa.J = ell ? p->d_ell_J : p->d_J;
    sa.nnz = p->nnz;
    sa.ell_D = p->ell_D;
    sa.state_bytes = buf ? (uint32_t)(cells * 4) : 0u;
    sa.call = call;
    sa.n = n;
    sa.R = R;
    sa.Rp = Rp;
    sa.q = cfg->q;
    for (sa.lr_shift = 0; packed && (1 << sa.lr_shift) < Rp;) ++sa.lr_shift;
    sa.gx = gx;
    // the state after local step s is in buffer (s + 1) % 2; after the run,
    // in buffer steps % 2
    uint32_t* const Ufinal = (steps & 1) ? U1 : U0;
    ReadArgs ra{p->d_row_ptr, p->d_col, p->d_J, Ufinal, part, call, 0, n, Rp, cfg->q};
    BestArgs ba{};
    ba.part = part;
    ba.nblocks = rblocks;
    ba.U = Ufinal;
    ba.best = best;
    ba.best_at = best_at;
    ba.call = call;
    ba.M = M;
    ba.n = n;
    ba.R = R;
    ba.Rp = Rp;
    ba.q = cfg->q;
    // colours by the best kernel: at a stride, but without a launch more
    // (64 steps with 8 readouts, 64 replicas, n = 1000 308 and 291 us, n = 6000
    // 371 and 363, n = 15000 497 and 513)
    ba.colours = n <= 8192;

    // Record one chunk: step kernels (with readouts where due) and the base
    // advance.  Buffer parity alternates per step (step s reads buffer s % 2);
    // an odd chunk flips it from one replay to the next, so it has a graph
    // for each parity.
    auto record_chunk = [&](hipStream_t s, bool parity) -> int {
        for (int k = 0; k < chunk; ++k) {
            const bool odd = ((k & 1) != 0) != parity;
            sa.Uin = odd ? U1 : U0;
            sa.Uout = odd ? U0 : U1;
            ra.U = sa.Uout;
            ba.U = sa.Uout;
            sa.k = k;
            hipLaunchKernelGGL(fn, step_grid, dim3(256), 0, s, sa);
            int rc = check_launch("stepwise_step_kernel");
            if (rc) return rc;
            if (M > 0 && (k + 1) % M == 0) {
                ra.k = k;
                hipLaunchKernelGGL(stepwise_readout_kernel, read_grid, dim3(256), 0, s, ra);
                if ((rc = check_launch("stepwise_readout_kernel"))) return rc;
                ba.k = k;
                hipLaunchKernelGGL(stepwise_best_kernel, dim3(R), dim3(256), 0, s, ba);
                if ((rc = check_launch("stepwise_best_kernel"))) return rc;
                if (!ba.colours) hipLaunchKernelGGL(stepwise_colour_kernel, tiles, dim3(256), 0, s, ba);
                if ((rc = check_launch("stepwise_colour_kernel"))) return rc;
            }
        }
        hipLaunchKernelGGL(advance_base_kernel, dim3(1), dim3(1), 0, s, call, chunk);
        return check_launch("advance_base_kernel");
    };

    const bool flip = (chunk & 1) != 0;
    const int replays = (steps + chunk - 1) / chunk;
    hipError_t e = hipSuccess;
    if (!graph) {
        for (int c = 0; c < replays; ++c)
            if ((st = record_chunk(stream, flip && (c & 1)))) return st;
    } else {
        PlanCache& cache = *static_cast<PlanCache*>(p->step_plans);
        Plan* plan = nullptr;
        for (int i = 0; i < cache.count; ++i) {
            Plan& c = cache.plans[i];
            if (c.q == cfg->q && c.R == R && c.M == M && c.chunk == chunk &&
                c.global_addr == sh.global_addr && c.work == work) {
                plan = &c;
                break;
            }
        }
        if (!plan) {
            // capture a new plan, evicting the least recently used one if full
            int slot = cache.count;
            if (cache.count == PlanCache::kMax) {
                slot = 0;
                for (int i = 1; i < cache.count; ++i)
                    if (cache.plans[i].last_use < cache.plans[slot].last_use) slot = i;
                destroy_plan(cache.plans[slot]);
            } else {
                ++cache.count;
            }
            Plan& pl = cache.plans[slot];
            pl = Plan{};
            hipStream_t cap = nullptr;
            e = hipStreamCreateWithFlags(&cap, hipStreamNonBlocking);
            if (e != hipSuccess) st = hip_error(e, "capture stream");
            for (int par = 0; par < (flip ? 2 : 1) && !st; ++par) {
                e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
                if (e != hipSuccess) {
                    st = hip_error(e, "hipStreamBeginCapture");
                    break;
                }
                st = record_chunk(cap, par == 1);
                e = hipStreamEndCapture(cap, &pl.g[par]);
                if (!st && e != hipSuccess) st = hip_error(e, "hipStreamEndCapture");
                if (!st && (e = hipGraphInstantiate(&pl.x[par], pl.g[par], nullptr, nullptr, 0)) != hipSuccess)
                    st = hip_error(e, "hipGraphInstantiate");
            }
            if (cap) (void)hipStreamDestroy(cap);
            if (!st && (e = hipEventCreateWithFlags(&pl.done, hipEventDisableTiming)) != hipSuccess)
                st = hip_error(e, "plan event");
            if (st) {
                destroy_plan(pl);
                // keep the cache dense: move the last plan into the freed slot
                if (slot != cache.count - 1) {
                    pl = cache.plans[cache.count - 1];
                    cache.plans[cache.count - 1] = Plan{};
                }
                --cache.count;
                return st;
            }
            pl.q = cfg->q;
            pl.R = R;
            pl.M = M;
            pl.chunk = chunk;
            pl.global_addr = sh.global_addr;
            pl.work = work;
            plan = &pl;
        }
        plan->last_use = ++cache.clock;
        for (int c = 0; c < replays; ++c) {
            e = hipGraphLaunch(plan->x[flip ? (c & 1) : 0], stream);
            if (e != hipSuccess) return hip_error(e, "hipGraphLaunch");
        }
        e = hipEventRecord(plan->done, stream);
        if (e != hipSuccess) return hip_error(e, "plan event record");
    }
    // readout after the last step when steps is not a multiple of M
    if (M > 0 && steps % M != 0) {
        ReadArgs rl = ra;
        rl.k = -1;
        rl.U = Ufinal;
        BestArgs bl = ba;
        bl.k = -1;
        bl.U = Ufinal;
        hipLaunchKernelGGL(stepwise_readout_kernel, read_grid, dim3(256), 0, stream, rl);
        if ((st = check_launch("stepwise_readout_kernel"))) return st;
        hipLaunchKernelGGL(stepwise_best_kernel, dim3(R), dim3(256), 0, stream, bl);
        if ((st = check_launch("stepwise_best_kernel"))) return st;
        if (!bl.colours) hipLaunchKernelGGL(stepwise_colour_kernel, tiles, dim3(256), 0, stream, bl);
        if ((st = check_launch("stepwise_colour_kernel"))) return st;
    }
    if (ro && M > 0 && steps > 0) {
        if (ro->best_h) {
            e = hipMemcpyAsync(ro->best_h, best, sizeof(double) * R, hipMemcpyDeviceToDevice, stream);
            if (e != hipSuccess) return hip_error(e, "best_h copy");
        }
        if (ro->best_step) {
            e = hipMemcpyAsync(ro->best_step, best_at, sizeof(int32_t) * R, hipMemcpyDeviceToDevice, stream);
            if (e != hipSuccess) return hip_error(e, "best_step copy");
        }
    }
    hipLaunchKernelGGL(stepwise_final_kernel, tiles, tile_tb, 0, stream, Ufinal, theta, phase, n, R,
                       Rp);
    return check_launch("stepwise_final_kernel");
}

}  // namespace

size_t stepwise_workspace_bytes(const Problem* p, const oim_run_cfg* cfg) {
    return shape_of(p, cfg).bytes;
}

int launch_stepwise_sparse(Problem* p, const oim_run_cfg* cfg, const float* K, const float* Ks,
                           const float* sigma, const uint64_t* seeds, int64_t step0,
                           float* theta, uint32_t* phase, const oim_readout* ro,
                           hipStream_t stream) {
    const size_t need = stepwise_workspace_bytes(p, cfg);
    if (p->work_bytes < need) {
        clear_plans(p);  // they were captured on the old workspace
        (void)hipFree(p->d_work);
        p->d_work = nullptr;
        p->work_bytes = 0;
        hipError_t e = hipMalloc(&p->d_work, need);
        if (e != hipSuccess) {
            p->d_work = nullptr;
            return e == hipErrorOutOfMemory ? set_error(OIM_E_NOMEM, "stepwise workspace")
                                            : hip_error(e, "hipMalloc stepwise workspace");
        }
        p->work_bytes = need;
    }
    return run_stepwise(p, cfg, K, Ks, sigma, seeds, step0, theta, phase, ro, stream, p->d_work,
                        true);
}

int launch_stepwise_sparse_ws(Problem* p, const oim_run_cfg* cfg, const float* K, const float* Ks,
                              const float* sigma, const uint64_t* seeds, int64_t step0,
                              float* theta, uint32_t* phase, const oim_readout* ro,
                              hipStream_t stream, void* work) {
    return run_stepwise(p, cfg, K, Ks, sigma, seeds, step0, theta, phase, ro, stream, work,
                        false);
}

}  // namespace oim
