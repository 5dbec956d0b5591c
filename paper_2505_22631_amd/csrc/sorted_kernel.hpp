// sorted_kernel.hpp -- the LDS-resident loop of persistent_kernel.hpp for
// shapes of one slice per wave group (instances of at most 4096
// oscillators): the same state, arithmetic and results, bit for bit, with the
// rows dealt to lanes by length.
//
// Such instances are small, so a step is a chain of latencies and LDS reads
// rather than a stream of work, and a run of 64 rows walks the longest of
// them.  So here
//  - rows are sorted by length, in 16-byte groups of entries, and dealt to
//    lanes 64 at a time (SortedRows); rows of one length keep the order of
//    their table slots, so a run's table writes spread over the banks;
//  - the first groups of every row's entries and its own (sin, cos) stay in
//    registers, and two tables are read and written in turn, one barrier per
//    step;
//  - each quad's noise is drawn once, a step ahead, and handed to its rows
//    through LDS (two buffers), by waves without rows where there are enough
//    of them, or else by the waves of the shortest rows;
//  - only waves that have rows or draw noise are launched.
//
// What bounds it: with one workgroup per CU and short rows the chain LDS
// reads -> sums -> update -> barrier, with long ones the LDS reads (8 bytes per
// entry from random banks; G(800, 0.06) 13 waves x 48 reads of 6 to 9 cycles).
// us per step of the shapes that walked each slice's longest row with two
// barriers, and now, one replica: n = 200 of degree 10 unit weights 1.03 ->
// 0.61, real weights 1.31 -> 0.60; n = 500 of degree 10 1.25 -> 0.64, real 1.60
// -> 0.63; G(800, 0.06) 3.13 -> 1.78, real 4.72 -> 2.12; n = 2000 of degree 10
// 2.41 -> 1.73, real 3.00 -> 1.52; n = 4000 of degree 6 real weights 4.5 ->
// 2.9.  Of that the noise drawn once by waves of their own gave 0.85 -> 0.60 us
// (n = 200, unit weights), the sorting 2.97 -> 2.20 (real 3.97 -> 2.32) on
// G(800, 0.06), whose runs' longest rows sum to 1.05 times the entries where
// whole slices' took 1.4, and the second copy of the table 2.20 -> 1.78 (real
// 2.32 -> 2.12; n = 2000 1.95 -> 1.73, real 1.81 -> 1.52).
#pragma once
#include <type_traits>

#include "persistent_kernel.hpp"

#pragma clang fp contract(off)

namespace oim {

namespace persist {

struct SortedArgs {
    PersistArgs p;
    const int4* entries;  // SortedRows entries
    const int2* run;      // per run: (first group, groups per row)
    const int2* row;      // per run and lane: (oscillator, upper start | length << 16)
    const int32_t* run0;  // per instance: its first run
    uint32_t bytes;       // of entries
};

// The same entry as one 64-bit word (sine below).
__device__ __forceinline__ uint64_t sc_word(int byte_off) {
    typedef __attribute__((address_space(3))) const uint64_t lds_u64;
    return *reinterpret_cast<lds_u64*>((uint32_t)byte_off);
}

// Split-row shapes keep every (sin, cos) twice, the second time in an order of
// its own, and each entry points at the copy that leaves the LDS banks less
// contended (see sorted_rows_kernel).
__host__ __device__ constexpr int copies(int rpl) { return rpl < 4 ? 2 : 1; }
// Where the second copy holds slot s: the same 32 slots, permuted by their
// number, so that its bank says nothing about the first copy's.
__host__ __device__ constexpr int second_slot(int s, int plane) {
    return 4 * plane + (s ^ ((s >> 5) & 31));
}

// Layout of a table: the copies of (sin, cos), of the colours, the zero entry
// at byte 36 * copies * plane.  The second table of a shape of C slices starts
// past the first one of its largest instance, a constant so that a read's
// table is part of its instruction.
__host__ __device__ constexpr int sorted_table1(int C, int cp) { return 36 * cp * 64 * C + 16; }

// LDS of a launch: the tables, the noise buffers, the readout's sums.
inline size_t sorted_lds(int C, int rpl, int plane) {
    const int cp = copies(rpl);
    return (size_t)sorted_table1(C, cp) + 36 * (size_t)cp * plane + 16 + 32 * (size_t)plane +
           16 * sizeof(double);
}

// Waves of this kernel share LDS alone, so its barriers wait for LDS alone: a
// readout's stores to memory drain while the next steps run.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// C slices of capacity, RPL rows per lane: wave w holds runs w * RPL ..
// w * RPL + RPL - 1, and waves past the last run draw noise.
template <int C, int RPL, int QM, bool UWT>
__global__ __launch_bounds__(1024, 4) void sorted_kernel(SortedArgs sa) {
    extern __shared__ __align__(16) unsigned char smem[];
    const PersistArgs& a = sa.p;
    // workgroup -> (instance, replica) as in persistent_sparse_kernel
    int grp, r;
    {
        const int b = blockIdx.x;
        const int I8 = a.I / 8 * 8;
        const int head = a.R * I8;
        if (b < head) {
            const int c = b & 7, k = b >> 3;
            grp = c + 8 * (k / a.R);
            r = k % a.R;
        } else {
            grp = I8 + (b - head) / a.R;
            r = (b - head) % a.R;
        }
    }
    const int inst_id = a.order[grp];
    const int4 idesc = a.inst[inst_id];
    const int S = idesc.y, off = idesc.z, n = idesc.w;
    const int plane = S * 64;
    const int runs = (n + 63) >> 6;
    const int run0 = sa.run0[inst_id];
    constexpr int CP = copies(RPL);
    constexpr int T1 = sorted_table1(C, CP);
    constexpr int E = UWT ? 4 : 2;      // entries per 16-byte group
    constexpr int GB = 4 / RPL;         // groups of a row read together
    constexpr int NV = 2 * GB;          // resident groups per row
    float2* sc = reinterpret_cast<float2*>(smem);
    unsigned char* col8 = smem + (size_t)32 * CP * plane;
    // (0, 0) in each table, what padding entries read
    float2* zero_entry = reinterpret_cast<float2*>(smem + (size_t)36 * CP * plane);
    float* nz = reinterpret_cast<float*>(smem + T1 + 36 * CP * plane + 16);  // [2][4 * plane]
    double* red = reinterpret_cast<double*>(nz + 8 * plane);            // [16]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = blockDim.x >> 6;
    const int row_waves = (runs + RPL - 1) / RPL;
    const int q = QM ? QM : a.q;
    const uint64_t seed = a.seeds[r];
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    float* th = a.theta + (int64_t)r * a.n_total + off;
    uint32_t* pw = a.phase ? a.phase + (int64_t)r * a.n_total + off : nullptr;
    const int out_id = r * a.I + inst_id;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)sa.entries, (short)0, (int)sa.bytes, 0x00020000);
    const int voff = lane * 16;

    // the lane's rows: oscillator (past n: none), table slot, (first group,
    // groups), phase, (sin, cos)
    int osc[RPL], slot[RPL], slot2[RPL], base[RPL], D[RPL];
    int ul[RPL];  // upper start | length << 16
    uint32_t ph[RPL];
    float2 own_sc[RPL];
    int4 res[RPL][NV];
    const bool rows = wave < row_waves;
    auto have = [&](int jj) { return wave * RPL + jj < runs; };
    // group h of row jj; past its last, the run's padding group
    auto load_group = [&](int jj, int h) __attribute__((always_inline)) {
        return load_pair(rsrc, voff, (base[jj] + (h < D[jj] ? h : D[jj])) * 1024);
    };
#pragma unroll
    for (int jj = 0; jj < RPL; ++jj) {
        // (a run past the last holds padding alone)
        const int run = have(jj) ? wave * RPL + jj : runs - 1;
        const int2 d = sa.run[run0 + run];
        D[jj] = __builtin_amdgcn_readfirstlane(have(jj) ? d.y : 0);
        base[jj] = __builtin_amdgcn_readfirstlane(have(jj) ? d.x : d.x + d.y);
        const int2 row = sa.row[(run0 + run) * 64 + lane];
        const int i = row.x;
        if constexpr (UWT) ul[jj] = have(jj) ? row.y : 0;
        osc[jj] = have(jj) ? i : n;
        slot[jj] = (i & 3) * plane + (i >> 2);
        slot2[jj] = CP > 1 ? second_slot(slot[jj], plane) : 0;
        const uint32_t u = osc[jj] < n ? (pw ? pw[osc[jj]] : phase_from_theta(th[osc[jj]])) : 0u;
        ph[jj] = u;
        own_sc[jj] = make_float2(sin_turn(u), cos_turn(u));
        if (have(jj)) {
            sc[slot[jj]] = own_sc[jj];
            if constexpr (CP > 1) sc[slot2[jj]] = own_sc[jj];
        }
#pragma unroll
        for (int h = 0; h < NV; ++h) res[jj][h] = load_group(jj, h);
    }

    // the slices whose noise this wave draws: duty, duty + duty_step, ... < S
    const int spare = nwaves - row_waves;
    const bool helpers = 3 * spare >= S;
    const int duty = helpers ? (rows ? S : wave - row_waves) : (rows ? row_waves - 1 - wave : S);
    const int duty_step = helpers ? spare : row_waves;
    // the normals of step t of their quads, into buffer `buf`
    auto draw = [&](uint32_t t, int buf) __attribute__((always_inline)) {
        for (int sl = duty; sl < S; sl += duty_step) {
            // (re-materialised every step, so that partial Philox rounds are
            // not precomputed and kept live in registers)
            uint32_t mm = (uint32_t)(sl * 64 + lane), kk0 = k0, kk1 = k1;
            asm volatile("" : "+v"(mm), "+s"(kk0), "+s"(kk1));
            float z4[4];
            normals4(mm, t, (uint32_t)inst_id, kk0, kk1, z4);
#pragma unroll
            for (int j = 0; j < 4; ++j) nz[buf * 4 * plane + j * plane + sl * 64 + lane] = z4[j];
        }
    };
    draw((uint32_t)a.step0, 0);
    if (threadIdx.x == 0) zero_entry[0] = zero_entry[T1 / 8] = make_float2(0.f, 0.f);
    double best_h = DBL_MAX;
    int best_at = -1;
    lds_barrier();

    const float sqrt_dt = __builtin_sqrtf(a.dt);
    const int64_t sched_off = (int64_t)r * a.sched_stride;
    auto sched = [&](const float* v, int c) {
        const int i = c * 64 + lane;
        return i < a.steps ? v[sched_off + i] : 0.0f;
    };
    float cK = sched(a.K, 0), cKs = sched(a.Ks, 0), cS = sched(a.sigma, 0);
    float nK = sched(a.K, 1), nKs = sched(a.Ks, 1), nS = sched(a.sigma, 1);

    // One step: the resident groups' LDS reads go out at once, with the
    // noise drawn while they are in flight; the rest of a long row is
    // streamed, its first loads issued before the resident groups are used.
    // Groups are read GB at a time, padding adding +-0.  Step s reads table
    // s % 2 and writes the other.
    auto step = [&](auto odd, uint32_t t, float kc, float ks, float ns) __attribute__((always_inline)) {
        constexpr int rd = decltype(odd)::value ? T1 : 0, wr = decltype(odd)::value ? 0 : T1;
        float A[RPL], B[RPL], z[RPL];
#pragma unroll
        for (int jj = 0; jj < RPL; ++jj) A[jj] = B[jj] = 0.f;
        const int D0 = D[0];  // the longest of the lane's rows
        int4 str[RPL][GB];
        auto stream = [&](int h0) __attribute__((always_inline)) {
#pragma unroll
            for (int jj = 0; jj < RPL; ++jj)
#pragma unroll
                for (int h = 0; h < GB; ++h) str[jj][h] = load_group(jj, h0 + h);
        };
        uint64_t p[RPL][GB][E];
        auto read = [&](int jj, int h, const int4& v) __attribute__((always_inline)) {
            p[jj][h][0] = sc_word(v.x + rd);
            if constexpr (UWT) {
                p[jj][h][1] = sc_word(v.y + rd);
                p[jj][h][2] = sc_word(v.z + rd);
                p[jj][h][3] = sc_word(v.w + rd);
            } else {
                p[jj][h][1] = sc_word(v.z + rd);
            }
        };
        // the reads' results arrive here, not before
        auto arrive = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int jj = 0; jj < RPL; ++jj)
#pragma unroll
                for (int h = 0; h < GB; ++h)
#pragma unroll
                    for (int x = 0; x < E; ++x) asm volatile("" : "+v"(p[jj][h][x]));
        };
        auto add = [&](int jj, int h, const int4& v) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < E; ++x) {
                const float ps = __uint_as_float((uint32_t)p[jj][h][x]);
                const float pc = __uint_as_float((uint32_t)(p[jj][h][x] >> 32));
                if constexpr (UWT) {
                    A[jj] = A[jj] + pc;
                    B[jj] = B[jj] + ps;
                } else {
                    const float w = __int_as_float(x == 0 ? v.y : v.w);
                    A[jj] = __builtin_fmaf(w, pc, A[jj]);
                    B[jj] = __builtin_fmaf(w, ps, B[jj]);
                }
            }
        };
        if (D0 > NV) stream(NV);
#pragma unroll
        for (int c = 0; c < NV; c += GB) {
            if (c > 0 && c >= D0) break;
#pragma unroll
            for (int jj = 0; jj < RPL; ++jj)
#pragma unroll
                for (int h = 0; h < GB; ++h) read(jj, h, res[jj][c + h]);
            if (c == 0) {
#pragma unroll
                for (int jj = 0; jj < RPL; ++jj)
                    z[jj] = nz[(decltype(odd)::value ? 4 * plane : 0) + slot[jj]];
                draw(t + 1u, decltype(odd)::value ? 0 : 1);
            }
            arrive();
#pragma unroll
            for (int jj = 0; jj < RPL; ++jj)
#pragma unroll
                for (int h = 0; h < GB; ++h) add(jj, h, res[jj][c + h]);
        }
        for (int h0 = NV; h0 < D0; h0 += GB) {
            int4 cur[RPL][GB];
#pragma unroll
            for (int jj = 0; jj < RPL; ++jj)
#pragma unroll
                for (int h = 0; h < GB; ++h) {
                    cur[jj][h] = str[jj][h];
                    read(jj, h, cur[jj][h]);
                }
            if (h0 + GB < D0) stream(h0 + GB);
            arrive();
#pragma unroll
            for (int jj = 0; jj < RPL; ++jj)
#pragma unroll
                for (int h = 0; h < GB; ++h) add(jj, h, cur[jj][h]);
        }
#pragma unroll
        for (int jj = 0; jj < RPL; ++jj) {
            if constexpr (UWT) {
                // (-1) x (a chain of roundings) equals the chain of roundings
                // of the negated terms, up to the sign of a zero sum, which no
                // phase update can tell apart
                A[jj] = a.w0 * A[jj];
                B[jj] = a.w0 * B[jj];
            }
            const float inc = increment<QM>(own_sc[jj], A[jj], B[jj], ph[jj], q, kc, ks, ns, z[jj]);
            const uint32_t u = advance(ph[jj], inc);
            ph[jj] = u;
            own_sc[jj] = make_float2(sin_turn(u), cos_turn(u));
            if (have(jj)) {
                sc[wr / 8 + slot[jj]] = own_sc[jj];
                if constexpr (CP > 1) sc[wr / 8 + slot2[jj]] = own_sc[jj];
            }
        }
    };

    for (int s = 0; s < a.steps; ++s) {
        const uint32_t t = (uint32_t)(a.step0 + s);
        // schedules arrive 64 steps at a time, one step per lane, the next
        // chunk's loads in flight
        if (s > 0 && (s & 63) == 0) {
            cK = nK;
            cKs = nKs;
            cS = nS;
            const int c = (s >> 6) + 1;
            nK = sched(a.K, c);
            nKs = sched(a.Ks, c);
            nS = sched(a.sigma, c);
        }
        const int sl = s & 63;
        const float Kt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cK), sl));
        const float Kst = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cKs), sl));
        const float St = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cS), sl));
        const float kc = -a.dt * Kt * kTurnScale;
        const float ks = -a.dt * Kst * kTurnScale;
        const float ns = St * sqrt_dt * kTurnScale;
        if (rows) {
            if (s & 1) step(std::true_type{}, t, kc, ks, ns);
            else step(std::false_type{}, t, kc, ks, ns);
        } else {
            draw(t + 1u, (s + 1) & 1);
        }
        lds_barrier();

        // ---- optional readout: threshold, Eq. 1 / Eq. 2, best-so-far ----
        if (a.M > 0 && ((s + 1) % a.M == 0 || s + 1 == a.steps)) {
            int own_c[RPL];
#pragma unroll
            for (int jj = 0; jj < RPL; ++jj) {
                own_c[jj] = nearest_state(ph[jj], q);
                if (have(jj)) {
                    col8[slot[jj]] = (unsigned char)own_c[jj];
                    if constexpr (CP > 1) col8[slot2[jj]] = (unsigned char)own_c[jj];
                }
                if constexpr (!UWT) ul[jj] = have(jj) ? sa.row[(run0 + wave * RPL + jj) * 64 + lane].y : 0;
            }
            lds_barrier();
            // Each row sums its terms over j > i in column order (its entries
            // from its upper start to its length).  With one weight on every
            // entry the terms are +-w0 or 0 and their sum is exact in any
            // order: counts, summed as integers.  Otherwise the rows' FP64
            // sums meet in the table that the next step overwrites, by table
            // slot, and fold as (r0 + r1) + (r2 + r3) per quad, by the xor
            // butterfly (partner distance 1, 2, ..., 32) over a slice's 64
            // quads, and pairwise over the slices: the library's fixed order.
            // (A readout of G(800, 0.06) with unit weights took 9 us: each
            // group's reads waited for, barriers for the stores too.  Now 4.)
            [[maybe_unused]] double* rowsum = reinterpret_cast<double*>(smem + ((s & 1) ? T1 : 0));
            [[maybe_unused]] int cnt = 0, all = 0;  // matching neighbours j > i, all of them
            if (rows) {
#pragma unroll
                for (int jj = 0; jj < RPL; ++jj) {
                    const int up = ul[jj] & 0xffff, len = ul[jj] >> 16;
                    if constexpr (UWT) {
                        // GB groups' colours are read together; what padding
                        // reads (past the colours, within the LDS) is not counted
                        auto terms = [&](const int4* v, int h0) __attribute__((always_inline)) {
                            int c[GB][4];
                            auto colour = [&](int at) __attribute__((always_inline)) {
                                // (kept here: hoisted out of the run, the
                                // resident entries' addresses would spill)
                                asm volatile("" : "+v"(at));
                                return (int)col8[(uint32_t)at >> 3];
                            };
#pragma unroll
                            for (int h = 0; h < GB; ++h) {
                                c[h][0] = colour(v[h].x);
                                c[h][1] = colour(v[h].y);
                                c[h][2] = colour(v[h].z);
                                c[h][3] = colour(v[h].w);
                            }
#pragma unroll
                            for (int h = 0; h < GB; ++h)
#pragma unroll
                                for (int x = 0; x < 4; ++x) {
                                    const bool in = (uint32_t)(4 * (h0 + h) + x - up) < (uint32_t)(len - up);
                                    cnt += in && own_c[jj] == c[h][x] ? 1 : 0;
                                }
                        };
#pragma unroll
                        for (int c = 0; c < NV; c += GB) {
                            if (c > 0 && c >= D[jj]) break;
                            terms(&res[jj][c], c);
                        }
                        for (int h0 = NV; h0 < D[jj]; h0 += GB) {
                            int4 v[GB];
#pragma unroll
                            for (int h = 0; h < GB; ++h) v[h] = load_group(jj, h0 + h);
                            terms(v, h0);
                        }
                        all += len - up;
                    } else {
                        double rs = 0.0;
                        auto terms = [&](const int4& v, int h) __attribute__((always_inline)) {
                            const int o2[2] = {v.x, v.z};
                            const float w2[2] = {__int_as_float(v.y), __int_as_float(v.w)};
#pragma unroll
                            for (int x = 0; x < 2; ++x) {
                                const int idx = 2 * h + x;
                                const bool in = idx >= up && idx < len;
                                const bool eq = own_c[jj] == col8[in ? o2[x] >> 3 : 0];
                                const float tt = eq ? w2[x] : (q == 2 ? -w2[x] : 0.f);
                                rs += in ? (double)tt : 0.0;
                            }
                        };
#pragma unroll
                        for (int h = 0; h < NV; ++h) {
                            if (h >= D[jj]) break;
                            terms(res[jj][h], h);
                        }
#pragma unroll 2
                        for (int h = NV; h < D[jj]; ++h) terms(load_group(jj, h), h);
                        if (have(jj)) rowsum[slot[jj]] = rs;
                    }
                }
            }
            double total;
            if constexpr (UWT) {
                // q = 2: +1 for a match, -1 for any other
                if (q == 2) cnt = 2 * cnt - all;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) cnt += __shfl_xor(cnt, o, 64);
                int* sums = reinterpret_cast<int*>(red);
                if (lane == 0) sums[wave] = cnt;
                lds_barrier();
                int c = lane < nwaves ? sums[lane] : 0;
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) c += __shfl_xor(c, o, 64);
                c = __builtin_amdgcn_readfirstlane(c);
                total = c ? (double)a.w0 * (double)c : 0.0;
            } else {
                // rows that no run holds
                for (int i = runs * 64 + threadIdx.x; i < 4 * plane; i += blockDim.x)
                    rowsum[(i & 3) * plane + (i >> 2)] = 0.0;
                lds_barrier();
                for (int k = wave; k < S; k += nwaves) {
                    const double* x = rowsum + k * 64 + lane;
                    double v = (x[0] + x[plane]) + (x[2 * plane] + x[3 * plane]);
                    for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
                    if (lane == 0) red[k] = v;
                }
                lds_barrier();
                // S <= 16 slices: two per lane, zero-padded
                const double v0 = 2 * lane < S ? red[2 * lane] : 0.0;
                const double v1 = 2 * lane + 1 < S ? red[2 * lane + 1] : 0.0;
                double v = v0 + v1;
                for (int o = 1; o < 16; o <<= 1) v = v + __shfl_down(v, o, 64);
                total = __shfl(v, 0, 64);
            }
            const double H = -total;
            if (threadIdx.x == 0 && a.trace) {
                const int kread = (s + a.M) / a.M - 1;
                a.trace[(int64_t)kread * a.R * a.I + out_id] = H;
            }
            if (H < best_h) {
                best_h = H;
                best_at = (int32_t)(a.step0 + s + 1);
                if (a.best_colour && rows) {
                    int8_t* bc = a.best_colour + (int64_t)r * a.n_total + off;
#pragma unroll
                    for (int jj = 0; jj < RPL; ++jj)
                        if (osc[jj] < n) bc[osc[jj]] = (int8_t)own_c[jj];
                }
            }
        }
    }

    // ---- final phases ----
#pragma unroll
    for (int jj = 0; jj < RPL; ++jj) {
        if (rows && osc[jj] < n) {
            th[osc[jj]] = theta_from_phase(ph[jj]);
            if (pw) pw[osc[jj]] = ph[jj];
        }
    }
    if (threadIdx.x == 0) {
        if (a.best_h) a.best_h[out_id] = best_at >= 0 ? best_h : __builtin_inf();
        if (a.best_step) a.best_step[out_id] = best_at;
    }
}

using SortedFn = void (*)(SortedArgs);

// The shapes (slices of capacity, rows per lane) and their instantiations by
// SHIL order class (generic, 2, 3).
#define OIM_SORTED_SHAPES(X)                                                             \
    X(1, 4) X(2, 4) X(4, 4) X(8, 4) X(16, 4) X(2, 2) X(4, 2) X(8, 2) X(1, 1) X(2, 1) X(4, 1)
struct SortedShape {
    int C, rpl;
    SortedFn fn[3];
};
#define OIM_SORTED_ONE(C, RPL) +1
constexpr int kSortedCount = 0 OIM_SORTED_SHAPES(OIM_SORTED_ONE);
extern const SortedShape kSorted[kSortedCount];         // general weights
extern const SortedShape kSortedUniform[kSortedCount];  // uniform unit weights

}  // namespace persist
}  // namespace oim
