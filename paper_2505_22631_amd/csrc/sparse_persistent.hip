// sparse_persistent.hip -- launch variants of the LDS-resident kernel
// (persistent_kernel.hpp), the default choice, the launch and the autotuner.
#include <float.h>

#include <algorithm>

#include "sorted_kernel.hpp"

namespace oim {

namespace {

using namespace persist;


struct Variant {
    int tb, ms, rpl;
    KernelFn fn[3];  // QM = 0 (generic), 2, 3
    // slices covered: (waves / waves per slice) x slices per wave group
    int covers() const { return (tb / 64) / (4 / rpl) * ms; }
};

#define OIM_VARIANT_ENTRY(TB, MS, RPL)                                                   \
    Variant{TB, MS, RPL,                                                                 \
            {persistent_sparse_kernel<TB, MS, 0, RPL, false>,                            \
             persistent_sparse_kernel<TB, MS, 2, RPL, false>,                            \
             persistent_sparse_kernel<TB, MS, 3, RPL, false>}},

const Variant kVariants[kVariantCount] = {OIM_PERSIST_VARIANTS(OIM_VARIANT_ENTRY)};

constexpr size_t kLdsLimit = 160 * 1024;

// LDS of a launch; with slice_sums, room for the readout's per-slice sums
// (slices covered by the variant) too.
size_t lds_bytes(int plane, int tb, int ms, int rpl, int covered = 0) {
    size_t b = (size_t)8 * 4 * plane;                 // (sin, cos) table
    b += (size_t)4 * plane + 16;                      // colours for readout, zero entry
    b += sizeof(double) * (tb / 64 + kSliceTreeLevels) + 32;  // reduction, tree levels, readout state
    if (rpl < 4) b += sizeof(double) * (size_t)tb;    // quads' partial row sums (readout)
    b += sizeof(double) * (size_t)covered;            // per-slice sums (readout), if used
    return b;
}

constexpr uint64_t kMaxSellBytes = 0x7fffffffull;

// The variant of `tb` threads and `rpl` rows per lane with the fewest slices
// per wave group that covers S slices, or null.
const Variant* covering(int tb, int rpl, int S) {
    const Variant* best = nullptr;
    for (const Variant& v : kVariants)
        if (v.tb == tb && v.rpl == rpl && v.covers() >= S && (!best || v.ms < best->ms)) best = &v;
    return best;
}

// The whole-quad variant with the fewest waves that cover S slices, preferring
// 8 waves per workgroup, among blocks of at least 256 threads (tb_hint: of
// that many).
const Variant* fewest_waves(int S, int tb_hint) {
    const Variant* best = nullptr;
    for (const Variant& v : kVariants) {
        const int W = v.tb / 64;
        if (v.rpl != 4) continue;
        if (tb_hint ? v.tb != tb_hint : v.tb < 256) continue;
        if (W * v.ms < S) continue;
        if (!best) { best = &v; continue; }
        // smallest ms*W (least idle), then the preferred block size
        const int cv = W * v.ms, cb = (best->tb / 64) * best->ms;
        const int pv = v.tb == 512 ? 0 : 1, pb = best->tb == 512 ? 0 : 1;
        if (cv < cb || (cv == cb && pv < pb)) best = &v;
    }
    return best;
}

// Whether a CU holds `groups` workgroups of `waves` waves at once at this
// kernel's registers, four waves per SIMD: a workgroup's waves go to the SIMDs
// in turn (three of five waves do not fit: n = 200 real weights, 600 replicas,
// 0.87 us per step with four waves each, 1.25 with five).
bool cu_holds(int64_t groups, int64_t waves) {
    return waves > 4 ? groups * ((waves + 3) / 4) <= 4 : groups * waves <= 16;
}

// Instances far below the largest one (a ragged batch): the mean under 0.65 of it.
bool ragged(const Problem* p) {
    return p->n_inst > 1 && 20 * (int64_t)p->n < 13 * (int64_t)p->n_inst * p->max_inst_n;
}

bool long_rows(const Problem* p) { return p->nnz / p->n >= 24; }

const Variant* find_variant(int tb, int ms, int rpl) {
    for (const Variant& v : kVariants)
        if (v.tb == tb && v.ms == ms && v.rpl == rpl) return &v;
    return nullptr;
}

// Whole quads of five slices and more: see default_variant.
int quad_threads(const Problem* p, int q, int M, int64_t per_cu) {
    const int S = p->max_slices;
    const int64_t deg = p->nnz / p->n;
    const bool often = M > 0 && M <= 16;  // readouts that weigh
    if (S <= 8) {
        if (!p->d_sell_uw) return 256;
        if (per_cu == 2) return 512;
        return S <= 6 && !ragged(p) && per_cu >= 5 && (per_cu <= 7 || q != 2) ? 128 : 256;
    }
    if (S <= 16) {
        if (per_cu == 1) return 1024;
        if (p->d_sell_uw && long_rows(p) && often && per_cu <= 3) return 1024;
        if (p->d_sell_uw)
            return S <= 12 && (per_cu == 3 || (per_cu >= 4 && q != 2) || (per_cu >= 5 && S >= 10)) ? 256 : 512;
        if (S > 12) return ragged(p) && per_cu >= 4 ? 512 : 1024;
        if (S <= 10 && per_cu == 3) return 256;
        if (S == 9 && per_cu == 2) return 512;
        if (often && per_cu >= 5) return 256;
        if (deg >= 12 || (S >= 11 && deg >= 6)) return 1024;
        return per_cu >= 3 && per_cu != 4 ? 256 : 512;
    }
    if (p->d_sell_uw && q != 2 && S <= 24 && per_cu >= 2) return 512;
    return p->d_sell_uw || S <= 32 ? 1024 : S <= 48 ? 768 : 512;
}

// Default choice without tuning, from the slices of the largest instance (S),
// the workgroups a CU holds at once (per_cu) and the rows' mean length (deg).
// All figures are us per step.
//  - A step's latency is shared by the waves of a workgroup, so the rows are
//    split over as many waves as the CU holds with its other workgroups
//    (cu_holds), short unit-weight rows with room for the noise's waves: 4, 2
//    and 1 rows per lane, n = 800 of degree 10, one replica 2.0, 0.93, 1.04
//    (real weights 2.1, 1.26, 0.96), 500 replicas 2.4, 1.63, 2.2 (real 3.0,
//    1.54, 2.2); G(800, 0.06) one replica 4.0, 2.2, 1.8.
//  - Past that two rows per lane stay the better choice for real weights and
//    longer rows, whose entries weigh more than the noise that every wave of a
//    split waits for, and the sorted rows keep them in registers: a batch of
//    256 graphs of 100 to 1000, degree 8, real, 8 replicas 5.9 and 7.4 in whole
//    quads; of 1024 graphs of 100 to 500, degree 20, unit, 2 replicas 4.6 and
//    8.0; n = 400 of degree 14, unit, 2048 replicas 3.9 and 4.1; n = 1500 of
//    degree 7, real, 1536 replicas 8.3 and 10.5.  Long real rows up to three and
//    four slices even take one row per lane (n = 600 of degree 20, 2048
//    replicas 10.5, 11.4 with two).
//  - Whole quads draw their own noise: unit weights with short rows take them,
//    on the general kernel (on_sorted_rows), about sixteen waves per CU: n = 400
//    of degree 4, 2048 replicas 2.4 on two waves (3.3 split); n = 600 of degree
//    7, 1024 replicas 2.9 on four (two 3.6, split 4.4), 2048 replicas 4.8 on two
//    (5.1, 7.2), 8192 replicas, q = 3, readouts every 10 steps 20.0 on one (two
//    24.0, four 21.8); n = 1500 of degree 4, 512 replicas 2.6 on eight (split
//    3.3), 1536 replicas 5.8 on two (6.8 on four, split 9.4).  A ragged batch's
//    workgroups are mostly small: 256 graphs of 100 to 1000, degree 4, 8
//    replicas 3.6 on two waves, 4.0 on four.
//  - Real weights do so with the shortest rows of three slices (64 graphs of
//    100 to 600, degree 4.6, 16 replicas 2.5 on four waves, split 3.0; 32
//    replicas 4.2 on two, split 5.1), unless few replicas share general images
//    that pass the L2s (1024 such graphs, one replica 3.0 split, 5.4), and in
//    ragged batches of five to eight (40 graphs of 300 to 1400, degree 4, 38
//    replicas 6.0, split 7.0), and with nine or ten split waves of short rows,
//    which leave SIMDs idle (n = 1100 of degree 4, 5000 replicas 19, split 23).
//  - Nine to sixteen slices take sixteen waves of sorted rows for one workgroup
//    per CU. Real weights do at any number from thirteen slices and with longer
//    rows (n = 3000 of degree 14, 1536 replicas 27, 32 on four or eight waves),
//    unless readouts weigh (every 10 steps 35 and 36, n = 2500 33 and 30) or
//    the batch is ragged (40 graphs of 500 to 4000, degree 4, 38 replicas 14.8,
//    13.9 on eight); unit weights with long rows only where readouts weigh (n =
//    2500 of degree 30, 300 replicas 14.0, 15.4 on eight; without 11.6 and
//    11.4). The others take eight waves, or four where those fit the CU better
//    or the SHIL order is not 2 and its term so the longer (n = 3000 of degree
//    7, unit, 1024 replicas 9.9 on eight, 11.2 on four, q = 3 with readouts
//    12.7 and 11.1; n = 2500 of degree 4, real, 1536 replicas 12.8 and 12.3).
//  - Instances of more slices take sixteen waves of whole quads: n = 3500 of
//    degree 10 4.1 -> 3.1 us (1024 x 1), n = 10000 of degree 5 8.6 -> 6.0
//    (1024 x 3); the general image, which holds more registers, twelve waves of
//    four slices for 33 to 48 (10.8 -> 9.3, against 9.75 with sixteen) and eight
//    beyond (n = 16000 of degree 4, 300 replicas 30 on eight, 37 on sixteen).
//    Up to 24 slices of unit weights and another SHIL order than 2 take eight
//    for more workgroups than CUs (n = 4100 of degree 6, 2000 replicas, q = 3:
//    23.4 us on 512 x 3, 27.8 on 1024 x 2, q = 2: 35.5 and 27.4).
const Variant* default_variant(const Problem* p, int q, int M, int R) {
    const int S = p->max_slices;
    const int64_t per_cu = ((int64_t)R * p->n_inst + 255) / 256, deg = p->nnz / p->n;
    const bool uw = p->d_sell_uw != nullptr, lng = long_rows(p);
    // waves of the split shapes with 1 and 2 rows per lane
    const int64_t w1 = (p->max_inst_n + 63) / 64, w2 = (w1 + 1) / 2;
    // the general images pass the L2s (4 MiB on each of 8 XCDs), read by few replicas
    const bool streams = p->n_inst > 1 && R < 4 && p->sell_entries * 8 > (28 << 20);
    int rpl = 4, tb = 0, ms = 0;
    if (w1 <= 16 && (cu_holds(per_cu, w1 + (uw && S > 1 && deg < 16 ? S : 0)) ||
                     (!uw && (lng || (S == 3 && deg >= 16))))) {
        rpl = 1;
    } else if (w2 <= 16 && cu_holds(per_cu, w2)) {
        rpl = 2;
    } else if (S == 1) {
        if (uw && !lng && per_cu >= 12) tb = 64;
        else rpl = 2;
    } else if (S == 2) {
        if (uw && deg < 9 && per_cu >= 6) tb = 128;
        else rpl = 2;
    } else if (S == 3 && uw) {
        if (lng && per_cu < 12 && per_cu != 4) rpl = 2;
        else if (lng || per_cu <= 5) tb = 256;
        else if (per_cu <= 10) tb = 128;
        else tb = q != 2 ? 64 : ragged(p) ? 128 : 256;
    } else if (S == 3 && deg < 5 && per_cu > 3) {
        if (streams && per_cu <= 5) rpl = 2;
        else if (streams) tb = 256;
        else if (per_cu <= 5) tb = 256, ms = 2;
        else tb = 128;
    } else if (S == 3) {
        if (deg >= 5 && (per_cu == 4 || per_cu >= 12)) tb = 256;
        else rpl = 2;
    } else if (S == 4) {
        if (!uw || deg >= 16 || per_cu <= 2 || (deg >= 12 && per_cu <= 5)) rpl = 2;
        else tb = ragged(p) && per_cu >= 6 ? 128 : 256;
    } else if (w2 <= 16) {
        if (uw ? deg >= 16 || per_cu == 1 || (deg >= 8 && per_cu <= 3 && w2 > 10)
               : !(ragged(p) && deg < 5 && per_cu >= 3) &&
                     !(w2 >= 9 && w2 <= 10 && deg < 8 && per_cu >= 4))
            rpl = 2;
    }
    if (rpl == 1) tb = S == 1 ? 256 : S == 2 ? 512 : 1024;
    else if (rpl == 2) tb = S <= 2 ? 256 : S <= 4 ? 512 : 1024;
    else if (!tb) tb = quad_threads(p, q, M, per_cu);
    const Variant* v = ms ? find_variant(tb, ms, rpl) : covering(tb, rpl, S);
    return v && lds_bytes(S * 64, v->tb, v->ms, v->rpl) <= kLdsLimit ? v : fewest_waves(S, 0);
}

// Whether a shape runs on the sorted rows.  Those of one slice per wave group
// do, but for whole quads of few slices with short rows and unit weights: their
// resident entries fill the registers, and the general kernel's quads draw
// their own noise (n = 1000 of degree 4, 600 replicas 3.4 us per step sorted,
// 2.5 so).
bool on_sorted_rows(const Problem* p, const Variant& v) {
    if (v.ms != 1 || !p->d_sorted) return false;
    return !(v.rpl == 4 && p->max_slices <= 8 && !long_rows(p) && p->d_sell_uw);
}

int env_int(const char* name, int dflt) {
    const char* v = getenv(name);
    return v ? atoi(v) : dflt;
}

// The variant covers every slice of the largest instance and its LDS fits.
bool variant_ok(const Problem* p, const Variant& v) {
    return v.covers() >= p->max_slices &&
           lds_bytes(p->max_slices * 64, v.tb, v.ms, v.rpl) <= kLdsLimit;
}

// Whether one launch holds a workgroup of v.tb threads for every replica and
// instance: a grid dimension ends at 2^32 threads, past which a launch wraps
// without an error.
bool launch_holds(const Problem* p, int R, const Variant& v) {
    return (int64_t)R * p->n_inst < ((int64_t)1 << 32) / v.tb;
}

int q_class(int q) { return q == 2 ? 1 : q == 3 ? 2 : 0; }

// The variant a run uses: the tuned one for this SHIL order if set, else an
// OIM_PERSIST_TB block-size hint, else the default choice -- unless that one's
// launch would not hold the workgroups: then the one of the fewest threads.
const Variant* run_variant(const Problem* p, int q, int M, int R) {
    const int qc = q_class(q);
    const Variant* v = nullptr;
    if (p->tuned_tb[qc]) {
        v = find_variant(p->tuned_tb[qc], p->tuned_ms[qc], p->tuned_rpl[qc]);
        if (v && !variant_ok(p, *v)) v = nullptr;
    }
    const int hint = env_int("OIM_PERSIST_TB", 0);
    if (!v && hint) v = fewest_waves(p->max_slices, hint);
    if (!v) v = default_variant(p, q, M, R);
    if (!v || launch_holds(p, R, *v)) return v;
    for (const Variant& k : kVariants)
        if (variant_ok(p, k) && k.tb < v->tb) v = &k;
    return v;
}

}  // namespace

bool persistent_variant_fits(const Problem* p, int tb, int ms, int rpl) {
    const Variant* v = find_variant(tb, ms, rpl);
    return v && variant_ok(p, *v);
}

bool persistent_sparse_fits(const Problem* p) {
    if (p->dense || p->max_slices == 0) return false;
    if (lds_bytes(p->max_slices * 64, 1024, 5, 4) > kLdsLimit) return false;
    if ((uint64_t)p->sell_entries * 8 > kMaxSellBytes) return false;
    return fewest_waves(p->max_slices, 0) != nullptr;
}

namespace {
// A shape of one slice per wave group on the sorted rows: the waves that hold
// rows of the largest instance and up to one more per slice to draw its noise,
// as long as the CU holds them beside its other workgroups (cu_holds: the
// sixteen waves of this kernel's registers).
int launch_sorted(const Problem* p, const Variant& v, const PersistArgs& a, int qi,
                  hipStream_t stream) {
    SortedArgs sa{};
    sa.p = a;
    sa.entries = copies(v.rpl) > 1 ? p->d_sorted2 : p->d_sorted;
    sa.run = p->d_sorted_run;
    sa.row = p->d_sorted_row;
    sa.run0 = p->d_sorted_run0;
    sa.bytes = p->sorted_bytes;
    const int S = p->max_slices;
    const SortedShape* shape = nullptr;
    for (const SortedShape& k : p->d_sell_uw ? kSortedUniform : kSorted)
        if (k.C == v.covers() && k.rpl == v.rpl) shape = &k;
    if (!shape) return set_error(OIM_E_UNSUPPORTED, "no sorted-rows shape");
    const int64_t per_cu = ((int64_t)a.R * p->n_inst + 255) / 256;
    int waves = ((p->max_inst_n + 63) / 64 + v.rpl - 1) / v.rpl;
    for (int k = 0; k < S && cu_holds(per_cu, waves + 1); ++k) ++waves;
    const size_t lds = sorted_lds(shape->C, v.rpl, S * 64);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(shape->fn[qi]),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_error(e, "hipFuncSetAttribute");
    hipLaunchKernelGGL(shape->fn[qi], dim3(a.R * p->n_inst), dim3(64 * waves), lds, stream, sa);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "sorted_kernel launch");
    return OIM_OK;
}

// sched_stride: the row length of per-replica schedules ([R][sched_stride]),
// or 0 for one schedule shared by every replica.
int launch_variant(const Problem* p, const oim_run_cfg* cfg, const float* K, const float* Ks,
                   const float* sigma, const uint64_t* seeds, int64_t step0, float* theta,
                   uint32_t* phase, const oim_readout* ro, hipStream_t stream,
                   const Variant* forced, int32_t sched_stride) {
    const int S = p->max_slices;
    const Variant* v = forced ? forced : run_variant(p, cfg->q, cfg->readout_every, cfg->R);
    if (!v || !persistent_sparse_fits(p) || !variant_ok(p, *v))
        return set_error(OIM_E_UNSUPPORTED, "replica does not fit the LDS-resident kernel");
    PersistArgs a{};
    a.sell = reinterpret_cast<const int4*>(p->d_sell);
    a.row_split = p->d_row_split;
    a.desc = p->d_sell_desc;
    a.sell_bytes = (uint32_t)(p->sell_entries * 8);
    a.inst = p->d_inst;
    a.order = p->d_order;
    a.I = p->n_inst;
    a.n_total = p->n;
    const int plane = S * 64;
    a.q = cfg->q;
    a.steps = cfg->steps;
    a.M = cfg->readout_every;
    a.step0 = step0;
    a.dt = cfg->dt;
    a.K = K;
    a.Ks = Ks;
    a.sigma = sigma;
    a.seeds = seeds;
    a.theta = theta;
    a.phase = phase;
    a.trace = ro ? ro->trace : nullptr;
    a.best_h = ro ? ro->best_h : nullptr;
    a.best_step = ro ? ro->best_step : nullptr;
    a.best_colour = ro ? ro->best_colour : nullptr;
    a.R = cfg->R;
    a.sched_stride = sched_stride;
    const int qi = cfg->q == 2 ? 1 : cfg->q == 3 ? 2 : 0;
    if (!launch_holds(p, cfg->R, *v)) return set_error(OIM_E_ARG, "R * instances too large");
    a.w0 = p->uniform_w;
    if (on_sorted_rows(p, *v)) return launch_sorted(p, *v, a, qi, stream);
    KernelFn fn = v->fn[qi];
    if (p->d_sell_uw) {
        a.sell_uw = reinterpret_cast<const int4*>(p->d_sell_uw);
        a.sell_uw_bytes = (uint32_t)(p->sell_entries * 4);
        fn = kUniformKernels[v - kVariants][qi];
    }
    // the readout keeps per-slice sums in LDS when there is room for them
    const size_t lds_fast = lds_bytes(plane, v->tb, v->ms, v->rpl, v->covers());
    a.slice_sums = (a.M > 0 && lds_fast <= kLdsLimit) ? 1 : 0;
    const size_t lds = a.slice_sums ? lds_fast : lds_bytes(plane, v->tb, v->ms, v->rpl);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_error(e, "hipFuncSetAttribute");
    hipLaunchKernelGGL(fn, dim3(cfg->R * p->n_inst), dim3(v->tb), lds, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "persistent_sparse_kernel launch");
    return OIM_OK;
}
}  // namespace

int launch_persistent_sparse(const Problem* p, const oim_run_cfg* cfg, const float* K,
                             const float* Ks, const float* sigma, const uint64_t* seeds,
                             int64_t step0, float* theta, uint32_t* phase,
                             const oim_readout* ro, hipStream_t stream) {
    return launch_variant(p, cfg, K, Ks, sigma, seeds, step0, theta, phase, ro, stream, nullptr,
                          (cfg->flags & OIM_SCHED_PER_REPLICA) ? cfg->steps : 0);
}

// Autotuner: every variant whose waves cover the largest instance runs the
// first trial_steps steps of the caller's schedule on a scratch copy of
// theta (no readout), twice; the faster of the two timings (HIP events on the
// caller's stream) ranks it.  The four fastest then run three times on up to
// twice as many steps, and the smallest median wins.  The winner is recorded
// in the problem for this SHIL order.  Results do not depend on the variant:
// every oscillator's arithmetic is the same in all of them.
int tune_persistent(Problem* p, const oim_run_cfg* cfg, const float* K, const float* Ks,
                    const float* sigma, const uint64_t* seeds, const float* theta,
                    int32_t trial_steps, oim_tune_report* rep, hipStream_t stream) {
    if (!persistent_sparse_fits(p))
        return set_error(OIM_E_UNSUPPORTED, "replica does not fit the LDS-resident kernel");
    const size_t bytes = (size_t)cfg->R * p->n * sizeof(float);
    float* scratch = nullptr;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&scratch), bytes);
    if (e != hipSuccess) {
        return e == hipErrorOutOfMemory ? set_error(OIM_E_NOMEM, "autotune scratch: out of device memory")
                                        : hip_error(e, "autotune scratch");
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int st = OIM_OK;
    if ((e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess)
        st = hip_error(e, "autotune events");
    oim_run_cfg c = *cfg;
    c.readout_every = 0;
    // per-replica schedules keep the caller's row length while the trials
    // run a prefix of each row
    const int32_t stride = (cfg->flags & OIM_SCHED_PER_REPLICA) ? cfg->steps : 0;
    // times one variant `reps` times on `steps` steps of the schedule
    auto time_variant = [&](const Variant& v, int steps, int reps, float* out) {
        c.steps = steps;
        for (int rep_i = 0; rep_i < reps && !st; ++rep_i) {
            if ((e = hipMemcpyAsync(scratch, theta, bytes, hipMemcpyDeviceToDevice, stream)) != hipSuccess ||
                (e = hipEventRecord(e0, stream)) != hipSuccess) {
                st = hip_error(e, "autotune copy");
                break;
            }
            st = launch_variant(p, &c, K, Ks, sigma, seeds, 0, scratch, nullptr, nullptr, stream, &v,
                                stride);
            if (st) break;
            float ms = 0.f;
            if ((e = hipEventRecord(e1, stream)) != hipSuccess ||
                (e = hipEventSynchronize(e1)) != hipSuccess ||
                (e = hipEventElapsedTime(&ms, e0, e1)) != hipSuccess) {
                st = hip_error(e, "autotune timing");
                break;
            }
            out[rep_i] = ms;
        }
    };
    // first pass: every covering variant, best of two short trials
    constexpr int kFinalists = 4;
    const Variant* fin[kFinalists] = {};
    float fin_ms[kFinalists] = {};
    int tried = 0;
    for (const Variant& v : kVariants) {
        if (st) break;
        if (!variant_ok(p, v) || !launch_holds(p, cfg->R, v)) continue;
        float t[2] = {0.f, 0.f};
        time_variant(v, trial_steps, 2, t);
        if (st) break;
        const float t_min = t[0] < t[1] ? t[0] : t[1];
        if (rep && tried < OIM_TUNE_MAX) {
            rep->block[tried] = v.tb;
            rep->slices_per_wave[tried] = v.ms;
            rep->rows_per_lane[tried] = v.rpl;
            rep->ms[tried] = t_min;
        }
        ++tried;
        // keep the kFinalists fastest, sorted
        for (int f = 0; f < kFinalists; ++f) {
            if (!fin[f] || t_min < fin_ms[f]) {
                for (int g2 = kFinalists - 1; g2 > f; --g2) {
                    fin[g2] = fin[g2 - 1];
                    fin_ms[g2] = fin_ms[g2 - 1];
                }
                fin[f] = &v;
                fin_ms[f] = t_min;
                break;
            }
        }
    }
    // second pass: the finalists on trials twice as long (within the schedule),
    // three times each; the smallest median wins (short trials alone picked
    // variants up to 15 % apart from run to run on the 1024-graph batch)
    const Variant* best = nullptr;
    float best_ms = 0.f;
    const int final_steps = 2 * trial_steps < cfg->steps ? 2 * trial_steps : cfg->steps;
    for (int f = 0; f < kFinalists && fin[f] && !st; ++f) {
        float t[3] = {0.f, 0.f, 0.f};
        time_variant(*fin[f], final_steps, 3, t);
        if (st) break;
        const float lo = t[0] < t[1] ? t[0] : t[1], hi = t[0] < t[1] ? t[1] : t[0];
        const float med = t[2] < lo ? lo : (t[2] > hi ? hi : t[2]);
        if (!best || med < best_ms) {
            best = fin[f];
            best_ms = med;
        }
    }
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
    hipFree(scratch);
    if (st) return st;
    if (!best) return set_error(OIM_E_UNSUPPORTED, "no variant covers the largest instance");
    const int qc = q_class(cfg->q);
    p->tuned_tb[qc] = (int16_t)best->tb;
    p->tuned_ms[qc] = (int16_t)best->ms;
    p->tuned_rpl[qc] = (int16_t)best->rpl;
    if (rep) {
        rep->n_tried = tried < OIM_TUNE_MAX ? tried : OIM_TUNE_MAX;
        rep->chosen_block = best->tb;
        rep->chosen_slices_per_wave = best->ms;
        rep->chosen_rows_per_lane = best->rpl;
        rep->chosen_ms = best_ms;
    }
    return OIM_OK;
}

}  // namespace oim
