// readout.hip -- thresholding and objective readouts.
//
//   round      nearest stable phase k = floor(q theta / 2pi + 1/2) mod q, the
//              "phase threshold kernel" of Sec. III-B, FP32 decision
//   cut        max-cut value sum_{i<j} w_ij [k_i != k_j] with w = -J (Sec. II-C)
//   conflicts  colouring conflicts #{i<j : J_ij != 0, k_i == k_j}
//   energy     Eq. 1 (q = 2) or Eq. 2 (q >= 3) at the colours, and Eq. 6 with
//              w = -J at the continuous phases, FP64
//
// Every FP64 sum follows one fixed order, the same in every readout of the
// library: each row i sums its terms over j > i in ascending column order,
// from +0, and the row sums are combined by the pairwise tree over rows
// (zero-padded to a power of two, adjacent pairs first, the lower rows on the
// left).  A lane owns one row of a block of 64; the block's tree runs over
// lanes (xor butterfly, partner distance 1, 2, ..., 32), the blocks' sums meet
// in LDS and one wave folds them by the same tree.  Results that are whole
// numbers by definition (the int64 cut, the conflicts) are exact in any order.
#include <type_traits>

#include "dense_pairs.hpp"
#include "internal.hpp"
#include "phase.hpp"
#include "tree.hpp"

// products and sums of the readouts are rounded one by one, as written
#pragma clang fp contract(off)

namespace oim {

namespace {

__global__ __launch_bounds__(256) void round_kernel(int64_t count, const float* theta, int q,
                                                    float scale, int8_t* colour) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * blockDim.x) {
        const float th = theta[k];
        int8_t c = -1;
        if (__builtin_isfinite(th) && __builtin_fabsf(th) < 1048576.0f) {
            const int x = (int)__builtin_floorf(__builtin_fmaf(th, scale, 0.5f));
            int m = x % q;
            if (m < 0) m += q;
            c = (int8_t)m;
        }
        colour[k] = c;
    }
}

__global__ __launch_bounds__(256) void phase_convert_kernel(int64_t count, const float* theta_in,
                                                            uint32_t* phase_out,
                                                            const uint32_t* phase_in,
                                                            float* theta_out) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * blockDim.x) {
        if (theta_in) {
            const float th = theta_in[k];
            phase_out[k] = phase_from_theta(th);
        } else {
            theta_out[k] = theta_from_phase(phase_in[k]);
        }
    }
}

// ---- dense coupling (dense_pairs.hpp) ----

// Cut (kDiffer), conflicts (kCount) or Eq. 1 / Eq. 2 (kIsing / kSame) of
// colours [R][n] with the pair's weight -J; NR replicas per workgroup.
template <int NR, int KIND, bool INTS, int WAVES>
__global__ __launch_bounds__(dpair::kTB) void dense_pair_kernel(int n, int R, const float* J,
                                                                const int8_t* colour,
                                                                int64_t* out_i64, double* out_f64) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int ld = dpair::code_stride(n), nblk = dpair::row_blocks(n);
    double* bs = reinterpret_cast<double*>(smem + (size_t)NR * ld);
    int64_t* bi = reinterpret_cast<int64_t*>(bs + (size_t)NR * nblk);
    const int r0 = blockIdx.x * NR;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int8_t* k = colour + (int64_t)(r0 + r < R ? r0 + r : R - 1) * n;
        for (int j = threadIdx.x; j < ld; j += blockDim.x)
            smem[r * ld + j] = j < n ? (unsigned char)k[j] : 0;
    }
    __syncthreads();
    dpair::block_sums<NR, KIND, true, INTS, WAVES>(J, n, smem, bs, bi);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int r = threadIdx.x >> 6; r < NR && r0 + r < R; r += blockDim.x >> 6) {
        const double v = dpair::fold_blocks(bs + r * nblk, nblk);
        if (lane == 0 && out_f64) out_f64[r0 + r] = v;
        if constexpr (INTS) {
            const int64_t vi = dpair::fold_blocks_int(bi + r * nblk, nblk);
            if (lane == 0 && out_i64) out_i64[r0 + r] = vi;
        }
    }
}

// Eq. 6 at the continuous phases [R][n]: the same walk with one FP64 cosine
// per pair, which bounds it; one replica per workgroup.  KIND: Eq. 1 or Eq. 2 at
// the colours too, after it (in the cosines' own loop it cost more), or kNone.
constexpr int kNone = -1;

template <int KIND>
__global__ __launch_bounds__(dpair::kTB) void dense_energy_kernel(int n, const float* __restrict__ J,
                                                                  const float* __restrict__ theta,
                                                                  const int8_t* __restrict__ colour,
                                                                  double* h_eq6, double* h_model) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nblk = dpair::row_blocks(n), ld = dpair::code_stride(n), waves = blockDim.x >> 6;
    double* bs = reinterpret_cast<double*>(KIND != kNone ? smem + ld : smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float* th = theta + (int64_t)blockIdx.x * n;
    if constexpr (KIND != kNone) {
        const int8_t* k = colour + (int64_t)blockIdx.x * n;
        for (int j = threadIdx.x; j < ld; j += blockDim.x) smem[j] = j < n ? (unsigned char)k[j] : 0;
        __syncthreads();
    }
    for (int t = 0; t * waves < nblk; ++t) {
        const int blk = t * waves + ((t & 1) ? waves - 1 - wave : wave);
        if (blk >= nblk) continue;
        const int i = blk * 64 + lane, ic = i < n ? i : n - 1;
        const double ti = (double)th[ic];
        double acc = 0.0;
        for (int j = blk * 64 + 1; j < n; ++j) {
            const double c = cos(ti - (double)th[j]);
            const double term = -(double)J[(size_t)j * n + ic] * c;
            acc += j > i ? term : 0.0;
        }
        double v = i < n ? acc : 0.0;
        for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) bs[blk] = v;
    }
    if constexpr (KIND != kNone) dpair::block_sums<1, KIND, true, false, 0>(J, n, smem, bs + nblk, nullptr);
    __syncthreads();
    if (threadIdx.x < 64) {
        const double v = dpair::fold_blocks(bs, nblk);
        if (threadIdx.x == 0) h_eq6[blockIdx.x] = v;
        if constexpr (KIND != kNone) {
            const double vk = dpair::fold_blocks(bs + nblk, nblk);
            if (threadIdx.x == 0) h_model[blockIdx.x] = vk;
        }
    }
}

// ---- sparse coupling ----

// Upper-triangle entries of row i: fn(valid, gathered, w) for each, in column
// order.  BATCH 4: four at a time, so that their columns and weights, then what
// the caller gathers at those columns, are in flight together, for launches
// that leave the chip idle; with LPR lanes per row (whole-number sums only),
// lane `sub` of them takes every LPR-th group of four.  BATCH 1: one at a time,
// gathering for the upper entries alone, for launches that fill it.
template <int LPR, int BATCH, class Gather, class Fn>
__device__ __forceinline__ void upper_entries(const int64_t* __restrict__ row_ptr,
                                              const int32_t* __restrict__ col,
                                              const float* __restrict__ J, int i, int sub,
                                              Gather gather, Fn fn) {
    const int64_t e1 = row_ptr[i + 1];
    if constexpr (BATCH == 1) {
        for (int64_t e = row_ptr[i]; e < e1; ++e) {
            const int j = col[e];
            if (j > i) fn(true, gather(j), J[e]);
        }
        return;
    }
    for (int64_t e = row_ptr[i] + 4 * sub; e < e1; e += 4 * LPR) {
        int j[4];
        float w[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int64_t ee = e + x < e1 ? e + x : e1 - 1;
            j[x] = col[ee];
            w[x] = J[ee];
        }
        decltype(gather(0)) g[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) g[x] = gather(j[x]);
#pragma unroll
        for (int x = 0; x < 4; ++x) fn(e + x < e1 && j[x] > i, g[x], w[x]);
    }
}

// Whole-number results alone: the cut of integer weights (CUT) or the
// conflicts.  LPR lanes share a row, and the rows of a replica are split over
// gridDim.x workgroups whose sums meet in out (zeroed before, unless one
// workgroup holds all rows) by integer atomics.  One workgroup per replica,
// a lane per row, left the chip idle for few replicas of a large graph: the
// conflicts of 256 colouring graphs (86 928 oscillators) x 8 replicas took
// 1642 us, now 42; the cut of a 200 x 300 torus x 64 replicas 549, now 38; of
// G(800, 0.06) x 1 replica 79, now 5 (and 5 for the zeroing).
__global__ void zero_kernel(int R, int64_t* out) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < R) out[r] = 0;
}

template <bool CUT, int LPR, int BATCH>
__global__ __launch_bounds__(1024) void sparse_int_kernel(
    int n, int rows, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
    const float* __restrict__ J, const int8_t* __restrict__ colour, int64_t* out) {
    __shared__ int64_t red[16];
    const int r = blockIdx.y;
    const int8_t* k = colour + (int64_t)r * n;
    int64_t acc = 0;
    const int64_t i0 = (int64_t)blockIdx.x * rows;
    const int64_t i1 = i0 + rows < n ? i0 + rows : n;
    for (int64_t i = i0 + threadIdx.x / LPR; i < i1; i += blockDim.x / LPR) {
        const int ki = k[i];
        upper_entries<LPR, BATCH>(row_ptr, col, J, (int)i, threadIdx.x % LPR,
                           [&](int j) { return (int)k[j]; },
                           [&](bool on, int kj, float w) {
                               if (CUT) acc += on && ki != kj ? (int64_t)(-w) : 0;
                               else acc += on && w != 0.0f && ki == kj ? 1 : 0;
                           });
    }
    for (int o = 1; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t tot = 0;
        for (int w = 0; w < (int)blockDim.x / 64; ++w) tot += red[w];
        if (gridDim.x == 1) out[r] = tot;
        else atomicAdd(reinterpret_cast<unsigned long long*>(out + r), (unsigned long long)tot);
    }
}

// FP64 results: one workgroup of 1 to 16 waves per replica.  A wave takes every
// so manieth block of 64 rows, one row per lane, without a barrier; the block sums
// of a round of kRoundBlocks blocks meet in LDS, where a wave folds each
// result's by the pairwise tree, and the rounds (a power of two of rows
// each) are folded in order.  STAGE: the replica's colours and phases are
// copied to LDS first, so a neighbour's value is an LDS read.  Bound by the
// latency of the row bounds and entries (and, for Eq. 6, the FP64 cosines).
// 100 x 100 torus, real weights, 64 replicas: cut 73 -> 25 us, both energies
// 130 -> 42 us against four waves with two to four barriers per 256 rows.  For
// many replicas a workgroup of sixteen waves was far too much (n = 10, 20000
// replicas, both energies 64 -> 288 us; n = 800 of degree 48, 1000 replicas,
// Eq. 1 123 -> 281): their waves follow from the replicas and the rows, and
// full chips take the entries one by one (41 and 110 us).
constexpr int kSumTB = 1024;
constexpr int kSumWaves = kSumTB / 64;
constexpr int kRoundBlocks = 1024;

struct Gathered {
    int k;
    float th;
};

// MODE 0: cut (FP64 and, when out_i64, int64), 2: energies.  WAVES: the waves of
// a workgroup, 0 as launched (the constant: 100 x 100 torus, real weights, 64
// replicas, cut 25.1 -> 24.8 us).
template <int MODE, bool STAGE, int BATCH, int WAVES>
__global__ __launch_bounds__(kSumTB) void sparse_sum_kernel(
    int n, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
    const float* __restrict__ J, const int8_t* __restrict__ colour,
    const float* __restrict__ theta, int q, int64_t* out_i64, double* out_a, double* out_b) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double stack[2][TreeAcc::kLevels];
    const int nblk = (n + 63) / 64;
    const int room = nblk < kRoundBlocks ? nblk : kRoundBlocks;
    double* const bs[2] = {reinterpret_cast<double*>(smem), reinterpret_cast<double*>(smem) + room};
    const int waves = WAVES ? WAVES : blockDim.x >> 6;  // MODE 0: at most nblk
    const int r = blockIdx.x;
    const int8_t* k = colour ? colour + (int64_t)r * n : nullptr;
    const float* th = theta ? theta + (int64_t)r * n : nullptr;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool want_a = out_a != nullptr, want_b = MODE == 2 && out_b != nullptr;
    const bool want_i = MODE == 0 && out_i64 != nullptr;
    float* th_lds = reinterpret_cast<float*>(bs[1] + (MODE == 2 ? room : 0));
    int8_t* k_lds = reinterpret_cast<int8_t*>(th_lds + (th ? n : 0));
    if constexpr (STAGE) {
        for (int i = threadIdx.x; i < n; i += 64 * waves) {
            if (th) th_lds[i] = th[i];
            if (k) k_lds[i] = k[i];
        }
        __syncthreads();
    }
    auto gather = [&](int j) __attribute__((always_inline)) {
        Gathered g{0, 0.f};
        if constexpr (STAGE) {
            if (k) g.k = k_lds[j];
            if (th) g.th = th_lds[j];
        } else {
            if (k) g.k = k[j];
            if (th) g.th = th[j];
        }
        return g;
    };
    TreeAcc tree_a(stack[0]), tree_b(stack[1]);
    const int wave_b = waves > 1 ? 1 : 0;  // the one that folds the second result
    int64_t tot_i = 0;
    for (int b0 = 0; b0 < nblk; b0 += kRoundBlocks) {
        const int nb = nblk - b0 < kRoundBlocks ? nblk - b0 : kRoundBlocks;
        for (int b = wave; b < nb; b += waves) {
            const int i = (b0 + b) * 64 + lane;
            int64_t acc_i = 0;
            double acc_a = 0.0, acc_b = 0.0;
            if (i < n) {
                const Gathered own = gather(i);
                const double ti = (double)own.th;
                upper_entries<1, BATCH>(row_ptr, col, J, i, 0, gather, [&](bool on, Gathered g, float w) {
                    if (!on) return;
                    if (MODE == 0) {
                        if (own.k != g.k) {
                            acc_i += (int64_t)(-w);
                            acc_a += -(double)w;
                        }
                    } else {
                        if (k) {
                            if (q == 2) acc_a += (own.k == g.k) ? -(double)w : (double)w;
                            else if (own.k == g.k) acc_a += -(double)w;
                        }
                        if (th) {
                            const double c = cos(ti - (double)g.th);
                            const double term = -(double)w * c;
                            acc_b += term;
                        }
                    }
                });
            }
            if (MODE == 0 && want_i) {
                for (int o = 1; o < 64; o <<= 1) acc_i += __shfl_xor(acc_i, o, 64);
                tot_i += acc_i;
            }
            if (want_a) {
                for (int o = 1; o < 64; o <<= 1) acc_a += __shfl_xor(acc_a, o, 64);
                if (lane == 0) bs[0][b] = acc_a;
            }
            if (want_b) {
                for (int o = 1; o < 64; o <<= 1) acc_b += __shfl_xor(acc_b, o, 64);
                if (lane == 0) bs[1][b] = acc_b;
            }
        }
        __syncthreads();
        if (wave == 0 && want_a) {
            const double v = dpair::fold_blocks(bs[0], nb);
            if (lane == 0) tree_a.push(v);
        }
        if (wave == wave_b && want_b) {
            const double v = dpair::fold_blocks(bs[1], nb);
            if (lane == 0) tree_b.push(v);
        }
        __syncthreads();
    }
    if (wave == 0 && lane == 0 && want_a) out_a[r] = tree_a.finish();
    if (wave == wave_b && lane == 0 && want_b) out_b[r] = tree_b.finish();
    if (MODE == 0 && want_i) {
        int64_t* ti = reinterpret_cast<int64_t*>(bs[0]);
        if (lane == 0) ti[wave] = tot_i;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t t = 0;
            for (int w = 0; w < waves; ++w) t += ti[w];
            out_i64[r] = t;
        }
    }
}

int launched(const char* what) {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? OIM_OK : hip_error(e, what);
}

// More than 64 KiB of LDS has to be asked for: the dynamic part, which with
// the kernel's static arrays may not pass the CU's 160 KiB.
int allow_lds(const void* fn, size_t bytes, size_t fixed = 0) {
    if (bytes + fixed <= 64 * 1024) return OIM_OK;
    const hipError_t e =
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    return e == hipSuccess ? OIM_OK : hip_error(e, "hipFuncSetAttribute");
}

// Workgroups of 1024 threads in one launch: a grid dimension ends at 2^32
// threads, past which the launch wraps without an error, so more replicas go
// in several launches.
constexpr int64_t kMaxGroups = (int64_t)1 << 21;

template <typename T>
T* offset(T* p, int64_t k) {
    return p ? p + k : nullptr;
}

template <int KIND, bool INTS>
int launch_dense_pairs(const Problem* p, int R, const int8_t* colour, int64_t* oi, double* of,
                       hipStream_t s) {
    // (sixteen waves as a constant: the cut of n = 6000 took 1550 us with their
    // number read, 1390 so)
    const int waves = dpair::group_waves(p->n);
    const int nr = dpair::replicas_per_group(p->n, R, INTS, waves);
    const size_t lds = dpair::lds_bytes(p->n, nr, INTS);
    auto pick = [&](auto w) {
        constexpr int W = decltype(w)::value;
        return nr == 4   ? dense_pair_kernel<4, KIND, INTS, W>
               : nr == 2 ? dense_pair_kernel<2, KIND, INTS, W>
                         : dense_pair_kernel<1, KIND, INTS, W>;
    };
    auto fn = waves == dpair::kWaves ? pick(std::integral_constant<int, dpair::kWaves>{})
                                     : pick(std::integral_constant<int, 0>{});
    if (int st = allow_lds(reinterpret_cast<const void*>(fn), lds)) return st;
    for (int64_t r0 = 0; r0 < R; r0 += nr * kMaxGroups) {
        const int count = (int)(R - r0 < nr * kMaxGroups ? R - r0 : nr * kMaxGroups);
        hipLaunchKernelGGL(fn, dim3((count + nr - 1) / nr), dim3(64 * waves), lds, s, p->n, count,
                           p->d_Jdense, colour + r0 * p->n, offset(oi, r0), offset(of, r0));
    }
    return launched("readout launch");
}

// The smallest power of two from `lo` on that is at least x, at most 1024.
int pow2_from(int lo, int64_t x) {
    while (lo < x && lo < 1024) lo *= 2;
    return lo;
}

template <bool CUT>
int launch_sparse_int(const Problem* p, int R, const int8_t* colour, int64_t* out, hipStream_t s) {
    // lanes per row: about one group of four entries each at the mean degree
    const int64_t n = p->n, deg = p->nnz / n;
    int lpr = deg > 32 ? 16 : deg > 8 ? 4 : 1;
    // A replica of at most 6 passes of 1024 threads stays in one workgroup,
    // which saves the zeroing launch (about 5 us; a pass is latency, 1 to 2
    // us).  Beyond, workgroups of 256 threads take one pass each while that
    // gives at most 2048 of them (eight per CU), else more.
    int tb = 1024, chunks = 1, batch = 4;
    int64_t rows = n;
    if (deg > 14 && R >= 256) {
        // Longer rows, replicas that nearly fill the chip: four lanes per row, a
        // workgroup each for up to two per CU and from 1000; a lane per row and its upper
        // entries alone while 1024 threads per CU hold all replicas (us with
        // sixteen lanes split over workgroups, four lanes, one: n = 698 of degree
        // 71, 300 replicas 64, 46, 120; 2000 294, 243, 202; 9000 1303, 1076, 1420;
        // n = 2031 of degree 22, 1000 replicas 161, 111, 113).
        lpr = 4;
        if (R >= 1536 && R <= 6144) {
            lpr = batch = 1;
            tb = pow2_from(64, (256 << 10) / R / 2 + 1);
        } else if (R > 6144 && deg <= 18) {
            lpr = batch = 1;
            tb = 256;
        } else if (n <= 64) {
            tb = 256;
        } else if (n > 256 && R < 1000 && !(R > 384 && R <= 512)) {
            tb = 256;
            const int64_t passes = (n + 63) / 64;
            int64_t per_group = passes * R / 4096;
            per_group = per_group < 1 ? 1 : per_group > 4 ? 4 : per_group;
            chunks = (int)((passes + per_group - 1) / per_group);
            rows = per_group * 64;
        }
    } else if (R >= (deg > 8 ? 512 : 256) && deg <= 14 && n * R >= (256 << 10)) {
        // Replicas that fill the chip: a workgroup each, a lane per row, upper
        // entries alone, threads enough for 1024 per CU and 20 passes (us in
        // groups of four split over workgroups, and so: n = 200 of degree 10,
        // 4000 replicas 29 and 21; n = 3000 of degree 8, 300 replicas 39 and 28,
        // 4000 284 and 203; n = 60000 of degree 4, 2000 replicas 6630 and 1630);
        // groups of four where 1024 rows' entries pass the L1 (n = 25000 of
        // degree 12, 2000 replicas 2290 one by one, 1720).
        tb = pow2_from(64, (256 << 10) / R);
        tb = pow2_from(tb, n / 20);
        if (n < tb) tb = pow2_from(64, n);
        if (tb < 1024 || n <= 8192 || deg <= 8) lpr = batch = 1;
    } else if (n * lpr > 6 * 1024) {
        tb = 256;
        const int64_t per_pass = tb / lpr;
        const int64_t passes = (n + per_pass - 1) / per_pass;
        const int64_t per_group = passes * R / 2048 > 1 ? passes * R / 2048 : 1;
        chunks = (int)((passes + per_group - 1) / per_group);
        rows = per_group * per_pass;
    } else if (n * lpr <= 256) {
        tb = 256;
    }
    auto fn = batch == 1  ? sparse_int_kernel<CUT, 1, 1>
              : lpr == 16 ? sparse_int_kernel<CUT, 16, 4>
              : lpr == 4  ? sparse_int_kernel<CUT, 4, 4>
                          : sparse_int_kernel<CUT, 1, 4>;
    for (int64_t r0 = 0; r0 < R; r0 += 65535) {  // grid.y limit
        const int nr = (int)(R - r0 < 65535 ? R - r0 : 65535);
        if (chunks > 1)
            hipLaunchKernelGGL(zero_kernel, dim3((nr + 255) / 256), dim3(256), 0, s, nr, out + r0);
        hipLaunchKernelGGL(fn, dim3(chunks, nr), dim3(tb), 0, s, p->n, (int)rows, p->d_row_ptr,
                           p->d_col, p->d_J, colour + r0 * p->n, out + r0);
    }
    return launched("readout launch");
}

template <int MODE>
int launch_sparse_sum(const Problem* p, int R, const int8_t* colour, const float* theta, int q,
                      int64_t* oi, double* oa, double* ob, hipStream_t s) {
    // block sums and, where they fit beside them, the staged copies
    constexpr size_t kFixed = 2 * 1024;
    const int nblk = (p->n + 63) / 64;
    const size_t sums = (size_t)(nblk < kRoundBlocks ? nblk : kRoundBlocks) * 8 * (MODE == 2 ? 2 : 1);
    const size_t copies = (size_t)p->n * ((theta ? 4 : 0) + (colour ? 1 : 0));
    const bool stage = copies + sums + kFixed <= dpair::kLdsLimit;
    const size_t lds = sums + (stage ? copies : 0);
    // Waves per replica: about 12288 in all (16384 with cosines), sixteen at most;
    // where rows are long, whose lines the waves of a CU take from each other's
    // L1, few (us: n = 1500 of degree 40, cut, 500 replicas 99 with three, 118 with
    // four; 1500 182 with three, 226 with one; 3000 262 with two, 369 with one; n =
    // 500, both energies, 500 replicas 59 with four, 70 with eight); enough for 32
    // per CU beside the copies.
    const int64_t deg = p->nnz / p->n;
    const bool long_rows = deg >= 24;
    auto within = [](int64_t v, int lo, int hi) { return (int)(v < lo ? lo : v > hi ? hi : v); };
    int waves = 1;
    if (long_rows) {
        waves = R > 6000   ? 1
                : R > 1920 ? 2
                : R >= 700 ? 3
                : R < 64   ? kSumWaves
                : theta    ? within(2048 / R, 4, nblk <= 32 ? 8 : kSumWaves)
                           : within(800 / R, 3, 8);
        while (waves < kSumWaves && waves * 5120 < (int64_t)(copies + sums)) ++waves;
    } else {
        const int64_t share = (theta && R >= 2048 ? 16384 : 12288) / R;
        while (waves < kSumWaves && (2 * waves <= share || waves * 5120 < (int64_t)(copies + sums)))
            waves *= 2;
    }
    // no more than there are blocks of rows, but one for each result (n = 25, 88
    // replicas, both energies 14.4 us with one wave, 13.0 with two)
    if (waves > nblk) waves = oa && ob && nblk == 1 && R <= 4096 ? 2 : nblk;
    // Entries one by one once the waves fill the chip (not with short rows
    // whose lines then pass the L1, nor for colours alone with the shortest).
    const int64_t total = (int64_t)R * waves;
    const bool one = long_rows ? total >= 2048
                               : (MODE == 0 || theta || deg >= 16) && total >= 4000 && waves * deg <= 60;
    auto fn = stage ? (one                  ? sparse_sum_kernel<MODE, true, 1, 0>
                       : waves == kSumWaves ? sparse_sum_kernel<MODE, true, 4, kSumWaves>
                                            : sparse_sum_kernel<MODE, true, 4, 0>)
                    : (one                  ? sparse_sum_kernel<MODE, false, 1, 0>
                       : waves == kSumWaves ? sparse_sum_kernel<MODE, false, 4, kSumWaves>
                                            : sparse_sum_kernel<MODE, false, 4, 0>);
    if (int st = allow_lds(reinterpret_cast<const void*>(fn), lds, kFixed)) return st;
    for (int64_t r0 = 0; r0 < R; r0 += kMaxGroups) {
        const int count = (int)(R - r0 < kMaxGroups ? R - r0 : kMaxGroups);
        hipLaunchKernelGGL(fn, dim3(count), dim3(64 * waves), lds, s, p->n, p->d_row_ptr, p->d_col, p->d_J,
                           offset(colour, r0 * p->n), offset(theta, r0 * p->n), q, offset(oi, r0),
                           offset(oa, r0), offset(ob, r0));
    }
    return launched("readout launch");
}

}  // namespace

int launch_round(int32_t q, int64_t count, const float* theta, int8_t* colour, hipStream_t s) {
    if (count == 0) return OIM_OK;
    const float scale = (float)((double)q / 6.283185307179586476925286766559);
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(round_kernel, dim3((unsigned)blocks), dim3(256), 0, s, count, theta, q,
                       scale, colour);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "round launch");
    return OIM_OK;
}

int launch_phase_convert(int64_t count, const float* theta_in, uint32_t* phase_out,
                         const uint32_t* phase_in, float* theta_out, hipStream_t s) {
    if (count == 0) return OIM_OK;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(phase_convert_kernel, dim3((unsigned)blocks), dim3(256), 0, s, count,
                       theta_in, phase_out, phase_in, theta_out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "phase conversion launch");
    return OIM_OK;
}

int launch_cut(const Problem* p, int32_t R, const int8_t* colour, int64_t* cut_i64,
               double* cut_f64, hipStream_t s) {
    if (p->dense)
        return cut_i64 ? launch_dense_pairs<dpair::kDiffer, true>(p, R, colour, cut_i64, cut_f64, s)
                       : launch_dense_pairs<dpair::kDiffer, false>(p, R, colour, nullptr, cut_f64, s);
    if (!cut_f64) return launch_sparse_int<true>(p, R, colour, cut_i64, s);
    return launch_sparse_sum<0>(p, R, colour, nullptr, 2, cut_i64, cut_f64, nullptr, s);
}

int launch_conflicts(const Problem* p, int32_t R, const int8_t* colour, int64_t* conflicts,
                     hipStream_t s) {
    if (p->dense) return launch_dense_pairs<dpair::kCount, true>(p, R, colour, conflicts, nullptr, s);
    return launch_sparse_int<false>(p, R, colour, conflicts, s);
}

int launch_energy(const Problem* p, int32_t q, int32_t R, const float* theta,
                  const int8_t* colour, double* h_model, double* h_eq6, hipStream_t s) {
    if (!p->dense)
        return launch_sparse_sum<2>(p, R, h_model ? colour : nullptr, h_eq6 ? theta : nullptr, q,
                                    nullptr, h_model, h_eq6, s);
    // Waves: as many for each SIMD, two where the chip is full without more (n =
    // 621, 1330 replicas, Eq. 6: 655 us with eight, 685 with twelve, 816 with ten,
    // one per block of rows; n = 400, 3000 replicas: 572 with eight, 670 with
    // seven; n = 960, 3000: 2855 with twelve, 3248 with fifteen).
    const int nblk = dpair::row_blocks(p->n);
    const int waves = nblk <= 2                ? nblk
                      : nblk <= 4              ? 4
                      : nblk <= 8              ? 8
                      : nblk <= 11 && R > 256  ? 8
                      : nblk < dpair::kWaves   ? 12
                                               : dpair::kWaves;
    // Both in one launch (us in two and in one: n = 10, 32 replicas 14.2 and
    // 11.5; n = 500 161 and 156; n = 814, 1330 replicas 1213 and 1182), not where
    // the pair sums of many replicas share columns (n = 500, 3000 replicas 910
    // and 952) or the cosines alone take fewer registers (sixteen waves: n = 2000,
    // 1500 replicas 6840 and 8400).
    const bool both = h_model && h_eq6 &&
                      (R <= 256 || (waves < dpair::kWaves && (R <= 1000 || nblk <= 2 || nblk > 8)));
    if (h_model && !both) {
        const int st = q == 2
                           ? launch_dense_pairs<dpair::kIsing, false>(p, R, colour, nullptr, h_model, s)
                           : launch_dense_pairs<dpair::kSame, false>(p, R, colour, nullptr, h_model, s);
        if (st) return st;
    }
    if (h_eq6) {
        auto fn = !both    ? dense_energy_kernel<kNone>
                  : q == 2 ? dense_energy_kernel<dpair::kIsing>
                           : dense_energy_kernel<dpair::kSame>;
        const size_t sums = sizeof(double) * dpair::row_blocks(p->n);
        const size_t lds = both ? dpair::code_stride(p->n) + 2 * sums : sums;
        if (int st = allow_lds(reinterpret_cast<const void*>(fn), lds)) return st;
        for (int64_t r0 = 0; r0 < R; r0 += kMaxGroups) {
            const int count = (int)(R - r0 < kMaxGroups ? R - r0 : kMaxGroups);
            hipLaunchKernelGGL(fn, dim3(count), dim3(64 * waves), lds, s, p->n,
                               p->d_Jdense, theta + r0 * p->n, offset(colour, r0 * p->n), h_eq6 + r0,
                               offset(h_model, r0));
        }
        return launched("readout launch");
    }
    return OIM_OK;
}

}  // namespace oim
