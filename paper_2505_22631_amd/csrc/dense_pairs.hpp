// dense_pairs.hpp -- FP64 sums over the pairs i < j of a dense coupling, in
// the library's fixed order, for the in-run readout of the dense loop
// (dense.hip) and the standalone readouts (readout.hip).
//
// Order: row i sums its terms over j > i in ascending j, from +0; the row
// sums are combined by the pairwise tree over rows (zero-padded to a power of
// two).  A term that does not count adds +0, which leaves a partial sum as it
// is (no partial sum is -0).
//
// One workgroup of up to 16 waves takes NR replicas.  A wave owns a block of 64
// rows, one per lane, and walks the columns upwards: J is symmetric bit for
// bit (checked at upload), so the 64 rows' entries of column j are the 256
// contiguous bytes J[j][i0 .. i0 + 63], one coalesced load shared by the NR
// replicas, and 16 columns are loaded before the first is used.  (A thread
// per row reading along its own row, 64 cache lines per load, is what this
// replaces.)  The replicas' colours sit in LDS, one byte
// per oscillator, read 16 columns at a time at a wave-uniform address.  The
// blocks are dealt to the waves longest first, back and forth, since block b
// has n - 64 b columns.  Bound by the vector instructions (a conversion per
// column, and per term a compare, a select and an FP64 add: requesting the
// next 16 columns ahead of the current ones changed nothing).  Eq. 1, before
// (that thread per row, one workgroup of 256 per replica) and now: n = 4096,
// 512 replicas 15 963 -> 840 us; n = 2000, 128 replicas 3535 -> 164 us;
// n = 777, 24 replicas 406 -> 34 us.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace oim {
namespace dpair {

constexpr int kTB = 1024;            // threads per workgroup
constexpr int kWaves = kTB / 64;
constexpr int kCols = 16;            // columns per iteration
constexpr size_t kLdsLimit = 160 * 1024;

// What a pair adds: weight v of the pair when its colours are equal / differ.
enum Kind {
    kIsing,     // equal: v, differ: -v        (Eq. 1)
    kSame,      // equal: v, differ: 0         (Eq. 2)
    kDiffer,    // equal: 0, differ: v         (cut)
    kCount      // equal and v != 0: 1         (conflicts)
};

__host__ __device__ constexpr int code_stride(int n) { return (n + 63) / 64 * 64; }
__host__ __device__ constexpr int row_blocks(int n) { return (n + 63) / 64; }

// LDS: colours [NR][code_stride], then block sums FP64 [NR][row_blocks] and,
// for the exact integer result, int64 [NR][row_blocks].
inline size_t lds_bytes(int n, int nr, bool ints) {
    return (size_t)nr * code_stride(n) + (size_t)nr * row_blocks(n) * (ints ? 16 : 8);
}

// Waves of a workgroup: as many as there are row blocks, sixteen at most.
inline int group_waves(int n) { return row_blocks(n) < kWaves ? row_blocks(n) : kWaves; }

// Replicas per workgroup of `waves` waves: sharing a column load and its
// conversion among replicas pays once the chip is full without it (64 waves per
// CU for four: n = 100, 1500 replicas 12.5, 10.7 and 16.5 us with 1, 2 and 4;
// 20000 replicas 87, 53, 45) and the colours of two workgroups fit the LDS.
inline int replicas_per_group(int n, int R, bool ints, int waves = kWaves) {
    const int64_t total = (int64_t)R * waves;
    if (total > 16384 && 2 * lds_bytes(n, 4, ints) <= kLdsLimit) return 4;
    if (R > 256 && total > 2048 && 2 * lds_bytes(n, 2, ints) <= kLdsLimit) return 2;
    return 1;
}

// The term of one column: `w` the (signed) weight as FP64.
template <int KIND>
__device__ __forceinline__ double term(bool same, double w) {
    if constexpr (KIND == kIsing) {
        // the sign bit alone
        const uint64_t b = __builtin_bit_cast(uint64_t, w);
        const uint32_t hi = (uint32_t)(b >> 32);
        const uint32_t h2 = same ? hi : hi ^ 0x80000000u;
        return __builtin_bit_cast(double, ((uint64_t)h2 << 32) | (uint32_t)b);
    } else if constexpr (KIND == kSame) {
        return same ? w : 0.0;
    } else if constexpr (KIND == kDiffer) {
        return same ? 0.0 : w;
    } else {
        return same && w != 0.0 ? 1.0 : 0.0;
    }
}

// Block sums of the workgroup's NR replicas into LDS: bs[r][block], and with
// INTS the same as int64 (every row sum is then an exact integer).  NEG: the
// pair's weight is -J instead of J.  `code` as staged by the caller (and
// published by a barrier); ends without one.  WAVES 0: as many as were launched.
template <int NR, int KIND, bool NEG, bool INTS, int WAVES = kWaves>
__device__ __forceinline__ void block_sums(const float* __restrict__ J, int n,
                                           const unsigned char* code, double* bs, int64_t* bi) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nblk = row_blocks(n), ld = code_stride(n);
    const int waves = WAVES ? WAVES : (int)blockDim.x >> 6;
    for (int t = 0; t * waves < nblk; ++t) {
        const int blk = t * waves + ((t & 1) ? waves - 1 - wave : wave);
        if (blk >= nblk) continue;
        const int i = blk * 64 + lane;
        const float* col = J + (i < n ? i : n - 1);
        uint32_t ci[NR];
        double acc[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            ci[r] = code[r * ld + i];
            acc[r] = 0.0;
        }
        // columns j0 .. j0 + 15; EDGE: those with j <= i or j >= n add nothing
        auto columns = [&](int j0, auto edge) __attribute__((always_inline)) {
            constexpr bool EDGE = decltype(edge)::value;
            float w[kCols];
#pragma unroll
            for (int x = 0; x < kCols; ++x) {
                const int j = EDGE && j0 + x >= n ? n - 1 : j0 + x;
                w[x] = col[(size_t)j * n];
            }
            uint4 cj[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) cj[r] = *reinterpret_cast<const uint4*>(code + r * ld + j0);
#pragma unroll
            for (int x = 0; x < kCols; ++x) {
                const double wd = NEG ? -(double)w[x] : (double)w[x];
                const bool on = !EDGE || (j0 + x > i && j0 + x < n);
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const uint32_t c4 = x < 4 ? cj[r].x : x < 8 ? cj[r].y : x < 12 ? cj[r].z : cj[r].w;
                    const bool same = ((c4 >> (8 * (x & 3))) & 0xffu) == ci[r];
                    const double v = term<KIND>(same, wd);
                    acc[r] += EDGE ? (on ? v : 0.0) : v;
                }
            }
        };
        int j0 = blk * 64;
        for (; j0 < n && j0 < blk * 64 + 64; j0 += kCols) columns(j0, std::true_type{});
        for (; j0 + kCols <= n; j0 += kCols) columns(j0, std::false_type{});
        if (j0 < n) columns(j0, std::true_type{});
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            double v = i < n ? acc[r] : 0.0;
            if constexpr (INTS) {
                int64_t vi = (int64_t)v;
                for (int o = 1; o < 64; o <<= 1) vi += __shfl_xor(vi, o, 64);
                if (lane == 0) bi[r * nblk + blk] = vi;
            }
            for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
            if (lane == 0) bs[r * nblk + blk] = v;
        }
    }
}

// One wave folds nblk <= 1024 block sums by the pairwise tree (zero-padded);
// the result is in lane 0.
__device__ __forceinline__ double fold_blocks(const double* bs, int nblk) {
    const int lane = threadIdx.x & 63;
    int per = 1;  // values per lane
    while (per * 64 < nblk) per <<= 1;
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int b = lane * per + k;
        v[k] = k < per && b < nblk ? bs[b] : 0.0;
    }
#pragma unroll
    for (int len = 16; len > 1; len >>= 1)
#pragma unroll
        for (int k = 0; k < len / 2; ++k) v[k] = v[2 * k] + v[2 * k + 1];
    for (int o = 1; o < 64; o <<= 1) v[0] += __shfl_xor(v[0], o, 64);
    return v[0];
}

__device__ __forceinline__ int64_t fold_blocks_int(const int64_t* bi, int nblk) {
    int64_t v = 0;
    for (int b = threadIdx.x & 63; b < nblk; b += 64) v += bi[b];
    for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}

}  // namespace dpair
}  // namespace oim
