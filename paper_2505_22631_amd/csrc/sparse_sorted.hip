// sparse_sorted.hip -- the image of the sorted-rows kernel, and that kernel's
// instantiations for general weights.
#include "sorted_kernel.hpp"

namespace oim {
namespace persist {

#define OIM_SORTED_ENTRY(C, RPL)                                                         \
    {C, RPL,                                                                             \
     {sorted_kernel<C, RPL, 0, false>, sorted_kernel<C, RPL, 2, false>,                  \
      sorted_kernel<C, RPL, 3, false>}},

const SortedShape kSorted[kSortedCount] = {OIM_SORTED_SHAPES(OIM_SORTED_ENTRY)};

}  // namespace persist

namespace {

using persist::second_slot;

// The LDS serves an 8-byte read 32 lanes at a time from 32 pairs of banks, in as
// many passes as the most lanes that ask one pair for different entries: about
// 3.5 for random neighbours, 9.5 cycles per read of 64 lanes, against 5.2
// without conflicts and 6.5 with two lanes on each pair.  So the image of the
// split-row shapes points each entry at one of two copies: lane after lane of
// the 32 takes the less loaded of its two pairs, and twice more each takes the
// better one given all others.
__device__ void choose_copies(short* slots, int plane, unsigned char* load) {
    for (int b = 0; b < 32; ++b) load[b] = 0;
    for (int pass = 0; pass < 3; ++pass) {
        for (int l = 0; l < 32; ++l) {
            int s = slots[l];
            if (s < 0) continue;
            if (pass > 0) {  // off its present pair
                --load[s & 31];
                if (s >= 4 * plane) {  // (its own inverse)
                    s -= 4 * plane;
                    s ^= (s >> 5) & 31;
                }
            }
            const int s2 = second_slot(s, plane);
            const int to = load[s2 & 31] < load[s & 31] ? s2 : s;
            ++load[to & 31];
            slots[l] = (short)to;
        }
    }
}

// A workgroup per run, sixteen groups of its rows at a time: lane l of every
// wave takes row l.  Group d.y of a row is padding.
__global__ __launch_bounds__(256) void sorted_rows_kernel(const int64_t* row_ptr, const int32_t* col,
                                                          const float* J, const int4* inst,
                                                          const int2* run, const int32_t* osc,
                                                          const int32_t* inst_of, int uw, int2* row,
                                                          int4* entries, int4* entries2) {
    __shared__ short slots[16 * 4][64];
    __shared__ unsigned char load[16 * 4 * 2][36];
    const int4 id = inst[inst_of[blockIdx.x]];
    const int plane = id.y * 64, off = id.z, n = id.w;
    const int lane = threadIdx.x & 63;
    const int i = osc[blockIdx.x * 64 + lane];
    const int64_t rb = i < n ? row_ptr[off + i] : 0;
    const int len = i < n ? (int)(row_ptr[off + i + 1] - rb) : 0;
    const int2 d = run[blockIdx.x];
    const int per = uw ? 4 : 2;
    auto store = [&](int4* to, int h, int hh, int zero) {
        int at[4];
        float w[2] = {0.f, 0.f};
        for (int x = 0; x < per; ++x) {
            const int s = slots[hh * per + x][lane], e = h * per + x;
            at[x] = s < 0 ? zero : 8 * s;
            if (!uw && s >= 0) w[x] = J[rb + e];
        }
        to[((int64_t)d.x + h) * 64 + lane] =
            uw ? make_int4(at[0], at[1], at[2], at[3])
               : make_int4(at[0], __float_as_int(w[0]), at[1], __float_as_int(w[1]));
    };
    for (int h0 = 0; h0 <= d.y; h0 += 16) {
        const int count = d.y + 1 - h0 < 16 ? d.y + 1 - h0 : 16;
        for (int k = threadIdx.x >> 6; k < count * per; k += 4) {
            const int e = h0 * per + k;
            int s = -1;
            if (e < len) {
                const int c = col[rb + e] - off;
                s = (c & 3) * plane + (c >> 2);
            }
            slots[k][lane] = (short)s;
        }
        __syncthreads();
        for (int hh = threadIdx.x >> 6; hh < count; hh += 4) store(entries, h0 + hh, hh, 36 * plane);
        __syncthreads();
        if (entries2) {
            if ((int)threadIdx.x < count * per * 2)
                choose_copies(&slots[threadIdx.x >> 1][(threadIdx.x & 1) * 32], plane, load[threadIdx.x]);
            __syncthreads();
            for (int hh = threadIdx.x >> 6; hh < count; hh += 4)
                store(entries2, h0 + hh, hh, 2 * 36 * plane);
            __syncthreads();
        }
    }
    if (threadIdx.x < 64) {
        int up = 0, hi = len;  // columns ascend along a row
        while (up < hi) {
            const int mid = (up + hi) / 2;
            if (col[rb + mid] - off <= i) up = mid + 1;
            else hi = mid;
        }
        row[blockIdx.x * 64 + lane] = make_int2(i, up | len << 16);
    }
}

}  // namespace

int sorted_build(const Problem* p, int32_t runs) {
    hipLaunchKernelGGL(sorted_rows_kernel, dim3(runs), dim3(256), 0, 0, p->d_row_ptr, p->d_col, p->d_J,
                       p->d_inst, p->d_sorted_run, p->d_sorted_osc, p->d_sorted_inst,
                       p->d_sell_uw ? 1 : 0, p->d_sorted_row, p->d_sorted, p->d_sorted2);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? OIM_OK : hip_error(e, "sorted_rows_kernel launch");
}

}  // namespace oim
