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

// A workgroup per run: lane l of every wave takes row l, wave k groups k,
// k + 4, ... of the row and, at the end, padding.
__global__ __launch_bounds__(256) void sorted_rows_kernel(const int64_t* row_ptr, const int32_t* col,
                                                          const float* J, const int4* inst,
                                                          const int2* run, const int32_t* osc,
                                                          const int32_t* inst_of, int uw, int2* row,
                                                          int4* entries) {
    const int4 id = inst[inst_of[blockIdx.x]];
    const int plane = id.y * 64, off = id.z, n = id.w;
    const int lane = threadIdx.x & 63;
    const int i = osc[blockIdx.x * 64 + lane];
    const int64_t rb = i < n ? row_ptr[off + i] : 0;
    const int len = i < n ? (int)(row_ptr[off + i + 1] - rb) : 0;
    const int2 d = run[blockIdx.x];
    const int zero = 36 * plane, per = uw ? 4 : 2;
    for (int h = threadIdx.x >> 6; h <= d.y; h += 4) {
        int at[4] = {zero, zero, zero, zero};
        float w[2] = {0.f, 0.f};
        for (int x = 0; x < per; ++x) {
            const int e = h * per + x;
            if (e >= len) continue;
            const int c = col[rb + e] - off;
            at[x] = 8 * ((c & 3) * plane + (c >> 2));
            if (!uw) w[x] = J[rb + e];
        }
        entries[((int64_t)d.x + h) * 64 + lane] =
            uw ? make_int4(at[0], at[1], at[2], at[3])
               : make_int4(at[0], __float_as_int(w[0]), at[1], __float_as_int(w[1]));
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
                       p->d_sell_uw ? 1 : 0, p->d_sorted_row, p->d_sorted);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? OIM_OK : hip_error(e, "sorted_rows_kernel launch");
}

}  // namespace oim
