// sparse_sorted_uw.hip -- the sorted-rows kernel's instantiations for uniform
// unit weights (see sparse_persistent_uw.hip).
#include "sorted_kernel.hpp"

namespace oim {
namespace persist {

#define OIM_SORTED_ENTRY(C, RPL)                                                         \
    {C, RPL,                                                                             \
     {sorted_kernel<C, RPL, 0, true>, sorted_kernel<C, RPL, 2, true>,                  \
      sorted_kernel<C, RPL, 3, true>}},

const SortedShape kSortedUniform[kSortedCount] = {OIM_SORTED_SHAPES(OIM_SORTED_ENTRY)};

}  // namespace persist
}  // namespace oim
