// sparse_sorted.hip -- the sorted-rows kernel's instantiations for general
// weights.
#include "sorted_kernel.hpp"

namespace oim {
namespace persist {

#define OIM_SORTED_ENTRY(C, RPL)                                                         \
    {C, RPL,                                                                             \
     {sorted_kernel<C, RPL, 0, false>, sorted_kernel<C, RPL, 2, false>,                  \
      sorted_kernel<C, RPL, 3, false>}},

const SortedShape kSorted[kSortedCount] = {OIM_SORTED_SHAPES(OIM_SORTED_ENTRY)};

}  // namespace persist
}  // namespace oim
