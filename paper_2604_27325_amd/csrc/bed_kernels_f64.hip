// bed_kernels_f64.hip -- binary64 instantiations of the n <= 64 solver's kernels.
#include "bed_kernels.hpp"

namespace bed {

BED_KERNELS_OF(, double)

}  // namespace bed
