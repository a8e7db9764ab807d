// The site-parallel dslash kernels on FP64 fields.
#include "dslash_site.h"

namespace ov {

template hipError_t launch_dslash<double2>(const DsArgs<double2> &, bool, bool, int, int, int, hipStream_t);

}  // namespace ov
