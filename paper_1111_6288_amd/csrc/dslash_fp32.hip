// The site-parallel dslash kernels on FP32 fields.
#include "dslash_site.h"

namespace ov {

template hipError_t launch_dslash<float2>(const DsArgs<float2> &, bool, bool, int, int, int, hipStream_t);

}  // namespace ov
