// The site-parallel dslash kernels on BF16 fields.
#include "dslash_site.h"

namespace ov {

template hipError_t launch_dslash<uint32_t>(const DsArgs<uint32_t> &, bool, bool, int, int, int, hipStream_t);

}  // namespace ov
