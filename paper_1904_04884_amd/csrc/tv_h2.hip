// TV pass kernels of fusion depth 2.
#include "tv_device.h"

namespace rihvr {
template void launch_tv_depth<2>(const TvSelect&, dim3, const TvPassArgs*, const BatchMap&, hipStream_t);
}  // namespace rihvr
