// The wide tile kernel's binary32 instantiations (a translation unit of their own: they compile beside the rest).
#include "nuts_wide.h"

namespace nuts {
void wide_launch_f32(const WideArgs& wa, const DevSample& sa, int nc, int blocks, hipStream_t stream)
{
    wide_launch<float>(wa, sa, nc, blocks, stream);
}
}  // namespace nuts
