// The one-launch decode kernels of groups of 3 and 4 heads.
#include "ds_device.h"

namespace ds {
DS_TRACE_BUFFER
}

#include "ds_decode_core.h"

namespace ds {
DS_DEFINE_DECODE_FN(4)
DS_DEFINE_TRACE_READ(4)
}  // namespace ds
