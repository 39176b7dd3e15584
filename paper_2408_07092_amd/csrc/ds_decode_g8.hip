// The one-launch decode kernels of groups of 5 to 8 heads.
#include "ds_device.h"

namespace ds {
DS_TRACE_BUFFER
}

#include "ds_decode_core.h"

namespace ds {
DS_DEFINE_DECODE_FN(8)
DS_DEFINE_TRACE_READ(8)
}  // namespace ds
