// The one-launch decode kernels of larger groups.
#include "ds_device.h"

namespace ds {
DS_TRACE_BUFFER
}

#include "ds_decode_core.h"

namespace ds {
DS_DEFINE_DECODE_FN(16)
DS_DEFINE_TRACE_READ(16)
}  // namespace ds
