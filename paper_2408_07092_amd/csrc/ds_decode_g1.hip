// The one-launch decode kernels of single heads.
#include "ds_device.h"

namespace ds {
DS_TRACE_BUFFER
}

#include "ds_decode_core.h"

namespace ds {
DS_DEFINE_DECODE_FN(1)
DS_DEFINE_TRACE_READ(1)
}  // namespace ds
