#include <hip/hip_runtime.h>

#include "core.hip"

static const bool registered = (emu::add_kernel(gcol::core_wide_kernel<2, 8, 1024>),
                                emu::add_kernel(gcol::core_wide_kernel<3, 12, 512>), emu::add_kernel(gcol::core_kernel),
                                true);
