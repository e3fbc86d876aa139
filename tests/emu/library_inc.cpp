#include <hip/hip_runtime.h>

#include "inc.hip"

static const bool registered = (emu::add_kernel(gcol::inc_tail_kernel), true);
