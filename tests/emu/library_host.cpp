// The whole library on the CPU: with the other sources of the package, compiled
// the same way, this makes a shared object with the C interface of
// graphcolor.h on host memory.
#define EMU_MAIN
#include <hip/hip_runtime.h>

// One workgroup of every kernel per CU is taken to be resident.
extern "C" void emu_start(int hardware_queues, int cus, uint64_t order) {
  emu::cus = cus;
  emu::seed = order;
  emu::start_queues(hardware_queues);
}
extern "C" void emu_stop() { emu::stop_queues(); }
