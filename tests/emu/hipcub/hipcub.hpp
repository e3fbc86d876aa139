// Host emulation: the device-wide scan that inc.hip calls, on the host.
#pragma once

#include <hip/hip_runtime.h>

namespace hipcub {

struct DeviceScan {
  template <typename T>
  static hipError_t ExclusiveSum(void* tmp, size_t& bytes, const T* in, T* out, int n, hipStream_t) {
    bytes = 1;
    if (!tmp) return hipSuccess;
    T sum = 0;
    for (int i = 0; i < n; ++i) {
      const T x = in[i];
      out[i] = sum;
      sum += x;
    }
    return hipSuccess;
  }
};

}  // namespace hipcub
