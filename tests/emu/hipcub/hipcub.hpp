// Host emulation: the device-wide scan and sort that the library calls.
#pragma once

#include <hip/hip_runtime.h>

namespace hipcub {

struct DeviceScan {
  template <typename T>
  static hipError_t ExclusiveSum(void* tmp, size_t& bytes, const T* in, T* out, int n, hipStream_t s) {
    bytes = 1;
    if (!tmp) return hipSuccess;
    emu::enqueue(s, [=] {
      T sum = 0;
      for (int i = 0; i < n; ++i) {
        const T x = in[i];
        out[i] = sum;
        sum += x;
      }
    });
    return hipSuccess;
  }
};

struct DeviceRadixSort {
  template <typename K, typename V>
  static hipError_t SortPairs(void* tmp, size_t& bytes, const K* keys, K* keys_out, const V* values, V* values_out, int n,
                              int = 0, int = 0, hipStream_t s = nullptr) {
    bytes = 1;
    if (!tmp) return hipSuccess;
    emu::enqueue(s, [=] {
      std::vector<int> by(n);
      std::iota(by.begin(), by.end(), 0);
      std::stable_sort(by.begin(), by.end(), [=](int a, int b) { return keys[a] < keys[b]; });
      for (int i = 0; i < n; ++i) {
        keys_out[i] = keys[by[i]];
        values_out[i] = values[by[i]];
      }
    });
    return hipSuccess;
  }
};

}  // namespace hipcub
