// Scratch of the allocation-free Krylov entry point (krylov_expv_static), with
// room for the vectors that the single-pass steps use more than the limit counts: a
// file-scope device array that each GPU holds for the life of the process.  In
// host code the array's name is only a stand-in; its device address comes from
// hipGetSymbolAddress, taken once per device with that device current and kept
// per device.

#include <hip/hip_runtime.h>

#include <mutex>

#include "kg_internal.h"

namespace kg {

namespace {

__device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kStepMaxD * kStepExtra + 3 * 256];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

hipError_t static_scratch(void** ptr) {
  *ptr = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace kg
