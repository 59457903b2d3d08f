// Stands in for the calls of the HIP runtime that the library makes: a program that includes this and is linked with -rdynamic
// has them come first in the symbol lookup.  Nothing runs and no GPU is needed.  The calls are counted, and the one it is told to
// refuse is refused as the runtime does it: the status is returned and stays behind as the thread's last error until somebody asks
// for it, whatever succeeds in between.
#pragma once
#define __HIP_PLATFORM_AMD__
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <map>
#include <string>

namespace fake {

inline int calls = 0, refused = -1, launches_after = 0;
inline hipError_t pending = hipSuccess;
alignas(256) inline char scratch[256];
inline std::string launched;   // the kernels launched, one a line

inline std::map<const void*, std::string>& names() {   // (filled while the library is loaded, before any constructor here)
  static std::map<const void*, std::string> all;
  return all;
}

inline hipError_t answer(const void* kernel) {
  if (refused >= 0 && calls > refused && kernel) ++launches_after;
  if (calls++ != refused) {
    if (kernel) launched += names()[kernel] + "\n";
    return hipSuccess;
  }
  return pending = hipErrorLaunchFailure;
}

template <typename T = void>
T* at(int n) { return reinterpret_cast<T*>((uintptr_t)(n + 1) << 28); }   // an argument, never read

}  // namespace fake

extern "C" {
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) { return fake::answer(f); }
hipError_t hipGetLastError() {
  const hipError_t e = fake::pending;
  fake::pending = hipSuccess;
  return e;
}
hipError_t hipPeekAtLastError() { return fake::pending; }
hipError_t hipGetDevice(int* device) { *device = 0; return fake::answer(nullptr); }
hipError_t hipGetDeviceCount(int* count) { *count = 2; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return fake::answer(nullptr); }
hipError_t hipGetSymbolAddress(void** at, const void*) { *at = fake::scratch; return fake::answer(nullptr); }
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int status = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  fake::names()[f] = plain ? plain : name;
  std::free(plain);
}
}
