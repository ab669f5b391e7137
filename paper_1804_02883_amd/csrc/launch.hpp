// Kernel launches as every translation unit makes them.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

namespace epdlb {

// Profiling: while the profiler has room, the next kernel launch records a
// start/stop event pair at the kernel's own start and end (AMD's extended
// launch), so the times are kernel durations even when the host is slower
// than the GPU.  Recording never blocks.
inline thread_local hipEvent_t tl_ev_start = nullptr;
inline thread_local hipEvent_t tl_ev_stop = nullptr;

template <typename F, typename... Args>
void launch_k(F kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, Args... args) {
  if (tl_ev_start) {
    hipExtLaunchKernelGGL(kernel, grid, block, uint32_t(lds), s, tl_ev_start, tl_ev_stop, 0u, args...);
    tl_ev_start = tl_ev_stop = nullptr;  // one launch per armed pair
  } else {
    hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
  }
}

template <typename K>
hipError_t prep_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}

inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

}  // namespace epdlb
