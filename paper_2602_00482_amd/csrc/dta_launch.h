// Kernel launches of the attention calls.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "dta_internal.h"

namespace dta {

// Launches a kernel on the call's stream.  `last`: no launch of the call follows, so the
// event that says when the tree's device copies are free can be the kernel's own
// completion.  An event recorded after it is a packet of its own, which the next kernel
// waits behind: 1480 calls of a leaf-order plan over short segments take 25.6 ms that way,
// 22.2 ms with the event on the kernel, 20.9 ms without any event.
template <typename... P, typename... A>
inline void launch(const LaunchArgs& a, bool last, void (*kernel)(P...), size_t grid, unsigned block, A... args) {
  const hipStream_t st = (hipStream_t)a.stream;
  if (last && a.done_event != nullptr) {
    hipExtLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(block), 0, st, nullptr, (hipEvent_t)a.done_event, 0,
                          static_cast<P>(args)...);
    *a.done_recorded = true;
  } else {
    kernel<<<(unsigned)grid, block, 0, st>>>(static_cast<P>(args)...);
  }
}

}  // namespace dta
