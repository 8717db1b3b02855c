// How the launchers put a kernel on its stream.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <tuple>
#include <utility>

namespace fp {

// The event that stands for the kernels this thread launches while it is set: each one carries it as the completion
// signal of its own dispatch, so that it completes with the last of them.  An event recorded behind a kernel is a packet of
// its own, which the next kernel waits for.  By itself, one kernel over and over, us per launch: 16.0 and 28.9 without an event,
// 19.0 and 32.0 with one recorded, 16.1 and 29.1 with one carried.  In the layers, all operators of a pass without a bound and with
// two operators in flight: recorded 1354 -> 1373 (4096 packed tokens) and 1531 -> 1555 (8192 tokens, mixture of experts), carried
// 1344 -> 1341 and 1516 -> 1513.  (A profiler's trace shows 4.7 us behind every kernel that carries an event, and none without a
// bound: those are the profiler's own.)
struct CarriedEvent {
  hipEvent_t event = nullptr;
  bool taken = false;       // a kernel has been launched with it
};
CarriedEvent& carried_event();

template <typename... P, typename... A, size_t... I>
void launch_with(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t s, std::index_sequence<I...>, A&&... a) {
  std::tuple<P...> params{static_cast<P>(a)...};
  void* at[] = {const_cast<void*>(static_cast<const volatile void*>(&std::get<I>(params)))...};
  CarriedEvent& c = carried_event();
  // (an error stays with hipGetLastError, as after <<<>>>)
  if (c.event) {
    c.taken = hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, at, lds_bytes, s, nullptr, c.event, 0) == hipSuccess;
  } else {
    (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, at, lds_bytes, s);
  }
}

template <typename... P, typename... A>
void launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t s, A&&... a) {
  static_assert(sizeof...(P) == sizeof...(A), "one argument for every parameter");
  launch_with(kernel, grid, block, lds_bytes, s, std::index_sequence_for<P...>{}, std::forward<A>(a)...);
}

}  // namespace fp
