// Work in slices on host threads (no HIP: also compiled by the host compiler
// alone).
#pragma once

#include <thread>

namespace finger {

constexpr int kMaxSlices = 8;

// fn(0) .. fn(slices - 1), a thread each, all ended on return; false if a
// thread could not be had (then some slices have not run).  Starting a thread
// can throw std::system_error and, for its state, std::bad_alloc: nothing may
// leave this function while a started thread is joinable.  fn must not throw.
template <typename F>
bool run_sliced(int slices, const F& fn) noexcept {
  std::thread th[kMaxSlices];
  bool all = slices <= kMaxSlices;
  try {
    for (int i = 0; all && i < slices; ++i) th[i] = std::thread([&fn, i] { fn(i); });
  } catch (...) {
    all = false;
  }
  for (std::thread& t : th)
    if (t.joinable()) t.join();
  return all;
}

}  // namespace finger
