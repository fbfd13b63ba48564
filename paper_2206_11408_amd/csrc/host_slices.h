// Work in slices on host threads (no HIP: also compiled by the host compiler
// alone).
#pragma once

#include <cstddef>
#include <thread>

namespace finger {

constexpr int kMaxSlices = 8;

// Slices of a copy of `bytes` to the host: four from 64 MB on, else the plain
// copy.  The slices' streams cost 2 to 3 ms a call in all (their queues; the
// calls behind them pay part of it), and about 10 once per process, so below
// that they lose what the threads save: an export with 10 MB of codes took
// 6.0 ms in slices and takes 3.6 in one copy, 20 MB 10.5 and 7.9, 41 MB 11.8
// and 11.7; 82 MB 16.0 and 18.5.
constexpr int copy_slices(std::size_t bytes) { return bytes >= (std::size_t)64 << 20 ? 4 : 1; }

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
