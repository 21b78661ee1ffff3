// Independent pieces of a mesh's host work, side by side.
#pragma once

#include <exception>
#include <thread>
#include <vector>

namespace ebe {

// f(0) .. f(n - 1), each on a thread of its own; the first exception is rethrown after all have ended
template <class F>
void parallel(int n, F f) {
  std::vector<std::exception_ptr> err(n);
  std::vector<std::thread> threads;
  threads.reserve(n);
  auto run = [&](int t) {
    try {
      f(t);
    } catch (...) {
      err[t] = std::current_exception();
    }
  };
  int started = 1;  // f(0) runs here, and what no thread could be started for
  try {
    for (; started < n; ++started) threads.emplace_back(run, started);
  } catch (...) {
  }
  run(0);
  for (int t = started; t < n; ++t) run(t);
  for (auto& t : threads) t.join();
  for (auto& e : err)
    if (e) std::rethrow_exception(e);
}

}  // namespace ebe
