// Independent host work over a few threads.
#pragma once

#include <algorithm>
#include <atomic>
#include <thread>
#include <vector>

namespace almbm {

// f(0), ..., f(count - 1), each at most once, over up to eight threads (one per four
// calls); f's calls must not share what they write.  False if one of them threw (out of
// memory): an exception must not leave a thread, nor the C entry point above.
template <typename F> bool host_parallel(int count, F&& f) {
  const int nt = std::min({8, (int)std::thread::hardware_concurrency(), count / 4});
  std::atomic<int> next{0};
  std::atomic<bool> threw{false};
  auto work = [&]() {
    try {
      for (int t = next++; t < count; t = next++) f(t);
    } catch (...) {
      threw = true;
    }
  };
  std::vector<std::thread> pool;
  try {
    for (int t = 1; t < nt; ++t) pool.emplace_back(work);
  } catch (...) {
    // fewer threads then: the caller's own takes what is left
  }
  work();
  for (std::thread& t : pool) t.join();
  return !threw;
}

}  // namespace almbm
