// Host work on two threads.
#pragma once

#include <exception>
#include <thread>

namespace thor {

// Runs a() here and b() on a second thread; where no thread is to be had, or
// no memory for one, b() follows a().  Neither may throw, and nothing does.
template <typename A, typename B>
void run_both(A a, B b) noexcept {
  std::thread t;
  try {
    t = std::thread([&b] { b(); });
  } catch (const std::exception &) {
  }
  a();
  if (t.joinable()) t.join();
  else b();
}

}  // namespace thor
