// run_both (two_threads.h) where the second thread is to be had, where its
// state's allocation fails, and where the system gives no thread: both parts
// run once each, and nothing is thrown.
#include <sys/resource.h>

#include <cstdio>
#include <cstdlib>
#include <new>

#include "two_threads.h"

static bool deny = false;

void *operator new(std::size_t n) {
  void *p = deny ? nullptr : std::malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

static int check(const char *what, bool other_thread) {
  int a = 0, b = 0;
  const std::thread::id here = std::this_thread::get_id();
  std::thread::id there;
  thor::run_both([&] { a += 1; }, [&] { b += 1; there = std::this_thread::get_id(); });
  const bool ok = a == 1 && b == 1 && (there != here) == other_thread;
  std::printf("%s: a %d b %d %s\n", what, a, b, ok ? "ok" : "WRONG");
  return ok ? 0 : 1;
}

int main() {
  int bad = 0;
  // no address space left for a thread's stack (before one is kept for reuse)
  rlimit lim{}, none{};
  if (getrlimit(RLIMIT_AS, &lim) == 0) {
    none = lim;
    none.rlim_cur = 1;
    if (setrlimit(RLIMIT_AS, &none) == 0) bad += check("no thread", false);
    setrlimit(RLIMIT_AS, &lim);
  }
  bad += check("thread", true);
  deny = true;
  bad += check("no memory", false);
  deny = false;
  return bad;
}
