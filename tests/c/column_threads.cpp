// The column check of a large map where a thread of it cannot be started: for
// want of memory for its state, or because the system refuses it.  The check
// is then done by the calling thread; nothing leaves it but its answer.
//
// Usage: column_threads
#include <pthread.h>

#include <cerrno>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "tc_plan.h"

static int g_allow = -1;    // allocations that still succeed; < 0: all
static int g_threads = -1;  // threads that still start; < 0: all
static int g_started = 0;

void* operator new(std::size_t n) {
  if (g_allow == 0) throw std::bad_alloc();
  if (g_allow > 0) --g_allow;
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

extern "C" int __real_pthread_create(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
extern "C" int __wrap_pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*),
                                     void* arg) {
  if (g_threads == 0) return EAGAIN;
  if (g_threads > 0) --g_threads;
  ++g_started;
  return __real_pthread_create(t, a, f, arg);
}

int main() {
  const int32_t W = 4096, H = 1100;   // above the size from which threads share it
  int fails = 0;
  for (int bad = 0; bad < 2; ++bad) {
    std::vector<uint8_t> F((size_t)W * H, 9), B((size_t)W * H, 0), T((size_t)W * H, 0);
    const int32_t bx = 4001, by = 777;
    if (bad) {
      T[(size_t)by * W + bx] = 1;
      T[(size_t)(H - 1) * W] = 1;   // (a later one: the first is reported)
    }
    for (int kind = 0; kind < 2; ++kind)
      for (int ok = -1; ok < 8; ++ok) {
        int32_t x = -1, y = -1;
        (kind ? g_threads : g_allow) = ok;
        const bool valid = tci::columns_valid(F.data(), B.data(), T.data(), W, H, W, &x, &y);
        g_allow = g_threads = -1;
        const bool right = bad ? !valid && x == bx && y == by : valid;
        if (!right) {
          std::printf("kind %d ok %d: valid %d at (%d, %d)\n", kind, ok, valid, x, y);
          ++fails;
        }
      }
  }
  std::printf("%d threads started, %d failures\n", g_started, fails);
  return fails != 0;
}
