// Tile lists where threads or memory are refused: without threads the same lists, without memory std::bad_alloc
// in the caller.  argv: pattern file (n, w, slot-major columns), halo depth, tile side.
#include <dlfcn.h>
#include <pthread.h>

#include <atomic>
#include <cerrno>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <thread>
#include <vector>

#include "tiles.hpp"

static std::atomic<int> no_threads{0}, no_memory{0};
static const std::thread::id main_id = std::this_thread::get_id();

extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*fn)(void*), void* arg) {
  if (no_threads) return EAGAIN;
  using Fn = int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
  static const Fn next = reinterpret_cast<Fn>(dlsym(RTLD_NEXT, "pthread_create"));
  return next(t, a, fn, arg);
}
void* operator new(std::size_t b) {   // the workers' lists are refused
  if (no_memory && b > 4096 && std::this_thread::get_id() != main_id) throw std::bad_alloc();
  if (void* p = std::malloc(b ? b : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  std::FILE* f = std::fopen(argv[1], "rb");
  int h[2];
  if (!f || std::fread(h, sizeof(int), 2, f) != 2) return 2;
  const int n = h[0], w = h[1], KM = std::atoi(argv[2]), side = std::atoi(argv[3]);
  std::vector<int> col((size_t)n * w);
  if (std::fread(col.data(), sizeof(int), col.size(), f) != col.size()) return 2;
  std::fclose(f);
  mgl::TilePlan a, b;
  if (!mgl::build_tiles(n, n, w, col.data(), KM, side, side, a, 4, 8)) return 1;
  no_threads = 1;
  if (!mgl::build_tiles(n, n, w, col.data(), KM, side, side, b, 4, 8) || !mgl::check_tiles(n, n, col.data(), b, 8))
    return 1;
  if (a.node != b.node || a.lcol != b.lcol || a.toff != b.toff || a.cnt != b.cnt) return 1;
  no_threads = 0;
  no_memory = 1;
  try {
    (void)mgl::build_tiles(n, n, w, col.data(), KM, side, side, b, 4, 8);
    if (std::thread::hardware_concurrency() > 1) return 1;
  } catch (const std::bad_alloc&) {
  }
  no_memory = 0;
  std::printf("ok %d\n", a.ntiles);
  return 0;
}
