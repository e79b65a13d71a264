// workspace_grow against a device with a fixed amount of free memory.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "workspace.h"

static size_t free_bytes;
static std::map<void*, size_t> live;
static int allocs, frees;
static bool capture;

static bool grow(Workspace& w, size_t need, size_t full) {
  return workspace_grow(
      w, need, full, 4, [] { return capture; },
      [](size_t n) -> void* {
        if (capture) std::abort();
        ++allocs;
        if (n > free_bytes) return nullptr;
        free_bytes -= n;
        void* p = std::malloc(1);
        live[p] = n;
        return p;
      },
      [](void* p) {
        if (capture) std::abort();
        ++frees;
        free_bytes += live[p];
        live.erase(p);
        std::free(p);
      });
}

#define CHECK(x)                                              \
  do {                                                        \
    if (!(x)) return std::printf("line %d: %s\n", __LINE__, #x), 1; \
  } while (0)

int main() {
  Workspace w;
  free_bytes = 1000;
  // a wish with a quarter more; a slightly larger batch does not allocate
  CHECK(grow(w, 100, 400) && w.bytes == 500);
  CHECK(grow(w, 110, 490) && w.bytes == 500 && allocs == 1);
  // under capture room for what is needed is enough
  capture = true;
  CHECK(grow(w, 450, 700) && w.bytes == 500);
  capture = false;
  // a wish that does not fit: what was there is there again
  CHECK(grow(w, 450, 1100) && w.bytes >= 500 && w.refused == 1100);
  // ... and the same wish is not tried again, a smaller one is
  int a = allocs;
  CHECK(grow(w, 450, 1100) && allocs == a);
  CHECK(grow(w, 450, 900) && allocs > a && w.bytes == 900 && w.refused == 1100);
  // once memory is there a call that must allocate wishes again
  free_bytes += 4000;
  CHECK(grow(w, 950, 1200) && w.bytes == 1500);
  // room for the need alone when nothing more is left
  free_bytes = 0;
  CHECK(grow(w, 1500, 1500) && w.bytes == 1500);
  const size_t f = frees;
  CHECK(!grow(w, 1501, 1501) && w.p == nullptr && w.bytes == 0);
  CHECK(frees == (int)f + 1);
  CHECK(grow(w, 1400, 1400) && w.bytes == 1400);
  // no wish (full == need) never counts as refused
  Workspace v;
  free_bytes = 100;
  CHECK(grow(v, 90, 90) && v.bytes == 90 && v.refused == (size_t)-1);
  for (auto& x : live) std::free(x.first);
  std::printf("ok\n");
  return 0;
}
