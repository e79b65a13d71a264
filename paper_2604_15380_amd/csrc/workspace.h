// Growth of a device workspace (host code without HIP).
#pragma once

#include <stddef.h>

struct Workspace {
  void* p = nullptr;
  size_t bytes = 0;
  size_t refused = (size_t)-1;   // smallest wish that could not be allocated
};

// Make room for a call that needs `need` bytes and runs best with `full` (at
// least `need`).  Room for `need` is enlarged for the wish's sake only where
// the stream may allocate (capturing() false: asked only then) and no smaller
// wish has been refused; a call that has to allocate anyway wishes again.  A
// wish comes with 1 / slack more, so that batches a little larger do not
// allocate again.  Where it is refused the call gets what it needs, at least
// what was there before.  False: not even `need` could be allocated.
template <class Capturing, class Alloc, class Release>
bool workspace_grow(Workspace& w, size_t need, size_t full, int slack, Capturing&& capturing, Alloc&& alloc,
                    Release&& release) {
  if (full <= w.bytes) return true;
  if (need <= w.bytes && (full >= w.refused || capturing())) return true;
  const size_t had = w.bytes;
  if (w.p) release(w.p);
  w.p = nullptr;
  w.bytes = 0;
  const size_t least = need > had ? need : had;
  const size_t tries[] = {full + full / slack, full, least + least / slack, least, need};
  for (int k = 0; k < 5; ++k) {
    if (k == 2 && full > need && full < w.refused) w.refused = full;
    if ((w.p = alloc(tries[k]))) {
      w.bytes = tries[k];
      return true;
    }
  }
  return false;
}
