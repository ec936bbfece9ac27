// The context's workspace: one device block that grows. Host code only; Dev gives the memory (alloc: null when there is
// none, free, sync, available: bytes of free memory), so that the rules can be checked without a device.
#pragma once

#include <cstddef>

namespace dfi {

struct Workspace {
  void* ptr = nullptr;
  size_t bytes = 0;
  bool frozen = false;       // a call captured into a caller's graph holds it: never reallocated
  size_t refused = 0;        // the smallest size that there was no memory for ...
  size_t refused_free = 0;   // ... when this much was free
};

template <class Dev>
void ws_release(Workspace& w, Dev& dev) {
  if (!w.ptr) return;
  dev.sync();
  dev.free(w.ptr);
  w.ptr = nullptr;
  w.bytes = 0;
}

// At least `bytes`, or no workspace at all (and false).
template <class Dev>
bool ws_need(Workspace& w, size_t bytes, Dev& dev) {
  if (bytes <= w.bytes) return true;
  if (w.frozen) return false;
  ws_release(w, dev);
  w.ptr = dev.alloc(bytes);
  w.bytes = w.ptr ? bytes : 0;
  return w.ptr != nullptr;
}

// `bytes` if there is the memory; false: the caller makes do with a smaller layout, `least` bytes of its last resort. Beside
// the present workspace first, which then stays as it is when there is no room; in its place where it has to grow
// anyway, or where that looks like enough. A refused size is not tried again until more memory is free than then: a program
// that runs at the limit of the memory pays for the attempt once, not on every call.
template <class Dev>
bool ws_want(Workspace& w, size_t bytes, size_t least, Dev& dev) {
  if (bytes <= w.bytes) return true;
  if (w.frozen) return false;
  if (w.refused != 0 && bytes >= w.refused && dev.available() <= w.refused_free) return false;
  if (void* p = dev.alloc(bytes)) {
    ws_release(w, dev);
    w.ptr = p;
    w.bytes = bytes;
    return true;
  }
  if (least > w.bytes || dev.available() + w.bytes >= bytes) {
    if (ws_need(w, bytes, dev)) return true;
  }
  w.refused = bytes;
  w.refused_free = dev.available();
  return false;
}

// The first of `levels` layouts, in order of preference, that there is the memory for; need(l) sets the caller's state to
// layout l and returns its bytes. `can_grow` false: out of the present workspace only. Returns false when there is no memory
// for the last one either; the state is then its.
template <class Dev, class F>
bool ws_levels(Workspace& w, int levels, bool can_grow, F need, Dev& dev) {
  if (need(0) <= w.bytes) return true;
  const size_t least = need(levels - 1);
  for (int l = 0; l + 1 < levels; ++l) {
    const size_t bytes = need(l);
    if (can_grow ? ws_want(w, bytes, least, dev) : bytes <= w.bytes) return true;
  }
  need(levels - 1);
  return can_grow ? ws_need(w, least, dev) : least <= w.bytes;
}

}  // namespace dfi
