// Bookkeeping of the internal workspace of ozaki2_dgemm and
// ozaki2_dgemm_strided_batched on one device: one grow-only buffer, and the
// buffers that captured graphs still hold.  Device memory comes from Mem
// (alloc, free, sync: HIP's in api.cpp).
#pragma once
#include <stddef.h>

#include <new>

struct Oz2Pool {
  struct Held {
    void* ptr;
    Held* next;
  };
  void* ptr = nullptr;
  size_t bytes = 0;
  bool captured = false;    // a stream capture has taken ptr: a graph may replay on it
  Held* held = nullptr;     // outgrown buffers that captures have taken

  enum Status { kOk, kNoMem, kDevice };

  // A buffer of at least `need` bytes.  Growing frees the old one once the
  // device has finished with it, unless a capture has taken it: a graph replays
  // on the addresses it was captured with, so that buffer stays until release().
  // Where no larger one can be had it also stays the current one.
  template <class Mem>
  Status get(size_t need, bool capturing, Mem& mem, void** out) {
    if (bytes < need) {
      const size_t grow = need > ((size_t)1 << 20) ? need : (size_t)1 << 20;
      void* p = nullptr;
      if (ptr && captured) {
        Held* h = new (std::nothrow) Held{ptr, held};
        if (!h || !mem.alloc(&p, grow)) {
          delete h;
          return kNoMem;
        }
        held = h;
      } else {
        if (ptr) {
          if (!mem.sync()) return kDevice;
          mem.free(ptr);
          ptr = nullptr;
          bytes = 0;
        }
        if (!mem.alloc(&p, grow)) return kNoMem;
      }
      ptr = p;
      bytes = grow;
      captured = false;
    }
    captured |= capturing;
    *out = ptr;
    return kOk;
  }

  // frees everything; the caller has synchronised the device
  template <class Mem>
  void release(Mem& mem) {
    if (ptr) mem.free(ptr);
    ptr = nullptr;
    bytes = 0;
    captured = false;
    while (held) {
      Held* h = held;
      held = h->next;
      mem.free(h->ptr);
      delete h;
    }
  }
};
