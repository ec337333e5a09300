// Device allocations of one context or trainer (plain C++ over Dev, which allocates, frees and clears the
// error that a failed allocation leaves).
#pragma once
#include <algorithm>
#include <cstddef>
#include <vector>

namespace best {

template <class Dev>
struct ArenaT {
  std::vector<void*> ptrs;
  // A buffer kept for speed alone, and its size: given back when another allocation fails.
  char** spare = nullptr;
  size_t* spare_size = nullptr;

  template <class T>
  bool alloc(T** p, size_t n) {
    *p = nullptr;
    if (n == 0) n = 1;
    void* q = nullptr;
    bool ok = Dev::alloc(&q, n * sizeof(T));
    if (!ok && spare && *spare) {
      release(*spare);
      *spare_size = 0;
      ok = Dev::alloc(&q, n * sizeof(T));
    }
    if (!ok) return false;
    ptrs.push_back(q);
    *p = (T*)q;
    return true;
  }
  // Frees *p if it is an allocation of the arena.  p ends as null: a stale pointer could be the address of
  // a later allocation, which the next release of it would free.
  template <class T>
  void release(T*& p) {
    auto it = std::find(ptrs.begin(), ptrs.end(), (void*)p);
    if (it != ptrs.end()) {
      Dev::free(*it);
      ptrs.erase(it);
    }
    p = nullptr;
  }
  void free_all() {
    for (void* p : ptrs) Dev::free(p);
    ptrs.clear();
  }
};

}  // namespace best
