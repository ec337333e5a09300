// The arena over a fake device with a byte budget that hands out the lowest free address: released
// pointers are null, a failed growth leaves nothing that a later release could free twice or in another
// buffer's place, the spare buffer is given back for an allocation that needs its bytes, and nothing leaks.
// Built and run by tests/test_arena_cpu.py.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "../paper_2606_04895_amd/csrc/arena.hpp"

static std::map<char*, size_t> live;  // address -> bytes
static size_t budget = 1000;
static int bad_frees = 0;

struct Fake {
  static bool alloc(void** p, size_t n) {
    size_t used = 0;
    for (auto& a : live) used += a.second;
    if (used + n > budget) return false;
    char* at = (char*)0x1000;
    for (auto& a : live)
      if (at + n <= a.first) break;
      else at = a.first + a.second;
    live[at] = n;
    *p = at;
    return true;
  }
  static void free(void* p) {
    if (!live.erase((char*)p)) ++bad_frees;
  }
};

#define REQUIRE(c)                                          \
  do {                                                      \
    if (!(c)) {                                             \
      std::printf("FAIL %d: %s\n", __LINE__, #c);           \
      return 1;                                             \
    }                                                       \
  } while (0)

int main() {
  best::ArenaT<Fake> m;
  char *a = nullptr, *b = nullptr, *c = nullptr;
  REQUIRE(m.alloc(&a, 100) && m.alloc(&b, 100));
  // a buffer that cannot grow: released, not replaced, then its address goes to another buffer
  m.release(a);
  REQUIRE(a == nullptr);
  REQUIRE(!m.alloc(&a, 2000) && a == nullptr);
  REQUIRE(m.alloc(&c, 100) && c == (char*)0x1000);
  m.release(a);  // what the next call of the failed one does first
  REQUIRE(live.count(c) == 1 && live.size() == 2 && bad_frees == 0);
  // the spare is given back, and only when needed
  char* met = nullptr;
  size_t met_cap = 600;
  m.spare = &met;
  m.spare_size = &met_cap;
  REQUIRE(m.alloc(&met, 600));
  char* d = nullptr;
  REQUIRE(m.alloc(&d, 150) && met && met_cap == 600);
  char* e = nullptr;
  REQUIRE(m.alloc(&e, 500) && !met && met_cap == 0);
  REQUIRE(!m.alloc(&a, 900) && a == nullptr);  // no spare left: refused
  m.free_all();
  REQUIRE(live.empty() && bad_frees == 0);
  std::printf("ok\n");
  return 0;
}
