"""The arena of an intermediate-bounds call on a card with little memory left: networks that fit one after the other
on buffers of their own also fit in one call."""


from test_launch_rules_cpu import _run, pytestmark  # noqa: F401

ARENA = r"""
#include "call_arena.h"
#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>
#include <set>
struct Mem {
  static inline size_t cap = 0, used = 0;
  static inline std::map<char*, size_t> live;
  static inline char* next = (char*)4096;
  static char* try_alloc(size_t n) {
    if (used + n > cap) return nullptr;
    char* p = next;
    next += n + 4096;
    live[p] = n;
    used += n;
    return p;
  }
  static char* alloc(size_t n) {
    char* p = try_alloc(n);
    if (!p) throw std::bad_alloc();
    return p;
  }
  static void free(char* p) {
    if (!live.count(p)) abort();
    used -= live[p];
    live.erase(p);
  }
  static void wait() {}
  static void clear(void*, size_t) {}
};
struct Scope {
  gcp::CallArena<Mem> arena;
  bool in = true;
  bool on() const { return in; }
  void off() { arena.give_back(); in = false; }
};
constexpr size_t MB = 1 << 20;
// one network: its buffers, in the arena or on their own, all dropped at the end
static int network(Scope& s, const std::vector<size_t>& sizes) {
  std::vector<char*> own;
  int rc = 0;
  try {
    for (size_t n : sizes) {
      if (s.on()) s.arena.take(n);
      else own.push_back(Mem::alloc(n));
    }
  } catch (const std::bad_alloc&) {
    rc = -4;
  }
  for (char* p : own) Mem::free(p);
  return rc;
}
int main() {
  // a large network, then one of small buffers (which come to lie in its chunk) and a larger one
  const std::vector<std::vector<size_t>> nets = {{40 * MB, 2000 * MB}, {1 * MB, 20 * MB, 30 * MB, 2500 * MB}, {2600 * MB, 1 * MB}};
  for (size_t cap : {(size_t)2601 * MB, (size_t)8000 * MB}) {
    Mem::cap = cap;
    int plain = 0, again = 0, alone = 0;
    {
      Scope s;
      s.off();
      for (auto& n : nets) plain |= network(s, n);
    }
    {
      Scope s;
      for (auto& n : nets) {
        s.arena.rewind();
        alone |= network(s, n);
      }
    }
    {
      Scope s;
      for (auto& n : nets) {
        s.arena.rewind();
        again |= gcp::in_arena(s, -4, [&] { return network(s, n); });
      }
      printf("%d %d %d %d\n", plain, alone, again, (int)s.on());
    }
    if (Mem::used) return 1;
  }
  // what does not fit by itself still fails, after one more try
  Mem::cap = 2000 * MB;
  Scope s;
  int tries = 0;
  const int rc = gcp::in_arena(s, -4, [&] { ++tries; return network(s, nets[1]); });
  printf("%d %d %d\n", rc, tries, (int)s.on());
}
"""


def test_networks_that_fit_by_themselves_fit_in_a_call(tmp_path):
    tight, roomy, none = [tuple(map(int, x.split())) for x in _run(tmp_path, ARENA)]
    assert tight == (0, -4, 0, 0)      # the arena by itself runs out; the call goes on without it
    assert roomy == (0, 0, 0, 1)
    assert none == (-4, 2, 0)
