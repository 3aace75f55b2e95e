// Device memory of one call that makes and drops whole networks (intermediate
// bounds), by what allocates it (Mem: the HIP runtime; a test's own).
#pragma once
#include <stddef.h>

#include <algorithm>
#include <vector>

namespace gcp {

// Buffers are cut from chunks that are kept until the call ends, zero-filled
// when they are made and again by rewind(), which the caller runs once nothing
// of the previous network is left, on the device or the host.  The
// intermediate bounds of the CNN (three prefix networks) spent 5.7 of 9.7 ms
// in 133 allocations and frees; with the arena they take 5.9 ms.
template <class Mem>
class CallArena {
  struct Chunk { char* p; size_t bytes, used; };
  std::vector<Chunk> chunks;
  static constexpr size_t kChunk = (size_t)32 << 20, kAlign = 256;
 public:
  CallArena() = default;
  CallArena(const CallArena&) = delete;
  CallArena& operator=(const CallArena&) = delete;
  ~CallArena() { give_back(); }
  void give_back() {
    if (chunks.empty()) return;
    Mem::wait();                      // an error may have left work in flight
    for (Chunk& c : chunks) Mem::free(c.p);
    chunks.clear();
  }
  void* take(size_t n) {
    n = (n + kAlign - 1) / kAlign * kAlign;
    for (Chunk& c : chunks)
      if (c.bytes - c.used >= n) {
        void* q = c.p + c.used;
        c.used += n;
        return q;
      }
    Chunk c{nullptr, std::max(n, kChunk), n};
    c.p = Mem::try_alloc(c.bytes);
    if (!c.p) {                       // give back what this network does not use, ask for n alone
      for (size_t i = chunks.size(); i-- > 0;)
        if (chunks[i].used == 0) {
          Mem::free(chunks[i].p);
          chunks.erase(chunks.begin() + i);
        }
      c.bytes = n;
      c.p = Mem::alloc(n);
    }
    chunks.push_back(c);
    Mem::clear(c.p, c.bytes);
    return c.p;
  }
  void rewind() {
    for (Chunk& c : chunks) {
      if (c.used) Mem::clear(c.p, c.used);
      c.used = 0;
    }
  }
};

// Runs network(), which returns a status and leaves nothing behind, with its
// buffers in the arena of `scope`.  A chunk of an earlier network that a small
// buffer sits in keeps all its bytes, so memory can run out where the network
// alone fits: it then runs once more without the arena (scope.off() gives
// everything back; this network's buffers, and those of the ones that follow,
// are allocations of their own).
template <class Scope, class Network>
int in_arena(Scope& scope, int no_memory, Network network) {
  const int rc = network();
  if (rc != no_memory || !scope.on()) return rc;
  scope.off();
  return network();
}

}  // namespace gcp
