// The pool of idle device blocks (bh_pool.h) over a scripted device, on the CPU.  A scenario
// prints "<name> ok".
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "bh_pool.h"

#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);             \
      std::exit(1);                                                   \
    }                                                                 \
  } while (0)

// Memory of `room` bytes; `busy` blocks may still be used by queued work until a wait succeeds.
struct Memory {
  std::mutex mu;
  size_t room = (size_t)8 << 30, in_use = 0;
  std::map<void*, size_t> live;
  std::vector<void*> freed;
  bool refuse_wait = false;
  int allocs = 0, waits = 0;
};

struct Fake {
  Memory* m;
  bool alloc(void** p, size_t bytes) {
    std::lock_guard<std::mutex> g(m->mu);
    if (m->in_use + bytes > m->room) return false;
    static size_t next = 0x1000;
    *p = (void*)next;
    next += 0x1000;
    m->live[*p] = bytes;
    m->in_use += bytes;
    ++m->allocs;
    return true;
  }
  void free(void* p) {
    std::lock_guard<std::mutex> g(m->mu);
    auto it = m->live.find(p);
    CHECK(it != m->live.end());
    m->in_use -= it->second;
    m->live.erase(it);
    m->freed.push_back(p);
  }
  bool wait() {
    std::lock_guard<std::mutex> g(m->mu);
    ++m->waits;
    return !m->refuse_wait;
  }
};

using Pool = bh::BlockPool<Fake>;
constexpr size_t MiB = (size_t)1 << 20;

static void reuse() {
  Memory m;
  Pool::Peers peers;
  Pool pool(Fake{&m}, peers);
  void *a, *b;
  CHECK(pool.alloc(&a, 10 * MiB));
  {
    Pool::Release give_back(pool);
    give_back(a, 10 * MiB);
  }
  CHECK(pool.alloc(&b, 10 * MiB - 1000) && b == a && m.allocs == 1);  // the same size step
  CHECK(pool.alloc(&a, 10 * MiB) && a != b && m.allocs == 2);
  pool.free(a);
  pool.free(b);
  pool.drop();
  CHECK(m.live.empty());
}

// A wait that is refused does not make a block idle: it goes to the device, not to the next build.
static void refused_wait() {
  Memory m;
  Pool::Peers peers;
  Pool pool(Fake{&m}, peers);
  void *a, *b;
  CHECK(pool.alloc(&a, 4 * MiB));
  m.refuse_wait = true;
  {
    Pool::Release give_back(pool);
    give_back(a, 4 * MiB);
  }
  CHECK(m.waits == 1 && m.freed.size() == 1 && m.freed[0] == a);
  CHECK(pool.alloc(&b, 4 * MiB) && b != a);
  m.refuse_wait = false;
  {
    Pool::Release give_back(pool);
    give_back(b, 4 * MiB);
  }
  CHECK(m.freed.size() == 1 && pool.alloc(&a, 4 * MiB) && a == b);
  pool.free(a);
  CHECK(m.live.empty());
}

// A failing allocation first gives the kept blocks back, then does without the rounding.
static void allocation_failure() {
  Memory m;
  m.room = 64 * MiB;
  Pool::Peers peers;
  Pool pool(Fake{&m}, peers);
  void *a, *b;
  CHECK(pool.alloc(&a, 40 * MiB));
  pool.recycle(a, 40 * MiB);
  CHECK(m.in_use == 40 * MiB);
  CHECK(pool.alloc(&b, 60 * MiB) && m.in_use == 60 * MiB);
  pool.free(b);
  const size_t odd = 63 * MiB;  // its size step is 64 MiB
  m.room = odd;
  CHECK(pool.alloc(&b, odd) && m.in_use == odd);
  pool.recycle(b, odd);         // smaller than its step: not kept
  CHECK(m.live.empty());
  m.room = MiB;
  CHECK(!pool.alloc(&b, 2 * MiB) && b == nullptr);
}

// A full pool: blocks that are no longer asked for make room after a while, so later builds find
// theirs again; the bound on what is kept holds, and a block above it is never kept.
static void full_pool() {
  Memory m;
  Pool::Peers peers;
  Pool pool(Fake{&m}, peers);
  std::vector<void*> old;
  for (int k = 0; k < 8; ++k) {  // 8 x 128 MiB: full
    void* p;
    CHECK(pool.alloc(&p, 128 * MiB));
    old.push_back(p);
  }
  for (void* p : old) pool.recycle(p, 128 * MiB);
  CHECK(m.in_use == bh::kKeepMost);
  int before_last = 0;
  const int rounds = (int)bh::kStale;
  for (int r = 0; r < rounds; ++r) {  // a session of other sizes
    void *a, *b;
    before_last = m.allocs;
    CHECK(pool.alloc(&a, 288 * MiB) && pool.alloc(&b, 60 * MiB));
    pool.recycle(a, 288 * MiB);
    pool.recycle(b, 60 * MiB);
    CHECK(m.in_use <= bh::kKeepMost);
  }
  CHECK(m.allocs == before_last);  // found both kept
  void* big;
  m.room = (size_t)16 << 30;
  CHECK(pool.alloc(&big, bh::kKeepMost + 1));
  const size_t before = m.in_use;
  pool.recycle(big, bh::kKeepMost + 1);
  CHECK(m.in_use < before && m.in_use <= bh::kKeepMost);
  pool.drop();
  CHECK(m.live.empty());
}

// Builds that need more in all than is kept: what is kept is found every time, and is not put out
// by the rest.
static void larger_cycle() {
  Memory m;
  Pool::Peers peers;
  Pool pool(Fake{&m}, peers);
  int allocs = 0;
  const int rounds = 200;
  for (int r = 0; r < rounds; ++r) {
    void *scratch, *map, *bits;
    CHECK(pool.alloc(&scratch, 360 * MiB) && pool.alloc(&map, bh::kKeepMost) &&
          pool.alloc(&bits, 53 * MiB));
    pool.recycle(scratch, 360 * MiB);
    pool.recycle(map, bh::kKeepMost);
    pool.recycle(bits, 53 * MiB);
    CHECK(m.in_use <= bh::kKeepMost);
    if (r == 0) allocs = m.allocs;
  }
  CHECK(m.allocs == allocs + rounds - 1);  // the map alone is allocated again
  pool.drop();
  CHECK(m.live.empty());
}

// The blocks that other pools of the device keep are given back too, for a block of any kind, and
// a pool that is gone is not asked.
static void peers() {
  Memory m;
  m.room = 100 * MiB;
  Pool::Peers all;
  Pool one(Fake{&m}, all);
  void *a, *b;
  {
    Pool two(Fake{&m}, all);
    CHECK(two.alloc(&a, 80 * MiB));
    two.recycle(a, 80 * MiB);
    CHECK(one.alloc(&b, 64 * MiB) && m.in_use == 64 * MiB);
    one.free(b);
    CHECK(two.alloc(&a, 80 * MiB));
    two.recycle(a, 80 * MiB);
    CHECK(one.alloc_exact(&b, 30 * MiB + 5) && m.in_use == 30 * MiB + 5);
    one.free(b);
    CHECK(two.alloc(&a, 80 * MiB));
    two.free(a);
  }
  m.room = MiB;
  CHECK(!one.alloc_exact(&b, 2 * MiB) && b == nullptr && m.live.empty());
}

// With a budget nothing is rounded or kept.
static void budget() {
  Memory m;
  Pool::Peers peers;
  Pool pool(Fake{&m}, peers);
  pool.keeps = false;
  void* a;
  CHECK(pool.alloc(&a, 9 * MiB + 1) && m.in_use == 9 * MiB + 1);
  pool.recycle(a, 9 * MiB + 1);
  CHECK(m.live.empty());
}

static void threads() {
  Memory m;
  Pool::Peers peers;
  Pool pool(Fake{&m}, peers);
  std::mutex mu;
  std::map<void*, int> held;
  std::vector<std::thread> ts;
  for (int t = 0; t < 4; ++t)
    ts.emplace_back([&, t] {
      for (int r = 0; r < 2000; ++r) {
        const size_t bytes = (size_t)(1 + (r * 7 + t * 3) % 40) * MiB;
        void* p;
        CHECK(pool.alloc(&p, bytes));
        {
          std::lock_guard<std::mutex> g(mu);
          CHECK(held[p]++ == 0);  // one owner at a time
        }
        if (r % 97 == 0) pool.drop();
        {
          std::lock_guard<std::mutex> g(mu);
          --held[p];
        }
        Pool::Release give_back(pool);
        give_back(p, bytes);
      }
    });
  for (auto& t : ts) t.join();
  pool.drop();
  CHECK(m.live.empty());
}

int main(int argc, char** argv) {
  const struct {
    const char* name;
    void (*run)();
  } all[] = {{"reuse", reuse},
             {"refused_wait", refused_wait},
             {"allocation_failure", allocation_failure},
             {"full_pool", full_pool},
             {"larger_cycle", larger_cycle},
             {"peers", peers},
             {"budget", budget},
             {"threads", threads}};
  for (const auto& s : all)
    if (argc > 1 && !std::strcmp(argv[1], s.name)) {
      s.run();
      std::printf("%s ok\n", s.name);
      return 0;
    }
  return 2;
}
