// Host checks of the memory kept between calls (csrc/workspace.hpp) against the stand-in runtime.
#include <cstdio>
#include <cstring>

#include "../../paper_1510_06897_amd/csrc/workspace.hpp"

using namespace ovl;

static int failed = 0;
#define CHECK(c)                                            \
  do {                                                      \
    if (!(c)) {                                             \
      std::printf("line %d: %s\n", __LINE__, #c);           \
      ++failed;                                             \
    }                                                       \
  } while (0)

constexpr size_t MB = (size_t)1 << 20;

// a handle that ends while work on some stream still reads its memory
static void destroy_refused() {
  ihipStream s;
  fake().streams.insert(&s);
  Block b;
  CHECK(block_cache().take(64 * MB, &s, b) == hipSuccess);
  void *const p = b.p;
  ++s.issued;  // a kernel that reads the block, on a stream the null stream does not wait for
  fake().sync_refused = true;
  block_cache().retire(b);
  fake().sync_refused = false;
  CHECK(b.p == nullptr);
  CHECK(fake().live.count(p) == 0);  // hipFree, which waits: not kept for another user
  Block c;
  CHECK(block_cache().take(64 * MB, nullptr, c) == hipSuccess && c.p != p);
  // and one that ends as it should: kept, no wait left for its next user
  void *const q = c.p;
  block_cache().retire(c);
  const int waits = fake().waits;
  CHECK(block_cache().take(64 * MB, &s, c) == hipSuccess && c.p == q && fake().waits == waits);
  block_cache().retire(c);
  fake().streams.erase(&s);
}

// a handle of device 1 that ends while device 0 is current: the wait is for device 1
static void destroy_elsewhere() {
  ihipStream s;
  s.device = 1;
  fake().streams.insert(&s);
  fake().device = 1;
  Block b;
  CHECK(block_cache().take(64 * MB, &s, b) == hipSuccess);
  ++s.issued;
  fake().device = 0;
  block_cache().retire(b);
  CHECK(fake().device == 0 && s.ended == s.issued);
  fake().streams.erase(&s);
}

// a handle made on a captured stream takes no kept block, whatever there is; nor does a small one
static void create() {
  Block b;
  CHECK(block_cache().take_handle(64 * MB, nullptr, b) == hipSuccess && b.evt);
  void *const kept = b.p;
  block_cache().retire(b);
  ihipStream s;
  fake().streams.insert(&s);
  s.capturing = true;
  const int waits = fake().waits;
  CHECK(block_cache().take_handle(64 * MB, &s, b) == hipSuccess && b.p != kept && fake().waits == waits);
  CHECK(fake().live[b.p] == 64 * MB);
  s.capturing = false;
  void *const p = b.p;
  block_cache().retire(b);
  CHECK(fake().live.count(p) == 0);
  CHECK(block_cache().take_handle(MB / 8, &s, b) == hipSuccess && fake().live[b.p] == MB / 8);
  void *const q = b.p;
  block_cache().retire(b);
  CHECK(fake().live.count(q) == 0 && fake().live.count(kept) == 1);
  // given back half made
  CHECK(block_cache().take_handle(MB / 8, &s, b) == hipSuccess);
  block_cache().give(b, &s);
  CHECK(b.p == nullptr && fake().live.size() == 1);
  CHECK(block_cache().take_handle(64 * MB, &s, b) == hipSuccess && b.p == kept);
  block_cache().give(b, &s);
  fake().streams.erase(&s);
}

// every allocation of the library that runs out of memory gets what is kept, in blocks and in the pool
static void room() {
  Block b, c;
  CHECK(block_cache().take(6000 * MB, nullptr, b) == hipSuccess);
  block_cache().give(b, nullptr);
  CHECK(fake().live.size() == 1);
  fake().free -= 1000 * MB;  // freed into the pool, which keeps it
  fake().pool_free = 1000 * MB;
  size_t all = fake().total;
  auto fill = [&](size_t left) {  // other allocators take the rest
    void *p = nullptr;
    CHECK(hipMalloc(&p, fake().free - left) == hipSuccess);
    return p;
  };
  void *rest = fill(100 * MB), *p = nullptr;
  // a deflation basis or a graph's vector, out of the kept block
  CHECK(block_cache().with_room([&] { return hipMalloc(&p, 5000 * MB); }) == hipSuccess);
  CHECK(fake().live.size() == 2 && fake().pool_free == 0);
  (void)hipFree(p);
  // work space out of the pool's free memory; a small one from the pool itself out of a kept block
  fake().pool_free = 1000 * MB, fake().free -= 1000 * MB;
  (void)hipFree(rest);
  rest = fill(100 * MB);
  CHECK(block_cache().take(1000 * MB, nullptr, c) == hipSuccess);
  block_cache().give(c, nullptr);
  void *rest2 = fill(0);
  CHECK(block_cache().with_room([&] { return hipMallocAsync(&p, MB, nullptr); }) == hipSuccess);
  (void)hipFreeAsync(p, nullptr);
  // a handle's memory, kept or plain
  for (size_t n : {MB, 64 * MB}) {
    Block k, h;
    CHECK(block_cache().take(500 * MB, nullptr, k) == hipSuccess);
    block_cache().give(k, nullptr);
    void *r = fill(0);
    CHECK(block_cache().take_handle(n, nullptr, h) == hipSuccess);
    block_cache().retire(h);
    (void)hipFree(r);
  }
  // what cannot be had is an error, with nothing left behind
  Block none;
  CHECK(block_cache().take(2 * all, nullptr, none) == hipErrorOutOfMemory && !none.p && !none.evt);
  CHECK(block_cache().take_handle(2 * all, nullptr, none) == hipErrorOutOfMemory && !none.p);
  (void)hipFree(rest);
  (void)hipFree(rest2);
  // on request, and no more than an eighth of the device is kept without one
  for (int i = 0; i < 5; ++i) {
    Block k;
    CHECK(block_cache().take((i + 1) * 1000 * MB, nullptr, k) == hipSuccess);
    block_cache().give(k, nullptr);
  }
  size_t kept = 0;
  for (auto &m : fake().live) kept += m.second;
  CHECK(kept <= all / 8 && kept > 0);
  block_cache().release();
  CHECK(fake().live.empty() && fake().free == all && fake().mode == hipStreamCaptureModeGlobal);
}

// independent streams whose calls overlap use different blocks, within the limit
static void streams() {
  ihipStream s1, s2;
  fake().streams.insert(&s1);
  fake().streams.insert(&s2);
  auto call = [](hipStream_t s, size_t bytes) {  // take, enqueue, give back at once: as a library call does
    Block b;
    CHECK(block_cache().take(bytes, s, b) == hipSuccess);
    void *const p = b.p;
    ++s->issued;
    block_cache().give(b, s);
    return p;
  };
  auto ended = [](hipStream_t s) { s->ended = s->issued; };
  const int waits = fake().waits;
  void *const p1 = call(&s1, 64 * MB), *const p2 = call(&s2, 64 * MB);
  CHECK(p1 != p2 && fake().waits == waits);
  for (int i = 0; i < 8; ++i) CHECK(call(&s1, 64 * MB) == p1 && call(&s2, 64 * MB) == p2);
  CHECK(fake().live.size() == 2);
  // a third stream waits for nobody; once the first has ended its block is taken
  ihipStream s3;
  fake().streams.insert(&s3);
  ended(&s1);
  const int w = fake().waits;
  CHECK(call(&s3, 64 * MB) == p1 && fake().waits == w && fake().live.size() == 2);
  // above the limit (8 GB here) the pending block is waited for, and below it when there is no memory
  ended(&s1), ended(&s2), ended(&s3);
  block_cache().release();
  void *const q1 = call(&s1, 7000 * MB);
  CHECK(call(&s2, 7000 * MB) == q1 && fake().waits > w && fake().live.size() == 1);
  ended(&s1), ended(&s2);
  block_cache().release();
  void *const r1 = call(&s1, 1000 * MB);
  void *rest = nullptr;
  CHECK(hipMalloc(&rest, fake().free) == hipSuccess);
  CHECK(call(&s2, 1000 * MB) == r1);
  (void)hipFree(rest);
  ended(&s1), ended(&s2);
  block_cache().release();
  CHECK(fake().live.empty());
  for (ihipStream *s : {&s1, &s2, &s3}) fake().streams.erase(s);
}

int main(int argc, char **argv) {
  const char *what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "destroy")) {
    destroy_refused();
    destroy_elsewhere();
  } else if (!std::strcmp(what, "create")) {
    create();
  } else if (!std::strcmp(what, "room")) {
    room();
  } else if (!std::strcmp(what, "streams")) {
    streams();
  } else {
    std::printf("no check named '%s'\n", what);
    return 2;
  }
  std::printf("%d failed\n", failed);
  return failed != 0;
}
