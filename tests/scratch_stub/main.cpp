// Bookkeeping of the handle's scratch blocks (scratch.hpp) on the stand-in
// runtime.  Each argument names a test; the first failing check is printed.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../../paper_2109_13406_amd/csrc/scratch.hpp"

#define CHECK(x)                                             \
  do {                                                       \
    if (!(x)) {                                              \
      std::printf("line %d: %s\n", __LINE__, #x);            \
      return 1;                                              \
    }                                                        \
  } while (0)

using mpdd::ScratchCache;

static bool no_memory = false;
void* operator new(size_t n) {
  if (no_memory && n >= 320) throw std::bad_alloc();   // (a list of eight blocks or more)
  return std::malloc(n);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

// A failing get or put leaves no error pending and loses no block.
static int errors() {
  StubStream s;
  for (const char* what : {"wait", "event", "malloc"}) {
    ScratchCache c;
    void *p = nullptr, *q = nullptr;
    if (!std::strcmp(what, "wait")) {            // a kept block to wait for
      CHECK(c.get(&p, 1 << 20, &s) == hipSuccess);
      CHECK(c.put(p, &s) == hipSuccess);
    }
    if (!std::strcmp(what, "malloc")) stub::limit = 1 << 10;
    stub::fail.insert(what);
    CHECK(c.get(&p, 1 << 20, &s) != hipSuccess);
    CHECK(hipGetLastError() == hipSuccess);
    stub::fail.clear();
    stub::limit = SIZE_MAX;
    CHECK(c.get(&q, 1 << 20, &s) == hipSuccess);
    CHECK(c.put(q, &s) == hipSuccess);
    c.close();
    CHECK(stub::live.empty());
  }
  ScratchCache c;
  void* p = nullptr;
  CHECK(c.get(&p, 1 << 20, &s) == hipSuccess);
  stub::fail.insert("record");
  CHECK(c.put(p, &s) != hipSuccess);
  CHECK(hipGetLastError() == hipSuccess);
  c.close();
  CHECK(stub::live.empty());
  return 0;
}

// Free blocks: at most 8, and 8 GiB where they are more than one.
static int bounds() {
  const size_t GB = (size_t)1 << 30;
  {
    // streams at work at once, 3 GiB each: nobody's work is waited for
    ScratchCache c;
    StubStream s[6];
    std::vector<void*> p(6);
    for (int i = 0; i < 6; ++i) {
      CHECK(c.get(&p[i], 3 * GB, &s[i]) == hipSuccess);
      s[i].pending = true;
    }
    const int waits = stub::calls["wait"] + stub::calls["sync"] + stub::calls["event_sync"];
    for (int i = 0; i < 6; ++i) CHECK(c.put(p[i], &s[i]) == hipSuccess);
    CHECK(waits == stub::calls["wait"] + stub::calls["sync"] + stub::calls["event_sync"]);
    CHECK(stub::total() <= 8 * GB);
    c.close();
    CHECK(stub::live.empty());
  }
  {
    // one after the other on streams of their own: the newest stay
    ScratchCache c;
    StubStream s[20];
    void* p = nullptr;
    size_t last = 0;
    for (int i = 0; i < 20; ++i) {
      const size_t n = ((size_t)(20 + i)) << 26;     // 1.25 to 2.4 GiB, each too small for the next
      CHECK(c.get(&p, n, &s[i]) == hipSuccess);
      CHECK(c.put(p, &s[i]) == hipSuccess);
      last = n;
      CHECK(stub::total() <= 8 * GB && stub::live.size() <= 8);
    }
    const int mallocs = stub::calls["malloc"];
    CHECK(c.get(&p, last, &s[19]) == hipSuccess && stub::calls["malloc"] == mallocs);
    CHECK(c.put(p, &s[19]) == hipSuccess);
    // a single block beyond the bound is kept, and takes the others' place
    for (int rep = 0; rep < 3; ++rep) {
      CHECK(c.get(&p, 20 * GB, &s[0]) == hipSuccess);
      CHECK(c.put(p, &s[0]) == hipSuccess);
      CHECK(stub::live.size() == 1 && stub::total() >= 20 * GB);
    }
    CHECK(stub::calls["malloc"] == mallocs + 1);
    CHECK(c.get(&p, 1 << 20, &s[1]) == hipSuccess);  // (its block is used, not another)
    CHECK(c.put(p, &s[1]) == hipSuccess);
    CHECK(stub::live.size() == 1);
    c.close();
    CHECK(stub::live.empty());
  }
  {
    // many small ones, more in use than are kept
    ScratchCache c;
    StubStream s;
    std::vector<void*> p(30);
    for (auto& x : p) CHECK(c.get(&x, 1 << 20, &s) == hipSuccess);
    CHECK(stub::live.size() == 30);
    for (auto& x : p) CHECK(c.put(x, &s) == hipSuccess);
    CHECK(stub::live.size() == 8);
    // under capture: the pool itself
    s.capturing = true;
    void* q = nullptr;
    CHECK(c.get(&q, 1 << 20, &s) == hipSuccess);
    CHECK(stub::live.size() == 9);
    CHECK(c.put(q, &s) == hipSuccess);
    CHECK(stub::live.size() == 8);
    c.close();
    CHECK(stub::live.empty());
  }
  return 0;
}

// Scratch that the caller can do without: where there is no memory nothing that is
// kept is given up, nothing is waited for, and the driver is not asked every time.
static int optional() {
  const size_t MB = (size_t)1 << 20;
  ScratchCache c;
  StubStream s;
  void *p = nullptr, *q = nullptr;
  CHECK(c.get(&p, 4 * MB, &s) == hipSuccess);
  CHECK(c.put(p, &s) == hipSuccess);
  stub::limit = 64 * MB;
  auto asked = [] { return stub::calls["malloc"]; };
  auto waits = [] {
    return stub::calls["wait"] + stub::calls["sync"] + stub::calls["event_sync"] +
           stub::calls["free"];
  };
  int m = asked();
  const int w = waits();
  CHECK(c.get(&q, 100 * MB, &s, true) != hipSuccess);
  CHECK(hipGetLastError() == hipSuccess);
  CHECK(asked() == m + 1 && waits() == w && stub::live.size() == 1);
  for (int i = 0; i < 64; ++i) CHECK(c.get(&q, 100 * MB, &s, true) != hipSuccess);
  CHECK(asked() == m + 1 && waits() == w);
  CHECK(c.get(&q, 100 * MB, &s, true) != hipSuccess);      // asked again
  CHECK(asked() == m + 2 && waits() == w && stub::live.size() == 1);
  // smaller ones and required ones are not held up, and the kept block serves
  CHECK(c.get(&q, 2 * MB, &s, true) == hipSuccess && q == p);
  CHECK(c.put(q, &s) == hipSuccess);
  CHECK(c.get(&q, 32 * MB, &s, true) == hipSuccess);       // (in place of the small one)
  CHECK(stub::live.size() == 1);
  CHECK(c.put(q, &s) == hipSuccess);
  stub::limit = SIZE_MAX;
  CHECK(c.get(&q, 100 * MB, &s) == hipSuccess);
  CHECK(c.put(q, &s) == hipSuccess);
  CHECK(c.get(&q, 100 * MB, &s, true) == hipSuccess);      // its block is kept now
  CHECK(c.put(q, &s) == hipSuccess);
  c.close();
  CHECK(stub::live.empty());
  return 0;
}

// No host memory for the list of blocks: an error, not an exception.
static int host_memory() {
  StubStream s;
  ScratchCache c;
  std::vector<void*> p(40, nullptr);
  int failed = 0;
  for (auto& x : p) {
    no_memory = true;
    const hipError_t e = c.get(&x, 1 << 20, &s);
    no_memory = false;
    if (e != hipSuccess) {
      x = nullptr;
      ++failed;
      CHECK(hipGetLastError() == hipSuccess);
      CHECK(c.get(&x, 1 << 20, &s) == hipSuccess);
    }
  }
  CHECK(failed > 0 && stub::live.size() == 40);
  for (auto x : p) CHECK(c.put(x, &s) == hipSuccess);
  c.close();
  CHECK(stub::live.empty());
  return 0;
}

int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    if (!std::strcmp(argv[i], "errors") && errors()) return 1;
    if (!std::strcmp(argv[i], "bounds") && bounds()) return 1;
    if (!std::strcmp(argv[i], "optional") && optional()) return 1;
    if (!std::strcmp(argv[i], "host_memory") && host_memory()) return 1;
  }
  std::printf("ok\n");
  return 0;
}
