// Bookkeeping of the handle's scratch blocks (scratch.hpp) on the stand-in
// runtime.  Each argument names a test; the first failing check is printed.
#include <cstdio>
#include <cstring>
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

int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    if (!std::strcmp(argv[i], "errors") && errors()) return 1;
  }
  std::printf("ok\n");
  return 0;
}
