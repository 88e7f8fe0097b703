// Test driver for TableCache: commands on stdin, one answer per line.
//   get TAG A B JOIN   sizes of the table handed out, or "none", and how many were built
//   look TAG A B       the same without building
//   hold               keeps a reference to the last table handed out
//   drop               gives up all references kept
//   fail 0|1           builds fail from now on
//   clear
// After each: the cache's bytes, the bytes of the tables alive and those that went.
// Bytes are 76 A B (or 76 A for B = 0); limits are the two arguments.
#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <string>

#include "../../paper_1201_1548_amd/csrc/table_cache.hpp"

using namespace bires;

static size_t alive = 0;
struct Mem {
  size_t n;
  explicit Mem(size_t b) : n(b) { alive += n; }
  ~Mem() { alive -= n; }
};

int main(int, char** argv) {
  TableCache<Mem> c(strtoull(argv[1], nullptr, 10), strtoull(argv[2], nullptr, 10));
  auto size = [](int a, int b) { return (size_t)76 * a * (b ? b : 1); };
  std::vector<std::shared_ptr<Mem>> kept;
  std::shared_ptr<Mem> last;
  bool fail = false;
  int built = 0;
  std::string cmd;
  while (std::cin >> cmd) {
    size_t went = 0;
    {
      TableCache<Mem>::Gone gone;
      if (cmd == "get" || cmd == "look") {
        int tag, a, b, join = 0;
        std::cin >> tag >> a >> b;
        if (cmd == "get") std::cin >> join;
        auto build = [&](int x, int y) {
          if (fail) return std::shared_ptr<Mem>();
          ++built;
          return std::make_shared<Mem>(size(x, y));
        };
        const auto t = cmd == "get" ? c.get(tag, a, b, join, size, build, &gone) : c.look(tag, a, b);
        last = t.mem;
        if (t.mem)
          printf("%d %d", t.a, t.b);
        else
          printf("none 0");
      } else {
        if (cmd == "hold") kept.push_back(last);
        if (cmd == "drop") kept.clear();
        if (cmd == "fail") std::cin >> fail;
        if (cmd == "clear") c.clear(&gone);
        printf("- -");
      }
      went = gone.size();
      last = cmd == "get" || cmd == "look" ? last : nullptr;
    }
    std::shared_ptr<Mem> keep = cmd == "hold" ? nullptr : last;
    printf(" %d %zu %zu %zu\n", built, c.bytes(), alive, went);
  }
  return 0;
}
