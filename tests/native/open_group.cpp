// qa_open_group.h for tests/test_open_group.py: rows that end where the process's memory does.
#include <sys/mman.h>
#include <unistd.h>

#include <cstdio>

#include "qa_open_group.h"

struct Quad {
  float x, y, z, w;
};

int main() {
  const long page = sysconf(_SC_PAGESIZE);
  char* p = static_cast<char*>(mmap(nullptr, 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
  if (p == MAP_FAILED || mprotect(p + page, page, PROT_NONE) != 0) return 2;
  for (uint32_t live = 1; live <= 257; ++live) {
    float* g = reinterpret_cast<float*>(p + page) - live;
    for (uint32_t i = 0; i < live; ++i) g[i] = (float)(i + 1);
    for (uint32_t group = 0; 4 * group < live; ++group) {
      const Quad q = qa::load_group<Quad>(g, group, live);
      const float x[4] = {q.x, q.y, q.z, q.w};
      for (uint32_t e = 0; e < 4; ++e) {
        const uint32_t i = 4 * group + e;
        if (x[e] != (i < live ? (float)(i + 1) : 0.0f)) {
          printf("live %u, component %u: %g\n", live, i, x[e]);
          return 1;
        }
      }
    }
  }
  return 0;
}
