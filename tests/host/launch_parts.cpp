// for_each_launch over workgroup counts up to the most the launchers take,
// block sizes and steps: the parts follow each other, cover every workgroup
// once, begin at multiples of the step, and none is a launch that HIP refuses;
// an error ends the loop and is returned.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "grid.hpp"

#define CHECK(c)                                                          \
  do {                                                                    \
    if (!(c)) {                                                           \
      std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
      std::exit(1);                                                       \
    }                                                                     \
  } while (0)

int main() {
  const int64_t limit = int64_t(1) << 32, most_blocks = (int64_t(1) << 31) - 1;
  for (int threads : {64, 128, 256, 512, 1024}) {
    for (int64_t step : {int64_t(1), int64_t(1024)}) {
      const int64_t edge = limit / threads;
      for (int64_t blocks : {int64_t(0), int64_t(1), step, edge - 1, edge, edge + 1, edge + step, 2 * edge + 7, most_blocks}) {
        if (blocks > most_blocks) continue;
        int64_t next = 0, parts = 0;
        const rdf2v_status st = rdf2v::for_each_launch(blocks, threads, step, [&](int64_t first, int64_t count) {
          CHECK(first == next && first % step == 0 && count > 0);
          CHECK(count * threads < limit);
          next = first + count;
          ++parts;
          return RDF2V_OK;
        });
        CHECK(st == RDF2V_OK && next == blocks);
        CHECK(blocks >= edge || parts <= 2);
        CHECK(blocks > (edge - 1) / step * step || parts == (blocks > 0 ? 1 : 0));
        int calls = 0;
        const rdf2v_status bad = rdf2v::for_each_launch(blocks, threads, step, [&](int64_t, int64_t) {
          ++calls;
          return RDF2V_ERR_HIP;
        });
        CHECK(blocks == 0 ? bad == RDF2V_OK && calls == 0 : bad == RDF2V_ERR_HIP && calls == 1);
      }
    }
  }
  std::puts("launch parts: ok");
  return 0;
}
