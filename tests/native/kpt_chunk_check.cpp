// The k-points whose grids are held at a time, and the step down where an
// allocation fails: prints (case, result) pairs for the test.
#include <cstdio>

#include "../../paper_1603_02732_amd/csrc/launch.hpp"

int main() {
  // grids of every k, of some, of one larger than the limit
  for (size_t bytes : {(size_t)1, (size_t)17694720, (size_t)255999999, (size_t)256000001, (size_t)5000000000})
    std::printf("chunk %zu %d\n", bytes, sgo::kpt_grid_chunk(32, bytes));
  // an allocator that grants `room` bytes; 100 bytes beside 10 a k-point
  for (size_t room : {1000u, 420u, 419u, 200u, 110u, 109u}) {
    size_t asked = 0;
    const int c = sgo::largest_chunk(
        32, [](int chunk) { return (size_t)(100 + 10 * chunk); },
        [&](size_t n) {
          asked = n;
          return n <= room;
        });
    std::printf("fit %zu %d %zu\n", room, c, asked);
  }
  return 0;
}
