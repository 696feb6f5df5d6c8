// Host check of the graph kernels' index arithmetic at the end of the int32 range: entry_ahead against 64-bit
// sums, and the pieces of make_pieces (csrc/host_prep.cpp) on rows that end at 2^31 - 1. Built with the
// undefined-behaviour sanitizer, which ends the program at a signed overflow.
#include <algorithm>
#include <cstdio>
#include <cstdint>
#include <vector>

#include "qpg_internal.hpp"

using namespace qpg;

#define FAIL(...)             \
  do {                        \
    std::printf(__VA_ARGS__); \
    std::printf("\n");        \
    return 1;                 \
  } while (0)

int main() {
  // k: the first entry of a batch, by: as far as the kernels look ahead (two batches of 1024 and a lane)
  for (int64_t last : {(int64_t)0, (int64_t)700, (int64_t)INT32_MAX - 1, (int64_t)INT32_MAX})
    for (int64_t back : {0, 1, 63, 511, 512, 1023, 1024, 2047, 2048, 4000})
      for (uint32_t by = 0; by < 4096; ++by) {
        const int64_t k = last - back;
        if (k < 0) continue;
        if ((int64_t)entry_ahead((uint32_t)k, by, (uint32_t)last) != std::min(k + (int64_t)by, last)) FAIL("entry %ld + %u", (long)k, by);
      }
  // rows of every kind, the last one ending at 2^31 - 1
  const std::vector<std::vector<int64_t>> cases = {
      {5, 16, 17, 256, 257, 2048, 2049, 3}, {0, 0, 1}, {kPieceNnz - 1}, {kPieceNnz}, {kPieceNnz + 1}, {3, 0}, {INT32_MAX}};
  for (const auto& lens : cases) {
    std::vector<int32_t> ptr(lens.size() + 1);
    int64_t at = INT32_MAX;
    for (size_t r = lens.size(); r-- > 0;) {
      ptr[r + 1] = (int32_t)at;
      at -= lens[r];
    }
    ptr[0] = (int32_t)at;
    const PiecePlan p = make_pieces(ptr.data(), ptr.data() + 1, ptr.data(), (int32_t)lens.size());
    std::vector<int64_t> covered(lens.size(), 0);
    for (size_t i = 0; i < p.pieces.size(); ++i) {
      const Piece& q = p.pieces[i];
      if ((q.k1 < 0) != ((int32_t)i < p.packs)) FAIL("piece %zu is in the wrong part", i);
      if (q.k1 < 0) {
        for (int32_t r = q.row; r < q.k0; ++r) covered[r] += lens[r];
        continue;
      }
      if (q.k0 < ptr[q.row] || q.k0 >= q.k1 || q.k1 > ptr[q.row + 1] || q.k1 - q.k0 > kPieceNnz) FAIL("piece %zu", i);
      covered[q.row] += q.k1 - q.k0;
    }
    for (size_t r = 0; r < lens.size(); ++r)
      if (covered[r] != lens[r]) FAIL("row %zu: %ld of %ld entries", r, (long)covered[r], (long)lens[r]);
  }
  return 0;
}
