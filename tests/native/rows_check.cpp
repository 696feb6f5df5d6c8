// Host check of segments_are_rows (csrc/qpg_internal.hpp) on the work list of a matrix: against the entries
// themselves (the row of every segment's first entry) instead of the list's row slots.
// Reads <prefix>_ptr.bin / <prefix>_col.bin (int32); prints the rows, the segments and the flag.
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <string>
#include <vector>

#include "qpg_internal.hpp"

using namespace qpg;

static std::vector<int32_t> read_all(const std::string& f) {
  std::ifstream in(f, std::ios::binary | std::ios::ate);
  const size_t n = (size_t)in.tellg();
  in.seekg(0);
  std::vector<int32_t> v(n / sizeof(int32_t));
  in.read(reinterpret_cast<char*>(v.data()), (std::streamsize)n);
  return v;
}

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  const std::string pre = argv[1];
  const auto rp = read_all(pre + "_ptr.bin"), col = read_all(pre + "_col.bin");
  const int nrows = (int)rp.size() - 1;
  const TilePlan t = make_tiles(rp, col.data(), nrows, std::atoi(argv[2]),
                                TileParams{8192, kTileNnz, kPlainNnz, kTileMaxRows});
  // the segment that row r would own as number r, and how many segments each row has
  std::vector<int32_t> place((size_t)std::max<int64_t>(t.nslot, 1), -1), count((size_t)nrows + 1, 0);
  for (size_t q = 0; q < t.slotidx.size(); ++q) place[t.slotidx[q]] = (int32_t)q;
  bool rows = t.nslot == nrows;
  for (size_t j = 0; j < t.segslot.size(); ++j) {
    if (t.segslot[j] < 0 || t.llen[j] <= 0) continue;
    int r = 0;
    while (rp[r + 1] <= t.lstart[j]) ++r;
    ++count[r];
    if (place[t.segslot[j]] != r) rows = false;
  }
  for (int r = 0; r < nrows; ++r) rows = rows && count[r] <= 1;
  std::printf("rows %d segments %ld flag %d entries %d\n", nrows, (long)t.nslot, (int)segments_are_rows(t), (int)rows);
  return 0;
}
