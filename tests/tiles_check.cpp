// Host check of rgc_tiles.h: which decompression calls the tables can hold, for lists of equal layers and messages.
#include <cstdio>
#include <initializer_list>

#include "../paper_1808_04357_amd/csrc/rgc_tiles.h"

using namespace rgc;

namespace {

int faults = 0;

void expect(const char* what, bool got, bool want) {
  if (got == want) return;
  std::printf("%s: %d, expected %d\n", what, got, want);
  ++faults;
}

bool accepted(int64_t layers, int64_t n, int32_t workers, int64_t entries_each) {
  const uint32_t log = tile_log_for(layers * n, layers * workers * entries_each, workers);
  const uint64_t tiles = static_cast<uint64_t>(layers * ((n + (int64_t(1) << log) - 1) >> log));
  const uint64_t blocks = needs_offset_table(workers) ? static_cast<uint64_t>(layers * workers * ((entries_each + 1023) / 1024)) : 0u;
  return tables_reach(tiles, tiles + static_cast<uint64_t>(layers), blocks, workers);
}

}  // namespace

int main() {
  // The largest buffers a card holds, in any tile size: up to 256 workers no table stands against them.
  const int64_t n = int64_t(1) << 30;
  for (int32_t workers : {1, 64, 65, 128, 129, 256})
    for (int64_t per_8192 : {1, 12, 15, 25, 70}) {
      char what[80];
      std::snprintf(what, sizeof what, "64 layers of 2^30, %d workers, %d entries in 8192", workers, static_cast<int>(per_8192));
      expect(what, accepted(64, n, workers, (n >> kTileShift) * per_8192), true);
    }
  // With more workers the table has a word per worker and column, numbered in 32 bits.
  expect("257 workers, 2^23 tiles", accepted(64, n, 257, 1000), true);
  expect("511 workers, 2^23 tiles", accepted(64, n, 511, 1000), true);
  expect("512 workers, 2^23 tiles", accepted(64, n, 512, 1000), false);
  // Where tiles of 4096 positions begin to be the faster ones (entries of a worker in 8192 positions).
  const struct { int32_t workers; double at_13, at_12; } lines[] = {{65, 16.4, 20.5}, {80, 15.6, 18.8}, {96, 15.6, 17.2}, {112, 15.5, 17.2}, {128, 13.9, 16.4},
                                                                    {144, 13.9, 17.2}, {160, 13.9, 15.6}, {180, 13.9, 15.6}, {200, 12.3, 16.4}, {256, 11.5, 13.9}};
  for (const auto& l : lines) {
    char what[80];
    std::snprintf(what, sizeof what, "%d workers, tiles of 8192 at %.1f and of 4096 at %.1f", l.workers, l.at_13, l.at_12);
    const auto log = [&](double per) { return tile_log_for(int64_t(100) << 20, static_cast<int64_t>(per * 12800.0 * l.workers), l.workers); };
    expect(what, log(l.at_13) == 13 && log(l.at_12) == 12, true);
  }
  // Stores at once, by the entries of all workers in 8192 positions: 0 where a tile is not paced.
  const struct { int64_t elements; int32_t workers; double in_8192; uint32_t log, want; } paces[] = {
      {64 << 20, 3, 4.0, 13, 0}, {64 << 20, 3, 5.0, 13, 1}, {64 << 20, 16, 13.0, 13, 2}, {64 << 20, 64, 52.0, 13, 4}, {64 << 20, 64, 66.0, 13, 0},
      {64 << 20, 2, 33.0, 12, 1}, {64 << 20, 3, 49.0, 12, 0}, {64 << 20, 1, 33.0, 11, 0}, {64 << 20, 65, 53.0, 13, 1}, {64 << 20, 128, 105.0, 13, 2},
      {64 << 20, 100, 164.0, 13, 0}, {64 << 20, 129, 53.0, 13, 0}, {48 << 20, 3, 5.0, 13, 1}, {(48 << 20) - 1, 3, 5.0, 13, 0}, {0, 1, 0.0, 13, 0}};
  for (const auto& p : paces) {
    char what[80];
    std::snprintf(what, sizeof what, "%d workers, %.0f entries in 8192 of %lld", p.workers, p.in_8192, static_cast<long long>(p.elements));
    expect(what, stores_at_once(p.elements, static_cast<int64_t>(p.in_8192 * static_cast<double>(p.elements) / kTile), p.workers, p.log) == p.want, true);
  }
  std::printf(faults == 0 ? "tiles_check ok\n" : "tiles_check: %d faults\n", faults);
  return faults == 0 ? 0 : 1;
}
