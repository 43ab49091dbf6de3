// How a decompression call is cut into tiles, and which calls its tables can hold.  No HIP in here: the host tests compile it by itself.
#pragma once

#include <stdint.h>

namespace rgc {

// 8192 positions unless the messages are dense or the call is small (tile_log_for()): most of a tile's instructions
// (window checks, map clearing, barriers) are paid per tile, not per position; 16384 leaves room for one workgroup per CU only.
constexpr int kTileShift = 13;
constexpr int kTile = 1 << kTileShift;            // dense positions owned by one workgroup (any number of workers)
// The tile kernel comes in three sizes, four lanes a worker: 256 threads for up to 64 workers, 512 for up to 128, 1024 for up to
// 256.  ResNet-50 set, 256 workers, 0.1 %: 76 us against 257 us in the kernel for any number of workers
// plus 36 us for the table it needs.  256 threads / 512: 16 workers on the VGG16 set 107 / 125 us, on 20 M elements at 0.4 % 32 / 53.
constexpr uint32_t kFewWorkers = 64, kFastWorkers = 128, kFastWorkersMax = 256;

// Positions a decompression tile (its logarithm).  A worker has 17 to 32 of its entries in registers; a tile that holds more of them
// fetches the rest from memory one round trip after the other, and has more colliding positions than rows.  A smaller tile in turn
// pays the steps of a tile more often, 512 threads more dearly than 256.  us per call with 2048 / 4096 / 8192 positions, 20 M
// elements: 8 workers 0.2 % 45 / 22 / 31, 0.4 % 47 / 30 / 66, 0.8 % 70 / 68 / 136, 6 % 947 / 995 / 2979; 64 workers 0.05 % 48 / 24 / 24,
// 0.2 % 54 / 28 / 39, 0.4 % 59 / 44 / 92; 128 workers 0.05 % 67 / 42 / 27, 0.2 % 78 / 50 / 52, 0.4 % 85 / 113 / 135; 200 workers
// 0.2 % 150 / 91 / 123, 10 M elements 0.4 % 95 / 124 / 157.  At 0.1 % and up to 64 workers it is the number of workgroups: ten tensors
// of 2 M elements 8.7 / 7.8 / 8.9, ResNet-50 set (26 M) - / 25.9 / 26.9, 64 M - / 59 / 55.
// From 65 workers on, where 4096 and 8192 positions meet moves with the workers, whose entries collide: entries of each in 8192 positions,
// us with 4096 / 8192, ResNet-50 set: 65 workers 13.9 48.1 / 42.7, 16.4 51.1 / 48.2, 20.5 54.6 / 64.2; 100 workers 13.9 54.8 / 48.7, 16.4
// 56.4 / 60.2; 128 workers 13.9 59.1 / 52.6, 16.4 61.9 / 64.7; 160 workers 13.9 96 / 86, 15.6 99 / 111; 200 workers 11.5 106 / 78, 13.9 108 / 103,
// 16.4 112 / 158; 256 workers 11.5 119 / 101, 13.9 123 / 165; VGG16 set, 65 workers 16.4 208 / 194.
inline uint32_t tile_log_for(int64_t elements, int64_t entries, int32_t workers) {
  if (workers < 1 || workers > static_cast<int32_t>(kFastWorkersMax)) return kTileShift;
  const double per = static_cast<double>(entries) * kTile / (static_cast<double>(elements) * workers);   // entries of a worker in 8192 positions
  if (workers <= static_cast<int32_t>(kFewWorkers)) return per > 64.0 ? 11 : per > 11.0 || elements < (int64_t(32) << 20) ? 12 : 13;
  return per > 22.0 ? 11 : per > 18.4 - workers / 48.0 ? 12 : 13;
}

// How many 16-byte stores a lane of the tile kernel has under way before it waits for them (0: as the kernel does without such a rule).
// Where a tile is little more than its stores and the dense buffers outgrow the memory-side cache, the memory takes them the faster the
// fewer come at once, down to what keeps it busy, and that depends on the time the tile's entries take.  us without the rule / with 1 / 2 /
// 4 / 8 stores, VGG16 set: 3 workers 0.02 % (5 entries of all workers in 8192 positions) 121 / 112 / 117 / 121 / 123, 16 workers 0.01 % (13)
// 123 / 118 / 108 / 121 / 123, 4 workers 0.05 % (16) 120 / 125 / 111 / 104 / 111, 16 workers 0.02 % (26) 121 / 124 / 109 / 104 / 117, 64 workers
// 0.01 % (52) 122 / 131 / 116 / 108 / 115, 8 workers 0.1 % (66) 103 / 131 / 117 / 110 / 106; tiles of 4096, 2 workers 0.2 % (33) 125 / 111 /
// 121 / 125; from 65 workers on 65 of 0.01 % (53) 131 / 111 / 119 / 124, 128 of 0.01 % (105) 132 / 129 / 122 / 118, 100 of 0.02 % (164) 109 / 129 /
// 122 / 118.  66 M elements: 16 workers 0.02 % 66 / 64 / 58 / 65.  Smaller buffers, without / with the rule: 50 M elements, 4 workers 0.05 %
// 48.2 / 45.8, 2 workers 47.2 / 47.3, 44 M 41.3 / 42.9, 41.7 / 44.4, 36 M 33.8 / 36.4, 34.6 / 37.7.
inline uint32_t stores_at_once(int64_t elements, int64_t entries, int32_t workers, uint32_t tile_log) {
  if (elements < (int64_t(48) << 20) || workers < 1 || workers > static_cast<int32_t>(kFastWorkers)) return 0;
  const double in_8192 = static_cast<double>(entries) * kTile / static_cast<double>(elements);   // entries of all workers in 8192 positions
  if (workers > static_cast<int32_t>(kFewWorkers)) return tile_log != 13 || in_8192 > 120.0 ? 0 : in_8192 > 90.0 ? 2 : 1;
  if (tile_log == 12) return in_8192 > 40.0 ? 0 : 1;
  return tile_log != 13 || in_8192 < 4.5 || in_8192 > 60.0 ? 0 : in_8192 > 30.0 ? 4 : in_8192 > 9.0 ? 2 : 1;
}

// Only the kernel for any number of workers reads the offset table (a word per worker and tile), which one workgroup per 1024 entries
// of a message builds.
constexpr bool needs_offset_table(int32_t workers) { return workers > static_cast<int32_t>(kFastWorkersMax); }

// Whether the tables' 32-bit offsets reach: `columns` are the tiles and one more per layer, `blocks` the workgroups that build the table.
constexpr bool tables_reach(uint64_t tiles, uint64_t columns, uint64_t blocks, int32_t workers) {
  const uint64_t words = needs_offset_table(workers) ? columns * static_cast<uint64_t>(workers) : 0u;
  return tiles <= 0x7FFFFFFFull && columns <= 0xFFFFFFFFull && blocks <= 0x7FFFFFFFull && words <= 0xFFFFFFFFull;
}

}  // namespace rgc
