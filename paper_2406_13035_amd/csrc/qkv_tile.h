// Geometry of the projection's operand tiles: which bytes of X and W every lane loads and where in
// LDS they land.  Plain constexpr functions, used by the kernel in qkv.hip and, without a GPU, by the test
// that enumerates every load of ragged tiles (tests/test_qkv_tile_loads.py).
#pragma once
#include <cstdint>

namespace d2o {
namespace qkv {

constexpr int kBM = 256, kBN = 128, kBK = 64;  // rows and columns (of X or W) of a k-tile; kBN: one head
constexpr int kHeadsPerWg = 2, kThreads = 256;
constexpr int kLd = kBK;                     // LDS pitch (elements) of the operand tiles: 128 bytes = eight 16-byte chunks,
                                             // chunk k of row r stored at position k ^ ((r >> 1) & 7): the 16 lanes of a
                                             // 128-bit access phase then cover all 64 banks once
constexpr int kLoads = 8;                    // loads per wavefront, k-tile and operand; one fills 8 rows (64 lanes x 16 bytes)

// The part of a load's offset that no loop changes: this lane's row in load 0 (the first of the wavefront's 64) and
// its chunk, which depends on the load's parity only.
constexpr uint32_t lane_offset(int w, int lane, bool odd, uint32_t row_bytes) {
  return uint32_t(w * 64 + (lane >> 3)) * row_bytes + uint32_t((((lane & 7) ^ (lane >> 4)) ^ (odd ? 4 : 0)) << 4);
}
// What load i (0..7) of k-tile kt adds to it, the same for all lanes.  A buffer load compares only the
// lane's offset with the buffer's size, not the scalar one, so this belongs in the lane's.
constexpr uint32_t load_step(int i, int kt, uint32_t row_bytes) {
  return uint32_t(kt) * (kBK * 2) + uint32_t(i * 8) * row_bytes;
}
// The LDS element at which the wavefront's 64 chunks of load i begin, one after the other by lane.
constexpr int lds_start(int w, int i) { return (w * kLoads + i) * 8 * kLd; }
// Bytes of a buffer over `rows` rows.
constexpr uint32_t buffer_bytes(int rows, uint32_t row_bytes) { return uint32_t(rows) * row_bytes; }
// Rows up to this wide keep a tile's offsets within 31 bits.
constexpr int kMaxBufferHidden = (1 << 22) - kBK;
// Wider ones: the same load's byte from the tile's first row on, held inside the tile's `rows` rows (a row or column
// behind them is replaced by the last one and never used).
constexpr int64_t wide_offset(int w, int lane, int i, int kt, int rows, int64_t row_bytes) {
  const int row = w * 64 + i * 8 + (lane >> 3), last = rows - 1;
  const int64_t col = int64_t(kt) * (kBK * 2) + ((((lane & 7) ^ (lane >> 4)) ^ (i & 1 ? 4 : 0)) << 4);
  return (row < last ? row : last) * row_bytes + (col < row_bytes - 16 ? col : row_bytes - 16);
}

}  // namespace qkv
}  // namespace d2o
