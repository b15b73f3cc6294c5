// Numbers of a tree's cells, for the host and the device.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define OCTGRAV_HD __host__ __device__
#else
#define OCTGRAV_HD
#endif

namespace octgrav {

// Most cells of a tree: the walks' queue entries hold cell id << 3.
constexpr int64_t kMaxCells = (int64_t(1) << 29) - 1;

// Cells before a block's cells of a level.  A valid input may have more than
// 2^31 (one particle per leaf and 3.5e8 particles of which every two coincide:
// 12 chain cells per pair), so they are added up in 64 bits, and the count that
// the host refuses such a tree by is exact.
using CellSum = int64_t;

// The number the block's first of them is written under: past the limit the
// limit itself, which no cell array holds, so that the numbers that follow it
// (at most a block's particles more) stay positive and outside every array.
OCTGRAV_HD inline int32_t cell_number(CellSum before) {
  return before < kMaxCells ? (int32_t)before : (int32_t)kMaxCells;
}

}  // namespace octgrav
