// Host-side sizes of the rows that go by cells of output columns (dense.hip):
// cells, the table of long columns and the launches.  Plain C++ (no HIP), so
// that they can be checked on any host.
#pragma once

#include <cstdint>

namespace spsyrk {

constexpr int kCellBits = 13;
constexpr int kCell = 1 << kCellBits;  // output columns per cell
constexpr int kSymCells = 16;          // cells per workgroup of the symbolic pass
constexpr int kDenseThreads = 512;     // threads per workgroup
constexpr int64_t kDenseMaxRows = int64_t(1) << 22;  // rows (and output columns) of the matrix, at most: 512 cells

constexpr int dense_cells(int64_t m) { return int((m + kCell - 1) >> kCellBits); }

// log2 of the positions per block of the table of long columns, for an index
// of `positions` entries over m rows (a table of at most 64 MB), and its blocks
constexpr int dense_block_log(int64_t positions, int64_t m) {
    int b = 4;
    while (((positions >> b) + 2) * int64_t(dense_cells(m)) > (int64_t(1) << 24)) ++b;
    return b;
}
constexpr int64_t dense_blocks(int64_t positions, int blk_log) { return (positions >> blk_log) + 2; }

// Workgroups of the passes over (row, cell) units: the rows in x, the cells
// (groups of kSymCells in the symbolic pass) in y.  x runs fastest, so units
// start cell by cell.  A launch takes fewer than 2^32 threads per dimension
// and 2^16 workgroups in y: one dimension would hold 2^23 units only (65,536
// rows of 2^20), while x takes every row up to 2^23 - 1 and y at most 512.
struct DenseGrid {
    uint32_t x, y;
};
constexpr DenseGrid dense_grid(int64_t nrows, int ncells, bool symbolic) {
    return {uint32_t(nrows), uint32_t(symbolic ? (ncells + kSymCells - 1) / kSymCells : ncells)};
}

}  // namespace spsyrk
