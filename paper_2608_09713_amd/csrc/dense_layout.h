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
constexpr uint64_t kDenseProducts = uint64_t(1) << 17;  // products of a row that may go by cells, at least
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

// Whether the `rows` rows of at least kDenseProducts products, with so many
// entries and products in all, go by cells in a matrix of m rows and nnz
// entries.  Every cell of a row looks up every entry of the row, so the
// lookups are not to outnumber the products; the products are to outnumber
// the matrix's entries (a lower bound of them), as the table of long columns
// takes a pass over those.  (All such rows or none: the few that would be left
// to one workgroup each would set the time.  Heavy rows' passes with cells
// against one workgroup per row, by lookups per product: R-MAT scale 18 in f32
// (0.09) 13.1 against 18.4 ms, scale 19 (0.13) 37.1 against 35.2; rows of 4,096
// and 8,192 entries of 2^18 rows (0.6, 0.8) 7.7 and 7.9 against 8.5 and 9.9, of
// 2^20 rows (0.7, 1.3, 1.8) 101, 65 and 28 against 95, 59 and 15; rows of 8,192
// entries of 2^22 rows (7) 71 against 19.)
constexpr bool dense_rows_pay(int64_t rows, uint64_t entries, uint64_t products, int64_t nnz, int64_t m) {
    return rows > 0 && m <= kDenseMaxRows && entries * uint64_t(dense_cells(m)) <= products &&
           rows * int64_t(kDenseProducts) >= nnz;
}

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
