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
// Rows that may go by cells: those of at least kDenseProducts products, which
// one workgroup would hold for long, and shorter ones that fill their cells,
// of at least kDenseFew products and kDenseFill per lookup.
constexpr uint64_t kDenseProducts = uint64_t(1) << 17;
constexpr uint64_t kDenseFew = uint64_t(1) << 14;
constexpr uint64_t kDenseFill = 64;
constexpr uint64_t kDenseTotal = uint64_t(1) << 25;  // products of the shorter ones in all, at least
constexpr int kDenseSplit = 8;         // cells of a row that pay even for a few rows
constexpr uint64_t kDenseUnits = 512;  // (row, cell) units with fewer cells, at least
constexpr int64_t kDenseMaxRows = int64_t(1) << 22;  // rows (and output columns) of the matrix, at most: 512 cells

constexpr int dense_cells(int64_t m) { return int((m + kCell - 1) >> kCellBits); }

// whether a row may go by cells
constexpr bool dense_row(uint64_t products, uint64_t entries, int ncells) {
    return products >= kDenseProducts || (products >= kDenseFew && entries * uint64_t(ncells) * kDenseFill <= products);
}

// log2 of the positions per block of the table of long columns, for an index
// of `positions` entries over m rows (a table of at most 64 MB), and its blocks
constexpr int dense_block_log(int64_t positions, int64_t m) {
    int b = 4;
    while (((positions >> b) + 2) * int64_t(dense_cells(m)) > (int64_t(1) << 24)) ++b;
    return b;
}
constexpr int64_t dense_blocks(int64_t positions, int blk_log) { return (positions >> blk_log) + 2; }

// What of the rows that may go by cells does, in a matrix of m rows and nnz
// entries: nothing (0), the rows of kDenseProducts products and more (1), the
// shorter ones too (2).
//
// Every cell of a row looks up every entry of the row, so the lookups are not
// to outnumber the products; the products are to outnumber the matrix's
// entries (rows * kDenseProducts is a lower bound of them), as the table of
// long columns takes a pass over those.  (All rows of a kind or none: the few
// that would be left to one workgroup each would set the time.  Heavy rows'
// passes with cells against one workgroup per row, by lookups per product:
// R-MAT scale 18 in f32 (0.09) 13.1 against 18.4 ms, scale 19 (0.13) 37.1
// against 35.2; rows of 4,096 and 8,192 entries of 2^18 rows (0.6, 0.8) 7.7 and
// 7.9 against 8.5 and 9.9, of 2^20 rows (0.7, 1.3, 1.8) 101, 65 and 28 against
// 95, 59 and 15; rows of 8,192 entries of 2^22 rows (7) 71 against 19.)
//
// The shorter rows go too where their cells are full, and where there are
// enough of them to pay for the path's six launches.  (Whole calls in f32,
// without the shorter rows and with them: 4096 rows of 300 entries in 2000
// columns 2.13 and 1.73 ms, 2^14 rows of 100 in 3000 3.44 and 2.82, 2^15 of 100
// in 3000 11.5 and 8.9; 35 to 41 M products 0.92 and 0.91.  Taken at 16 and 32
// products per lookup instead of 64: rows of 100 entries of 2^16 rows, 10,000
// columns, 14.1 and 14.5 against 16.7 ms, but R-MAT scale 18 16.1 and 14.2
// against 13.6.  R-MAT scale 12 to 14 with 2^14 products each and no total:
// 0.43 to 0.81 ms become 0.51 to 0.92.)
//
// Few cells split a row into few units, and then a few rows are not worth the
// passes of their own, which leave most of the device idle while the other
// rows wait: two workgroups per compute unit at least.  (64 rows of 32,768
// entries in 2^18 columns, one cell, 24 rows of 2^17 products and more: 2.70 ms
// in f64 by cells and 1.87 whole, 2.50 and 1.74 as counts; 1000 of 8192 in
// 2^18, 480 rows, 2.31 and 2.22; 4000 of 4096, 2000 rows, 4.28 and 4.79.)
struct DenseSums {
    uint64_t rows, entries, products;
};
constexpr int dense_kinds(DenseSums top, DenseSums few, int64_t nnz, int64_t m) {
    const uint64_t cells = uint64_t(dense_cells(m));
    if (m > kDenseMaxRows || top.entries * cells > top.products) return 0;
    const bool both = few.products >= kDenseTotal && top.products + few.products >= 2 * uint64_t(nnz);
    const uint64_t rows = top.rows + (both ? few.rows : 0);
    if (cells < kDenseSplit && rows * cells < kDenseUnits) return 0;
    if (both) return 2;
    return top.rows > 0 && top.rows * kDenseProducts >= uint64_t(nnz) ? 1 : 0;
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
