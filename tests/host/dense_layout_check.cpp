// Host check of the launches over (row, cell) units of dense.hip: every unit
// is one workgroup of the grid, and no dimension passes what a launch takes
// (fewer than 2^32 threads, fewer than 2^16 workgroups in y), for any number
// of rows and cells the path accepts; and of the rule that takes rows there.
#include <cstdio>
#include <initializer_list>

#include "dense_layout.h"

int main() {
    using namespace spsyrk;
    long checked = 0;
    for (int64_t m : {int64_t(1), int64_t(8192), int64_t(8193), int64_t(1) << 19, int64_t(1) << 20, int64_t(1) << 21,
                      kDenseMaxRows - 1, kDenseMaxRows}) {
        const int cells = dense_cells(m);
        if (int64_t(cells) * kCell < m || int64_t(cells - 1) * kCell >= m) return 1;
        for (int64_t rows : {int64_t(1), int64_t(41454), int64_t(65536), int64_t(131073), m}) {
            if (rows > m) continue;
            for (bool symbolic : {false, true}) {
                const DenseGrid g = dense_grid(rows, cells, symbolic);
                const int64_t per = symbolic ? kSymCells : 1;
                if (int64_t(g.x) != rows || int64_t(g.y) * per < cells || (int64_t(g.y) - 1) * per >= cells) {
                    std::printf("units lost: %lld rows, %d cells\n", (long long)rows, cells);
                    return 1;
                }
                if (int64_t(g.x) * kDenseThreads >= (int64_t(1) << 32) || g.y >= 65536) {
                    std::printf("launch too large: %lld rows, %d cells\n", (long long)rows, cells);
                    return 1;
                }
                ++checked;
            }
        }
    }
    // the table of long columns stays within 64 MB and has a block for every column start
    for (int64_t positions : {int64_t(1), int64_t(1000), int64_t(1) << 24, (int64_t(1) << 31) - 1})
        for (int64_t m : {int64_t(9000), int64_t(1) << 20, kDenseMaxRows}) {
            const int b = dense_block_log(positions, m);
            const int64_t blocks = dense_blocks(positions, b);
            if (blocks * dense_cells(m) > (int64_t(1) << 24) || ((positions + (int64_t(1) << b) - 1) >> b) >= blocks) return 1;
            ++checked;
        }
    // R-MAT's rows go by cells (scale 19 and 20: rows, entries, products), few
    // rows of many entries and few partners do not: more lookups than products
    const DenseSums no{0, 0, 0};
    if (dense_kinds({5408, 3323000, 1674000000}, no, 7970000, int64_t(1) << 19) != 1) return 1;
    if (dense_kinds({14859, 8180000, 5470000000}, no, 16090000, int64_t(1) << 20) != 1) return 1;
    if (dense_kinds({64, 64 * 131072, 64 * uint64_t(131072)}, no, 2 * 64 * 131072, kDenseMaxRows)) return 1;
    if (dense_kinds({63, 6300000, 206000000}, no, 6500000, kDenseMaxRows)) return 1;
    // never: no rows, too many rows in all, entries that outnumber the products
    if (dense_kinds(no, no, 0, 1000) || dense_kinds({1, 10, 1 << 20}, no, 10, kDenseMaxRows + 1) ||
        dense_kinds({1, 10, 1 << 17}, no, (1 << 17) + 1, 1000))
        return 1;
    // a row just within, and just past, its lookups
    if (dense_kinds({1, (1 << 17) / 512, 1 << 17}, no, 1000, kDenseMaxRows) != 1 ||
        dense_kinds({1, (1 << 17) / 512 + 1, 1 << 17}, no, 1000, kDenseMaxRows))
        return 1;
    // shorter rows: enough products in all, for the matrix's entries too, and
    // not beside longer rows with more lookups than products
    const DenseSums few{1000, 100000, kDenseTotal};
    if (dense_kinds(no, few, 1000, 8192) != 2 || dense_kinds({1, 10, 1 << 17}, few, 1000, 8192) != 2 ||
        dense_kinds(no, {1000, 100000, kDenseTotal - 1}, 1000, 8192) ||
        dense_kinds(no, few, int64_t(kDenseTotal / 2) + 1, 8192) || dense_kinds(no, few, 1000, kDenseMaxRows + 1) ||
        dense_kinds({1, 1 << 17, 1 << 17}, few, 1000, 8193))
        return 1;
    // of fewer than eight cells, not a few rows: their units, of either kind, fill the device
    for (int64_t m : {int64_t(100), int64_t(8192), int64_t(8193), int64_t(7 * 8192), int64_t(7 * 8192 + 1)}) {
        const uint64_t least = m > 7 * 8192 ? 1 : (512 + dense_cells(m) - 1) / dense_cells(m);
        for (uint64_t r : {least - 1, least}) {
            if (r == 0) continue;
            const uint64_t p = r << 17;
            if (dense_kinds({r, r, p}, no, 1000, m) != int(r >= least) ||
                dense_kinds({r - r / 2, r - r / 2, p}, {r / 2, r / 2, kDenseTotal}, 1000, m) != 2 * int(r >= least))
                return 1;
        }
    }
    // a row of kDenseProducts products in any case, a shorter one that fills its cells
    if (!dense_row(kDenseProducts, kDenseProducts, 512) || dense_row(kDenseFew - 1, 1, 1) ||
        !dense_row(kDenseFew, kDenseFew / kDenseFill, 1) || dense_row(kDenseFew, kDenseFew / kDenseFill + 1, 1) ||
        dense_row(kDenseFew, kDenseFew / kDenseFill, 2))
        return 1;
    std::printf("ok %ld\n", checked);
    return 0;
}
