// Gustavson accumulation of the rows with the most products (power-law
// graphs: rows of hundreds to thousands of entries that meet hub columns) and
// of rows that fill their columns, lower mode.
//
// A row of the first kind is too long for one workgroup: on R-MAT scale 19 (f32) the
// largest rows alone (20,000 entries, 6 million products) kept a workgroup
// busy for 57 ms, the length of the whole pass, through hundreds of value
// tiles that each search the ends of every entry's stretch.  Here (12 ms for
// 1.7 G products) the unit of work is a (row, cell) pair, a cell being kCell =
// 2^13 output columns:
//
//   * the accumulator is dense over the cell (these rows fill 10 to 50% of
//     it), so products need no rank, one walk both marks and adds, and the
//     columns come out in order;
//   * a table of the columns with many entries keeps the position of every
//     cell's first entry, so the ends of a stretch are two reads instead of
//     two binary searches (short columns are searched);
//   * units go cell by cell, so that all workgroups read one slab of the
//     column index at a time, which an XCD's L2 holds (1 MB of keys and
//     values of R-MAT scale 19);
//   * a symbolic pass counts every unit's columns, so each unit knows where
//     its outputs start.
#include "common.h"
#include "dense_layout.h"
#include "internal.h"
#include "lookup.h"
#include "stretches.h"

namespace spsyrk {
namespace {

constexpr int kDB = kDenseThreads;
constexpr int kDW = kDB / kWave;
constexpr int kDU = 4;          // registers of products in flight per wavefront
constexpr uint32_t kNoColumn = 0xffffffffu;

// A column of more than blk entries holds the first multiple of blk at or
// after its start, and no other such column does: that block's number names
// the column in the table.
__device__ inline uint32_t block_of(uint32_t start, int blk_log) { return (start + (1u << blk_log) - 1u) >> blk_log; }

// owner[b] = the start of the long column named by block b
__global__ __launch_bounds__(kBlock) void own_blocks(const RunTab run, int64_t nnz, int blk_log,
                                                     uint32_t* __restrict__ owner) {
    for (int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x; e < nnz; e += int64_t(gridDim.x) * kBlock) {
        const uint2 r = run_of(run, e);
        if (r.y - r.x == (1u << blk_log)) owner[block_of(r.x, blk_log)] = r.x;  // (one entry per column)
    }
}

// cells[b * ncells + g] = the position of the long column's first entry with
// a row of g * kCell or more, up to the cell of its last entry.  Every entry
// (one per lane; its row from the row pointers by the tile's wavefront) but
// the column's first fills the cells after its predecessor's up to its own.
__global__ __launch_bounds__(kBlock) void fill_cells(const RunTab run, const int64_t* __restrict__ rp, int64_t m,
                                                     int64_t nnz, const uint32_t* __restrict__ key, uint32_t rowmask,
                                                     int blk_log, const uint32_t* __restrict__ owner, int ncells,
                                                     uint32_t* __restrict__ cells) {
    // a wavefront per row, rows in turn
    const int lane = lane_id();
    const int64_t waves = int64_t(gridDim.x) * (kBlock / kWave);
    for (int64_t i = int64_t(blockIdx.x) * (kBlock / kWave) + threadIdx.x / kWave; i < m; i += waves) {
        for (int64_t e = rp[i] + lane; e < rp[i + 1]; e += kWave) {
            const uint2 r = run_of(run, e);
            if (r.y == r.x) continue;
            const uint32_t b = block_of(r.x, blk_log);
            if (owner[b] != r.x) continue;
            const uint32_t before = key[r.y - 1] & rowmask;
            uint32_t* c = cells + size_t(b) * size_t(ncells);
            uint32_t g = before >> kCellBits;
            if (r.y - r.x == 1)  // the column's second entry also fills those up to the first's
                for (uint32_t q = 0; q <= g; ++q) c[q] = r.x;
            const uint32_t last = uint32_t(i) >> kCellBits;
            for (++g; g <= last; ++g) c[g] = r.y;
        }
    }
}

// The part of the run r of an entry of row i that falls into the cells
// [g, g + n): {first, end} position.  (Every row of the run is below i; the
// entry itself or one before it filled its column's cells up to its own.)
__device__ inline uint2 cell_stretch(const DenseArgs& a, uint2 r, int64_t i, int64_t g, int n, uint32_t rowmask) {
    const int64_t x0 = g * kCell, x1 = (g + n) * kCell;
    const bool open = x1 >= i;  // (the run ends inside)
    const uint32_t len = r.y - r.x;
    if (len > (1u << a.blk_log)) {
        const uint32_t* c = a.cells + size_t(block_of(r.x, a.blk_log)) * size_t(a.ncells) + size_t(g);
        return make_uint2(g == 0 ? r.x : (x0 >= i ? r.y : c[0]), open ? r.y : c[n]);
    }
    // both ends of a short run searched side by side
    uint32_t lo = r.x, lon = len, hi = r.x, hin = len;
    while (lon | hin) {
        const uint32_t lm = lon / 2, hm = hin / 2;
        const uint32_t lk = lon ? a.cx.key[lo + lm] & rowmask : 0u, hk = hin ? a.cx.key[hi + hm] & rowmask : 0u;
        if (lon) {
            if (lk < uint32_t(x0)) {
                lo += lm + 1;
                lon -= lm + 1;
            } else {
                lon = lm;
            }
        }
        if (hin) {
            if (int64_t(hk) < x1) {
                hi += hm + 1;
                hin -= hm + 1;
            } else {
                hin = hm;
            }
        }
    }
    return make_uint2(lo, hi);
}

// Columns of kSymCells consecutive cells of a row: count[d * ncells + g].
__global__ __launch_bounds__(kDB) void dense_symbolic_kernel(DenseArgs a) {
    __shared__ uint32_t bits[kSymCells * kCell / 32];
    __shared__ Stretches<float, false, kDB, kDU> S;
    const int d = int(blockIdx.x);
    const int64_t g0 = int64_t(blockIdx.y) * kSymCells;
    const int64_t i = a.rows[d];
    if (g0 * kCell >= i) return;
    const int lane = lane_id();
    const uint32_t rowmask = a.cx.rowbits >= 32 ? 0xffffffffu : ((1u << a.cx.rowbits) - 1u);
    const int64_t B0 = g0 * kCell;
    for (int x = threadIdx.x; x < kSymCells * kCell / 32; x += kDB) bits[x] = 0;
    const int64_t e0 = a.rp[i], e1 = a.rp[i + 1];
    for (int64_t c0 = e0; c0 < e1; c0 += kDB) {
        const int64_t e = c0 + threadIdx.x;
        uint32_t lo = 0, hi = 0;
        if (e < e1) {
            const uint2 c = cell_stretch(a, run_of(a.run, e), i, g0, kSymCells, rowmask);
            lo = c.x;
            hi = c.y;
        }
        S.products(lo, hi, 0.0f, [&](uint32_t t, uint32_t te, const uint32_t(&pos)[kDU], const float(&)[kDU]) {
            uint32_t j[kDU];
#pragma unroll
            for (int u = 0; u < kDU; ++u) j[u] = t + uint32_t(u * kWave) + lane < te ? a.cx.key[pos[u]] & rowmask : 0u;
#pragma unroll
            for (int u = 0; u < kDU; ++u)
                if (t + uint32_t(u * kWave) + lane < te) {
                    const uint32_t x = j[u] - uint32_t(B0);
                    atomicOr(&bits[x >> 5], 1u << (x & 31));
                }
        });
    }
    // a cell's words by kDB / kSymCells threads
    constexpr int kPer = kDB / kSymCells;
    const int g = threadIdx.x / kPer;
    uint32_t s = 0;
    for (int x = threadIdx.x % kPer; x < kCell / 32; x += kPer) s += uint32_t(__popc(bits[g * (kCell / 32) + x]));
#pragma unroll
    for (int dd = 1; dd < kPer; dd <<= 1) s += __shfl_xor(s, dd, kWave);
    static_assert(kWave % kPer == 0, "a cell's threads lie in one wavefront");
    if (threadIdx.x % kPer == 0 && g0 + g < a.ncells) a.count[size_t(d) * size_t(a.ncells) + size_t(g0 + g)] = s;
}

// counts of a row's cells into its first output of every cell (relative to
// the row), and the row's length with its diagonal; a wavefront per row
__global__ __launch_bounds__(kWave) void dense_offsets(DenseArgs a) {
    const int d = blockIdx.x;
    const int64_t i = a.rows[d];
    uint32_t* c = a.count + size_t(d) * size_t(a.ncells);
    uint32_t carry = 0;
    for (int g0 = 0; g0 < a.ncells; g0 += kWave) {
        const int g = g0 + lane_id();
        const uint32_t v = g < a.ncells && int64_t(g) * kCell < i ? c[g] : 0u;
        const uint32_t inc = wsort::inclusive_sum(v);
        if (g < a.ncells) c[g] = carry + inc - v;
        carry += uint32_t(__builtin_amdgcn_readlane(int(inc), kWave - 1));
    }
    if (lane_id() == 0) a.row_nnz[i] = int64_t(carry) + 1;
}

// One cell of a row (64 KiB of f64 accumulators: two workgroups per compute
// unit, so that one's walk runs during the other's searches and output; cells
// of 2^14 columns with 1024 threads measure the same, 2^12 with 256 threads
// 25% slower).
template <int SR>
__global__ __launch_bounds__(kDB) void dense_numeric_kernel(DenseArgs a) {
    using Tr = SrTraits<SR>;
    using In = typename Tr::In;
    using Acc = typename Tr::Acc;
    using Out = typename Tr::Out;
    constexpr bool kVal = (SR == kF64 || SR == kF32);
    __shared__ __align__(16) Acc acc[kCell];
    __shared__ uint64_t bits[kCell / 64];
    __shared__ uint32_t first[kCell / 64];
    __shared__ Stretches<In, kVal, kDB, kDU> S;
    const int d = int(blockIdx.x);
    const int64_t g = blockIdx.y;
    const int64_t i = a.rows[d];
    const int64_t B0 = g * kCell;
    if (B0 > i) return;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const uint32_t rowmask = a.cx.rowbits >= 32 ? 0xffffffffu : ((1u << a.cx.rowbits) - 1u);
    const int64_t e0 = a.rp[i], e1 = a.rp[i + 1];
    const int64_t out = a.c_rp[i] + int64_t(a.count[size_t(d) * size_t(a.ncells) + size_t(g)]);
    for (int x = tid; x < kCell * int(sizeof(Acc)) / 16; x += kDB)
        reinterpret_cast<uint4*>(acc)[x] = make_uint4(0u, 0u, 0u, 0u);
    for (int x = tid; x < kCell / 64; x += kDB) bits[x] = 0;
    for (int64_t c0 = e0; c0 < e1; c0 += kDB) {
        const int64_t e = c0 + tid;
        uint32_t lo = 0, hi = 0;
        In val = In(0);
        if (e < e1) {
            const uint2 c = cell_stretch(a, run_of(a.run, e), i, g, 1, rowmask);
            lo = c.x;
            hi = c.y;
            if constexpr (kVal) val = static_cast<const In*>(a.val)[e];
        }
        S.products(lo, hi, val, [&](uint32_t t, uint32_t te, const uint32_t(&pos)[kDU], const In(&av)[kDU]) {
            uint32_t j[kDU];
            In bv[kDU];
#pragma unroll
            for (int u = 0; u < kDU; ++u) {
                const bool in = t + uint32_t(u * kWave) + lane < te;
                j[u] = in ? a.cx.key[pos[u]] & rowmask : 0u;
                bv[u] = In(0);
                if constexpr (kVal) bv[u] = in ? static_cast<const In*>(a.cx.val)[pos[u]] : In(0);
            }
#pragma unroll
            for (int u = 0; u < kDU; ++u) {
                if (t + uint32_t(u * kWave) + lane < te) {
                    const uint32_t x = j[u] - uint32_t(B0);
                    atomicOr(reinterpret_cast<uint32_t*>(bits) + (x >> 5), 1u << (x & 31));
                    if constexpr (kVal)
                        atomicAdd(&acc[x], double(av[u]) * double(bv[u]));
                    else
                        atomicAdd(&acc[x], 1);
                }
            }
        });
    }
    // the cell's columns in order: ranks of 64 columns at a time
    uint32_t total;
    static_assert(kCell / 64 <= kDB, "a thread per 64 columns");
    const uint32_t off = S.scan(tid < kCell / 64 ? uint32_t(__popcll(bits[tid < kCell / 64 ? tid : 0])) : 0u, &total);
    if (tid < kCell / 64) first[tid] = off;
    __syncthreads();
    const int64_t E = e1 - e0;
    for (int q = tid / kWave; q < kCell / 64; q += kDW) {
        const uint64_t b = bits[q];
        if (!((b >> lane) & 1u)) continue;
        const int x = 64 * q + lane;
        const int64_t p = out + first[q] + __popcll(b & lanemask_lt());
        const int32_t j = int32_t(B0 + x);
        SPSYRK_CHECK(p < a.c_rp[i + 1], kDbgHeavyOut);
        a.c_ci[p] = j;
        Out ov;
        if constexpr (kVal)
            ov = Out(acc[x]);
        else if constexpr (SR == kCount)
            ov = acc[x];
        else
            ov = jaccard(acc[x], E, a.rp[j + 1] - a.rp[j]);
        static_cast<Out*>(a.c_val)[p] = ov;
    }
    // the diagonal ends the row: the unit of its cell writes it
    if (B0 + kCell > i) {
        Out dv;
        if constexpr (kVal) {
            // fixed-order sum of the squared entries
            double s = 0.0;
            for (int64_t e = e0 + tid; e < e1; e += kDB) {
                const double v = double(static_cast<const In*>(a.val)[e]);
                s += v * v;
            }
            s = wave_reduce_sum(s);
            __syncthreads();
            double* ws = reinterpret_cast<double*>(acc);  // (every output is written)
            if (lane == 0) ws[tid / kWave] = s;
            __syncthreads();
            double t = 0.0;
            for (int q = 0; q < kDW; ++q) t += ws[q];
            dv = Out(t);
        } else if constexpr (SR == kCount) {
            dv = int32_t(E);
        } else {
            dv = jaccard(int32_t(E), E, E);
        }
        if (tid == 0) {
            SPSYRK_CHECK(out + total + 1 == a.c_rp[i + 1], kDbgHeavyCount);
            a.c_ci[out + total] = int32_t(i);
            static_cast<Out*>(a.c_val)[out + total] = dv;
        }
    }
}

}  // namespace

void dense_table(const DenseArgs& a, int64_t m, int64_t nnz, uint32_t* owner, hipStream_t s) {
    fill_u32(owner, dense_blocks(nnz, a.blk_log), kNoColumn, s);
    int64_t grid = (nnz + kBlock - 1) / kBlock;
    if (grid > 8192) grid = 8192;
    own_blocks<<<unsigned(grid), kBlock, 0, s>>>(a.run, nnz, a.blk_log, owner);
    const uint32_t rowmask = a.cx.rowbits >= 32 ? 0xffffffffu : ((1u << a.cx.rowbits) - 1u);
    grid = (m + kBlock / kWave - 1) / (kBlock / kWave);
    if (grid > 8192) grid = 8192;
    fill_cells<<<unsigned(grid), kBlock, 0, s>>>(a.run, a.rp, m, nnz, a.cx.key, rowmask, a.blk_log, owner, a.ncells,
                                                 a.cells);
}

void dense_symbolic(const DenseArgs& a, hipStream_t s) {
    if (a.nrows <= 0) return;
    const DenseGrid g = dense_grid(a.nrows, a.ncells, true);
    dense_symbolic_kernel<<<dim3(g.x, g.y), kDB, 0, s>>>(a);
    dense_offsets<<<unsigned(a.nrows), kWave, 0, s>>>(a);
}

void dense_numeric(const DenseArgs& a, hipStream_t s) {
    if (a.nrows <= 0) return;
    const DenseGrid g = dense_grid(a.nrows, a.ncells, false);
    const dim3 grid(g.x, g.y);
    switch (a.sr) {
        case kF64: dense_numeric_kernel<kF64><<<grid, kDB, 0, s>>>(a); break;
        case kF32: dense_numeric_kernel<kF32><<<grid, kDB, 0, s>>>(a); break;
        case kCount: dense_numeric_kernel<kCount><<<grid, kDB, 0, s>>>(a); break;
        default: dense_numeric_kernel<kJaccard><<<grid, kDB, 0, s>>>(a); break;
    }
}

}  // namespace spsyrk
