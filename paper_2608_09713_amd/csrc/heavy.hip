// Gustavson accumulation for rows with many products (rows of power-law
// graphs that meet hub columns): one workgroup per row, taken from a work
// queue.
//
// The row's output column range is swept in windows of kWin columns.  In a
// window the row's distinct columns are first marked in an LDS bitmap; a scan
// of the words' popcounts gives every marked column its rank, i.e. its
// position among the row's output entries, so the window's column indices are
// written straight from the bitmap, in order.  The values are then summed in
// LDS over the compacted ranks (tiles of kAcc ranks), so the accumulator only
// spans columns that occur.
//
// Every partner run is sorted by row, so the part of it that falls into a
// window or a tile is a stretch of consecutive positions: its end is found by
// binary search, and the stretches of the row's entries, laid end to end, are
// shared out evenly over the wavefronts (stretches.h).  What bounds a row are
// its chains of dependent loads (a search is about ten, each a miss in L2)
// and LDS traffic: marks and values run at about 300 G products/s each.  The
// rows of 2^17 products and more, and shorter ones that fill their columns, go
// to dense.hip in lower mode; together the
// two numeric passes take 30 ms on R-MAT scale 19 in f32 (57 ms with one
// workgroup for every row, whose largest rows set its length).
//
// The symbolic pass builds the bitmaps only and counts the row's columns; the
// numeric pass rebuilds them, writes the column indices and the values.
#include "common.h"
#include "internal.h"
#include "lookup.h"
#include "stretches.h"

namespace spsyrk {
namespace {

constexpr int kHB = kHeavySmall;         // threads per workgroup
constexpr int kHW = kHB / kWave;         // wavefronts per workgroup
constexpr uint32_t kNoRow = 0xffffffffu;  // (rows are below 2^31)
constexpr uint32_t kOwnMost = 64;        // products of a stretch that its wavefront walks by itself, at most
constexpr int kHeavyGroups = 1024;       // workgroups of a heavy-row launch

// Output columns per window and ranks per value tile: the symbolic pass
// holds a 32 KiB bitmap; the numeric pass a 16 KiB bitmap, the rank of every
// 128 columns' first column (4 KiB) and an 18 or 21 KiB value tile, 52 KiB
// with the stretches and bounds of kHB entries, so that three workgroups
// share a compute unit.
template <int SR, bool NUM>
struct HeavyCfg {
    using Acc = typename SrTraits<SR>::Acc;
    static constexpr int kWin = NUM ? (1 << 17) : (1 << 18);
    static constexpr int kWords = kWin / 32;
    static constexpr int kAcc = (SR == kF64 ? 18432 : 21504) / int(sizeof(Acc));
    // registers of products in flight (3 for all: R-MAT in f32 15% slower,
    // the symbolic pass of long rows 20%)
    static constexpr int kHU = NUM && SR != kF32 ? 3 : 2;
};

// first position in [lo, hi) whose row is at least x (hi if none)
__device__ inline uint32_t stretch_end(const uint32_t* __restrict__ key, uint32_t rowmask, uint32_t lo, uint32_t hi,
                                       int64_t x) {
    if (lo >= hi || int64_t(key[hi - 1] & rowmask) < x) return hi;
    uint32_t n = hi - 1;  // (the last one is at least x)
    while (lo < n) {
        const uint32_t mid = lo + (n - lo) / 2;
        if (int64_t(key[mid] & rowmask) < x)
            lo = mid + 1;
        else
            n = mid;
    }
    return lo;
}

// The same for U stretches side by side, hi becoming the position and row the
// row there (kNoRow at hi); known: every stretch's first row is below x.  Most
// ends lie near the front of a stretch, so its first rows are read at once,
// 16 bytes per lane (the keys are padded by kKeyPad words), and searched for
// only past them.  (1024 rows of 10,000 entries with nine partners each, 2^20
// columns, f64, whole call: 9.8 ms with searches from a stretch's ends, 8.3 so.)
template <int U>
__device__ inline void stretch_ends(const uint32_t* __restrict__ key, uint32_t rowmask, const uint32_t (&lo)[U],
                                    uint32_t (&hi)[U], uint32_t (&row)[U], int64_t x, bool known) {
    static_assert(kKeyPad >= 4, "four rows from any position, or the one after it");
    uint32_t k[U][4], at[U], n[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (lo[u] < hi[u]) __builtin_memcpy(k[u], key + lo[u] + (known ? 1u : 0u), 16);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        at[u] = n[u] = hi[u];
        row[u] = kNoRow;
        if (lo[u] >= hi[u]) continue;
        const uint32_t p = lo[u] + (known ? 1u : 0u);
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (p + j < hi[u]) {
                const uint32_t r = k[u][j] & rowmask;
                if (int64_t(r) < x)
                    c = j + 1;
                else
                    row[u] = min(row[u], r);  // (rows ascend: the first one)
            }
        at[u] = p + c;
        if (c < 4)
            n[u] = min(at[u], hi[u]);
        else if (at[u] < hi[u] && int64_t(key[hi[u] - 1] & rowmask) < x)
            at[u] = hi[u];
    }
    auto left = [&] {
        bool f = false;
#pragma unroll
        for (int u = 0; u < U; ++u) f |= at[u] < n[u];
        return f;
    };
    while (left()) {
        uint32_t m[U], v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            m[u] = at[u] + (n[u] - at[u]) / 2;
            v[u] = at[u] < n[u] ? key[m[u]] & rowmask : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (at[u] >= n[u]) continue;
            if (int64_t(v[u]) < x) {
                at[u] = m[u] + 1;
            } else {
                n[u] = m[u];
                row[u] = v[u];  // (the last such position read is the first one)
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) hi[u] = n[u];
}

// Three workgroups of the numeric pass share a compute unit by their LDS;
// that takes six wavefronts per SIMD, i.e. at most 80 VGPRs.
template <int SR, bool NUM, bool LOWER>
__global__ __launch_bounds__(kHB) __attribute__((amdgpu_waves_per_eu(NUM ? 6 : 8)))
void heavy_kernel(HeavyArgs a, int* queue) {
    using Tr = SrTraits<SR>;
    using In = typename Tr::In;
    using Acc = typename Tr::Acc;
    using Out = typename Tr::Out;
    constexpr int kAcc = HeavyCfg<SR, NUM>::kAcc;
    constexpr int kWin = HeavyCfg<SR, NUM>::kWin;
    constexpr int kWords = HeavyCfg<SR, NUM>::kWords;
    constexpr int kHU = HeavyCfg<SR, NUM>::kHU;
    constexpr bool kVal = (SR == kF64 || SR == kF32);
    // Batches of short stretches by their own wavefronts (long rows; counts of
    // eight rows of 2^18 entries, whole call: 11.4 ms shared out, 10.0 so; 200
    // rows of 16,384 0.99 and 0.87).  Not where values are added: the second
    // walk in that kernel costs R-MAT scale 17 in f32 5.7 -> 6.6 ms.
    constexpr bool kOwn = !(NUM && kVal);
    constexpr int kTiles = (kWin + kAcc - 1) / kAcc;  // value tiles of a window, at most

    __shared__ __align__(16) uint32_t bits[kWords];
    __shared__ uint32_t prefw[NUM ? kWords / 4 : 1];  // rank of the first column of each 4 words in the window
    __shared__ Acc acc[NUM ? kAcc : 1];
    // (the symbolic pass and the marks need no values; the numeric pass's are A's)
    __shared__ Stretches<In, NUM && kVal, kHB, kHU> S;
    __shared__ int32_t tile_col[NUM ? kTiles + 1 : 1];  // first column of every value tile
    // rows of up to kHB entries: ends of the entries' stretches in the next
    // windows, and in the next tiles of a window (boundary-major)
    __shared__ uint32_t win_end[kHB];
    __shared__ uint32_t tile_end[NUM ? kHB : 1];
    __shared__ int row_s;
    __shared__ int listed_s;  // (long rows) entries with a stretch in the window
    __shared__ double wtd[kHW];

    const int tid = threadIdx.x;
    const int w = tid / kWave;
    const int lane = lane_id();
    const uint32_t* __restrict__ key = a.cx.key;
    const uint32_t rowmask = a.cx.rowbits >= 32 ? 0xffffffffu : ((1u << a.cx.rowbits) - 1u);
    const int nheavy = *a.heavy_count;

    // rank of column B0 + x among the window's columns
    auto rank_of = [&](uint32_t x) -> uint32_t {
        if constexpr (!NUM) return 0u;  // (ranks exist in the numeric pass only)
        const uint4 q = reinterpret_cast<const uint4*>(bits)[x >> 7];
        const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
        const uint32_t k = (x >> 5) & 3u, mk = (1u << (x & 31)) - 1u;
        uint32_t r = prefw[x >> 7];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) r += i < k ? uint32_t(__popc(wd[i])) : (i == k ? uint32_t(__popc(wd[i] & mk)) : 0u);
        return r;
    };

    int next_row = -1;  // (thread 0)
    if (tid == 0) {
        const int h = a.heavy_first + atomicAdd(queue, 1);
        next_row = h < nheavy ? a.heavy_rows[h] : -1;
    }
    while (true) {
        if (tid == 0) row_s = next_row;
        __syncthreads();
        const int i = int(uniform(uint32_t(row_s)));
        __syncthreads();
        if (i < 0) break;
        if (tid == 0) next_row = a.heavy_first + atomicAdd(queue, 1);  // (the next row's place, used at this row's end)
        const int64_t e0 = a.rp[i], e1 = a.rp[i + 1];
        const int64_t E = e1 - e0;
        // Rows of up to kHB entries keep an entry per thread: the start of its
        // stretch stays in a register, and the idle threads search the ends in several windows or tiles at once (a
        // search is a chain of about ten loads, each of them a miss in L2).
        // Longer rows go through the entries, two per thread at a time, in
        // every window.  An entry's next position is kept in memory with the
        // row there, so that an entry with nothing in the window costs one
        // streamed read, and the numeric pass lists the entries that have
        // something: its value tiles go through those alone.  (2048 rows of
        // 5000 entries, 2^22 columns, f64, whole call: 12.6 ms with every
        // entry searched for in every window and tile, 8.6 so; one row of
        // 500,000 entries of one partner, 2^20 columns: 511 ms, 94 so.)
        const bool small = E <= kHB;
        uint32_t start = 0;  // (small rows) the stretch's start
        // The products of a batch of stretches.  Those of a long row, where all
        // are short, by their own wavefronts: a batch is too little work for
        // the barriers of sharing it out.  (The vote's barrier also orders what
        // was cleared before.)
        auto walk = [&](uint32_t l, uint32_t h, In v, auto use) {
            if constexpr (kOwn)
                if (!small && !__syncthreads_or(int(h - l > kOwnMost))) {
                    S.own_products(l, h, v, use);
                    return;
                }
            S.products(l, h, v, use);
        };

        // (two passes) partner runs
        if constexpr (!NUM) {
            if (!a.runs_ready) {
                uint64_t prod_local = 0;
                for (int64_t e = e0 + tid; e < e1; e += kHB) {
                    uint32_t st, len;
                    partner_run(key, a.cx.gptr, a.cx.gs, a.cx.rowbits, uint32_t(a.ci[e]), uint32_t(i), LOWER, st, len);
                    a.run.r8[e] = make_uint2(st, st + len);
                    prod_local += len;
                }
                const uint64_t tot = wave_reduce_sum(prod_local);
                if (lane == 0 && tot && a.products) atomicAdd(a.products, (unsigned long long)tot);
                __threadfence_block();
                __syncthreads();
            }
        }
        if (small && tid < E) start = run_of(a.run, e0 + tid).x;
        const int per_group = small ? kHB / int(E) : 1;  // boundaries searched at once

        const int64_t jmax = LOWER ? int64_t(i) : a.m_right;
        const int nwin = int((jmax + kWin - 1) / kWin);
        int64_t count = 0;                          // symbolic: distinct columns so far
        int64_t outp = NUM ? a.c_rp[i] : 0;         // numeric: first output slot of the window
        for (int k = 0; k < nwin; ++k) {
            const int64_t B0 = int64_t(k) * kWin;
            const int64_t B1 = min(jmax, B0 + int64_t(kWin));
            const int nw = int((B1 - B0 + 31) >> 5);
            for (int x = tid; x < nw; x += kHB) bits[x] = 0;
            if (NUM && tid == 0) listed_s = 0;
            // (each entry of a long row is one thread's in every window: its
            // own writes to the cursor are the ones it reads)
            const int kg = small ? int(k % per_group) : 0;  // the window in its group
            if (small && kg == 0 && k + 1 < nwin) {
                // ends at the next per_group window ends, the last one left
                // out: thread tid searches boundary tid / E for entry tid % E
                const int eg = tid / int(E), ee = tid - eg * int(E);
                if (eg < per_group && k + 1 + eg < nwin) {
                    const uint2 r = run_of(a.run, e0 + ee);
                    win_end[tid] = stretch_end(key, rowmask, r.x, r.y, int64_t(k + 1 + eg) * kWin);
                }
                __syncthreads();
            }

            // mark the window's columns; the numeric pass keeps the starts
            // for the values and notes where the window's stretch ends
            uint32_t wend = 0;
            auto mark = [&](uint32_t t, uint32_t te, const uint32_t(&pos)[kHU], const In(&)[kHU]) {
                uint32_t j[kHU];
#pragma unroll
                for (int u = 0; u < kHU; ++u) j[u] = t + uint32_t(u * kWave) + lane < te ? key[pos[u]] & rowmask : 0u;
#pragma unroll
                for (int u = 0; u < kHU; ++u) {
                    if (t + uint32_t(u * kWave) + lane < te) {
                        const uint32_t x = uint32_t(int64_t(j[u]) - B0);
                        atomicOr(&bits[x >> 5], 1u << (x & 31));
                    }
                }
            };
            // (two entries per thread at a time, whose loads go together; a
            // small row holds its one)
            for (int64_t c0 = e0; c0 < e1; c0 += 2 * kHB) {
                uint32_t lo[2] = {start, 0u}, hi[2] = {wend, 0u};
                if (small) {
                    if (tid < E) hi[0] = wend = k + 1 < nwin ? win_end[kg * int(E) + tid] : run_of(a.run, e0 + tid).y;
                } else {
                    uint32_t row[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int64_t e = c0 + u * kHB + tid;
                        lo[u] = hi[u] = 0;
                        if (e >= e1) continue;
                        const uint2 c = k ? a.cursor[e] : make_uint2(0u, 0u);
                        if (int64_t(c.y) >= B1) continue;  // nothing in the window
                        const uint2 r = run_of(a.run, e);
                        lo[u] = k ? c.x : r.x;
                        hi[u] = r.y;
                    }
                    if (k + 1 < nwin) {
                        stretch_ends<2>(key, rowmask, lo, hi, row, B1, k > 0);
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int64_t e = c0 + u * kHB + tid;
                            if (e < e1 && (k == 0 || lo[u] < hi[u])) a.cursor[e] = make_uint2(hi[u], row[u]);
                        }
                    }
                }
#pragma unroll 1
                for (int u = 0; u < 2 && c0 + u * kHB < e1; ++u) {
                    const uint32_t l = u ? lo[1] : lo[0], h = u ? hi[1] : hi[0];
                    walk(l, h, In(0), mark);
                    if (NUM && !small) {  // the stretches that are not empty, listed (a wavefront's in a row)
                        const uint64_t some = __ballot(l < h);
                        int at = 0;
                        if (lane == 0 && some) at = atomicAdd(&listed_s, __popcll(some));
                        at = __builtin_amdgcn_readfirstlane(at);
                        if (l < h)
                            a.list[e0 + at + __popcll(some & lanemask_lt())] = {uint32_t(c0 + u * kHB + tid), l, h, 0u};
                    }
                }
            }

            if (kOwn && !small) __syncthreads();  // (marks made without barriers)

            // ranks: every thread owns a contiguous stretch of words
            constexpr int kPer = (kWords + kHB - 1) / kHB;
            const int wlo = min(nw, tid * kPer), whi = min(nw, wlo + kPer);
            uint32_t s = 0;
#pragma unroll 4
            for (int x = wlo; x < whi; ++x) s += uint32_t(__popc(bits[x]));
            uint32_t Nw;
            uint32_t off = S.scan(s, &Nw);
            Nw = uniform(Nw);
            // entries whose values the tiles add, kHB at a time
            const int nadd = NUM && !small ? __builtin_amdgcn_readfirstlane(listed_s) : int(E);
            if constexpr (!NUM) {
                count += Nw;
                start = wend;
            } else {
                for (int x = wlo; x < whi; ++x) {
                    if ((x & 3) == 0) prefw[x >> 2] = off;
                    uint32_t b = bits[x];
                    // the window's column indices, in order
                    while (b) {
                        const int t = __ffs(b) - 1;
                        b &= b - 1;
                        SPSYRK_CHECK(outp + off < a.c_rp[i + 1], kDbgHeavyOut);
                        const int32_t j = int32_t(B0 + 32 * x + t);
                        a.c_ci[outp + off] = j;
                        if (off % uint32_t(kAcc) == 0) tile_col[off / uint32_t(kAcc)] = j;
                        ++off;
                    }
                }
                // (the barrier orders these writes for the workgroup's reads below)
                __syncthreads();

                // values over the compacted ranks, kAcc ranks at a time
                const int ntile = int((Nw + uint32_t(kAcc) - 1) / uint32_t(kAcc));
                for (int q = 0; q < ntile; ++q) {
                    const uint32_t T0 = uint32_t(q) * uint32_t(kAcc);
                    const uint32_t tl = min(Nw - T0, uint32_t(kAcc));
                    for (uint32_t x = tid; x < tl; x += kHB) acc[x] = Acc(0);
                    const bool last = q + 1 == ntile;
                    auto add = [&](uint32_t t, uint32_t te, const uint32_t(&pos)[kHU], const In(&av)[kHU]) {
                        uint32_t j[kHU];
                        In bv[kHU];
#pragma unroll
                        for (int u = 0; u < kHU; ++u) {
                            const bool in = t + uint32_t(u * kWave) + lane < te;
                            j[u] = in ? key[pos[u]] & rowmask : 0u;
                            bv[u] = In(0);
                            if constexpr (kVal) bv[u] = in ? static_cast<const In*>(a.cx.val)[pos[u]] : In(0);
                        }
#pragma unroll
                        for (int u = 0; u < kHU; ++u) {
                            if (t + uint32_t(u * kWave) + lane < te) {
                                const uint32_t rk = rank_of(uint32_t(int64_t(j[u]) - B0)) - T0;
                                SPSYRK_CHECK(rk < tl, kDbgHeavyOut);
                                if constexpr (kVal)
                                    atomicAdd(&acc[rk], double(av[u]) * double(bv[u]));
                                else
                                    atomicAdd(&acc[rk], 1);
                            }
                        }
                    };
                    const int qg = small ? q % per_group : 0;
                    if (small && qg == 0 && !last) {
                        const int eg = tid / int(E), ee = tid - eg * int(E);
                        if (eg < per_group && q + 1 + eg < ntile) {
                            const uint2 r = run_of(a.run, e0 + ee);
                            tile_end[tid] = stretch_end(key, rowmask, r.x, k + 1 < nwin ? win_end[kg * int(E) + ee] : r.y,
                                                        int64_t(tile_col[q + 1 + eg]));
                        }
                        __syncthreads();
                    }
                    for (int c0 = 0; c0 < nadd; c0 += kHB) {  // (once for a small row)
                        uint32_t lo = start, hi = wend;
                        In val = In(0);
                        if (small) {
                            if constexpr (kVal) {
                                // (opaque: the address is formed here, not
                                // held in registers across the row)
                                int t = tid;
                                asm volatile("" : "+v"(t));
                                if (t < nadd) val = static_cast<const In*>(a.val)[e0 + t];
                            }
                            if (!last && tid < nadd) hi = tile_end[qg * nadd + tid];
                            start = hi;
                        } else {
                            const int at = c0 + tid;
                            const int64_t x = last ? B1 : int64_t(tile_col[q + 1]);
                            HeavyStretch l{0u, 0u, 0u, kNoRow};
                            if (at < nadd) l = a.list[e0 + at];
                            lo = hi = l.pos;
                            if (int64_t(l.row) < x) {
                                hi = l.end;
                                if constexpr (kVal) val = static_cast<const In*>(a.val)[l.entry];
                            }
                            if (!last) {
                                const uint32_t from[1] = {lo};
                                uint32_t to[1] = {hi}, row[1];
                                stretch_ends<1>(key, rowmask, from, to, row, x, q > 0);
                                if (lo < hi) {
                                    a.list[e0 + at].pos = to[0];
                                    a.list[e0 + at].row = row[0];
                                }
                                hi = to[0];
                            }
                        }
                        walk(lo, hi, val, add);
                    }
                    if (kOwn && !small) __syncthreads();  // (sums made without barriers)
                    for (uint32_t x = tid; x < tl; x += kHB) {
                        const int64_t p = outp + T0 + x;
                        SPSYRK_CHECK(p < a.c_rp[i + 1], kDbgHeavyOut);
                        Out ov;
                        if constexpr (kVal) {
                            ov = Out(acc[x]);
                        } else if constexpr (SR == kCount) {
                            ov = acc[x];
                        } else {
                            const int32_t j = a.c_ci[p];
                            ov = jaccard(acc[x], E, a.rp_right[j + 1] - a.rp_right[j]);
                        }
                        static_cast<Out*>(a.c_val)[p] = ov;
                    }
                    __syncthreads();
                }
                outp += Nw;
            }
        }
        if constexpr (NUM) {
            if (tid == 0) SPSYRK_CHECK(outp + (LOWER ? 1 : 0) == a.c_rp[i + 1], kDbgHeavyCount);
        }
        if (tid == 0) next_row = next_row < nheavy ? a.heavy_rows[next_row] : -1;
        // diagonal (lower triangle only; a heavy row is never empty)
        if constexpr (!NUM) {
            if (tid == 0) {
                a.row_nnz[i] = count + (LOWER ? 1 : 0);
                if (a.nnz_total) atomicAdd(a.nnz_total, (unsigned long long)(count + (LOWER ? 1 : 0)));
            }
        } else if (LOWER) {
            Out dv;
            if constexpr (kVal) {
                // fixed-order reduction of the squared entries
                double s = 0.0;
                for (int64_t e = e0 + tid; e < e1; e += kHB) {
                    const double v = double(static_cast<const In*>(a.val)[e]);
                    s += v * v;
                }
                s = wave_reduce_sum(s);
                if (lane == 0) wtd[w] = s;
                __syncthreads();
                double t = 0.0;
                for (int q = 0; q < kHW; ++q) t += wtd[q];
                dv = Out(t);
                __syncthreads();
            } else if constexpr (SR == kCount) {
                dv = int32_t(E);
            } else {
                dv = jaccard(int32_t(E), E, E);
            }
            if (tid == 0) {
                SPSYRK_CHECK(outp < a.c_rp[i + 1], kDbgHeavyOut);
                a.c_ci[outp] = i;
                static_cast<Out*>(a.c_val)[outp] = dv;
            }
        }
        __syncthreads();
    }
}

template <int SR, bool NUM>
void launch(const HeavyArgs& a, int* queue, hipStream_t s) {
    if (a.heavy_max <= 0) return;
    (void)hipMemsetAsync(queue, 0, sizeof(int), s);
    const int64_t grid = a.heavy_max < kHeavyGroups ? a.heavy_max : kHeavyGroups;

    if (a.lower)
        heavy_kernel<SR, NUM, true><<<unsigned(grid), kHB, 0, s>>>(a, queue);
    else
        heavy_kernel<SR, NUM, false><<<unsigned(grid), kHB, 0, s>>>(a, queue);
}

template <bool NUM>
void dispatch(const HeavyArgs& a, int* queue, hipStream_t s) {
    switch (a.sr) {
        case kF64: launch<kF64, NUM>(a, queue, s); break;
        case kF32: launch<kF32, NUM>(a, queue, s); break;
        case kCount: launch<kCount, NUM>(a, queue, s); break;
        default: launch<kJaccard, NUM>(a, queue, s); break;
    }
}

}  // namespace

void heavy_symbolic(const HeavyArgs& a, int* queue, hipStream_t s) { dispatch<false>(a, queue, s); }
void heavy_numeric(const HeavyArgs& a, int* queue, hipStream_t s) { dispatch<true>(a, queue, s); }

}  // namespace spsyrk
