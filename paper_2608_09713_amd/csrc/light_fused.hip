// Single-pass Gustavson accumulation of the light rows.
//
// Work unit: a chunk of R consecutive rows per wavefront.  Each wavefront
// works alone in its own slice of LDS (no workgroup barriers), in batches of
// consecutive light rows of at most 1024 (with values 768) products:
//
//   1. the batch's entries, 64 at a time: the partner run of every entry
//      (written by the column-index build), a prefix sum of the run lengths,
//      and at every run's first product slot the run's start less that slot;
//   2. the batch's rows listed by size class (8, 16, 32 or 64 lanes, two
//      registers, more), so that one wavefront register holds several short
//      rows side by side;
//   3. per register: every lane is one product; the nearest marked slot at or
//      below its own gives its position in the column index (one ballot), all
//      keys are loaded together, and every row is sorted by (column, product
//      index) in registers (wave_sort.h), rows of more than 128 products 64
//      at a time with merges in LDS.  The first product of every column
//      takes the column's terms in product order; with no equal columns, the
//      usual case, each lane is one output, written at its place in the row;
//   4. diagonals and exact lengths, one row per lane.
//
// A scan of the exact lengths gives the row pointers and a streaming copy
// moves the rows into place, so no row waits for the lengths of earlier
// rows.  Rows with too many entries or products ("heavy") are left to the
// heavy-row kernels.
#include <type_traits>

#include "common.h"
#include "dense_layout.h"
#include "internal.h"
#include "lookup.h"
#include "wave_sort.h"

namespace spsyrk {
namespace {

constexpr int kFE = kFusedEntries;   // entries of a light row
constexpr int kFP = kFusedProducts;  // products of a light row
constexpr int kFR = kFusedRows;      // rows per chunk (upper limit: one per lane)
// product slots per batch
constexpr int slots(bool val) { return val ? 768 : 1024; }
constexpr int kWavesF = 2;           // wavefronts per workgroup
constexpr int64_t kDealtBelow = 98304;  // chunks below which they are dealt out (all_chunks)
constexpr int kOrdBits = 9;          // product index bits of a 32-bit plus-times key (column above them)
constexpr uint32_t kNoRun = 0x80000000u;  // a slot where no run starts (starts are below 2^31, slots below 2^11)
static_assert(kFR <= kWave, "one row per lane");
static_assert(kFP <= slots(true) && kFP <= slots(false), "a row fits a batch");
static_assert(kFP <= (1 << kOrdBits), "a product index must fit kOrdBits");
static_assert(slots(false) <= (1 << 11) && slots(true) <= (1 << 11) && kFP <= (1 << 10) && kFR <= (1 << 6), "fields of a listed row");
static_assert(kFR * kFE <= (1 << 16), "an entry's index in its batch must fit 16 bits");

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (5 KiB; with values 7.5 KiB, 64-bit keys 9.5: 20 and 16 wavefronts per
// compute unit)
template <bool VAL, typename Key>
struct WaveLds {
    // a long row's keys; without values 32-bit keys take the row's slots of d
    static constexpr int kCap = slots(VAL);
    static constexpr bool kOwnKeys = VAL || sizeof(Key) > 4;
    Key key[kOwnKeys ? kFP : 1];
    alignas(16) uint32_t d[kCap];  // start of the run that begins at the slot, less the slot; else kNoRun
    uint16_t x[VAL ? kCap : 2];    // the run's entry (index in the batch)
    int64_t out[kFR];              // first output slot of every row
    uint32_t ord[kFR];             // rows by size class: first slot | products << 11 | row << 21
    uint16_t cnt[kFR];             // outputs off the diagonal
    uint16_t len[kFR];             // entries of every light row
};

// WIDE: 64-bit sort keys.  Plus-times: column and product index, where both
// do not fit 32 bits.  Jaccard without packed words: column and the
// partner's length (packed words are sorted as they are; counts need the
// column only).
template <int SR, bool LOWER, bool WIDE>
struct Chunk {
    using Tr = SrTraits<SR>;
    using In = typename Tr::In;
    using Out = typename Tr::Out;
    using Key = typename std::conditional<WIDE, uint64_t, uint32_t>::type;
    static constexpr bool kVal = (SR == kF64 || SR == kF32);
    static constexpr int kCap = slots(kVal);
    static constexpr Key kDead = ~Key(0);  // sorts behind every product of its row

    const FusedArgs& a;
    WaveLds<kVal, Key>& L;
    const int lane0;
    uint32_t rowmask;
    uint32_t lenmax;  // saturated length in a key (Jaccard keys carrying lengths)
    int64_t r0 = 0;

    // The lane number, as a value the compiler does not know: what a passage
    // derives from it (masks, sides, addresses) is formed there again instead
    // of being held in registers through all the others (25 of them: one
    // wavefront per SIMD).
    __device__ int fresh_lane() const {
        int l = lane0;
        asm volatile("" : "+v"(l));
        return l;
    }
    __device__ static uint64_t lanes_upto(int lane) { return (uint64_t(2) << lane) - 1; }

    __device__ Chunk(const FusedArgs& a_, WaveLds<kVal, Key>& L_) : a(a_), L(L_), lane0(lane_id()) {
        rowmask = a.cx.rowbits >= 32 ? 0xffffffffu : ((1u << a.cx.rowbits) - 1u);
        lenmax = a.cx.lenbits > 0 ? ((a.cx.lenbits >= 32 ? 0xffffffffu : (1u << a.cx.lenbits) - 1u)) : 0u;
    }

    // sort key of the product with key word w at position pos, product index o of its row
    __device__ Key sort_key(uint32_t w, uint32_t o) const {
        const uint32_t j = w & rowmask;
        if constexpr (SR == kCount) {
            return Key(j);
        } else if constexpr (kVal) {
            if constexpr (WIDE)
                return (uint64_t(j) << 32) | o;
            else
                return (j << kOrdBits) | o;
        } else {
            // the partner's length from its key; saturated: from the row pointers
            uint32_t len = w >> a.cx.rowbits;
            if (len >= lenmax) len = uint32_t(a.rp_right[j + 1] - a.rp_right[j]);
            if constexpr (WIDE)
                return (uint64_t(j) << 32) | len;
            else
                return j * a.pack_rr + a.pack_r2 + len;
        }
    }
    __device__ static uint32_t index_of(Key k) { return WIDE ? uint32_t(k) : uint32_t(k) & ((1u << kOrdBits) - 1u); }
    // equal for two keys of a row exactly when their columns are equal
    __device__ static uint32_t column_of(Key k) {
        if constexpr (WIDE)
            return uint32_t(k >> 32);
        else
            return kVal ? uint32_t(k) >> kOrdBits : uint32_t(k);
    }

    // one output: slot p, sorted key k of the column's first product, its
    // terms' count and (plus-times) sum; len_i: the row's entries (Jaccard)
    __device__ void emit(int64_t p, Key k, uint32_t cnt, double sum, uint32_t len_i) const {
        if constexpr (SR == kCount) {
            if (a.pack_rr) {  // one staged word: column and count
                a.c_ci[p] = int32_t(uint32_t(k) * a.pack_rr + cnt);
                return;
            }
            a.c_ci[p] = int32_t(uint32_t(k));
            static_cast<Out*>(a.c_val)[p] = Out(cnt);
        } else if constexpr (kVal) {
            a.c_ci[p] = int32_t(column_of(k));
            static_cast<Out*>(a.c_val)[p] = Out(sum);
        } else if constexpr (WIDE) {
            a.c_ci[p] = int32_t(column_of(k));
            static_cast<Out*>(a.c_val)[p] = jaccard(int32_t(cnt), len_i, int64_t(uint32_t(k)));
        } else {  // the packed word holds one term already
            a.c_ci[p] = int32_t(uint32_t(k) + (cnt - 1u) * a.pack_r2);
        }
    }

    // ---- rows of up to 64 products, 64 / S of them side by side

    struct Group {  // one register of products, its loads in flight
        uint32_t info, key;
        uint32_t src;  // (plus-times) the partner's value: its place in right_values()
        bool live;
        In va;         // the entry's value
    };

    // The partners' values: by position in the column index, or, where the
    // index keeps entries instead (lower mode), by entry of A.
    __device__ const In* right_values() const {
        return static_cast<const In*>(LOWER && a.cx.ke ? a.val : a.cx.val);
    }
    // key word of a position, and (plus-times) where the partner's value is
    __device__ void partner(uint32_t pos, uint32_t& key, uint32_t& src) const {
        if constexpr (kVal && LOWER) {
            if (a.cx.ke) {
                const uint2 q = a.cx.ke[pos];
                key = q.x;
                src = q.y;
                return;
            }
        }
        key = a.cx.key[pos];
        src = pos;
    }

    template <int S>
    __device__ Group fetch(int lane, uint32_t g, uint32_t end, uint32_t ebase) const {
        Group f;
        const uint32_t idx = g + uint32_t(lane / S), o = uint32_t(lane % S);
        f.info = L.ord[min(idx, end - 1u)];
        const uint32_t p = (f.info >> 11) & 0x3ffu, slot = (f.info & 0x7ffu) + o;
        f.live = idx < end && o < p;
        const uint32_t d = f.live ? L.d[slot] : kNoRun;
        // the run that holds this product starts at the nearest marked lane
        // (a row's first product always starts one)
        const int src = 63 - __clzll((long long)(__ballot(d != kNoRun) & lanes_upto(lane)));
        const uint32_t pos = uint32_t(__shfl(int(d), src, kWave)) + slot;
        f.key = f.src = 0;
        f.va = In(0);
        if (f.live) {
            partner(pos, f.key, f.src);
            if constexpr (kVal) f.va = static_cast<const In*>(a.val)[ebase + L.x[slot - uint32_t(lane - src)]];
        }
        return f;
    }

    template <int S>
    __device__ void finish(int lane, const wsort::Sides& sides, const Group& f) const {
        const uint32_t o = uint32_t(lane % S);
        const uint32_t p = (f.info >> 11) & 0x3ffu, row = f.info >> 21;
        In vb = In(0);
        if constexpr (kVal) vb = f.live ? right_values()[f.src] : In(0);  // (in flight during the sort)
        Key k = f.live ? sort_key(f.key, o) : kDead;
        k = wsort::sort_segments<S>(k, sides);
        double v = 0.0;
        if constexpr (kVal)
            v = __shfl(double(f.va) * double(vb), int((uint32_t(lane) & ~uint32_t(S - 1)) | (index_of(k) & uint32_t(S - 1))),
                       kWave);
        // (the row's products fill its first p lanes before and after the sort)
        const uint32_t j = column_of(k);
        const uint32_t prev = wsort::from_lane_before(j, 0u);  // (with every lane active)
        const bool same = f.live && o > 0 && prev == j;
        const int64_t out = L.out[row];
        const uint32_t len_i = SR == kJaccard && WIDE ? L.len[row] : 0u;
        if (__ballot(same) == 0) {
            if (f.live) emit(out + o, k, 1u, v, len_i);
            if (f.live && o == 0) L.cnt[row] = uint16_t(p);
            return;
        }
        const bool head = f.live && !same;
        const uint64_t seg = S == 64 ? ~uint64_t(0) : ((uint64_t(1) << (S & 63)) - 1) << (lane & ~(S - 1));
        const uint64_t hm = __ballot(head) & seg;
        const uint32_t rank = uint32_t(__popcll(hm & lanes_upto(lane))) - 1u;  // (heads)
        const uint64_t above = (hm >> lane) >> 1;
        const uint32_t cnt = above ? uint32_t(__ffsll((long long)above)) : p - o;
        if constexpr (kVal) {
            const uint32_t most = wave_reduce_max(head ? cnt : 1u);
            const double first = v;
            for (uint32_t c = 1; c < most; ++c) {
                const double w = __shfl_down(first, c, kWave);
                if (head && c < cnt) v += w;
            }
        }
        if (head) emit(out + rank, k, cnt, v, len_i);
        if (f.live && o == 0) L.cnt[row] = uint16_t(__popcll(hm));
    }

    template <int S>
    __device__ void short_rows(uint32_t begin, uint32_t end, uint32_t ebase) const {
        if (begin >= end) return;
        constexpr uint32_t kSide = kWave / S;
        const int lane = fresh_lane();
        const wsort::Sides sides(lane);
        Group f = fetch<S>(lane, begin, end, ebase);
        for (uint32_t g = begin; g < end; g += kSide) {
            Group n = f;
            if (g + kSide < end) n = fetch<S>(lane, g + kSide, end, ebase);  // (in flight during the sort)
            finish<S>(lane, sides, f);
            f = n;
        }
    }

    // Key word and (plus-times) factors of product o of a row whose slots
    // start at s0, every lane of one register; dc and sc carry the last run
    // begun before this register (its word and slot).
    __device__ Group fetch_at(int lane, uint32_t s0, uint32_t o, uint32_t p, uint32_t ebase, uint32_t& dc, uint32_t& sc,
                              uint32_t& x) const {
        Group f;
        f.info = 0;
        f.live = o < p;
        const uint32_t slot = s0 + o;
        const uint32_t d = f.live ? L.d[slot] : kNoRun;
        const uint64_t marks = __ballot(d != kNoRun), lm = marks & lanes_upto(lane);
        const int src = 63 - __clzll((long long)lm);
        const uint32_t dd = uint32_t(__shfl(int(d), src, kWave));
        const uint32_t pos = (lm ? dd : dc) + slot;
        x = 0;
        f.key = f.src = 0;
        f.va = In(0);
        if (f.live) {
            partner(pos, f.key, f.src);
            if constexpr (kVal) x = L.x[lm ? slot - uint32_t(lane - src) : sc];
        }
        if (marks) {
            const int last = 63 - __clzll((long long)marks);
            dc = uint32_t(__builtin_amdgcn_readlane(int(d), last));
            sc = slot - uint32_t(lane) + uint32_t(last);
        }
        return f;
    }

    // ---- rows of 65 to 128 products, one at a time in two registers

    __device__ void pair_rows(uint32_t begin, uint32_t end, uint32_t ebase) const {
        if (begin >= end) return;
        const int lane = fresh_lane();
        const wsort::Sides sides(lane);
        for (uint32_t g = begin; g < end; ++g)
            pair_row(lane, sides, uint32_t(__builtin_amdgcn_readfirstlane(int(L.ord[g]))), ebase);
    }

    __device__ void pair_row(int lane, const wsort::Sides& sides, uint32_t info, uint32_t ebase) const {
        const uint32_t s0 = info & 0x7ffu, p = (info >> 11) & 0x3ffu, row = info >> 21;
        const uint32_t o1 = uint32_t(kWave + lane);
        Key k[2];
        double t[2] = {0.0, 0.0};
        {
            uint32_t dc = 0, sc = 0, x[2];
            Group f[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) f[u] = fetch_at(lane, s0, uint32_t(u * kWave + lane), p, ebase, dc, sc, x[u]);
            In vb[2] = {In(0), In(0)};
            if constexpr (kVal) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (f[u].live) {
                        f[u].va = static_cast<const In*>(a.val)[ebase + x[u]];
                        vb[u] = right_values()[f[u].src];
                    }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                k[u] = f[u].live ? sort_key(f[u].key, uint32_t(u * kWave + lane)) : kDead;
                if constexpr (kVal) t[u] = double(f[u].va) * double(vb[u]);
            }
        }
        wsort::sort_regs<2>(k, sides);
        double v[2] = {0.0, 0.0};
        if constexpr (kVal) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t o = index_of(k[u]);
                const double lo = __shfl(t[0], int(o & 63u), kWave), hi = __shfl(t[1], int(o & 63u), kWave);
                v[u] = (o & 64u) ? hi : lo;
            }
        }
        const int64_t out = L.out[row];
        const uint32_t len_i = SR == kJaccard && WIDE ? L.len[row] : 0u;
        const uint32_t j0 = column_of(k[0]), j1 = column_of(k[1]);
        const uint32_t prev0 = wsort::from_lane_before(j0, 0u);
        const uint32_t prev1 = wsort::from_lane_before(j1, uint32_t(__builtin_amdgcn_readlane(int(j0), kWave - 1)));
        const bool same0 = lane > 0 && prev0 == j0, same1 = o1 < p && prev1 == j1;
        if ((__ballot(same0) | __ballot(same1)) == 0) {
            emit(out + lane, k[0], 1u, v[0], len_i);
            if (o1 < p) emit(out + o1, k[1], 1u, v[1], len_i);
            if (lane == 0) L.cnt[row] = uint16_t(p);
            return;
        }
        const bool head0 = !same0, head1 = o1 < p && !same1;
        const uint64_t hm0 = __ballot(head0), hm1 = __ballot(head1);
        // every head's terms: up to the next head or the row's end
        const uint64_t up0 = (hm0 >> lane) >> 1, up1 = (hm1 >> lane) >> 1;
        const uint32_t next = hm1 ? uint32_t(kWave) + uint32_t(__ffsll((long long)hm1)) - 1u : p;
        const uint32_t cnt0 = up0 ? uint32_t(__ffsll((long long)up0)) : next - uint32_t(lane);
        const uint32_t cnt1 = up1 ? uint32_t(__ffsll((long long)up1)) : p - o1;
        if constexpr (kVal) {
            // terms of a column in product order: the sorted products moved
            // down one lane at a time
            const uint32_t most = wave_reduce_max(max(head0 ? cnt0 : 1u, head1 ? cnt1 : 1u));
            double w0 = v[0], w1 = v[1];
            for (uint32_t c = 1; c < most; ++c) {
                const double first1 = __shfl(w1, 0, kWave);
                w0 = __shfl_down(w0, 1, kWave);
                w1 = __shfl_down(w1, 1, kWave);
                if (lane == kWave - 1) w0 = first1;
                if (head0 && c < cnt0) v[0] += w0;
                if (head1 && c < cnt1) v[1] += w1;
            }
        }
        const uint32_t n0 = uint32_t(__popcll(hm0));
        if (head0) emit(out + __popcll(hm0 & lanes_upto(lane)) - 1, k[0], cnt0, v[0], len_i);
        if (head1) emit(out + n0 + uint32_t(__popcll(hm1 & lanes_upto(lane))) - 1, k[1], cnt1, v[1], len_i);
        if (lane == 0) L.cnt[row] = uint16_t(n0 + uint32_t(__popcll(hm1)));
    }

    // ---- rows of more than 128 products, one at a time: 64 products sorted
    // in a register at a time, merged in LDS (few registers, rolled loops)

    __device__ void long_rows(uint32_t begin, uint32_t end, uint32_t ebase) const {
        if (begin >= end) return;
        const int lane = fresh_lane();
        const wsort::Sides sides(lane);
        for (uint32_t g = begin; g < end; ++g) {
            wave_sync();
            long_row(lane, sides, uint32_t(__builtin_amdgcn_readfirstlane(int(L.ord[g]))), ebase);
        }
    }

    // value of a product (its entry and its partner's place kept at its slot)
    __device__ double term(uint32_t slot, uint32_t ebase) const {
        return double(static_cast<const In*>(a.val)[ebase + L.x[slot]]) *
               double(right_values()[L.d[slot]]);
    }

    __device__ void long_row(int lane, const wsort::Sides& sides, uint32_t info, uint32_t ebase) const {
        const uint32_t s0 = info & 0x7ffu, p = (info >> 11) & 0x3ffu, row = info >> 21;
        Key* K;
        if constexpr (WaveLds<kVal, Key>::kOwnKeys)
            K = L.key;
        else
            K = L.d + s0;
        uint32_t dc = 0, sc = 0;
#pragma unroll 1
        for (uint32_t o = uint32_t(lane); o < ((p + 63u) & ~63u); o += kWave) {
            uint32_t x;
            const Group f = fetch_at(lane, s0, o, p, ebase, dc, sc, x);
            Key k = f.live ? sort_key(f.key, o) : kDead;
            k = wsort::sort64(k, sides);
            if (f.live) {
                K[o] = k;
                if constexpr (kVal) {
                    L.d[s0 + o] = f.src;
                    // (a run reaching into the next registers is looked up
                    // at its slot again: its first slot keeps its entry)
                    L.x[s0 + o] = uint16_t(x);
                }
            }
        }
        // blocks of B sorted keys merged in pairs: mirror-image exchanges
        // across the pair, then half-cleaners; every block ascends, so the
        // keys past the row's end stay virtual
#pragma unroll 1
        for (uint32_t B = kWave; B < p; B <<= 1) {
            wave_sync();
#pragma unroll 1
            for (uint32_t q = uint32_t(lane); 2 * (q & ~(B - 1)) < p; q += kWave) {
                // (q counts the lower blocks' elements: element e of pair b)
                const uint32_t b = 2 * (q & ~(B - 1)), e = q & (B - 1);
                const uint32_t i = b + e, j = b + 2 * B - 1 - e;
                if (j < p) {
                    const Key u = K[i], w = K[j];
                    if (w < u) {
                        K[i] = w;
                        K[j] = u;
                    }
                }
            }
#pragma unroll 1
            for (uint32_t h = B >> 1; h >= uint32_t(kWave); h >>= 1) {
                wave_sync();
#pragma unroll 1
                for (uint32_t q = uint32_t(lane); 2 * (q & ~(h - 1)) < p; q += kWave) {
                    const uint32_t i = 2 * (q & ~(h - 1)) + (q & (h - 1)), j = i + h;
                    if (j < p) {
                        const Key u = K[i], w = K[j];
                        if (w < u) {
                            K[i] = w;
                            K[j] = u;
                        }
                    }
                }
            }
            wave_sync();
#pragma unroll 1
            for (uint32_t o = uint32_t(lane); o < ((p + 63u) & ~63u); o += kWave) {
                const Key k = wsort::merge64(o < p ? K[o] : kDead, sides);
                if (o < p) K[o] = k;
            }
        }
        wave_sync();
        const int64_t out = L.out[row];
        const uint32_t len_i = SR == kJaccard && WIDE ? L.len[row] : 0u;
        uint32_t heads = 0;
#pragma unroll 1
        for (uint32_t o = uint32_t(lane); o < ((p + 63u) & ~63u); o += kWave) {
            const Key k = o < p ? K[o] : kDead;
            const uint32_t j = column_of(k);
            const bool head = o < p && !(o > 0 && column_of(K[o - 1]) == j);
            const uint64_t hm = __ballot(head);
            if (head) {
                double v = 0.0;
                if constexpr (kVal) v = term(s0 + index_of(k), ebase);
                uint32_t cnt = 1;  // terms in product order
                for (; o + cnt < p; ++cnt) {
                    const Key n = K[o + cnt];
                    if (column_of(n) != j) break;
                    if constexpr (kVal) v += term(s0 + index_of(n), ebase);
                }
                emit(out + heads + uint32_t(__popcll(hm & lanes_upto(lane))) - 1, k, cnt, v, len_i);
            }
            heads += uint32_t(__popcll(hm));
        }
        if (lane == 0) L.cnt[row] = uint16_t(heads);
    }

    // Entries [eb, eb + ne) of the batch: their runs marked at their first
    // product slots (nprod slots).
    __device__ void mark_runs(uint32_t eb, int ne, int nprod) const {
        const int lane = fresh_lane();
        for (int q = 4 * lane; q < nprod; q += 4 * kWave)
            *reinterpret_cast<uint4*>(L.d + q) = make_uint4(kNoRun, kNoRun, kNoRun, kNoRun);
        wave_sync();
        constexpr int kU = 4;  // run words per lane in flight
        uint32_t carry = 0;
        for (int b = 0; b < ne; b += kU * kWave) {
            uint32_t w[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int q = b + u * kWave + lane;
                w[u] = q < ne ? a.run.r4[eb + q] : 0u;
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int q = b + u * kWave + lane;
                if (b + u * kWave >= ne) break;
                const uint2 r = q < ne ? run_from(a.run, w[u], int64_t(eb) + q) : make_uint2(0u, 0u);
                const uint32_t len = r.y - r.x;
                const uint32_t inc = wsort::inclusive_sum(len);
                const uint32_t slot = carry + inc - len;
                if (len) {
                    L.d[slot] = r.x - slot;
                    if constexpr (kVal) L.x[slot] = uint16_t(q);
                }
                carry += uint32_t(__builtin_amdgcn_readlane(int(inc), kWave - 1));
            }
        }
        wave_sync();
    }

    // A chunk's row pointers, product counts and staging slots (lane = row),
    // loaded in one round, ahead of the chunk.
    struct Head {
        int64_t ubv = 0;
        uint32_t pr = 0;  // (over the light rows' limit: kFP + 1)
        uint32_t rpv = 0, rpn = 0;  // the row's entries
    };
    __device__ Head head(int64_t c) const {
        const int lane = lane0;
        const int R = a.rows_per_chunk;
        const int64_t rs = c * R;
        const int nr = int(min(int64_t(R), a.m - rs));
        Head h;
        if (lane < nr) {
            h.rpv = uint32_t(a.rp[rs + lane]);  // (entries of A are below 2^31)
            h.rpn = uint32_t(a.rp[rs + lane + 1]);
            h.pr = uint32_t(min(a.prod[rs + lane], (unsigned long long)(kFP + 1)));
            h.ubv = a.ubp[rs + lane];
        }
        return h;
    }

    // Sum of the squares of every light row's entries (lane = row): eight
    // lanes per row, two groups of eight rows at a time, the first 32 entries
    // of each in one round of loads.
    __device__ double diagonals(uint32_t rpv, int nr) const {
        const int lane = fresh_lane();
        double mine = 0.0;
        const uint32_t sub = uint32_t(lane) & 7u;
        constexpr int kU = 4;
        for (int g = 0; g < nr; g += 16) {
            double t[2];
            In v[2][kU];
            uint32_t s[2], e[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int row = min(g + 8 * h + (lane >> 3), kFR - 1);
                s[h] = uint32_t(__shfl(int(rpv), row, kWave)) + sub;
                e[h] = s[h] - sub + (g + 8 * h + (lane >> 3) < nr ? uint32_t(L.len[row]) : 0u);
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    v[h][u] = s[h] + 8u * u < e[h] ? static_cast<const In*>(a.val)[s[h] + 8u * u] : In(0);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                t[h] = 0.0;
#pragma unroll
                for (int u = 0; u < kU; ++u) t[h] += double(v[h][u]) * double(v[h][u]);
                for (uint32_t q = s[h] + 8u * kU; q < e[h]; q += 8u) {
                    const double w = double(static_cast<const In*>(a.val)[q]);
                    t[h] += w * w;
                }
                t[h] = wsort::sum8(t[h]);
                const double got = __shfl(t[h], int(8u * sub), kWave);
                if ((lane >> 3) == (g >> 3) + h) mine = got;
            }
        }
        return mine;
    }

    __device__ void run(int64_t c, const Head& h) {
        const int lane = lane0;
        const int R = a.rows_per_chunk;
        r0 = c * R;
        const int nr = int(min(int64_t(R), a.m - r0));
        const uint32_t len = h.rpn - h.rpv;
        const bool light = lane < nr && h.pr <= uint32_t(kFP) && len <= uint32_t(kFE);
        const uint32_t p = light ? h.pr : 0u;
        L.out[lane] = h.ubv;
        L.cnt[lane] = 0;
        L.len[lane] = light ? uint16_t(len) : uint16_t(0);
        const uint32_t pinc = wsort::inclusive_sum(p), pexc = pinc - p;
        // batches of consecutive light rows, cut greedily: a batch opened at
        // row ra takes the following light rows while its products fit
        const uint64_t lightmask = __ballot(light);
        for (uint64_t rest = lightmask; rest;) {
            const int ra = __ffsll((unsigned long long)rest) - 1;
            const uint32_t pa = uint32_t(__builtin_amdgcn_readlane(int(pexc), ra));
            const uint64_t okm = __ballot(lane >= ra && light && pinc - pa <= uint32_t(kCap)) >> ra;
            const int rb = ~okm ? ra + __ffsll((unsigned long long)~okm) - 1 : kWave;
            rest = rb < kWave ? lightmask & (~uint64_t(0) << rb) : 0;
            const uint32_t nprod = uint32_t(__builtin_amdgcn_readlane(int(pinc), rb - 1)) - pa;
            if (nprod == 0) continue;
            const uint32_t eb = uint32_t(__builtin_amdgcn_readlane(int(h.rpv), ra));
            const uint32_t ee = uint32_t(__builtin_amdgcn_readlane(int(h.rpn), rb - 1));
            mark_runs(eb, int(ee - eb), int(nprod));
            // rows by size class
            const uint32_t q = lane >= ra && lane < rb ? p : 0u;
            const uint32_t info = (pexc - pa) | (p << 11) | (uint32_t(lane) << 21);
            constexpr uint32_t kMost[6] = {8, 16, 32, 64, 128, kFP};
            uint32_t at[7];
            at[0] = 0;
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const bool in = q > (k ? kMost[k ? k - 1 : 0] : 0u) && q <= kMost[k];
                const uint64_t m = __ballot(in);
                if (in) L.ord[at[k] + uint32_t(__popcll(m & lanes_upto(lane))) - 1u] = info;
                at[k + 1] = at[k] + uint32_t(__popcll(m));
            }
            wave_sync();
            short_rows<8>(at[0], at[1], eb);
            short_rows<16>(at[1], at[2], eb);
            short_rows<32>(at[2], at[3], eb);
            short_rows<64>(at[3], at[4], eb);
            pair_rows(at[4], at[5], eb);
            long_rows(at[5], at[6], eb);
            wave_sync();
        }
        wave_sync();
        double dv = 0.0;
        if constexpr (LOWER && kVal) dv = diagonals(h.rpv, nr);
        if (lane < nr) {
            // exact lengths; diagonals (lower triangle) end their rows
            int64_t cnt = light ? int64_t(L.cnt[lane]) : a.heavy_nnz[r0 + lane];
            if (LOWER && light && len > 0) {
                const int64_t at = h.ubv + cnt;
                const uint32_t i = uint32_t(r0 + lane);
                if constexpr (kVal) {
                    a.c_ci[at] = int32_t(i);
                    static_cast<Out*>(a.c_val)[at] = Out(dv);
                } else if constexpr (SR == kCount) {  // |S(i) and S(i)| = |S(i)|
                    emit(at, Key(i), len, 0.0, len);
                } else if constexpr (WIDE) {
                    emit(at, (uint64_t(i) << 32) | len, len, 0.0, len);
                } else {
                    emit(at, i * a.pack_rr + a.pack_r2 + len, len, 0.0, len);
                }
                ++cnt;
            }
            a.row_cnt[r0 + lane] = cnt;
        }
        wave_sync();
    }
};

// Persistent wavefronts.  Up to kDealtBelow chunks they are dealt out in turn
// (c, c + stride, ...).  Past that, the wavefronts take runs of consecutive
// chunks from a counter, so that every wavefront the device holds keeps busy
// however many of the launched ones are resident at once and however the
// chunks' costs vary: a run is a quarter of the chunks left per launched
// wavefront (as last seen), at least one, so the runs shrink towards the end.
// The next chunk is taken and its head loaded while the current chunk runs.
// The runs cost an atomic add on one address each, about 10 ns, 46,000 of them
// for 65,536 chunks: 0.5 ms, which only long launches hide, so the line lies
// at a number of chunks (64 rows each there), whatever the wavefronts.  (Dealt
// against counted: off-diagonal Jaccard, 2^20 rows in 65,536 chunks, whole call
// 0.96 and 1.38 ms; f64, 1.4 M rows in 87,500 chunks, 1.04 and 1.43.)
template <int SR, bool LOWER, bool WIDE>
__device__ void all_chunks(const FusedArgs& a) {
    using C = Chunk<SR, LOWER, WIDE>;
    __shared__ WaveLds<C::kVal, typename C::Key> lds[kWavesF];
    C ch(a, lds[threadIdx.x / kWave]);
    const int lane = lane_id();
    if (blockIdx.x == 0 && threadIdx.x == 0) a.row_cnt[a.m] = 0;  // (the scan's last input)
    const int64_t nwaves = int64_t(gridDim.x) * kWavesF;
    const bool dealt = a.nchunks < kDealtBelow;
    int64_t seen = 0, rend = 0;
    auto take = [&]() -> int64_t {
        if (dealt) {
            const int64_t c = seen ? rend + nwaves - 1 : int64_t(blockIdx.x) * kWavesF + threadIdx.x / kWave;
            seen = 1;
            rend = c + 1;
            return c;
        }
        int64_t g = (a.nchunks - seen) / (4 * nwaves);
        g = g < 1 ? 1 : g;
        unsigned long long c0 = 0;
        if (lane == 0) c0 = atomicAdd(a.chunk_counter, (unsigned long long)g);
        const int64_t c = int64_t(__shfl(c0, 0, kWave));
        seen = c + g;
        rend = c + g;
        return c;
    };
    int64_t c = take();
    if (c >= a.nchunks) return;
    auto h = ch.head(c);
    while (true) {
        const int64_t cn = c + 1 < rend ? c + 1 : take();
        decltype(h) hn;
        if (cn < a.nchunks) hn = ch.head(cn);
        ch.run(c, h);
        if (cn >= a.nchunks) break;
        c = cn;
        h = hn;
    }
}

// Wavefronts per SIMD: six (80 VGPRs), plus-times five (96); Jaccard off the
// diagonal, which has no packed words and so 64-bit keys of its own in LDS
// (9 KiB per wavefront), four.
constexpr int light_waves(int sr, bool lower) { return sr == kF64 || sr == kF32 ? 5 : (sr == kJaccard && !lower ? 4 : 6); }
template <int SR, bool LOWER>
__global__ __launch_bounds__(kWave* kWavesF) __attribute__((amdgpu_waves_per_eu(light_waves(SR, LOWER))))
void fused_kernel(FusedArgs a) {
    all_chunks<SR, LOWER, SR == kJaccard && !LOWER>(a);
}
template <int SR, bool LOWER>
__global__ __launch_bounds__(kWave* kWavesF) __attribute__((amdgpu_waves_per_eu(4)))
void fused_wide(FusedArgs a) {
    all_chunks<SR, LOWER, true>(a);
}

// Workgroups resident on the whole device at once (at least one).
template <typename K>
int resident_groups(K kernel) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, kWave * kWavesF, 0) != hipSuccess) return 1;
    const int g = cus * per;
    return g > 0 ? g : 1;
}

template <int SR, bool LOWER>
void launch(const FusedArgs& a, bool wide, int grid, hipStream_t s) {
    if constexpr (SR != kCount && !(SR == kJaccard && !LOWER)) {
        if (wide) {
            static const int res = resident_groups(fused_wide<SR, LOWER>);
            fused_wide<SR, LOWER><<<grid < res ? grid : res, kWave * kWavesF, 0, s>>>(a);
            return;
        }
    }
    static const int res = resident_groups(fused_kernel<SR, LOWER>);
    fused_kernel<SR, LOWER><<<grid < res ? grid : res, kWave * kWavesF, 0, s>>>(a);
}

template <int SR>
void launch(const FusedArgs& a, int grid, hipStream_t s) {
    // 64-bit sort keys where a column and a product index, or a Jaccard
    // word, do not fit 32 bits
    const bool wide = SR == kJaccard ? a.pack_rr == 0 : a.m_right > (int64_t(1) << (32 - kOrdBits));
    if (a.lower)
        launch<SR, true>(a, wide, grid, s);
    else
        launch<SR, false>(a, wide, grid, s);
}

__global__ __launch_bounds__(kBlock) void classify_kernel(const int64_t* __restrict__ rp,
                                                          const unsigned long long* __restrict__ prod, int64_t m,
                                                          bool lower, int32_t* __restrict__ heavy_rows,
                                                          int32_t* heavy_count, unsigned long long* light_cap,
                                                          unsigned long long* prod_sum, int64_t* __restrict__ ub,
                                                          unsigned long long* maxlen, unsigned long long* dense,
                                                          int ncells) {
    __shared__ unsigned long long wt[kWavesPerBlock][3];
    __shared__ unsigned long long dn[6];
    if (threadIdx.x < 6) dn[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long cap = 0, ps = 0, ml = 0;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < m; i += int64_t(gridDim.x) * kBlock) {
        const int64_t len = rp[i + 1] - rp[i];
        const unsigned long long pr = prod[i];
        ps += pr;
        ml = max(ml, (unsigned long long)len);
        int64_t u = 0;
        if (pr <= (unsigned long long)kFP && len <= kFE) {
            u = int64_t(pr) + ((lower && len > 0) ? 1 : 0);
            cap += u;
        } else {
            heavy_rows[atomicAdd(heavy_count, 1)] = int32_t(i);
            if (dense_row(pr, uint64_t(len), ncells)) {
                unsigned long long* d = dn + (pr >= kDenseProducts ? 0 : 3);
                atomicAdd(d, 1ull);
                atomicAdd(d + 1, (unsigned long long)len);
                atomicAdd(d + 2, pr);
            }
        }
        ub[i] = u;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ub[m] = 0;  // (the scan's last input)
    cap = wave_reduce_sum(cap);
    ps = wave_reduce_sum(ps);
    ml = wave_reduce_max(ml);
    if (lane_id() == 0) {
        wt[threadIdx.x / kWave][0] = cap;
        wt[threadIdx.x / kWave][1] = ps;
        wt[threadIdx.x / kWave][2] = ml;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long c = 0, p = 0, l = 0;
        for (int w = 0; w < kWavesPerBlock; ++w) {
            c += wt[w][0];
            p += wt[w][1];
            l = max(l, wt[w][2]);
        }
        if (c) atomicAdd(light_cap, c);
        if (p) atomicAdd(prod_sum, p);
        if (l && maxlen) atomicMax(maxlen, l);
    }
    if (dense && threadIdx.x < 6 && dn[threadIdx.x]) atomicAdd(dense + threadIdx.x, dn[threadIdx.x]);
}

}  // namespace

void classify_rows(const int64_t* rp, const unsigned long long* prod, int64_t m, bool lower, int32_t* heavy_rows,
                   int32_t* heavy_count, unsigned long long* light_cap, unsigned long long* prod_sum, int64_t* ub,
                   hipStream_t s, unsigned long long* maxlen, unsigned long long* dense) {
    if (m <= 0) return;
    int64_t grid = (m + kBlock - 1) / kBlock;
    if (grid > 1024) grid = 1024;
    classify_kernel<<<unsigned(grid), kBlock, 0, s>>>(rp, prod, m, lower, heavy_rows, heavy_count, light_cap,
                                                      prod_sum, ub, maxlen, dense, dense_cells(m));
}

void light_fused(const FusedArgs& a, hipStream_t s) {
    const int grid = int((a.nchunks + kWavesF - 1) / kWavesF);
    if (grid <= 0) return;
    switch (a.sr) {
        case kF64: launch<kF64>(a, grid, s); break;
        case kF32: launch<kF32>(a, grid, s); break;
        case kCount: launch<kCount>(a, grid, s); break;
        default: launch<kJaccard>(a, grid, s); break;
    }
}

}  // namespace spsyrk
