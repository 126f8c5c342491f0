// Walking the products of many stretches of the column index by one
// workgroup: the stretches, one per thread, are laid end to end and shared
// out evenly over the wavefronts, 64 consecutive products per register.
//
// A lane finds the stretch of its product from marks: the stretches that
// begin among the next KU * 64 products write their numbers at their first
// products' slots of a wavefront's own LDS bytes, and the nearest marked lane
// at or below (one ballot) names the stretch.  That costs the same for one
// stretch per register as for twenty; stepping through the beginnings one by
// one (scalar lane reads) took 9 of 14 ms of R-MAT's dense rows, whose
// stretches hold about 20 products.
#pragma once

#include "common.h"
#include "wave_sort.h"

namespace spsyrk {

// NT threads; VAL: with a value of type In per stretch; KU registers of
// products in flight per wavefront
template <typename In, bool VAL, int NT, int KU>
struct Stretches {
    static constexpr int kWaves = NT / kWave;
    static constexpr int kPiece = KU * kWave;
    static_assert(kPiece <= 256, "a mark is one byte");
    uint32_t off[NT + 1];  // first product of every stretch that is not empty, then their total
    uint32_t pos[NT];      // position less product
    In val[VAL ? NT : 1];
    uint32_t wt[kWaves];   // (a wavefront's products)
    uint32_t wn[kWaves];   // a wavefront's stretches that are not empty
    alignas(4) uint8_t mark[kWaves][kPiece];

    // exclusive scan over the workgroup's threads; *total gets the sum
    __device__ uint32_t scan(uint32_t v, uint32_t* total) {
        const int w = threadIdx.x / kWave;
        const uint32_t inc = wsort::inclusive_sum(v);
        if (lane_id() == kWave - 1) wt[w] = inc;
        __syncthreads();
        uint32_t before = 0, tot = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
            const uint32_t t = wt[q];
            if (q < w) before += t;
            tot += t;
        }
        __syncthreads();
        *total = tot;
        return before + inc - v;
    }

    __device__ static void wave_fence() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // The products of the stretches [lo, hi), one per thread (v: the
    // stretch's value): use(first product, end of the share, positions,
    // values) for every KU registers.  Called by all threads.
    template <typename F>
    __device__ void products(uint32_t lo, uint32_t hi, In v, F use) {
        // (an opaque lane number: what is derived from it is formed here, not
        // kept in registers across the caller's loops)
        int lane = lane_id();
        asm volatile("" : "+v"(lane));
        const uint32_t w = uniform(threadIdx.x / kWave);
        // the places and first products of the stretches that are not empty,
        // by one exchange of every wavefront's counts (the barriers below
        // order those words' next use)
        const uint32_t len = hi - lo;
        const uint64_t some = __ballot(len != 0);
        const uint32_t inc = wsort::inclusive_sum(len);
        if (lane == kWave - 1) {
            wt[w] = inc;
            wn[w] = uint32_t(__popcll(some));
        }
        __syncthreads();
        const uint32_t lens = lane < kWaves ? wt[lane] : 0u, nums = lane < kWaves ? wn[lane] : 0u;
        const uint32_t leni = wsort::inclusive_sum(lens), numi = wsort::inclusive_sum(nums);
        auto of = [](uint32_t v, uint32_t l) { return uint32_t(__builtin_amdgcn_readlane(int(v), int(l))); };
        const uint32_t n = of(numi, kWaves - 1), total = of(leni, kWaves - 1);
        const uint32_t at = of(numi, w) - of(nums, w) + uint32_t(__popcll(some & ((uint64_t(1) << lane) - 1)));
        const uint32_t first = of(leni, w) - of(lens, w) + inc - len;
        if (len) {
            off[at] = first;
            pos[at] = lo - first;
            if constexpr (VAL) val[at] = v;
        }
        if (threadIdx.x == 0) off[n] = total;
        __syncthreads();
        const uint32_t share = ((total + NT - 1) / NT) * kWave;
        const uint32_t ts = w * share, te = min(total, ts + share);
        if (ts < te) {
            // the stretch that holds product ts
            uint32_t cur = 0;
            for (uint32_t x = 0; x < n; x += kWave)
                cur += uint32_t(__popcll(__ballot(x + lane < n && off[min(x + lane, n)] <= ts)));
            cur = uniform(cur - 1);
            pieces(lane, w, n, ts, te, cur, use);
        }
        __syncthreads();
    }

    // The same by every wavefront for its own 64 stretches, with no barrier:
    // for batches of short stretches, too few products to share out over the
    // workgroup.  (Barriers order it before and after products.)
    template <typename F>
    __device__ void own_products(uint32_t lo, uint32_t hi, In v, F use) {
        int lane = lane_id();
        asm volatile("" : "+v"(lane));
        const uint32_t w = uniform(threadIdx.x / kWave);
        const uint32_t len = hi - lo;
        const uint64_t some = __ballot(len != 0);
        if (some == 0) return;
        const uint32_t inc = wsort::inclusive_sum(len);
        if (len) {
            const uint32_t at = w * kWave + uint32_t(__popcll(some & ((uint64_t(1) << lane) - 1)));
            off[at] = inc - len;
            pos[at] = lo - (inc - len);
            if constexpr (VAL) val[at] = v;
        }
        wave_fence();
        pieces(lane, w, w * kWave + uint32_t(__popcll(some)), 0u, uint32_t(__builtin_amdgcn_readlane(int(inc), kWave - 1)),
               w * kWave, use);
        wave_fence();
    }

  private:
    // Products [ts, te) by wavefront w; product ts lies in stretch cur, the
    // stretches end at n.
    template <typename F>
    __device__ void pieces(int lane, uint32_t w, uint32_t n, uint32_t ts, uint32_t te, uint32_t cur, F use) {
                    uint8_t* mk = mark[w];
                    const uint64_t upto = (uint64_t(2) << lane) - 1;
                    for (uint32_t t = ts; t < te; t += kPiece) {
                        // stretches that begin after product t, in this piece (marked)
                        // or right behind it (then the next piece's first)
                        if (4 * lane < kPiece) reinterpret_cast<uint32_t*>(mk)[lane] = 0;
                        wave_fence();
                        uint32_t begun = 0;
                        for (uint32_t x = 1; x <= uint32_t(kPiece); x += kWave) {
                            const uint32_t s = cur + x + lane;
                            const uint32_t d = s < n ? off[s] - t : ~0u;
                            if (d < uint32_t(kPiece)) mk[d] = uint8_t(x + lane);
                            const uint32_t c = uint32_t(__popcll(__ballot(d <= uint32_t(kPiece))));
                            begun += c;
                            if (c < uint32_t(kWave)) break;
                        }
                        wave_fence();
                        uint32_t p[KU];
                        In a[KU];
                        if (begun == 0) {  // one stretch holds the whole piece
                            const uint32_t base = pos[cur] + t + lane;
                            const In v = VAL ? val[VAL ? cur : 0] : In(0);
        #pragma unroll
                            for (int u = 0; u < KU; ++u) {
                                p[u] = base + uint32_t(u * kWave);
                                a[u] = v;
                            }
                        } else {
                            uint32_t carry = 0;
        #pragma unroll
                            for (int u = 0; u < KU; ++u) {
                                const uint32_t m = mk[u * kWave + lane];
                                const uint64_t has = __ballot(m != 0), below = has & upto;
                                const uint32_t mine = uint32_t(__shfl(int(m), 63 - __clzll((long long)below), kWave));
                                const uint32_t s = cur + (below ? mine : carry);
                                if (has) carry = uint32_t(__builtin_amdgcn_readlane(int(m), 63 - __clzll((long long)has)));
                                p[u] = pos[s] + t + uint32_t(u * kWave) + lane;
                                a[u] = In(0);
                                if constexpr (VAL) a[u] = val[s];
                            }
                        }
                        use(t, te, p, a);
                        cur += begun;
                    }
    }
};

}  // namespace spsyrk
