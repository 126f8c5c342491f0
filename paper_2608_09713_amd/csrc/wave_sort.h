// Sorting of short key lists in the registers of one wavefront.
//
// A bitonic network over lanes, every compare-exchange a cross-lane move and
// one median: med3(a, b, 0) is min(a, b) and med3(a, b, ~0) is max(a, b), so a
// lane's side of the exchange is a constant register instead of a select.
// Distances inside a row of 16 lanes are DPP moves (two for distance 4), 16
// and 32 the lane-swap instructions: no LDS and no address arithmetic.
// Sorting 16 keys per row costs 21 instructions, 32 keys 35, 64 keys 52, for
// the whole wavefront.
#pragma once

#include "common.h"

namespace spsyrk {
namespace wsort {

template <int CTRL, int BANKS = 0xf>
__device__ inline uint32_t dpp(uint32_t old, uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(int(old), int(v), CTRL, 0xf, BANKS, false));
}

constexpr int kXor1 = 0xB1;      // quad_perm [1, 0, 3, 2]
constexpr int kXor2 = 0x4E;      // quad_perm [2, 3, 0, 1]
constexpr int kFlip4 = 0x1B;     // quad_perm [3, 2, 1, 0]
constexpr int kFlip8 = 0x141;    // row_half_mirror
constexpr int kFlip16 = 0x140;   // row_mirror
constexpr int kXor8 = 0x128;     // row_ror:8
constexpr int kFrom4Up = 0x104;  // row_shl:4 (lane i reads lane i + 4)
constexpr int kFrom4Dn = 0x114;  // row_shr:4

// a permutation of the lanes (every lane is written: no old value)
template <int CTRL, int BANKS = 0xf>
__device__ inline uint32_t move(uint32_t v) {
    return uint32_t(__builtin_amdgcn_mov_dpp(int(v), CTRL, 0xf, BANKS, false));
}
__device__ inline uint32_t xor4(uint32_t v) { return dpp<kFrom4Dn, 0xA>(move<kFrom4Up, 0x5>(v), v); }
template <int CTRL>
__device__ inline uint64_t move(uint64_t v) {
    return (uint64_t(move<CTRL>(uint32_t(v >> 32))) << 32) | move<CTRL>(uint32_t(v));
}
__device__ inline uint64_t xor4(uint64_t v) {
    return (uint64_t(xor4(uint32_t(v >> 32))) << 32) | xor4(uint32_t(v));
}

// the two lanes' keys in both lanes: x of the pair's lower row (half), y of
// the upper one
__device__ inline void pair16(uint32_t v, uint32_t& x, uint32_t& y) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    x = r[0];
    y = r[1];
}
__device__ inline void pair32(uint32_t v, uint32_t& x, uint32_t& y) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    x = r[0];
    y = r[1];
}
__device__ inline void pair16(uint64_t v, uint64_t& x, uint64_t& y) {
    uint32_t xl, yl, xh, yh;
    pair16(uint32_t(v), xl, yl);
    pair16(uint32_t(v >> 32), xh, yh);
    x = (uint64_t(xh) << 32) | xl;
    y = (uint64_t(yh) << 32) | yl;
}
__device__ inline void pair32(uint64_t v, uint64_t& x, uint64_t& y) {
    uint32_t xl, yl, xh, yh;
    pair32(uint32_t(v), xl, yl);
    pair32(uint32_t(v >> 32), xh, yh);
    x = (uint64_t(xh) << 32) | xl;
    y = (uint64_t(yh) << 32) | yl;
}

// min(a, b) where c is 0, max(a, b) where c is ~0
__device__ inline uint32_t pick(uint32_t a, uint32_t b, uint32_t c) { return max(min(a, b), min(max(a, b), c)); }
__device__ inline uint64_t pick(uint64_t a, uint64_t b, uint32_t c) {
    const bool less = a < b;
    return less == (c == 0) ? a : b;
}
__device__ inline uint32_t flip(uint32_t v, uint32_t c) { return v ^ c; }
__device__ inline uint64_t flip(uint64_t v, uint32_t c) { return v ^ ((uint64_t(c) << 32) | c); }

// ~0 in the lanes whose number has the bit set
struct Sides {
    uint32_t b1, b2, b4, b8, b16, b32;
    __device__ explicit Sides(int lane) {
        const uint32_t l = uint32_t(lane);
        b1 = 0u - (l & 1u);
        b2 = 0u - ((l >> 1) & 1u);
        b4 = 0u - ((l >> 2) & 1u);
        b8 = 0u - ((l >> 3) & 1u);
        b16 = 0u - ((l >> 4) & 1u);
        b32 = 0u - ((l >> 5) & 1u);
    }
};

template <typename K>
__device__ inline K sort8(K v, const Sides& s) {
    v = pick(v, move<kXor1>(v), s.b1);
    v = pick(v, move<kFlip4>(v), s.b2);
    v = pick(v, move<kXor1>(v), s.b1);
    v = pick(v, move<kFlip8>(v), s.b4);
    v = pick(v, move<kXor2>(v), s.b2);
    return pick(v, move<kXor1>(v), s.b1);
}

template <typename K>
__device__ inline K merge16(K v, const Sides& s) {  // (v bitonic in every row)
    v = pick(v, move<kXor8>(v), s.b8);
    v = pick(v, xor4(v), s.b4);
    v = pick(v, move<kXor2>(v), s.b2);
    return pick(v, move<kXor1>(v), s.b1);
}

template <typename K>
__device__ inline K sort16(K v, const Sides& s) {
    v = sort8(v, s);
    v = pick(v, move<kFlip16>(v), s.b8);
    v = pick(v, xor4(v), s.b4);
    v = pick(v, move<kXor2>(v), s.b2);
    return pick(v, move<kXor1>(v), s.b1);
}

template <typename K>
__device__ inline K merge32(K v, const Sides& s) {
    K x, y;
    pair16(v, x, y);
    return merge16(pick(x, y, s.b16), s);
}

template <typename K>
__device__ inline K sort32(K v, const Sides& s) {
    // the upper row descends (its complement ascends), so the pair is bitonic
    return merge32(flip(sort16(flip(v, s.b16), s), s.b16), s);
}

template <typename K>
__device__ inline K merge64(K v, const Sides& s) {
    K x, y;
    pair32(v, x, y);
    return merge32(pick(x, y, s.b32), s);
}

template <typename K>
__device__ inline K sort64(K v, const Sides& s) {
    return merge64(flip(sort32(flip(v, s.b32), s), s.b32), s);
}

// ascending sort of every segment of S lanes
template <int S, typename K>
__device__ inline K sort_segments(K v, const Sides& s) {
    static_assert(S == 8 || S == 16 || S == 32 || S == 64, "segment size");
    if constexpr (S == 8)
        return sort8(v, s);
    else if constexpr (S == 16)
        return sort16(v, s);
    else if constexpr (S == 32)
        return sort32(v, s);
    else
        return sort64(v, s);
}

// ascending sort of N registers of 64 keys, element k * 64 + lane in v[k]
// (merge_regs: of a bitonic sequence)
template <int N, typename K>
__device__ inline void merge_regs(K* v, const Sides& s) {
    if constexpr (N == 1) {
        v[0] = merge64(v[0], s);
    } else {
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const K a = v[k], b = v[k + N / 2];
            v[k] = a < b ? a : b;
            v[k + N / 2] = a < b ? b : a;
        }
        merge_regs<N / 2>(v, s);
        merge_regs<N / 2>(v + N / 2, s);
    }
}
template <int N, typename K>
__device__ inline void sort_regs(K* v, const Sides& s) {
    if constexpr (N == 1) {
        v[0] = sort64(v[0], s);
    } else {
        sort_regs<N / 2>(v, s);
#pragma unroll
        for (int k = N / 2; k < N; ++k) v[k] = ~v[k];
        sort_regs<N / 2>(v + N / 2, s);
#pragma unroll
        for (int k = N / 2; k < N; ++k) v[k] = ~v[k];
        merge_regs<N>(v, s);
    }
}

// inclusive sum over the wavefront's lanes
__device__ inline uint32_t inclusive_sum(uint32_t v) {
    v += dpp<0x111>(0u, v);  // row_shr:1, 2, 4, 8
    v += dpp<0x112>(0u, v);
    v += dpp<0x114>(0u, v);
    v += dpp<0x118>(0u, v);
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xa, 0xf, false));  // row_bcast:15
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x143, 0xc, 0xf, false));  // row_bcast:31
    return v;
}

// the value of the lane before (lane 0: first)
__device__ inline uint32_t from_lane_before(uint32_t v, uint32_t first) {
    return uint32_t(__builtin_amdgcn_update_dpp(int(first), int(v), 0x138, 0xf, 0xf, false));  // wave_shr:1
}

// sum over every group of 8 lanes, in all of its lanes
__device__ inline double sum8(double v) {
    auto part = [](double x, auto mv) {
        const uint64_t b = uint64_t(__double_as_longlong(x));
        return __longlong_as_double((long long)mv(b));
    };
    v += part(v, [](uint64_t b) { return move<kXor1>(b); });
    v += part(v, [](uint64_t b) { return move<kXor2>(b); });
    v += part(v, [](uint64_t b) { return move<kFlip8>(b); });
    return v;
}

}  // namespace wsort
}  // namespace spsyrk
