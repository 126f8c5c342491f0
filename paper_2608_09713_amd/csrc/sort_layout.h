// Host-side choice of the column sort's path: passes over every bit, or passes
// over the high bits and a sort of the low ones inside groups of equal high
// bits.  Plain C++ (no HIP), so that the choice can be checked on any host.
#pragma once

#include <cstdint>

namespace spsyrk {

constexpr int kLBits = 12;      // low bits sorted inside groups, at most
constexpr int kLCap = 4096;     // records of a group sorted in LDS
constexpr int kSortDigit = 8;   // bits per pass, at most
constexpr int64_t kFewRecords = int64_t(1) << 16;

// Low bits sorted inside groups for n entries with nbits-bit columns (0:
// passes over every bit).  The high bits make groups of about 2048 records on
// average.  Used for wide columns over many entries, and for few entries,
// where it takes fewer launches and the passes are all latency (groups of
// about 512 records there, so that more workgroups share them): up to 2^16
// entries with columns of at most 20 bits, whose high bits take one pass of at
// most 256 groups (calls on 32,768 entries of 14 bits, f64: 193 us by full
// passes, 170 so; on 65,536 of 20 bits 222 and 167).  With wider columns the
// groups outnumber the entries and more passes follow (1000 entries of 31
// bits: 186 us by full passes, 301 in groups).  forced: 1 wherever it applies,
// 0 never, -1 by these rules.
constexpr int local_sort_bits(int64_t n, int nbits, int forced) {
    const bool force = forced == 1, few = n <= kFewRecords;
    if (forced == 0) return 0;
    if (!force && !(few ? nbits <= kLBits + kSortDigit : nbits >= 22 && n >= (int64_t(1) << 20))) return 0;
    int h = nbits - kLBits, hg = 0;
    for (uint64_t g = uint64_t(n / (few && !force ? 512 : 2048)); g; g >>= 1) ++hg;
    if (hg > h) h = hg;
    if (h < 1) h = 1;
    return nbits > h ? nbits - h : 0;
}

// Whether few entries' groups are looked at first (group_counts: the entries
// of each, as the validation counts them): a group past what LDS holds is
// sorted by one workgroup over memory, 256 records at a time, and then the
// passes over every bit are faster (60,000 entries in 4096 columns of 2^20: 805
// us so, 243 by full passes).
constexpr bool local_sort_checked(int64_t n, int forced) { return forced < 0 && n <= kFewRecords; }
inline bool local_groups_fit(const uint32_t* group_counts, int groups) {
    for (int g = 0; g < groups; ++g)
        if (group_counts[g] > uint32_t(kLCap)) return false;
    return true;
}

}  // namespace spsyrk
