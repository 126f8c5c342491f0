// Host check of the column sort's choice: few entries are sorted in groups only
// where one pass makes at most 256 of them; the groups' bits and the passes'
// make up the columns' bits; a group past what LDS holds is refused; many
// entries keep the rule of wide columns.
#include <cstdio>

#include "sort_layout.h"

int main() {
    using namespace spsyrk;
    long checked = 0;
    for (int nbits = 0; nbits <= 31; ++nbits)
        for (int64_t n = 1; n < (int64_t(1) << 31); n = n * 3 / 2 + 1)
            for (int64_t d = -1; d <= 1; ++d) {
                const int64_t e = n + d;
                if (e < 1) continue;
                ++checked;
                const int L = local_sort_bits(e, nbits, -1), h = nbits - L;
                if (L < 0 || L > kLBits || (L && h < 1) || local_sort_bits(e, nbits, 0) != 0) return 1;
                if (e <= kFewRecords && L && h > kSortDigit) {
                    std::printf("%lld entries of %d bits: 2^%d groups\n", (long long)e, nbits, h);
                    return 1;
                }
                if (e > kFewRecords && (L > 0) != (nbits >= 22 && e >= (1 << 20) && L > 0)) return 1;
                if (e >= (1 << 20) && nbits >= 22 && h > 8 && (int64_t(1) << h) > 4 * e) return 1;
            }
    uint32_t counts[256] = {};
    counts[3] = kLCap;
    if (!local_groups_fit(counts, 256)) return 1;
    counts[200] = kLCap + 1;
    if (local_groups_fit(counts, 256)) return 1;
    if (!local_sort_checked(kFewRecords, -1) || local_sort_checked(kFewRecords + 1, -1) || local_sort_checked(10, 1))
        return 1;
    std::printf("ok %ld\n", checked);
    return 0;
}
