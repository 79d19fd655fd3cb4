// The weights by which big_band_kernel shares a large node's bit positions among
// its bands.
#pragma once

#include <stdint.h>

namespace qd {

// A position that c of a node's m rows have set weighs (c >> shift) + 1.  The
// weights of all 4,096 positions add to at most 4096 * ((m >> shift) + 1), which
// this shift keeps within 2^31 + 2^12: the kernel adds them in 32 bits, and a sum
// that wrapped would give bands that are no runs of the popularity order, and
// with them a wrong cut.  8 up to 2^27 rows, one more for every doubling.
constexpr uint32_t band_weight_shift(uint32_t m) {
    uint32_t length = 0;  // bits of m
    for (uint32_t x = m; x; x >>= 1) length++;
    return length > 27 ? length - 19 : 8;
}

}  // namespace qd
