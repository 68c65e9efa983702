// Host helpers with no device code and no HIP types, so that they compile and
// are tested on their own.
#pragma once

#include <cstddef>
#include <cstdint>

namespace cube {

// Bits of a cell index: the smallest b with 2^b >= cells.
inline int key_bits(int64_t cells) {
    int b = 0;
    while (((int64_t)1 << b) < cells) ++b;
    return b;
}

}  // namespace cube
