// Host helpers with no device code and no HIP types, so that they compile and
// are tested on their own.
#pragma once

#include <cstddef>
#include <cstdint>
#include <utility>

namespace cube {

// Bits of a cell index: the smallest b with 2^b >= cells.
inline int key_bits(int64_t cells) {
    int b = 0;
    while (((int64_t)1 << b) < cells) ++b;
    return b;
}

// Copies that follow each other on both sides go as one (a view's planes are
// mostly rows of one array, and so are the context's): a copy costs 2 to 4 us
// whatever its size, and a state has seven arrays.  Only where
// one(dst, src, bytes) says that the run is one allocation on either side:
// separate ones can be neighbours by chance.  copy(dst, src, bytes) returns an
// error, of which the type's zero is none.
template <class Copy, class One>
struct CopyRuns {
    using Error = decltype(std::declval<Copy&>()(std::declval<void*>(), std::declval<const void*>(), size_t()));
    Copy copy;
    One one;
    char* dst = nullptr;
    const char* src = nullptr;
    size_t bytes = 0;

    CopyRuns(Copy c, One o) : copy(c), one(o) {}

    Error flush() {
        const size_t n = bytes;
        bytes = 0;
        return n ? copy(dst, src, n) : Error{};
    }
    Error add(void* d, const void* s, size_t n) {
        if (bytes && d == dst + bytes && s == src + bytes && one(dst, src, bytes + n)) {
            bytes += n;
            return Error{};
        }
        const Error e = flush();
        dst = static_cast<char*>(d);
        src = static_cast<const char*>(s);
        bytes = n;
        return e;
    }
};

}  // namespace cube
