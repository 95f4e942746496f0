// How a block of the bucket sort cuts its range of sorted positions: plain
// functions that the device code and a host program share.
#pragma once

#include <cstdint>

namespace bhx {

// The range [a, b) holds whole buckets (keys of equal top bits, key >> shift) in
// ascending order, of which only the last may end far from the block's tile. The
// end of the piece that starts at a: all of it where it fits `cap` keys, else the
// buckets before the last one, and then the last one alone. A piece beyond `cap`
// is sorted through global memory in passes whose intermediate orders other
// blocks can see; as one bucket it shares its top bits, so the top bits of every
// position stay what they were, and a block that looks for bucket boundaries at
// any time finds the same ones.
template <typename Keys>
__host__ __device__ inline int64_t piece_end(const Keys &keys, int64_t a, int64_t b, int64_t cap,
                                             int shift)
{
    if (b - a <= cap) return b;
    const uint64_t last = keys[b - 1] >> shift;
    int64_t lo = a, hi = b - 1;  // the last bucket's first position
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if ((keys[mid] >> shift) != last)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo > a ? lo : b;
}

}  // namespace bhx
