// How large a context's workspace becomes when a call needs more than it has.  (Host only)
#pragma once
#include <stddef.h>

#include <algorithm>

namespace agzo {

constexpr size_t kMapBytes = (size_t)2 << 20, kGrowBytes = (size_t)32 << 20;

// A context that needs more once will need more again (the layers of a model, one after the other): half as much again, at first more, up to
// the 2 MiB that device memory is mapped by (a page of it is some 10 us).  (A growth is up to 0.5 ms of a first pass: the dense estimator's over
// seven 0.6B-sized layers on 1131 tokens takes 0.97 ms growing by what a call needs, 1.24 by half, 0.77 so.)
// have: what it holds now, given back before; need: what the call cannot do without; wish: what the calls behind it will ask for.
// allocate(bytes) -> allocated.  Where that much is not left, what the call needs.  Returns the bytes it got, 0: not even those
template <typename F>
size_t grow(size_t have, size_t need, size_t wish, F allocate) {
    size_t bytes = std::max(need, wish);
    if (have) bytes = (std::max({bytes, have + have / 2, std::min(16 * have, have + kGrowBytes)}) + kMapBytes - 1) / kMapBytes * kMapBytes;
    if (allocate(bytes)) return bytes;
    return bytes > need && allocate(need) ? need : 0;
}

}  // namespace agzo
