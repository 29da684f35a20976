// Whether rows of two tensors share memory: what a call that reads one while it writes the other has to know.  (Host only)
#pragma once
#include <stdint.h>

namespace agzo {

// n rows of `bytes` bytes, `ld` bytes from one to the next (ld >= bytes)
struct Rows { uintptr_t at; int64_t ld, n, bytes; };

// Rows of one leading dimension (views into one wider tensor): exactly.  Of two: true where the ranges from first to last byte meet, so that a
// false answer is always right
inline bool rows_overlap(const Rows& a, const Rows& b) {
    if (a.n <= 0 || b.n <= 0 || a.bytes <= 0 || b.bytes <= 0) return false;
    const uintptr_t a_end = a.at + (uintptr_t)((a.n - 1) * a.ld + a.bytes), b_end = b.at + (uintptr_t)((b.n - 1) * b.ld + b.bytes);
    if (a_end <= b.at || b_end <= a.at) return false;
    if (a.ld != b.ld) return true;
    // b's row j starts in a's row j + q, behind rem bytes, and may reach into the one that follows
    const int64_t delta = (int64_t)(b.at - a.at), ld = a.ld;
    const int64_t q = delta >= 0 ? delta / ld : -((-delta + ld - 1) / ld), rem = delta - q * ld;
    auto meet = [&](int64_t shift) {      // some j of b with row j + shift of a
        const int64_t from = shift < 0 ? -shift : 0, to = a.n - shift < b.n ? a.n - shift : b.n;
        return from < to;
    };
    return (rem < a.bytes && meet(q)) || (rem + b.bytes > ld && meet(q + 1));
}

}  // namespace agzo
