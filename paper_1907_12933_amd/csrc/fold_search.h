// The job search of the folded enumeration, apart from how a wave compares.
#pragma once

namespace ibmc {

// The last of n >= 1 ordered entries that starts at or before a value, the
// first one doing so.  A round compares up to 64 entries at equal steps and goes
// on with the entries of the last step that does: one round to 64 entries, two
// to 4,096, three beyond.  count(first, step, n): how many of the entries first,
// first + step, ... below first + n start at or before the value.
template <class F>
constexpr int fold_search(int n, F count) {
    int first = 0;
    while (n > 1) {
        const int step = (n + 63) / 64, at = (count(first, step, n) - 1) * step;
        first += at;
        n = n - at < step ? n - at : step;
    }
    return first;
}

}  // namespace ibmc
