// Where the server's results go (dare_server.hip): which results a tick's kernels may write to their
// destinations themselves, and which ticks in flight its copies have to wait for.  Plain C++: the
// scheduler and the host tests use it.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace dare {

struct Destination {
    uintptr_t lo = 0, hi = 0;              // the result's bytes
    bool device = false;                   // device memory
    bool direct = false;                   // kernels may write it: the server's GPU, one allocation, aligned
};

// A tick's device results that overlap another's, of the same tick or of one in flight, lose `direct`:
// they are copied from their slots when the kernels are done, in request order within the tick, and
// after the ticks in flight that they overlap (`wait[s]`).  So the last request's values stand,
// however requests fall into ticks.  `flight[s]`: the device destinations of tick s.
inline void settle_destinations(std::vector<Destination>& tick, const std::vector<std::vector<Destination>>& flight,
                                std::vector<char>& wait) {
    struct Range {
        uintptr_t lo, hi;
        int slot;                          // -1: of the new tick
        size_t k;
    };
    std::vector<Range> all;
    for (size_t k = 0; k < tick.size(); ++k)
        if (tick[k].device && tick[k].hi > tick[k].lo) all.push_back({tick[k].lo, tick[k].hi, -1, k});
    for (size_t s = 0; s < flight.size(); ++s)
        for (const Destination& d : flight[s])
            if (d.hi > d.lo) all.push_back({d.lo, d.hi, (int)s, 0});
    std::sort(all.begin(), all.end(), [](const Range& a, const Range& b) { return a.lo < b.lo; });
    wait.assign(flight.size(), 0);
    // in order of their starts, a range overlaps an earlier one where that one reaches past its start;
    // of the tick's own ranges the one that reaches furthest is kept: any other that reaches so far
    // overlaps that one too, and so has lost `direct` already
    const Range* own = nullptr;
    std::vector<uintptr_t> top(flight.size(), 0);
    for (const Range& r : all) {
        const bool meets = own && r.lo < own->hi;
        if (meets) tick[own->k].direct = false;
        if (r.slot < 0) {
            if (meets) tick[r.k].direct = false;
            for (size_t s = 0; s < top.size(); ++s)
                if (r.lo < top[s]) {
                    tick[r.k].direct = false;
                    wait[s] = 1;
                }
            if (!own || r.hi > own->hi) own = &r;
        } else {
            if (meets) wait[r.slot] = 1;
            top[r.slot] = std::max(top[r.slot], r.hi);
        }
    }
}

}  // namespace dare
