// Host test of dare::settle_destinations against all pairs of ranges.
#include <cstdio>
#include <random>

#include "dare_destinations.h"

using namespace dare;

static bool meet(const Destination& a, const Destination& b) {
    return a.device && b.device && a.lo < b.hi && b.lo < a.hi && a.hi > a.lo && b.hi > b.lo;
}

int main() {
    std::mt19937 g(9);
    for (int trial = 0; trial < 60000; ++trial) {
        const int space = 1 + g() % (trial % 2 ? 60 : 2000), longest = 1 + g() % 40;
        auto make = [&](int n, bool flying) {
            std::vector<Destination> v(n);
            for (Destination& d : v) {
                d.lo = 1000 + g() % space;
                d.hi = d.lo + g() % (longest + 1);
                d.device = flying || g() % 5 != 0;
                d.direct = d.device && g() % 4 != 0;
            }
            return v;
        };
        std::vector<Destination> tick = make(g() % 9, false);
        std::vector<std::vector<Destination>> flight(g() % 4);
        for (auto& f : flight) f = make(g() % 6, true);
        std::vector<Destination> ref = tick;
        std::vector<char> wait, ref_wait(flight.size(), 0);
        for (size_t k = 0; k < ref.size(); ++k) {
            for (size_t m = 0; m < ref.size(); ++m)
                if (m != k && meet(tick[k], tick[m])) ref[k].direct = false;
            for (size_t s = 0; s < flight.size(); ++s)
                for (const Destination& d : flight[s])
                    if (meet(tick[k], d)) ref[k].direct = false, ref_wait[s] = 1;
        }
        settle_destinations(tick, flight, wait);
        bool same = wait == ref_wait;
        for (size_t k = 0; k < ref.size(); ++k) same = same && tick[k].direct == ref[k].direct;
        if (!same) {
            std::printf("trial %d differs\n", trial);
            return 1;
        }
    }
    std::printf("destinations host test ok\n");
    return 0;
}
