// The buckets that a search visits: prints, per kind and size of table, the least number of
// different ones among the first kMaxLdsProbe / 4 over many keys.
#include <stdio.h>

#include <set>

#include "../../paper_2409_03095_amd/csrc/walk_common.hpp"

using namespace mcmi::walkdev;
void other_lanes() {}

template <typename Tab>
void least(const char *name, uint32_t slots) {
    size_t fewest = 99;
    uint32_t key = 1;
    for (int t = 0; t < 20000; ++t) {
        key = (key * 1664525u + 1013904223u) & 0x7fffffffu;
        const int32_t k = t < 5000 ? t : (int32_t)key;
        uint32_t b = Tab::home(k, slots, 32 - __builtin_ctz(slots));
        std::set<uint32_t> seen;
        for (int p = 0; p < kMaxLdsProbe / 4; ++p) {
            if (b % 4 || b >= slots) fewest = 0;
            seen.insert(b);
            b = Tab::next(b, k, slots);
        }
        fewest = std::min(fewest, seen.size());
    }
    printf("%s %u: %zu different buckets\n", name, slots, fewest);
}

int main() {
    for (uint32_t n : {64u, 128u, 256u, 512u, 1024u, 8192u}) {
        least<Probe<true, true, false>>("scattered", n);
        least<Probe<true, false, false>>("plain", n);
    }
    for (uint32_t n : {64u, 100u, 128u, 512u, 848u}) least<Probe<false, false, true>>("any size", n);
    return 0;
}
