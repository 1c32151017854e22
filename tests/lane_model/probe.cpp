// A wavefront of 64 lanes that adds to one open-addressing table through Probe::add, as
// the walk kernels do: the home bucket of a key is read one step ahead, lanes take turns at
// every compare-and-swap. Keys that add() gives up on go to a spill set. Prints, per kind
// of table: tables filled, keys held by both table and spill set, keys twice in the
// table, sums that are not those of the additions, additions spilled.
#include <stdio.h>
#include <ucontext.h>

#include <map>
#include <random>
#include <set>
#include <vector>

#include "../../paper_2409_03095_amd/csrc/walk_common.hpp"

using namespace mcmi::walkdev;

namespace {

constexpr int kLanes = 64;
constexpr size_t kStack = 32768;
ucontext_t back, lane_ctx[kLanes];
std::vector<char> stacks(kLanes * kStack);
int now_on;
bool running[kLanes];

int32_t keys[1024];
double vals[1024];
std::map<int32_t, double> added, spilled;
std::vector<int32_t> universe;
uint32_t slots;
int steps;
std::mt19937 rng;
bool (*add_one)(uint32_t b, int32_t k[4], int32_t key);
uint32_t (*home_of)(int32_t key);

void lane() {
    int32_t key = universe[rng() % universe.size()], k[4];
    uint32_t b = home_of(key);
    read_bucket_wave(keys, b, k);
    other_lanes();
    for (int s = 0; s < steps; ++s) {
        added[key] += 1.0;
        if (!add_one(b, k, key)) spilled[key] += 1.0;
        key = universe[rng() % universe.size()];
        b = home_of(key);
        read_bucket_wave(keys, b, k);
        other_lanes();
    }
    running[now_on] = false;
    swapcontext(&lane_ctx[now_on], &back);
}

void wave() {
    for (int l = 0; l < kLanes; ++l) {
        getcontext(&lane_ctx[l]);
        lane_ctx[l].uc_stack.ss_sp = &stacks[l * kStack];
        lane_ctx[l].uc_stack.ss_size = kStack;
        lane_ctx[l].uc_link = nullptr;
        makecontext(&lane_ctx[l], lane, 0);
        running[l] = true;
    }
    for (bool any = true; any;) {
        any = false;
        for (int l = 0; l < kLanes; ++l)
            if (running[l]) {
                any = true;
                now_on = l;
                swapcontext(&back, &lane_ctx[l]);
            }
    }
}

template <bool kPow2, bool kScatter, bool kPeel>
void kind(uint32_t n, int tables) {
    using Tab = Probe<kPow2, kScatter, kPeel>;
    slots = n;
    add_one = [](uint32_t b, int32_t k[4], int32_t key) { return Tab::add(keys, vals, slots, b, k, key, 1.0); };
    home_of = [](int32_t key) { return Tab::home(key, slots, 32 - __builtin_ctz(slots)); };
    int both = 0, twice = 0, wrong = 0;
    double spills = 0;
    for (int t = 0; t < tables; ++t) {
        for (uint32_t s = 0; s < slots; ++s) {
            keys[s] = kEmpty;
            vals[s] = 0.0;
        }
        added.clear();
        spilled.clear();
        // 9/10 to 12/10 of the slots: tables that are nearly full or overflow
        universe.resize(slots * (9 + t % 4) / 10);
        for (int32_t &u : universe) u = (int32_t)(rng() & 0x7fffffffu);
        steps = (int)slots / 16;
        wave();
        std::set<int32_t> seen;
        std::map<int32_t, double> sums = spilled;
        for (uint32_t s = 0; s < slots; ++s)
            if (keys[s] != kEmpty) {
                twice += !seen.insert(keys[s]).second;
                both += spilled.count(keys[s]) != 0;
                sums[keys[s]] += vals[s];
            }
        wrong += sums != added;
        for (auto &e : spilled) spills += e.second;
    }
    printf("%d%d%d %u: %d tables, %d both, %d twice, %d wrong, %.0f spilled\n", kPow2, kScatter, kPeel, n, tables, both,
           twice, wrong, spills);
}

}  // namespace

void other_lanes() { swapcontext(&lane_ctx[now_on], &back); }

int main() {
    rng.seed(1);
    // the instances of the walk kernels: tables of any size, scattered, plain
    for (uint32_t n : {128u, 256u, 512u, 848u}) kind<false, false, true>(n, (int)(100000u / n));
    for (uint32_t n : {64u, 128u, 256u, 1024u}) kind<true, true, false>(n, (int)(100000u / n));
    for (uint32_t n : {64u, 128u, 256u, 1024u}) kind<true, false, false>(n, (int)(100000u / n));
    return 0;
}
