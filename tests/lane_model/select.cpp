// select_top (walk.hip) run by the 64 lanes of a modelled wavefront on random survivors, M
// filter and plain, with equal values and values that are zero (M_rc may underflow): the
// kept set is the one a sort gives, and nothing past the survivors is written.
#include <stdio.h>
#include <ucontext.h>

#include <numeric>
#include <random>
#include <vector>

#include "../../paper_2409_03095_amd/csrc/walk_common.hpp"

namespace mcmi {
using namespace walkdev;
#include SELECT_TOP
}  // namespace mcmi

namespace {

using namespace mcmi;

constexpr int kLanes = 64;
ucontext_t back, ctx[kLanes];
std::vector<char> stacks(kLanes * 65536);
int on;
bool done[kLanes];
uint64_t votes, result;
int voted;

WalkArgs args;
std::vector<int32_t> keys;
std::vector<double> vals;
int K;
int32_t own;
double chains;

void body() {
    select_top<false>(args, keys.data(), vals.data(), K, own, chains);
    done[on] = true;
    swapcontext(&ctx[on], &back);
}

void wave() {
    for (int l = 0; l < kLanes; ++l) {
        getcontext(&ctx[l]);
        ctx[l].uc_stack.ss_sp = &stacks[(size_t)l * 65536];
        ctx[l].uc_stack.ss_size = 65536;
        ctx[l].uc_link = nullptr;
        makecontext(&ctx[l], body, 0);
        done[l] = false;
    }
    // every lane to its next vote (or its end), then the votes' result to all
    while (!done[kLanes - 1]) {
        votes = 0;
        for (int l = 0; l < kLanes; ++l) {
            on = l;
            swapcontext(&back, &ctx[l]);
        }
        result = votes;
    }
}

}  // namespace

int __lane_id() { return on; }
uint64_t __ballot(int p) {
    if (p) votes |= 1ull << on;
    swapcontext(&ctx[on], &back);
    return result;
}
uint32_t mask_bits_below(uint64_t m) { return (uint32_t)__popcll(m & ((1ull << on) - 1)); }
void other_lanes() {}

int main() {
    std::mt19937 rng(3);
    int bad = 0, runs = 0;
    std::vector<double> diag(1 << 14);
    for (int t = 0; t < 600; ++t) {
        K = 2 + (int)(rng() % (t % 2 ? 511 : 100));
        args.topk = 1 + (int)(rng() % (K - 1));
        args.filter_m = t % 3 != 0;
        args.diag = diag.data();
        for (double &d : diag) d = t % 5 == 0 ? 1e308 : 0.5 + rng() % 3;
        chains = 4.0;
        keys.assign(K + 1024, -7);
        vals.assign(K + 1024, -7.0);
        std::vector<int32_t> pool(1 << 14);
        std::iota(pool.begin(), pool.end(), 0);
        std::shuffle(pool.begin(), pool.end(), rng);
        for (int i = 0; i < K; ++i) {
            keys[i] = pool[i];
            // few different values, some of which underflow when divided by 1e308
            vals[i] = (rng() & 1 ? 1.0 : -1.0) * ldexp(1.0, -(int)(rng() % (t % 4 ? 6 : 80)));
        }
        own = keys[rng() % K];
        std::vector<int> order(K);
        std::iota(order.begin(), order.end(), 0);
        const std::vector<int32_t> k0 = keys;
        const std::vector<double> v0 = vals;
        auto size = [&](int i) { return args.filter_m ? fabs(v0[i] / chains / diag[k0[i]]) : fabs(v0[i] / chains); };
        std::sort(order.begin(), order.end(), [&](int x, int y) {
            if ((k0[x] == own) != (k0[y] == own)) return k0[x] == own;
            if (size(x) != size(y)) return size(x) > size(y);
            return k0[x] < k0[y];
        });
        wave();
        std::vector<std::pair<int32_t, double>> got, want;
        for (int i = 0; i < args.topk; ++i) {
            got.push_back({keys[i], vals[i]});
            want.push_back({k0[order[i]], v0[order[i]] / chains});
        }
        std::sort(got.begin(), got.end());
        std::sort(want.begin(), want.end());
        bool ok = got == want;
        for (int i = K; i < K + 1024; ++i) ok = ok && keys[i] == -7 && vals[i] == -7.0;
        bad += !ok;
        ++runs;
    }
    printf("%d of %d selections wrong\n", bad, runs);
    return bad != 0;
}
