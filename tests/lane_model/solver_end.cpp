// A solve that breaks down in k_step (t = 0): workgroup 0 ends it between the moments at
// which two waves of workgroup 1 start. A workgroup is four threads here, lane 0 of each of
// its waves; LDS keeps what the workgroup before left in it. Whichever wave of workgroup 1
// comes first, x stays as it is.
#include <math.h>
#include <stdio.h>
#include <ucontext.h>

#include <string>
#include <vector>

#include "../../paper_2409_03095_amd/csrc/common.hpp"

// the kernels twice, each workgroup with LDS of its own
namespace g0 {
using namespace mcmi;
#include SOLVER_KERNELS
}
namespace g1 {
using namespace mcmi;
#include SOLVER_KERNELS
}

template <typename T>
T __shfl_xor(T, int, int) {
    return T(0);  // the other lanes hold nothing
}
void other_lanes() {}

dim3 threadIdx, blockIdx, blockDim = {256, 1, 1}, gridDim = {2, 1, 1};

namespace {

constexpr int kWaves = 4, kN = 512;
ucontext_t back, ctx[2][kWaves];
std::vector<char> stacks(2 * kWaves * 65536);
int group, wave;
enum { kRunning, kWaiting, kEnded };
int state[2][kWaves];

double x[kN], r[kN], v[kN], t[kN], sv[kN], phat[kN], shat[kN], rhat[kN], part[g0::kParts * g0::kDotBlocks];
g0::KState st;
int32_t host_status;

void body() {
    if (group == 0)
        g0::k_step(kN, 1, phat, shat, sv, t, rhat, x, r, {&st, part, &host_status, 1e-10});
    else
        g1::k_step(kN, 1, phat, shat, sv, t, rhat, x, r, {(g1::KState *)&st, part, &host_status, 1e-10});
    state[group][wave] = kEnded;
    swapcontext(&ctx[group][wave], &back);
}

// runs one wave up to its next barrier or its end
void turn(int g, int w) {
    if (state[g][w] != kRunning) return;
    group = g;
    wave = w;
    blockIdx.x = (unsigned)g;
    threadIdx.x = 64u * (unsigned)w;
    swapcontext(&back, &ctx[g][w]);
}

void start(int g) {
    for (int w = 0; w < kWaves; ++w) {
        getcontext(&ctx[g][w]);
        ctx[g][w].uc_stack.ss_sp = &stacks[(size_t)(g * kWaves + w) * 65536];
        ctx[g][w].uc_stack.ss_size = 65536;
        ctx[g][w].uc_link = nullptr;
        makecontext(&ctx[g][w], body, 0);
        state[g][w] = kRunning;
    }
}

// waves that have ended do not hold a barrier up
void finish(int g) {
    for (;;) {
        int live = 0;
        for (int w = 0; w < kWaves; ++w) turn(g, w);
        for (int w = 0; w < kWaves; ++w) {
            if (state[g][w] == kWaiting) state[g][w] = kRunning;
            live += state[g][w] == kRunning;
        }
        if (!live) return;
    }
}

}  // namespace

void __syncthreads() {
    state[group][wave] = kWaiting;
    swapcontext(&ctx[group][wave], &back);
}

int main() {
    int bad = 0;
    for (int first = 0; first < kWaves; ++first) {
        for (int i = 0; i < kN; ++i) {
            x[i] = 1.0;
            t[i] = 0.0;
            r[i] = v[i] = sv[i] = phat[i] = shat[i] = rhat[i] = 1.0 + i;
        }
        st = g0::KState{};
        st.status = g0::kRun;
        st.alpha = 0.5;
        st.bnrm = 1.0;
        // LDS as another kernel's sums left it
        for (double &p : part) p = 0.25;
        start(1);
        finish(1);
        // now the breakdown
        for (double &p : part) p = 0.0;
        for (int i = 0; i < kN; ++i) x[i] = 1.0;
        start(1);
        turn(1, first);
        start(0);
        finish(0);
        finish(1);
        if (st.status != g0::kBreakdown) ++bad;
        for (int i = 0; i < kN; ++i) bad += x[i] != 1.0;
    }
    printf("%d values changed\n", bad);
    return bad != 0;
}
