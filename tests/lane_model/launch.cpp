// Calls the library's launch_walk (address given) with a walk of one row and no buffers.
#include "../../paper_2409_03095_amd/csrc/walk_args.hpp"

extern "C" int try_launch(void *launch_walk, int f32, int slots, int lanes, int lane_chains, int topk) {
    mcmi::WalkArgs a;
    memset(&a, 0, sizeof(a));
    static uint32_t rec[8];
    a.rec = a.rec32 = rec;
    a.hash_slots = slots;
    a.row_lanes = lanes;
    a.lane_chains = lane_chains;
    a.topk = topk;
    return ((int (*)(const mcmi::WalkArgs &, bool, int, int, void *))launch_walk)(a, f32 != 0, 1, 4, nullptr);
}
