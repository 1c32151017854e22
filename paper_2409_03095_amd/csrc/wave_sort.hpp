// Sorting up to 256 32-bit words in the registers of one wavefront (internal).
//
// A bitonic network over 64 W words, lane l holding words l W .. l W + W - 1. Exchanges
// inside a lane are a min and a max; exchanges between lanes d = 1, 2, 4, 8 apart
// read the partner by DPP (no LDS, no address), 16 and 32 apart by the row swaps
// of gfx950. A network in LDS pays a round trip per one or two passes and
// two 64-bit LDS accesses per word and pass.
#pragma once
#include "common.hpp"

namespace mcmi {
namespace wavesort {

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, kCtrl, 0xf, 0xf, false);
}

// the word of lane (this lane ^ D), D in {1, 2, 4, 8}
template <int D>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
    if constexpr (D == 1) return dpp<0xB1>(v);   // quad_perm 1 0 3 2
    if constexpr (D == 2) return dpp<0x4E>(v);   // quad_perm 2 3 0 1
    if constexpr (D == 4) return dpp<0x1B>(dpp<0x141>(v));  // half-row mirror (^ 7), then quad_perm 3 2 1 0 (^ 3)
    return dpp<0x128>(v);                        // D = 8: rotate the row of 16 by 8
}

// smaller and larger word of the lanes l and l ^ D, the same on both
template <int D>
__device__ __forceinline__ void pair_minmax(uint32_t v, uint32_t &mn, uint32_t &mx) {
    uint32_t a = v, b;
    if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = r[0];
        b = r[1];
    } else if constexpr (D == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = r[0];
        b = r[1];
    } else {
        b = xor_lane<D>(v);
    }
    mn = a < b ? a : b;
    mx = a < b ? b : a;
}

__device__ __forceinline__ void exch32(uint32_t &a, uint32_t &b) {
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    a = lo;
    b = hi;
}

// The passes at distances J, J / 2, .. 1 of a merge whose runs are all ascending.
template <int W, int J>
__device__ __forceinline__ void merge_passes(uint32_t (&e)[W], int lane) {
    if constexpr (J >= W) {
        constexpr int D = J / W;
        const bool low = (lane & D) == 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            uint32_t mn, mx;
            pair_minmax<D>(e[q], mn, mx);
            e[q] = low ? mn : mx;
        }
    } else {
#pragma unroll
        for (int q = 0; q < W; ++q)
            if ((q & J) == 0) exch32(e[q], e[q | J]);
    }
    if constexpr (J > 1) merge_passes<W, J / 2>(e, lane);
}

// Merges of width K, 2 K, .. 64 W. Descending runs are sorted as ascending runs of the
// complemented words.
template <int W, int K>
__device__ __forceinline__ void merges(uint32_t (&e)[W], int lane) {
    if constexpr (K < W) {
        // runs inside a lane (W = 4, K = 2): the second pair descends
        exch32(e[0], e[1]);
        exch32(e[3], e[2]);
    } else {
        const uint32_t flip = K < 64 * W && (lane & (K / W)) != 0 ? ~0u : 0u;
#pragma unroll
        for (int q = 0; q < W; ++q) e[q] ^= flip;
        merge_passes<W, K / 2>(e, lane);
#pragma unroll
        for (int q = 0; q < W; ++q) e[q] ^= flip;
    }
    if constexpr (K < 64 * W) merges<W, 2 * K>(e, lane);
}

// Ascending sort of the wave's 64 W words (W = 1, 2 or 4).
template <int W>
__device__ __forceinline__ void sort_words(uint32_t (&e)[W], int lane) {
    static_assert(W == 1 || W == 2 || W == 4, "words per lane");
    merges<W, 2>(e, lane);
}

// Smallest / largest word of the wave (DPP row scans, then the last lane of each row
// on to the next).
template <bool kMax>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
    constexpr int kId = kMax ? 0 : -1;
    auto op = [](uint32_t a, uint32_t b) { return kMax ? (a > b ? a : b) : (a < b ? a : b); };
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(kId, (int)v, 0x111, 0xf, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(kId, (int)v, 0x112, 0xf, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(kId, (int)v, 0x114, 0xf, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(kId, (int)v, 0x118, 0xf, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(kId, (int)v, 0x142, 0xa, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(kId, (int)v, 0x143, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

}  // namespace wavesort
}  // namespace mcmi
