// Monte Carlo walks, per-row accumulation and finalize (gfx950).
//
// Section III-A, eq. (2): row r of (I - C)^-1 is estimated by the mean over N_r
// chains started at r of sum_j W_j e_{s_j}, with W_0 = 1 and
// W_j = W_{j-1} * c_{s_{j-1} s_j} / p_{s_{j-1} s_j} = W_{j-1} * sign * Shat.
// Section IV-A, phase 4 scales column c by 1 / d_c, and the filter keeps the
// diagonal and every entry with |N_rc| >= eps.
//
// Design (one wavefront owns one row at a time, or 64 / G rows of G lanes each when
// rows have few chains; persistent grid):
//  * rows come from eight work queues, one per XCD (workgroups are dispatched
//    round-robin over the XCDs, so blockIdx % 8 picks the XCD), each a contiguous
//    slice of the rows so that neighbouring rows share their L2; a wave whose
//    queue is empty steals from the next queue;
//  * each lane runs one chain at a time and starts the row's next unstarted chain
//    as soon as its chain stops, so short and long chains do not wait for each
//    other;
//  * a step draws one Philox word and reads the 64-byte alias bucket it names,
//    which also carries the next state's header: one random line per step;
//  * contributions go to an open-addressing hash per row in LDS (key = column,
//    value = float64 sum, LDS float64 atomics; the wave's table split among its
//    rows); a full neighbourhood spills to a per-row share of the wave's HBM hash;
//  * the rows of a wave start together and are finalized one after the other;
//  * at the end of the row the wave filters the slots with a ballot, compacts the
//    survivors in place, scales them by 1 / d_c, sorts them by column with a
//    bitonic network (in registers up to 256 of them, else in LDS) and appends them
//    to an output pool.
#include "common.hpp"
#include "walk_args.hpp"
#include "walk_common.hpp"
#include "wave_sort.hpp"

namespace mcmi {

namespace {

using namespace walkdev;

// Wave-uniform task fetch from the eight per-XCD queues.
// Rows are taken from the XCD queues kTaskChunk at a time (one atomic per chunk);
// [lo, hi) is the wave's current chunk. The chunk sets the locality of an XCD's
// rows in flight (about chunk x its wavefronts consecutive rows of the schedule)
// against the atomics on the queue counters: on the 160^3 27-point walk chunks of
// 2, 3, 4, 8 and 16 rows took 63.0, 61.9, 61.7, 62.2 and 71.5 ms. Binary64 walks that run at
// the DRAM's rate (lds_sort) take kTaskChunkDram: chunks of 2, 3 and 4 rows took 70.9, 69.2 and
// 69.7 ms there (160^3 27-point), 35.9, 35.3 and 35.4 (128^3), 60.8, 59.9 and 62.0 (2000^2 grid).
constexpr int kTaskChunk = 4, kTaskChunkDram = 3;

// Compare-exchange of a bitonic pass: a keeps the smaller word of an ascending
// pair (up), the larger of a descending one.
__device__ __forceinline__ void exch(uint64_t &a, uint64_t &b, bool up) {
    const uint64_t lo = a < b ? a : b, hi = a < b ? b : a;
    a = up ? lo : hi;
    b = up ? hi : lo;
}

// lane 0's value as a wave-uniform one
__device__ __forceinline__ int64_t first_lane(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <bool kF32>
__device__ __forceinline__ int64_t next_task(const WalkArgs &a, int &queue, int64_t &lo, int64_t &hi) {
    if (lo < hi) return lo++;
    const int chunk = !kF32 && a.lds_sort ? kTaskChunkDram : kTaskChunk;
    const int lane = lane_id();
    int64_t clo = -1, chi = -1;
    if (lane == 0) {
        for (int tries = 0; tries < 8; ++tries) {
            const int q = (queue + tries) & 7;
            const int64_t qlo = a.n_tasks * q / 8, qhi = a.n_tasks * (q + 1) / 8;
            if (qhi > qlo && __atomic_load_n(&a.queue_ctr[q * kQueueStride], __ATOMIC_RELAXED) < (uint32_t)(qhi - qlo)) {
                const uint32_t idx = atomicAdd(&a.queue_ctr[q * kQueueStride], (uint32_t)chunk);
                if ((int64_t)idx < qhi - qlo) {
                    clo = qlo + idx;
                    chi = qlo + (int64_t)idx + chunk < qhi ? qlo + (int64_t)idx + chunk : qhi;
                    queue = q;
                    break;
                }
            }
        }
    }
    clo = first_lane(clo);
    chi = first_lane(chi);
    queue = __builtin_amdgcn_readfirstlane(queue);
    if (clo < 0) return -1;
    lo = clo + 1;
    hi = chi;
    return clo;
}

// A row's ids, record offset and header, loaded ahead of its walk: row_ids issues
// the offset load, row_hdr (later, once that has arrived) the header load.
struct RowPre {
    int64_t task, slot;
    int32_t r, N;
    uint32_t r_off;
    StepHdr h0;
};

__device__ __forceinline__ void row_ids(const WalkArgs &a, int64_t task, RowPre &p) {
    p.task = task;
    if (task < 0) return;
    p.slot = a.task_map ? (int64_t)a.task_map[task] : task;
    p.r = a.rows ? a.rows[p.slot] : (int32_t)p.slot;
    p.N = a.chains_per_row ? a.chains_per_row[p.r] : a.chains;
    p.r_off = a.roff[p.r];
}

template <bool kF32, bool kCmp>
__device__ __forceinline__ void row_hdr(const WalkArgs &a, RowPre &p) {
    if (p.task < 0) return;
    if (kCmp)
        load_header_c(a.rec32, p.r_off, p.h0);
    else
        load_header<kF32>(a.rec, p.r_off, p.h0);
}

// One chain of a lane: its index in the row, state, weight and Philox block.
struct ChainSt {
    int32_t c;
    bool active;
    uint32_t off, j;
    double w64;
    float w32;
    StepHdr H;
    u32x4 blk;
    int32_t pk[4];  // the home bucket of the next contribution's key, read ahead
    uint32_t pb;
};

// One step of a chain: stop (and start the lane's next chain of the row, `stride`
// further on) or draw the next state, and add the current state's weight (j > 0).
// The next bucket's loads go out first; the weight's accumulation (from the copy of
// its key's home bucket read at the end of the previous step) and the Philox
// block of the next four steps run while they are in flight. `blk` holds the
// words of the chain's next draws (step j + 1 takes word j mod 4 of block j / 4).
template <bool kF32, bool kCmp, typename Tab>
__device__ __forceinline__ void chain_step(const WalkArgs &a, ChainSt &ch, int stride, int32_t N, uint32_t r_off,
                                           const StepHdr &H0, uint32_t prow, uint32_t ptag, uint32_t k0, uint32_t k1,
                                           int32_t *gkeys, double *gvals, uint32_t slots, int hshift, int32_t *gskeys,
                                           double *gsvals, int32_t *gsused, int *gspill, uint32_t smask,
                                           unsigned long long &trans, unsigned long long &spilled, bool &spill_full) {
    const uint4 h = ch.H.h0;  // row, m, W, Shat32
    const double s64 = kF32 ? 0.0 : header_shat64(ch.H);
    const double wcur = kF32 ? (double)ch.w32 : ch.w64;
    bool stop = (h.y == 0u) || (ch.j >= (uint32_t)a.lmax);
    double wn64 = 0.0;
    float wn32 = 0.0f;
    if (kF32) {
        wn32 = ch.w32 * __uint_as_float(h.w);
        stop = stop || (fabsf(wn32) < a.delta32);
    } else {
        wn64 = ch.w64 * s64;
        stop = stop || (fabs(wn64) < a.delta);
    }
    BucketLd bl;
    if (!stop) {
        const uint32_t u = ch.blk.x;
        ch.blk.x = ch.blk.y;
        ch.blk.y = ch.blk.z;
        ch.blk.z = ch.blk.w;
        if (kCmp)
            bucket_issue_c(a.rec32, ch.off, ch.H, u, bl);
        else
            bucket_issue<kF32>(a.rec, ch.off, ch.H, u, bl);
        // the last word of the block went to this draw: the next block now
        if ((ch.j & 3u) == 3u) ch.blk = philox4x32_10((ch.j + 1u) >> 2, (uint32_t)ch.c, prow, ptag, k0, k1);
    }
    if (ch.j > 0) {
        const int32_t key = (int32_t)h.x;  // the row, or its compact record offset
        if (!Tab::add(gkeys, gvals, slots, ch.pb, ch.pk, key, wcur)) {
            ++spilled;
            if (!spill_add_window(gskeys, gsvals, gsused, gspill, smask, key, wcur)) spill_full = true;
        }
    }
    if (stop) {
        trans += ch.j;
        ch.c += stride;
        if (ch.c < N) {
            ch.off = r_off;
            ch.H = H0;
            ch.j = 0;
            ch.w64 = 1.0;
            ch.w32 = 1.0f;
            ch.blk = philox4x32_10(0u, (uint32_t)ch.c, prow, ptag, k0, k1);
        } else {
            ch.active = false;
        }
    } else {
        StepHdr Nx;
        const uint32_t tgt = kCmp ? bucket_resolve_c(bl, Nx) : bucket_resolve<kF32>(bl, Nx);
        const bool neg = (tgt & kSignBit) != 0u;
        if (kF32)
            ch.w32 = neg ? -wn32 : wn32;
        else
            ch.w64 = neg ? -wn64 : wn64;
        ch.off = tgt & ~kSignBit;
        ch.H = Nx;
        ++ch.j;
        // the next step adds this state's weight: its key's home bucket is read
        // now, so that the read has a whole bucket load's latency to complete
        ch.pb = Tab::home((int32_t)Nx.h0.x, slots, hshift);
        read_bucket_wave(gkeys, ch.pb, ch.pk);
    }
}

// Top-k retention of a row's K survivors (keys tk, sums tv), topk < K <= 512: leaves the
// topk entries that come first in retention order, with N_rc for sums, in any order. The
// values stay in registers: a search from the top bit finds the largest threshold that
// at least topk values (as bits, which order like non-negative doubles) reach, ending as
// soon as exactly topk do; values equal to it are kept by ascending key. A bitonic sort of
// all survivors in LDS in that order took the walk of a 64^3 27-point matrix (32 chains,
// top 32) 18.3 ms against 15.6, of a 48^3 one in binary64 (top 16) 9.1 against 6.9.
template <bool kCmp>
__device__ __forceinline__ void select_top(const WalkArgs &a, int32_t *tk, double *tv, int K, int32_t kg, double nd) {
    constexpr int R = 8;
    const int lane = lane_id();
    const int want = a.topk;
    uint64_t b[R];
    int32_t key[R];
    double nh[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = lane + 64 * q;
        b[q] = 0;
        key[q] = 0;
        nh[q] = 0.0;
        if (i < K) {
            key[q] = tk[i];
            nh[q] = tv[i] / nd;
            double t = fabs(nh[q]);
            if (a.filter_m) t = fabs(nh[q] / (kCmp ? diag_of_c(a.rec32, (uint32_t)key[q]) : a.diag[key[q]]));
            // the diagonal first; 1 more than the value's bits, so that a value of zero (M_rc may
            // underflow) is not taken for one of the places past the survivors
            b[q] = key[q] == kg ? ~0ull >> 1 : (uint64_t)__double_as_longlong(t) + 1u;
        }
    }
    wave_sync();
    uint64_t T = 0;
    bool exact = false;
    for (int bit = 62; bit >= 0 && !exact; --bit) {
        const uint64_t cand = T | (1ull << bit);
        int c = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) c += __popcll(ballot(b[q] >= cand));
        if (c >= want) T = cand;
        exact = c == want;
    }
    int32_t last = INT32_MAX;  // largest key kept among the values equal to T
    if (!exact) {
        int above = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) above += __popcll(ballot(b[q] > T));
        last = 0;
        for (int bit = 30; bit >= 0; --bit) {
            const int32_t cand = last | (int32_t)(1u << bit);
            int c = above;
#pragma unroll
            for (int q = 0; q < R; ++q) c += __popcll(ballot(b[q] == T && key[q] < cand));
            if (c < want) last = cand;
        }
    }
    int n = 0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const bool keep = b[q] > T || (b[q] == T && (exact || key[q] <= last));
        const uint64_t km = ballot(keep);
        if (keep) {
            const int pos = n + mask_rank(km);
            tk[pos] = key[q];
            tv[pos] = nh[q];
        }
        n += __popcll(km);
    }
    wave_sync();
}

// Sorts the row's K <= 64 W survivors (keys tk, sums tv) by key into ps (positions in
// the low 8 bits) and turns keys and sums, in place, into columns and M_rc. False,
// with the survivors as they were, when the keys span 2^24 or more.
template <bool kCmp, int W>
__device__ __forceinline__ bool finish_sorted(const WalkArgs &a, int32_t *tk, double *tv, uint32_t *ps, int K,
                                              double nd, double ninv, bool pow2) {
    const int lane = lane_id();
    int32_t key[W];
    uint32_t mn = ~0u, mx = 0u;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const int i = lane * W + q;
        key[q] = i < K ? tk[i] : 0;
    }
    int32_t rw[W];
    double d[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        rw[q] = key[q];
        d[q] = 1.0;
        if (lane * W + q < K) {
            if (kCmp) {
                const uint32_t *h = a.rec32 + (size_t)(uint32_t)key[q] * kUnitWords32;
                rw[q] = (int32_t)h[0];
                d[q] = *(const double *)(h + 6);
            }
            mn = min(mn, (uint32_t)key[q]);
            mx = max(mx, (uint32_t)key[q]);
        }
    }
    mn = wavesort::wave_extreme<false>(mn);
    mx = wavesort::wave_extreme<true>(mx);
    if (mx - mn >= (1u << 24)) return false;
    uint32_t e[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const int i = lane * W + q;
        e[q] = i < K ? (((uint32_t)key[q] - mn) << 8) | (uint32_t)i : ~0u;
    }
    wavesort::sort_words<W>(e, lane);
#pragma unroll
    for (int q = 0; q < W; ++q) ps[lane * W + q] = e[q];
    if (!kCmp) {
        // d_c in column order: neighbours share lines (in table order a row of the 100^3
        // 27-point matrix touched a line per survivor, and the walk took 18.5 ms against 17.0)
        wave_sync();
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int i = lane + 64 * q;
            if (i < K) {
                const uint32_t p = ps[i] & 255u;
                const double acc = tv[p];
                const double nhat = pow2 ? acc * ninv : acc / nd;
                tv[p] = nhat / a.diag[tk[p]];
            }
        }
        wave_sync();
        return true;
    }
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const int i = lane * W + q;
        if (i < K) {
            const double acc = tv[i];
            const double nhat = pow2 ? acc * ninv : acc / nd;
            tk[i] = rw[q];
            tv[i] = nhat / d[q];
        }
    }
    wave_sync();
    return true;
}

// The 64 / kG rows of one wave (one per group of kG lanes; cur and nxt hold each
// lane's own group's row); each lane keeps kC of its row's chains in flight.
// kTop: with top-k retention (an instance of its own: its registers would not fit beside
// the walk's in the common one).
template <bool kF32, int kG, int kC, bool kCmp, bool kTop, bool kWide>
__device__ __forceinline__ void walk_rows(const WalkArgs &a, const RowPre &cur, RowPre &nxt, int &queue, int64_t &tlo,
                         int64_t &thi, int32_t *keys, double *vals, int *spill_cnt,
                         int32_t *skeys, double *svals, int32_t *sused, uint32_t k0, uint32_t k1,
                         unsigned long long &pcur, unsigned long long &pend, unsigned long long *wstats) {
    constexpr int P = 64 / kG;  // rows per wave
    const int lane = lane_id();
    const int grp = lane / kG;
    const int sub = lane & (kG - 1);
    const int Hg = a.hash_slots / P;  // slots per row
    const uint32_t slots = (uint32_t)Hg;
    constexpr int kLogP = P == 1 ? 0 : P == 2 ? 1 : P == 4 ? 2 : 3;
    const int hshift = a.hash_shift + kLogP;
    using Tab = Probe<!kWide, kC == 2 || !kF32, kWide>;
    const int Sg = a.spill_slots / P;
    const uint32_t smask = (uint32_t)Sg - 1u;
    int32_t *gkeys = keys + grp * Hg;
    double *gvals = vals + grp * Hg;
    int32_t *gskeys = skeys + (size_t)grp * Sg;
    double *gsvals = svals + (size_t)grp * Sg;
    int32_t *gsused = sused + (size_t)grp * Sg;
    const bool has = cur.task >= 0;
    const int32_t r = has ? cur.r : 0;
    const int32_t N = has ? cur.N : 0;
    const uint32_t r_off = has ? cur.r_off : 0u;
    uint32_t prow = 0, ptag = 0;
    if (has) philox_ids(a, r, prow, ptag);

    // j = 0: every chain contributes W_0 = 1 at (r, r); N ones sum exactly to N.
    // Keys are rows, or record offsets with compact records (turned into rows once
    // the kept set is known).
    const int32_t rkey = kCmp ? (int32_t)r_off : r;
    if (sub == 0 && has) {
        const uint32_t b = Tab::home(rkey, slots, hshift);
        int32_t k[4];
        read_bucket_wave(gkeys, b, k);
        Tab::add(gkeys, gvals, slots, b, k, rkey, (double)N);
    }
    wave_sync();

    // the row's own header (every chain starts there, loaded ahead); later
    // states' headers arrive with the bucket of the step that reaches them
    const StepHdr H0 = cur.h0;
    ChainSt ch[kC];
#pragma unroll
    for (int k = 0; k < kC; ++k) {
        ch[k].c = sub + k * kG;
        ch[k].active = has && ch[k].c < N;
        ch[k].off = r_off;
        ch[k].j = 0;
        ch[k].w64 = 1.0;
        ch[k].w32 = 1.0f;
        ch[k].H = H0;
        ch[k].blk = ch[k].active ? philox4x32_10(0u, (uint32_t)ch[k].c, prow, ptag, k0, k1) : u32x4{0, 0, 0, 0};
    }
    unsigned long long trans = 0, spilled = 0;
    bool spill_full = false;

    if constexpr (kC == 1 && kF32) {
        // one chain per lane: a lane leaves the loop with its last chain (1024^2 grid with
        // per-row chains 7.9 -> 7.5 ms, 33 x 31 grid 150 -> 140 us against a wave vote per step;
        // binary64 rows keep the vote: 100^3 27-point 18.5 -> 18.0 ms with it, 77^3 7.9 -> 7.8)
        while (ch[0].active)
            chain_step<kF32, kCmp, Tab>(a, ch[0], kG, N, r_off, H0, prow, ptag, k0, k1, gkeys, gvals, slots, hshift, gskeys,
                                   gsvals, gsused, spill_cnt + grp, smask, trans, spilled, spill_full);
    } else {
        while (true) {
            bool any = false;
    #pragma unroll
            for (int k = 0; k < kC; ++k) any |= ch[k].active;
            if (!__any(any)) break;
    #pragma unroll
            for (int k = 0; k < kC; ++k)
                if (ch[k].active)
                    chain_step<kF32, kCmp, Tab>(a, ch[k], kG * kC, N, r_off, H0, prow, ptag, k0, k1, gkeys, gvals, slots, hshift,
                                     gskeys, gsvals, gsused, spill_cnt + grp, smask, trans, spilled, spill_full);
        }
    }
    wave_sync();
    // the next rows' ids and record offsets load now, their headers during the
    // finalize: both latencies hide behind these rows' finalize
#pragma unroll
    for (int g = 0; g < P; ++g) {
        const int64_t t = next_task<kF32>(a, queue, tlo, thi);
        if (grp == g) row_ids(a, t, nxt);
    }

    // ---------------------------------------------------------- finalize, row by row
    bool hdr_issued = false;
#pragma unroll 1
    for (int g = 0; g < P; ++g) {
        if (__shfl((int)has, g * kG, 64) == 0) continue;  // no row in this group
        const int32_t rg = __shfl(r, g * kG, 64);
        const int32_t kg = kCmp ? __shfl(rkey, g * kG, 64) : rg;  // the row's own key
        const int32_t Ng = __shfl(N, g * kG, 64);
        const int64_t slot = (int64_t)(((uint64_t)(uint32_t)__shfl((int)(cur.slot >> 32), g * kG, 64) << 32) |
                                       (uint32_t)__shfl((int)(uint32_t)cur.slot, g * kG, 64));
        int32_t *tk = keys + g * Hg;
        double *tv = vals + g * Hg;
        int32_t *tsk = skeys + (size_t)g * Sg;
        double *tsv = svals + (size_t)g * Sg;
        const int32_t *tsu = sused + (size_t)g * Sg;
        const double nd = (double)Ng;
        // The eps test needs N_rc = fl(acc / N) only near the cutoff: |acc| above
        // hi = fl(fl(eps N) (1 + 2^-50)) gives fl(acc / N) >= eps for certain, below lo
        // = fl(fl(eps N) (1 - 2^-50)) gives < eps; in between (and for the M filter or
        // eps = 0) the quotient itself decides. Survivors keep acc until the kept set
        // is known.
        const bool exact = a.filter_m || !(a.eps > 0.0);
        const double en = a.eps * nd;
        const double hi = en * (1.0 + 0x1p-50), lo = en * (1.0 - 0x1p-50);
        auto keep_test = [&](int32_t key, double acc) -> bool {
            const double aa = fabs(acc);
            if (key == kg || (!exact && aa > hi)) return true;
            if (!exact && !(aa >= lo)) return false;
            const double nhat = acc / nd;
            const double test =
                a.filter_m ? fabs(nhat / (kCmp ? diag_of_c(a.rec32, (uint32_t)key) : a.diag[key])) : fabs(nhat);
            return nhat != 0.0 && test >= a.eps;
        };
        // Four consecutive slots per lane and round (16-byte LDS reads); the survivors
        // move to the front of the table in any order, they are sorted below. A round
        // writes only slots that it or an earlier round has read.
        const double hi_t = exact ? __builtin_huge_val() : hi, lo_t = exact ? 0.0 : lo;
        int K = 0;
        for (int base = 0; base < Hg; base += 256) {
            const int s = base + 4 * lane;
            i32x4v kk = {kEmpty, kEmpty, kEmpty, kEmpty};
            f64x2v va = {0.0, 0.0}, vb = {0.0, 0.0};
            if (s < Hg) {
                kk = *(const i32x4v *)(tk + s);
                va = *(const f64x2v *)(tv + s);
                vb = *(const f64x2v *)(tv + s + 2);
            }
            const int32_t key4[4] = {kk.x, kk.y, kk.z, kk.w};
            const double acc4[4] = {va.x, va.y, vb.x, vb.y};
            bool keep[4], near = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double aa = fabs(acc4[q]);
                keep[q] = key4[q] >= 0 && (aa > hi_t || key4[q] == kg);
                near |= key4[q] >= 0 && !keep[q] && aa >= lo_t;
            }
            if (__any(near)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) keep[q] = key4[q] >= 0 && keep_test(key4[q], acc4[q]);
            }
            wave_sync();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t km = ballot(keep[q]);
                if (keep[q]) {
                    const int pos = K + mask_rank(km);
                    tk[pos] = key4[q];
                    tv[pos] = acc4[q];
                }
                K += __popcll(km);
            }
        }
        wave_sync();
        if (!hdr_issued) {
            row_hdr<kF32, kCmp>(a, nxt);
            hdr_issued = true;
        }
        const int nsp = spill_cnt[g];
        bool stage_full = false;
        for (int base = 0; base < nsp; base += 64) {
            const int u = base + lane;
            bool keep = false;
            int32_t key = kEmpty;
            double acc = 0.0;
            if (u < nsp) {
                const int32_t sl = tsu[u];
                key = tsk[sl];
                acc = tsv[sl];
                keep = keep_test(key, acc);
                tsk[sl] = kEmpty;
                tsv[sl] = 0.0;
            }
            const uint64_t km = ballot(keep);
            if (keep) {
                const int pos = K + mask_rank(km);
                if (pos < Hg) {
                    tk[pos] = key;
                    tv[pos] = acc;
                } else {
                    stage_full = true;
                }
            }
            K += __popcll(km);
        }
        if (K > Hg) K = Hg;
        wave_sync();
        // the survivors: record offsets -> rows (compact records: row and d from the
        // header unit, loaded together), N_rc = acc / N, and without top-k at once
        // M_rc = N_rc / d_c; four entries per lane in flight
        double nd_now = nd;  // divisor of the sums that are left
        if (kTop && K > a.topk && K <= 512) {
            select_top<kCmp>(a, tk, tv, K, kg, nd);
            K = a.topk;
            nd_now = 1.0;
        }
        const bool scale_now = !kTop || K <= a.topk;
        // Up to 256 survivors without top-k: their keys (record offsets order like the
        // rows they start) are sorted in registers while the loads of their rows and
        // d_c are in flight; M_rc = (acc / N) / d_c and the columns then replace the
        // sums and keys in place and go out in the sorted order. A sorted word is
        // (key - smallest key) << 8 | position, so the keys must span less than 2^24
        // (on the 160^3 27-point matrix they span up to 9.7e6 units; rows that span more
        // take the general path below). With the 64-bit network in LDS (about 20 round
        // trips), one slot per lane and read in the filter, and two wave sums per row,
        // the walks took 55.3 ms (160^3), 23.3 ms (batched, 128 chains), 9.0 ms (77^3
        // binary64) and 9.4 ms (1024^2 grid, 1-96 chains) against 51.4, 21.6, 8.2 and 7.8.
        const int W = K <= 64 ? 1 : K <= 128 ? 2 : 4;
        uint32_t *ps = (uint32_t *)(tv + (Hg - 32 * W));
        bool early = scale_now && (kCmp || !a.lds_sort) && K <= 256 && K + 32 * W <= Hg;
        if (early) {
            const double ninv = 1.0 / nd_now;
            const bool pow2 = nd_now == 1.0 || (Ng & (Ng - 1)) == 0;  // acc / N = acc (1 / N) exactly
            if (W == 1)
                early = finish_sorted<kCmp, 1>(a, tk, tv, ps, K, nd_now, ninv, pow2);
            else if (W == 2)
                early = finish_sorted<kCmp, 2>(a, tk, tv, ps, K, nd_now, ninv, pow2);
            else
                early = finish_sorted<kCmp, 4>(a, tk, tv, ps, K, nd_now, ninv, pow2);
        }
        if (!early) {
            for (int i0 = lane; i0 < K; i0 += 256) {
                int32_t rw[4];
                double d[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + 64 * q;
                    rw[q] = i < K ? tk[i] : 0;
                    d[q] = 1.0;
                    if (i < K) {
                        if (kCmp) {
                            const uint32_t *h = a.rec32 + (size_t)(uint32_t)rw[q] * kUnitWords32;
                            rw[q] = (int32_t)h[0];
                            if (scale_now) d[q] = *(const double *)(h + 6);
                        } else if (scale_now) {
                            d[q] = a.diag[rw[q]];
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + 64 * q;
                    if (i < K) {
                        const double nhat = tv[i] / nd_now;
                        tk[i] = rw[q];
                        tv[i] = scale_now ? nhat / d[q] : nhat;
                    }
                }
            }
            wave_sync();

            // top-k retention: bitonic sort in retention order, keep the first topk,
            // then turn N_rc into M_rc = N_rc / d_c
            if (!scale_now) {
                if (K > a.topk) {
                    int PT = 1;
                    while (PT < K) PT <<= 1;
                    for (int s = K + lane; s < PT; s += 64) tk[s] = INT32_MAX;
                    wave_sync();
                    for (int k = 2; k <= PT; k <<= 1) {
                        for (int jj = k >> 1; jj > 0; jj >>= 1) {
                            for (int pr = lane; pr < (PT >> 1); pr += 64) {
                                const int i = ((pr & ~(jj - 1)) << 1) | (pr & (jj - 1));
                                const int ixj = i | jj;
                                const int32_t ka = tk[i], kb = tk[ixj];
                                const double va = tv[i], vb = tv[ixj];
                                if (top_after(a, rg, ka, va, kb, vb) == ((i & k) == 0)) {
                                    tk[i] = kb;
                                    tk[ixj] = ka;
                                    tv[i] = vb;
                                    tv[ixj] = va;
                                }
                            }
                            wave_sync();
                        }
                    }
                    K = a.topk;
                }
                for (int i0 = lane; i0 < K; i0 += 256) {
                    double d[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) d[q] = i0 + 64 * q < K ? a.diag[tk[i0 + 64 * q]] : 1.0;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (i0 + 64 * q < K) tv[i0 + 64 * q] = tv[i0 + 64 * q] / d[q];
                }
                wave_sync();
            }
        }

        // Bitonic sort by column in LDS. A pass has PS / 2 compare-exchange pairs, pair p
        // joining i (p with a zero bit inserted at jj) and i | jj, so every lane has a
        // pair. When the value slots past the survivors have room, the sort moves
        // one word per entry, (column << 13) | position, in that free part of the
        // value table, and the values stay where they are; otherwise it moves
        // (column, value) pairs.
        int PS = 1;
        while (PS < K) PS <<= 1;
        const bool packed = K + PS <= Hg;
        uint64_t *pk = (uint64_t *)(tv + (Hg - PS));
        if (early) {
        } else if (packed) {
            for (int s = lane; s < PS; s += 64) pk[s] = s < K ? ((uint64_t)(uint32_t)tk[s] << 13) | (uint64_t)s : ~0ull;
            wave_sync();
            for (int k = 2; k <= PS; k <<= 1) {
                int jj = k >> 1;
                // two passes per LDS round trip: a lane takes the four words b, b + h,
                // b + jj, b + jj + h (h = jj / 2; b with bits h and jj clear) and
                // applies the exchanges at distance jj, then at distance h
                for (; jj >= 2; jj >>= 2) {
                    const int h = jj >> 1;
                    const int ph = __builtin_ctz((unsigned)h);
                    for (int g = lane; g < (PS >> 2); g += 64) {
                        const int b = ((g >> ph) << (ph + 2)) | (g & (h - 1));
                        const bool up = (b & k) == 0;
                        uint64_t e0 = pk[b], e1 = pk[b + h], e2 = pk[b + jj], e3 = pk[b + jj + h];
                        exch(e0, e2, up);
                        exch(e1, e3, up);
                        exch(e0, e1, up);
                        exch(e2, e3, up);
                        pk[b] = e0;
                        pk[b + h] = e1;
                        pk[b + jj] = e2;
                        pk[b + jj + h] = e3;
                    }
                    wave_sync();
                }
                if (jj == 1) {
                    for (int pr = lane; pr < (PS >> 1); pr += 64) {
                        const int i = pr << 1;
                        uint64_t ea = pk[i], eb = pk[i + 1];
                        exch(ea, eb, (i & k) == 0);
                        pk[i] = ea;
                        pk[i + 1] = eb;
                    }
                    wave_sync();
                }
            }
        } else {
            // (column, value) pairs in place. Every exchange leaves the smaller column in the
            // lower slot (a merge of width k starts with the pairs i and k - 1 - i of its
            // run), so the words past the survivors need no slots: they would stay
            // where they are.
            for (int k = 2; k <= PS; k <<= 1) {
                for (int jj = k >> 1; jj > 0; jj >>= 1) {
                    for (int pr = lane; pr < (PS >> 1); pr += 64) {
                        const int i = ((pr & ~(jj - 1)) << 1) | (pr & (jj - 1));
                        const int ixj = jj == k >> 1 ? i ^ (k - 1) : i | jj;
                        if (ixj >= K) continue;
                        const int32_t ka = tk[i], kb = tk[ixj];
                        if (ka > kb) {
                            const double va = tv[i], vb = tv[ixj];
                            tk[i] = kb;
                            tk[ixj] = ka;
                            tv[i] = vb;
                            tv[ixj] = va;
                        }
                    }
                    wave_sync();
                }
            }
        }

        // append to the pool unless a table overflowed for this row (then it is rerun)
        const bool row_spill_full = __any(spill_full && grp == g);
        const bool row_stage_full = __any(stage_full);
        unsigned long long pos0 = 0;
        if (lane == 0 && !row_spill_full && !row_stage_full) {
            if (a.pool_chunk > 0) {
                // the wave's reservation: one global atomic per pool_chunk entries
                if (pcur + (unsigned long long)K > pend) {
                    const unsigned long long grab = (unsigned long long)(K > a.pool_chunk ? K : a.pool_chunk);
                    pcur = atomicAdd(a.pool_used, grab);
                    pend = pcur + grab;
                }
                pos0 = pcur;
                pcur += (unsigned long long)K;
            } else {
                pos0 = atomicAdd(a.pool_used, (unsigned long long)K);
            }
        }
        pos0 = __shfl(pos0, 0, 64);
        const bool fits = (int64_t)(pos0 + (unsigned long long)K) <= a.pool_cap;
        const bool ok = fits && !row_spill_full && !row_stage_full;
        if (ok) {
            for (int i = lane; i < K; i += 64) {
                int e = i;
                if (early)
                    e = (int)(ps[i] & 255u);
                else if (packed)
                    e = (int)(pk[i] & 8191u);
                if (kCmp) {
                    a.pool_col[pos0 + i] = tk[e];
                    a.pool_val[pos0 + i] = tv[e];
                } else {
                    // not kept in L2, which the full records want (100^3 27-point, binary64:
                    // 17.0 -> 16.9 ms; the batched FP32 walk lost 0.7 %, so not there)
                    __builtin_nontemporal_store(tk[e], a.pool_col + pos0 + i);
                    __builtin_nontemporal_store(tv[e], a.pool_val + pos0 + i);
                }
            }
        }
        // statistics per lane, summed over the wave when the kernel ends
        if (grp == g) {
            if (ok) wstats[0] += trans;
            wstats[1] += spilled;
        }
        if (lane == 0) {
            a.row_start[slot] = ok ? ((int64_t)pos0 | a.pool_tag) : -1;
            a.row_cnt[slot] = (uint32_t)K;
            uint32_t f = 0;
            if (!fits && !row_spill_full && !row_stage_full) f |= kFlagPool;
            if (row_spill_full) f |= kFlagSpill;
            if (row_stage_full) f |= kFlagStage;
            if (f) atomicOr(a.flags, f);
            if (ok) wstats[2] += (unsigned long long)Ng;
        }
        // clear this row's table for the next row of its group
        wave_sync();
        for (int s = 4 * lane; s < Hg; s += 256) *(i32x4v *)(tk + s) = i32x4v{kEmpty, kEmpty, kEmpty, kEmpty};
        for (int s = 2 * lane; s < Hg; s += 128) *(f64x2v *)(tv + s) = f64x2v{0.0, 0.0};
        if (lane == 0) spill_cnt[g] = 0;
        wave_sync();
    }
    if (!hdr_issued) row_hdr<kF32, kCmp>(a, nxt);
}

// kWide: at most 128 registers, for four waves per SIMD where the tables of a launch leave
// room for more than three (choose_shape).
template <bool kF32, int kG, int kC, bool kCmp, bool kTop, bool kWide>
__global__ void __launch_bounds__(256, kWide ? 4 : 3) k_walk(WalkArgs a) {
    constexpr int P = 64 / kG;
    extern __shared__ __align__(16) unsigned char smem[];
    const int waves = blockDim.x >> 6;
    const int w = threadIdx.x >> 6;
    const int lane = lane_id();
    const int H = a.hash_slots;
    // per wave: vals[H] (f64), keys[H] (i32), one spill counter per row (64 bytes)
    const size_t per_wave = (size_t)H * 12u + 64u;
    unsigned char *mine = smem + (size_t)w * per_wave;
    double *vals = (double *)mine;
    int32_t *keys = (int32_t *)(mine + (size_t)H * 8u);
    int *spill_cnt = (int *)(mine + (size_t)H * 12u);
    for (int s = lane; s < H; s += 64) {
        keys[s] = kEmpty;
        vals[s] = 0.0;
    }
    if (lane < P) spill_cnt[lane] = 0;
    wave_sync();
    const int64_t gw = (int64_t)blockIdx.x * waves + w;
    int32_t *skeys = a.spill_keys + gw * a.spill_slots;
    double *svals = a.spill_vals + gw * a.spill_slots;
    int32_t *sused = a.spill_used + gw * a.spill_slots;
    int queue = (int)(blockIdx.x & 7u);
    const uint32_t k0 = a.keys_dev ? a.keys_dev[0] : a.key0;
    const uint32_t k1 = a.keys_dev ? a.keys_dev[1] : a.key1;
    unsigned long long pcur = 0, pend = 0, wstats[3] = {0, 0, 0};
    int64_t tlo = 0, thi = 0;
    const int grp = lane / kG;
    RowPre cur;
#pragma unroll
    for (int g = 0; g < P; ++g) {
        const int64_t t = next_task<kF32>(a, queue, tlo, thi);
        if (grp == g) row_ids(a, t, cur);
    }
    row_hdr<kF32, kCmp>(a, cur);
    while (__any(cur.task >= 0)) {
        RowPre nxt;
        walk_rows<kF32, kG, kC, kCmp, kTop, kWide>(a, cur, nxt, queue, tlo, thi, keys, vals, spill_cnt, skeys, svals, sused, k0,
                                      k1, pcur, pend, wstats);
        cur = nxt;
    }
    // statistics: one set of atomics per wave
    wstats[0] = wave_sum(wstats[0]);
    wstats[1] = wave_sum(wstats[1]);
    if (lane == 0) {
        if (wstats[0]) atomicAdd(&a.stats[0], wstats[0]);
        if (wstats[1]) atomicAdd(&a.stats[1], wstats[1]);
        if (wstats[2]) atomicAdd(&a.stats[2], wstats[2]);
    }
}

}  // namespace

size_t walk_lds_bytes(int hash_slots, int waves) { return (size_t)waves * ((size_t)hash_slots * 12u + 64u); }

// Whether a launch uses the four-waves-per-SIMD instance (one row per wave, one chain per lane).
bool walk_wide(bool f32, bool top, int row_lanes, int lane_chains, int hash_slots) {
    return f32 && !top && (row_lanes == 0 || row_lanes == 64) && lane_chains != 2 && hash_slots <= kWideSlots;
}

using WalkKernel = void (*)(WalkArgs);

// FP32 walks read the compact records, FP64 walks the full ones (which carry Shat64).
template <bool kF32, bool kTop>
WalkKernel walk_kernel_t(int row_lanes, int lane_chains, int hash_slots) {
    switch (row_lanes) {
        case 8: return k_walk<kF32, 8, 1, kF32, kTop, false>;
        case 16: return k_walk<kF32, 16, 1, kF32, kTop, false>;
        case 32: return k_walk<kF32, 32, 1, kF32, kTop, false>;
        default: break;
    }
    if (lane_chains == 2) return k_walk<kF32, 64, 2, kF32, kTop, false>;
    if (walk_wide(kF32, kTop, row_lanes, lane_chains, hash_slots)) return k_walk<kF32, 64, 1, kF32, kTop, kF32 && !kTop>;
    return k_walk<kF32, 64, 1, kF32, kTop, false>;
}

// The instance that runs a launch; its registers and tables set how many workgroups a CU holds.
WalkKernel walk_kernel(bool f32, bool top, int row_lanes, int lane_chains, int hash_slots) {
    if (top)
        return f32 ? walk_kernel_t<true, true>(row_lanes, lane_chains, hash_slots)
                   : walk_kernel_t<false, true>(row_lanes, lane_chains, hash_slots);
    return f32 ? walk_kernel_t<true, false>(row_lanes, lane_chains, hash_slots)
               : walk_kernel_t<false, false>(row_lanes, lane_chains, hash_slots);
}

hipError_t launch_walk(const WalkArgs &a, bool f32, int blocks, int waves, hipStream_t s) {
    if (a.row_lanes != 0 && a.row_lanes != 8 && a.row_lanes != 16 && a.row_lanes != 32 && a.row_lanes != 64)
        return hipErrorInvalidValue;
    if (a.lane_chains == 2 && a.row_lanes != 0 && a.row_lanes != 64) return hipErrorInvalidValue;
    if (f32 && !a.rec32) return hipErrorInvalidValue;
    // only the small-table instance takes tables that are no power of two
    const bool top = a.topk > 0, wide = walk_wide(f32, top, a.row_lanes, a.lane_chains, a.hash_slots);
    if (a.hash_slots < 64 || ((a.hash_slots & (a.hash_slots - 1)) != 0 && !(wide && a.hash_slots % 4 == 0)))
        return hipErrorInvalidValue;
    const WalkKernel k = walk_kernel(f32, top, a.row_lanes, a.lane_chains, a.hash_slots);
    k<<<blocks, waves * 64, walk_lds_bytes(a.hash_slots, waves), s>>>(a);
    return hipGetLastError();
}

hipError_t walk_occupancy(bool f32, bool top, int row_lanes, int lane_chains, int hash_slots, int waves,
                          int *blocks_per_cu) {
    const WalkKernel k = walk_kernel(f32, top, row_lanes, lane_chains, hash_slots);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, waves * 64, walk_lds_bytes(hash_slots, waves));
}

}  // namespace mcmi
