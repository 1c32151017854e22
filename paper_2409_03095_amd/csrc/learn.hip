// Per-row inputs of the learned chain allocation (gfx950): row features and
// pilot-run variance.
//
// Features (8 per row, binary32, row-major), with p_ij = w_ij / W_i the
// quantized transition probabilities and S = Shat:
//   f0 = ln max(m_i, 1)      f1 = S_i               f2 = max_j |chat_ij|
//   f3 = sum_j p_ij S_j      f4 = max_j S_j          f5 = sum_j p_ij m_j
//   f6 = |sum_j chat_ij| / S_i (sign balance)        f7 = min(L_max, ln delta / ln S_i)
// (f3..f6 = 0 for an empty row; f7 = L_max when S_i >= 1 and 0 when S_i = 0).
//
// Pilot variance (the per-row target of the allocation): P chains per row on
// their own Philox streams (tag bit 31 set). Each chain's row estimate is the
// sparse vector X_c with X_c[s] = sum of its W_j at s (revisits merged);
// v_r = mean_c ||X_c||^2 - ||mean_c X_c||^2 and len_r = mean transitions per chain.
#include <string.h>

#include <algorithm>
#include <string>

#include "common.hpp"
#include "walk_args.hpp"
#include "walk_common.hpp"

namespace mcmi {

namespace {

using namespace walkdev;

// Features of row r by P lanes (sub: the lane's place among them), from the compact
// records: an entry's weight, target and the target's m from its bucket, Shat64 from the
// target's header. The sums are those of 64 strided partial sums per row added as a
// binary tree, of which a lane keeps 64 / P.
template <int P>
__device__ __forceinline__ void row_features(int64_t r, int sub, const uint32_t *__restrict__ rec32,
                                             const uint32_t *__restrict__ roff, double delta, int lmax,
                                             float *__restrict__ feat) {
    constexpr int T = 64 / P;
    const uint32_t *recp = rec32 + (size_t)roff[r] * kUnitWords32;
    const uint4 h = *(const uint4 *)recp;  // row, m, W, Shat32
    const uint32_t m = h.y, W = h.z;
    const double S = *(const double *)(recp + 4);
    double ps[T], pm[T], sgn[T], smax = 0.0;
    uint32_t wmax = 0;
#pragma unroll
    for (int t = 0; t < T; ++t) ps[t] = pm[t] = sgn[t] = 0.0;
    auto add = [&](int t, const uint4 &q0, uint32_t w, double St) {
        const double mt = (double)q0.z;
        ps[t] += (double)w * St;
        pm[t] += (double)w * mt;
        sgn[t] += (q0.y & kSignBit) ? -(double)w : (double)w;
        smax = St > smax ? St : smax;
        wmax = w > wmax ? w : wmax;
    };
    uint32_t k0 = 0;
    if (T == 1) {  // long rows: the loads of four entries in flight
        constexpr int U = 4;
        for (; k0 + U * 64u <= m; k0 += U * 64u) {
            uint4 q0[U];
            uint32_t w[U];
            double St[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t *e = recp + (size_t)(1u + k0 + u * 64u + sub) * kUnitWords32;
                q0[u] = *(const uint4 *)e;
                w[u] = e[4];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                St[u] = *(const double *)(rec32 + (size_t)(q0[u].y & ~kSignBit) * kUnitWords32 + 4);
#pragma unroll
            for (int u = 0; u < U; ++u) add(0, q0[u], w[u], St[u]);
        }
    }
    for (; k0 < m; k0 += 64) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const uint32_t k = k0 + (uint32_t)(t * P + sub);
            if (k < m) {
                const uint32_t *e = recp + (size_t)(1u + k) * kUnitWords32;
                const uint4 q0 = *(const uint4 *)e;  // T', target, m and Shat32 of the target's row
                add(t, q0, e[4], *(const double *)(rec32 + (size_t)(q0.y & ~kSignBit) * kUnitWords32 + 4));
            }
        }
    }
#pragma unroll
    for (int hh = T / 2; hh > 0; hh >>= 1)
#pragma unroll
        for (int t = 0; t < hh; ++t) {
            ps[t] += ps[t + hh];
            pm[t] += pm[t + hh];
            sgn[t] += sgn[t + hh];
        }
#pragma unroll
    for (int off = P / 2; off > 0; off >>= 1) {
        ps[0] += __shfl_xor(ps[0], off, P);
        pm[0] += __shfl_xor(pm[0], off, P);
        sgn[0] += __shfl_xor(sgn[0], off, P);
        const double so = __shfl_xor(smax, off, P);
        smax = so > smax ? so : smax;
        const uint32_t wo = (uint32_t)__shfl_xor((int)wmax, off, P);
        wmax = wo > wmax ? wo : wmax;
    }
    if (sub == 0) {
        const double Wd = (double)W;
        float4 f0, f1;
        f0.x = (float)log((double)(m > 1u ? m : 1u));
        f0.y = (float)S;
        f0.z = m ? (float)(S * (double)wmax / Wd) : 0.f;
        f0.w = m ? (float)(ps[0] / Wd) : 0.f;
        f1.x = (float)smax;
        f1.y = m ? (float)(pm[0] / Wd) : 0.f;
        f1.z = (m && S > 0.0) ? (float)(fabs(sgn[0]) / Wd) : 0.f;
        double f7;
        if (S > 0.0 && S < 1.0 && delta > 0.0) {
            const double l = log(delta) / log(S);
            f7 = l < (double)lmax ? l : (double)lmax;
        } else {
            f7 = S > 0.0 ? (double)lmax : 0.0;
        }
        f1.w = (float)f7;
        float *f = feat + 8 * r;
        f[0] = f0.x;
        f[1] = f0.y;
        f[2] = f0.z;
        f[3] = f0.w;
        f[4] = f1.x;
        f[5] = f1.y;
        f[6] = f1.z;
        f[7] = f1.w;
    }
}

// P lanes per row, several rows to a wavefront; a row of more than kFeatureWide entries is
// left to the whole wavefront. On the 1024^2 5-point grid 0.70 ms with a wavefront per row on
// the full records, whose build (0.22 ms there, 4.9 ms on the 160^3 matrix) this does
// without, against 0.09 ms. Random matrix of 20000 rows, one of 3000 entries: 23 us that way,
// 79 us with its 16 lanes for that row, 34 us with the wavefront, 17 us with four loads ahead.
constexpr uint32_t kFeatureWide = 256;

template <int P>
__global__ void __launch_bounds__(256) k_features(int64_t n, const uint32_t *__restrict__ rec32,
                                                  const uint32_t *__restrict__ roff, double delta, int lmax,
                                                  float *__restrict__ feat) {
    const int lane = threadIdx.x & 63, sub = threadIdx.x & (P - 1);
    const int64_t groups = ((int64_t)gridDim.x * blockDim.x) / P;
    int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / P;
    for (; r - lane / P < n; r += groups) {  // uniform over the wave
        bool wide = false;
        if (r < n) {
            wide = P < 64 && rec32[(size_t)roff[r] * kUnitWords32 + 1] > kFeatureWide;
            if (!wide) row_features<P>(r, sub, rec32, roff, delta, lmax, feat);
        }
        if (P < 64) {
            for (uint64_t left = __ballot(wide && sub == 0); left != 0; left &= left - 1)
                row_features<64>(r - lane / P + __builtin_ctzll(left) / P, lane, rec32, roff, delta, lmax, feat);
        }
    }
}

// One wavefront per row, one chain per lane (with refill). A chain's own estimate
// X_c is a small open-addressing table per lane in LDS (cap slots in buckets of
// four, laid out so that a lane's bank does not depend on its bucket: no bank
// conflicts), the row mean the wave's LDS hash (spilling to HBM like the walk). A
// step issues the next bucket's loads, then reads the state's bucket in both tables
// together and adds to both while they are in flight. The tables allow about three
// waves per CU, so a step's serial chain sets the time. On 200 5-point grids of 24-40
// points a side (binary64, 64 chains): 26.7 ms with a linear search of each lane's list
// of states (up to 48 dependent LDS reads per step), 18.9 ms with the tables and each
// chain's norm taken when it stops, 9.5 ms with the norms of the lanes' last chains
// taken together; with the sums in HBM (twice the waves, global atomics) 11.9 ms.
// FP32 walks read the compact records (keys are record offsets), FP64 walks the full ones.
template <bool kF32>
__global__ void __launch_bounds__(64) k_pilot(WalkArgs a, int pilot, int cap, double *__restrict__ var,
                                              double *__restrict__ len) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int H = a.hash_slots;
    const uint32_t nbk = (uint32_t)cap / 4u;  // buckets of a lane's table
    double *vals = (double *)smem;
    int32_t *keys = (int32_t *)(smem + (size_t)H * 8u);
    int *spill_cnt = (int *)(smem + (size_t)H * 12u);
    double *lv = (double *)(smem + (size_t)H * 12u + 16u);  // [slot][lane]
    i32x4v *lk = (i32x4v *)(smem + (size_t)H * 12u + 16u + (size_t)cap * 64u * 8u);  // [bucket][lane]
    const uint32_t smask = (uint32_t)a.spill_slots - 1u;
    const i32x4v none = {kEmpty, kEmpty, kEmpty, kEmpty};
    for (int s = lane; s < H; s += 64) {
        keys[s] = kEmpty;
        vals[s] = 0.0;
    }
    for (int s = 0; s < cap; ++s) lv[s * 64 + lane] = 0.0;
    for (uint32_t b = 0; b < nbk; ++b) lk[b * 64u + lane] = none;
    if (lane == 0) *spill_cnt = 0;
    wave_sync();
    int32_t *skeys = a.spill_keys + (int64_t)blockIdx.x * a.spill_slots;
    double *svals = a.spill_vals + (int64_t)blockIdx.x * a.spill_slots;
    int32_t *sused = a.spill_used + (int64_t)blockIdx.x * a.spill_slots;
    int queue = (int)(blockIdx.x & 7u);
    const uint32_t tag = a.tag | 0x80000000u;
    for (;;) {
        int64_t task = -1;
        if (lane == 0) {
            for (int tries = 0; tries < 8; ++tries) {
                const int q = (queue + tries) & 7;
                const int64_t lo = a.n_tasks * q / 8, hi = a.n_tasks * (q + 1) / 8;
                if (hi > lo && __atomic_load_n(&a.queue_ctr[q * kQueueStride], __ATOMIC_RELAXED) < (uint32_t)(hi - lo)) {
                    const uint32_t idx = atomicAdd(&a.queue_ctr[q * kQueueStride], 1u);
                    if ((int64_t)idx < hi - lo) {
                        task = lo + idx;
                        queue = q;
                        break;
                    }
                }
            }
        }
        task = __shfl(task, 0, 64);
        queue = __shfl(queue, 0, 64);
        if (task < 0) break;
        const int32_t r = (int32_t)task;
        const uint32_t r_off = a.roff[r];
        int32_t c = lane;
        bool active = c < pilot;
        uint32_t off = r_off, j = 0;
        double w64 = 1.0;
        float w32 = 1.0f;
        u32x4 blk = {0, 0, 0, 0};
        StepHdr H0;
        if (kF32)
            load_header_c(a.rec32, r_off, H0);
        else
            load_header<false>(a.rec, r_off, H0);
        StepHdr Hd = H0;  // header of the current state
        bool overflow = false, spill_full = false;
        double sq = 0.0;
        unsigned long long steps = 0;
        auto flush = [&]() {
#pragma unroll 8
            for (int q = 0; q < cap; ++q) {
                const double x = lv[q * 64 + lane];
                sq += x * x;
                lv[q * 64 + lane] = 0.0;
            }
            for (uint32_t q = 0; q < nbk; ++q) lk[q * 64u + lane] = none;
        };
        while (active) {
            const uint4 h = Hd.h0;
            const double s64 = kF32 ? 0.0 : header_shat64(Hd);
            const int32_t key = (int32_t)h.x;
            const double w = kF32 ? (double)w32 : w64;
            bool stop = (h.y == 0u) || (j >= (uint32_t)a.lmax);
            double wn64 = 0.0;
            float wn32 = 0.0f;
            if (kF32) {
                wn32 = w32 * __uint_as_float(h.w);
                stop = stop || (fabsf(wn32) < a.delta32);
            } else {
                wn64 = w64 * s64;
                stop = stop || (fabs(wn64) < a.delta);
            }
            BucketLd bl;
            if (!stop) {
                if ((j & 3u) == 0u) blk = philox4x32_10(j >> 2, (uint32_t)c, (uint32_t)r, tag, a.key0, a.key1);
                const uint32_t u = blk.x;
                blk.x = blk.y;
                blk.y = blk.z;
                blk.z = blk.w;
                if (kF32)
                    bucket_issue_c(a.rec32, off, Hd, u, bl);
                else
                    bucket_issue<false>(a.rec, off, Hd, u, bl);
            }
            // contribution (j = 0 included: the start state gets W_0 = 1)
            const uint32_t rb = Probe<true, true, false>::home(key, (uint32_t)H, a.hash_shift);
            uint32_t pb = __umulhi((uint32_t)key * 0x9E3779B1u, nbk);
            int32_t rk[4];
            read_bucket_wave(keys, rb, rk);
            i32x4v pv = lk[pb * 64u + lane];
            if (!Probe<true, true, false>::add(keys, vals, (uint32_t)H, rb, rk, key, w))
                if (!spill_add(skeys, svals, sused, spill_cnt, smask, key, w)) spill_full = true;
            uint32_t tries = 0;
#pragma unroll 1
            for (;;) {
                const int32_t pk[4] = {pv.x, pv.y, pv.z, pv.w};
                const int s = pick_slot(pk, key);
                if (s < 4) {
                    ((int32_t *)&lk[pb * 64u + lane])[s] = key;
                    atomicAdd(&lv[(pb * 4u + s) * 64u + lane], w);
                    break;
                }
                if (++tries == nbk) {
                    overflow = true;
                    break;
                }
                pb = pb + 1u == nbk ? 0u : pb + 1u;
                pv = lk[pb * 64u + lane];
            }
            if (stop) {
                steps += j;
                c += 64;
                if (c < pilot) {
                    // ||X_c||^2 now, as the lane's table serves its next chain (a lane's
                    // last chain waits for the others: chains stop in many different steps)
                    flush();
                    off = r_off;
                    Hd = H0;
                    j = 0;
                    w64 = 1.0;
                    w32 = 1.0f;
                } else {
                    active = false;
                }
            } else {
                StepHdr Nx;
                const uint32_t tgt = kF32 ? bucket_resolve_c(bl, Nx) : bucket_resolve<false>(bl, Nx);
                const bool neg = (tgt & kSignBit) != 0u;
                if (kF32)
                    w32 = neg ? -wn32 : wn32;
                else
                    w64 = neg ? -wn64 : wn64;
                off = tgt & ~kSignBit;
                Hd = Nx;
                ++j;
            }
        }
        flush();
        wave_sync();
        // ||mean||^2 over the row hash and the spilled columns
        const double P = (double)pilot;
        double msq = 0.0;
        for (int s = lane; s < H; s += 64) {
            if (keys[s] != kEmpty) {
                const double mu = vals[s] / P;
                msq += mu * mu;
            }
        }
        const int nsp = *spill_cnt;
        for (int u = lane; u < nsp; u += 64) {
            const int32_t sl = sused[u];
            const double mu = svals[sl] / P;
            msq += mu * mu;
            skeys[sl] = kEmpty;
            svals[sl] = 0.0;
        }
        msq = wave_sum(msq);
        sq = wave_sum(sq);
        steps = wave_sum(steps);
        const bool bad_cap = __any(overflow), bad_spill = __any(spill_full);
        if (lane == 0) {
            var[r] = sq / P - msq;
            len[r] = (double)steps / P;
            if (bad_cap) atomicOr(a.flags, kFlagStage);
            if (bad_spill) atomicOr(a.flags, kFlagSpill);
        }
        wave_sync();
        for (int s = lane; s < H; s += 64) {
            keys[s] = kEmpty;
            vals[s] = 0.0;
        }
        if (lane == 0) *spill_cnt = 0;
        wave_sync();
    }
}

// Neyman allocation target of each row: minimising sum_r v_r / N_r under
// sum_r N_r (len_r + 1) = T gives N_r proportional to sqrt(v_r / (len_r + 1)), so
// the network regresses y_r = (ln v_r - ln(len_r + 1)) / 2 (v floored at 1e-30 so
// that rows with a deterministic chain get a finite, very small share).
__global__ void __launch_bounds__(256) k_neyman_target(int64_t n, const double *__restrict__ var,
                                                       const double *__restrict__ len, float *__restrict__ y) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
        const double v = var[r] > 1e-30 ? var[r] : 1e-30;
        y[r] = (float)(0.5 * (log(v) - log(len[r] + 1.0)));
    }
}

// Budget units of one chain of each row: the states it visits when every row on
// its path has the row's own |C| row sum, 1 + floor(f7) (f7 = min(L_max,
// ln delta / ln S), the feature the network also sees); exact for matrices with
// equal row sums. Partial sums of the costs per workgroup, in 64-bit integers.
__global__ void __launch_bounds__(256) k_chain_cost(int64_t n, const float *__restrict__ feat,
                                                    int32_t *__restrict__ cost,
                                                    unsigned long long *__restrict__ total) {
    __shared__ unsigned long long red[4];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    unsigned long long sum = 0;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
        const float f7 = feat[8 * r + 7];
        const int32_t c = 1 + (int32_t)floorf(f7 > 0.f ? f7 : 0.f);
        cost[r] = c;
        sum += (unsigned long long)c;
    }
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(total, red[0] + red[1] + red[2] + red[3]);
}

}  // namespace

template <int P>
hipError_t launch_features_p(const mcmi_cdf *cdf, double delta, int lmax, float *feat, hipStream_t s) {
    int64_t blocks = (cdf->n * P + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    k_features<P><<<(unsigned)blocks, 256, 0, s>>>(cdf->n, cdf->rec32, cdf->roff, delta, lmax, feat);
    return hipGetLastError();
}

hipError_t launch_features(const mcmi_cdf *cdf, double delta, int lmax, float *feat, hipStream_t s) {
    const double per_row = cdf->n > 0 ? (double)cdf->nnz_c / (double)cdf->n : 0.0;
    if (per_row <= 10.0) return launch_features_p<4>(cdf, delta, lmax, feat, s);
    if (per_row <= 40.0) return launch_features_p<16>(cdf, delta, lmax, feat, s);
    return launch_features_p<64>(cdf, delta, lmax, feat, s);
}

size_t pilot_lds_bytes(int hash_slots, int cap) { return (size_t)hash_slots * 12u + 16u + (size_t)cap * 64u * 12u; }

hipError_t launch_pilot(const WalkArgs &a, bool f32, int pilot, int cap, int blocks, double *var, double *len,
                        hipStream_t s) {
    const size_t lds = pilot_lds_bytes(a.hash_slots, cap);
    if (f32)
        k_pilot<true><<<blocks, 64, lds, s>>>(a, pilot, cap, var, len);
    else
        k_pilot<false><<<blocks, 64, lds, s>>>(a, pilot, cap, var, len);
    return hipGetLastError();
}

hipError_t pilot_occupancy(bool f32, int hash_slots, int cap, int *bpc) {
    const size_t lds = pilot_lds_bytes(hash_slots, cap);
    if (f32) return hipOccupancyMaxActiveBlocksPerMultiprocessor(bpc, k_pilot<true>, 64, lds);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(bpc, k_pilot<false>, 64, lds);
}

}  // namespace mcmi

// ------------------------------------------------------------------ C ABI
using namespace mcmi;

extern "C" mcmi_status mcmi_row_features(const mcmi_cdf *cdf, double delta, int32_t max_len, float *feat_dev,
                                         void *stream) {
    if (!cdf || !feat_dev) return fail(MCMI_ERR_ARG, "mcmi_row_features: null argument");
    if (!(delta >= 0.0) || max_len < 0) return fail(MCMI_ERR_ARG, "mcmi_row_features: bad delta / max_len");
    int lmax = derive_lmax(cdf->norm_inf, delta, max_len);
    if (lmax < 0) lmax = max_len;  // not contractive and no max_len: f7 uses 0
    MCMI_HIP(launch_features(cdf, delta, lmax, feat_dev, (hipStream_t)stream));
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_pilot_variance(const mcmi_cdf *cdf, const mcmi_params *p, int32_t pilot_chains,
                                           double *var_dev, double *len_dev, void *stream) {
    if (!cdf || !p || !var_dev || !len_dev) return fail(MCMI_ERR_ARG, "mcmi_pilot_variance: null argument");
    if (pilot_chains < 1) return fail(MCMI_ERR_ARG, "mcmi_pilot_variance: pilot_chains must be >= 1");
    if (p->walk_prec != MCMI_WALK_F64 && p->walk_prec != MCMI_WALK_F32)
        return fail(MCMI_ERR_ARG, "mcmi_pilot_variance: walk_prec must be 64 or 32");
    const int lmax = derive_lmax(cdf->norm_inf, p->delta, p->max_len);
    if (lmax < 0) return fail(lmax == (int)MCMI_ERR_NOT_CONTRACTIVE ? MCMI_ERR_NOT_CONTRACTIVE : MCMI_ERR_ARG,
                              "mcmi_pilot_variance: ||Chat||_inf >= 1 needs max_len, or bad delta");
    hipStream_t s = (hipStream_t)stream;
    const bool f32 = p->walk_prec == MCMI_WALK_F32;
    int H = 1024, cap = lmax + 1 < 48 ? (lmax + 4) / 4 * 4 : 48, spill_slots = 4096;
    unsigned char *ctrl = nullptr;
    int32_t *sk = nullptr, *su = nullptr;
    double *sv = nullptr;
    const size_t ctrl_bytes = kCtrlBytes;
    auto cleanup = [&]() {
        for (void *t : {(void *)ctrl, (void *)sk, (void *)sv, (void *)su})
            if (t) dev_release(t, s);  // behind the last kernel that uses them
        ctrl = nullptr;
        sk = su = nullptr;
        sv = nullptr;
    };
    // FP64 pilot walks read the full records: build them before the arguments take their address
    if (!f32) {
        const hipError_t fe = ensure_full_records(cdf, s);
        if (fe != hipSuccess) return fail(MCMI_ERR_HIP, std::string("mcmi_pilot_variance: ") + hipGetErrorString(fe));
    }
    for (int attempt = 0; attempt < 6; ++attempt) {
        int bpc = 0;
        hipError_t e = pilot_occupancy(f32, H, cap, &bpc);
        if (e != hipSuccess || bpc < 1) {
            cleanup();
            return fail(MCMI_ERR_CAPACITY, "mcmi_pilot_variance: per-chain state lists do not fit in LDS");
        }
        const int64_t blocks = std::min<int64_t>((int64_t)bpc * device_cus(), cdf->n);
#define TRYP(call)                                                                              \
    do {                                                                                        \
        hipError_t _e = (call);                                                                 \
        if (_e != hipSuccess) {                                                                 \
            cleanup();                                                                          \
            return fail(MCMI_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(_e));       \
        }                                                                                       \
    } while (0)
        TRYP(dev_alloc((void **)&ctrl, ctrl_bytes, s));
        TRYP(dev_alloc((void **)&sk, (size_t)blocks * spill_slots * 4, s));
        TRYP(dev_alloc((void **)&sv, (size_t)blocks * spill_slots * 8, s));
        TRYP(dev_alloc((void **)&su, (size_t)blocks * spill_slots * 4, s));
        TRYP(hipMemsetAsync(ctrl, 0, ctrl_bytes, s));
        TRYP(hipMemsetAsync(sk, 0xFF, (size_t)blocks * spill_slots * 4, s));
        TRYP(hipMemsetAsync(sv, 0, (size_t)blocks * spill_slots * 8, s));
        WalkArgs a;
        memset(&a, 0, sizeof(a));
        a.rec = cdf->rec;
        a.rec32 = cdf->rec32;
        a.roff = cdf->roff;
        a.diag = cdf->diag;
        a.n_tasks = cdf->n;
        a.key0 = (uint32_t)(p->seed & 0xffffffffu);
        a.key1 = (uint32_t)(p->seed >> 32);
        a.tag = p->stream_tag;
        a.delta = p->delta;
        a.delta32 = (float)p->delta;
        a.lmax = lmax;
        a.hash_slots = H;
        a.hash_shift = 32 - __builtin_ctz((unsigned)H);
        a.queue_ctr = (uint32_t *)ctrl;
        a.stats = (unsigned long long *)(ctrl + kCtrlStats);
        a.flags = (uint32_t *)(ctrl + kCtrlFlags);
        a.spill_keys = sk;
        a.spill_vals = sv;
        a.spill_used = su;
        a.spill_slots = spill_slots;
        TRYP(launch_pilot(a, f32, pilot_chains, cap, (int)blocks, var_dev, len_dev, s));
        uint32_t hflags = 0;
        TRYP(hipMemcpyAsync(&hflags, a.flags, sizeof(hflags), hipMemcpyDeviceToHost, s));
        TRYP(hipStreamSynchronize(s));
#undef TRYP
        cleanup();
        if (!(hflags & (kFlagStage | kFlagSpill))) return MCMI_OK;
        if (hflags & kFlagStage) {
            if (cap >= lmax + 1 || cap >= 160) return fail(MCMI_ERR_CAPACITY, "mcmi_pilot_variance: state list overflow");
            cap = cap * 2 < lmax + 1 ? cap * 2 : (lmax + 4) / 4 * 4;  // whole buckets of four
            if (cap > 160) cap = 160;
        }
        if (hflags & kFlagSpill) spill_slots *= 4;
    }
    return fail(MCMI_ERR_CAPACITY, "mcmi_pilot_variance: tables still overflow");
}

extern "C" mcmi_status mcmi_neyman_target(const double *var_dev, const double *len_dev, int64_t n, float *y_dev,
                                          void *stream) {
    if (n < 0 || (n > 0 && (!var_dev || !len_dev || !y_dev)))
        return fail(MCMI_ERR_ARG, "mcmi_neyman_target: bad argument");
    if (n == 0) return MCMI_OK;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    k_neyman_target<<<(unsigned)blocks, 256, 0, (hipStream_t)stream>>>(n, var_dev, len_dev, y_dev);
    MCMI_HIP(hipGetLastError());
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_chain_cost(const float *feat_dev, int64_t n, int32_t *cost_dev, int64_t *total_host,
                                       void *stream) {
    if (n < 0 || (n > 0 && (!feat_dev || !cost_dev)))
        return fail(MCMI_ERR_ARG, "mcmi_chain_cost: bad argument");
    if (total_host) *total_host = 0;
    if (n == 0) return MCMI_OK;
    if (n > (int64_t)INT32_MAX * 4) return fail(MCMI_ERR_ARG, "mcmi_chain_cost: too many rows");
    hipStream_t s = (hipStream_t)stream;
    unsigned long long *tot = nullptr;
    MCMI_HIP(hipMallocAsync((void **)&tot, sizeof(unsigned long long), s));
    hipError_t e = hipMemsetAsync(tot, 0, sizeof(unsigned long long), s);
    // one atomic per workgroup on one address: 512 workgroups (1M rows: 4096 took 53 us)
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 512);
    if (e == hipSuccess) {
        k_chain_cost<<<(unsigned)blocks, 256, 0, s>>>(n, feat_dev, cost_dev, tot);
        e = hipGetLastError();
    }
    unsigned long long h = 0;
    if (e == hipSuccess && total_host) e = hipMemcpyAsync(&h, tot, sizeof(h), hipMemcpyDeviceToHost, s);
    const hipError_t ef = hipFreeAsync(tot, s);
    if (e == hipSuccess) e = ef;
    if (e == hipSuccess && total_host) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(MCMI_ERR_HIP, std::string("mcmi_chain_cost: ") + hipGetErrorString(e));
    if (total_host) *total_host = (int64_t)h;
    return MCMI_OK;
}
