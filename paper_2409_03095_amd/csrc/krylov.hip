// BiCGstab on the device around the sparse approximate inverse (gfx950).
//
// The paper uses M directly as a preconditioner of a Krylov solver (Section III-B,
// last paragraph; the solver experiments of Section VI). This is van der Vorst's
// BiCGstab with M applied on the right (solve B M y = b, x = M y): every step
// applies B and M once per half step (CSR SpMV), and each vector update also forms
// the partial sums of the inner products that follow it, which the last workgroup to
// arrive adds in index order (a fixed order: reruns give the same iterates). That
// workgroup then forms the step's scalars on the device, so an iteration is 7 launches (9
// with M) with no host round trip in it; every kernel returns at once when the
// solve has ended. The host queues up to kAhead iterations ahead and reads the status word
// that the last launch of an iteration leaves in host memory. On a 100 x 77 5-point
// grid (45 iterations) an inner product's two launches, copy and wait, six times
// per iteration, took 7.6 of 7.7 ms.
#include <math.h>
#include <string.h>

#include <mutex>
#include <string>
#include <vector>

#include "common.hpp"

namespace mcmi {
hipError_t spmv(int64_t n, int64_t nnz, const int64_t *rp, const int32_t *ci, const double *v, const double *x,
                double *y, const int32_t *stop, hipStream_t s);

namespace {

constexpr int kDotBlocks = 1024;  // most workgroups of an inner product
constexpr int kAhead = 3;         // iterations queued past the one whose status is read

enum Status : int32_t { kRun = 0, kConverged = 1, kHalf = 2, kBreakdown = 3, kZeroRhs = 4 };

// Scalars of a solve (device memory).
struct KState {
    int32_t status;  // kHalf: converged in the half step, x not yet updated
    uint32_t arrived;
    int64_t it, maxiter;
    double rtol, bnrm, rr, ss, rho, alpha, beta, omega;
};

// The workgroup's sums of acc[0 .. K) into part[k kDotBlocks + block]; true in the last
// workgroup of the grid, with the totals in tot (all threads), each added over
// the blocks in a fixed order.
template <int K>
__device__ __forceinline__ bool finish_sums(const double (&acc)[K], double *part, KState *st, double (&tot)[K]) {
    __shared__ double red[K][4];
    __shared__ int last;
    const int t = threadIdx.x, w = t >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double a = wave_sum(acc[k]);
        if ((t & 63) == 0) red[k][w] = a;
    }
    __syncthreads();
    if (t == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            __hip_atomic_store(part + k * kDotBlocks + blockIdx.x,
                               (red[k][0] + red[k][1]) + (red[k][2] + red[k][3]), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        last = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
               gridDim.x - 1u;
    }
    __syncthreads();
    if (!last) return false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double a = 0.0;
        for (int i = t; i < (int)gridDim.x; i += 256)
            a += __hip_atomic_load(part + k * kDotBlocks + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a = wave_sum(a);
        if ((t & 63) == 0) red[k][w] = a;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) tot[k] = (red[k][0] + red[k][1]) + (red[k][2] + red[k][3]);
    if (t == 0) st->arrived = 0u;
    return true;
}

// ||b||, and the solve's constants
__global__ void __launch_bounds__(256) k_norm_b(int64_t n, const double *__restrict__ b, double rtol, int64_t maxiter,
                                                double *part, KState *st) {
    double acc[1] = {0.0}, tot[1];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) acc[0] += b[i] * b[i];
    if (!finish_sums<1>(acc, part, st, tot) || threadIdx.x != 0) return;
    st->bnrm = sqrt(tot[0]);
    st->rtol = rtol;
    st->maxiter = maxiter;
    st->it = 0;
    st->alpha = st->omega = 1.0;
    st->beta = 0.0;
}

// r = b - y, rhat = r; ||r||^2
__global__ void __launch_bounds__(256) k_residual(int64_t n, const double *__restrict__ b,
                                                  const double *__restrict__ y, double *__restrict__ r,
                                                  double *__restrict__ rhat, double *part, KState *st) {
    double acc[1] = {0.0}, tot[1];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double v = b[i] - y[i];
        r[i] = v;
        rhat[i] = v;
        acc[0] += v * v;
    }
    if (!finish_sums<1>(acc, part, st, tot) || threadIdx.x != 0) return;
    st->rr = tot[0];
    st->rho = tot[0];  // rhat . r
    if (st->bnrm == 0.0)
        st->status = kZeroRhs;
    else if (sqrt(tot[0]) <= st->rtol * st->bnrm)
        st->status = kConverged;
}

// p = r + beta (p - omega v) (p = r in the first iteration); x = 0 when b = 0
__global__ void __launch_bounds__(256) k_dir(int64_t n, const double *__restrict__ r, const double *__restrict__ v,
                                             double *__restrict__ p, double *__restrict__ x,
                                             const KState *__restrict__ st) {
    const int32_t status = st->status;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (status == kZeroRhs)
        for (int64_t i = i0; i < n; i += stride) x[i] = 0.0;
    if (status != kRun) return;
    if (st->it == 0) {
        for (int64_t i = i0; i < n; i += stride) p[i] = r[i] + 0.0;
        return;
    }
    const double beta = st->beta, omega = st->omega;
    for (int64_t i = i0; i < n; i += stride) p[i] = r[i] + beta * (p[i] - omega * v[i]);
}

// alpha = rho / (rhat . v)
__global__ void __launch_bounds__(256) k_alpha(int64_t n, const double *__restrict__ rhat,
                                               const double *__restrict__ v, double *part, KState *st) {
    if (st->status != kRun) return;
    double acc[1] = {0.0}, tot[1];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) acc[0] += rhat[i] * v[i];
    if (!finish_sums<1>(acc, part, st, tot) || threadIdx.x != 0) return;
    st->it += 1;
    if (tot[0] == 0.0)
        st->status = kBreakdown;
    else
        st->alpha = st->rho / tot[0];
}

// s = r - alpha v; ||s||^2
__global__ void __launch_bounds__(256) k_half(int64_t n, const double *__restrict__ r, const double *__restrict__ v,
                                              double *__restrict__ sv, double *part, KState *st) {
    if (st->status != kRun) return;
    const double a = -st->alpha;
    double acc[1] = {0.0}, tot[1];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double s = r[i] + a * v[i];
        sv[i] = s;
        acc[0] += s * s;
    }
    if (!finish_sums<1>(acc, part, st, tot) || threadIdx.x != 0) return;
    st->ss = tot[0];
    if (sqrt(tot[0]) <= st->rtol * st->bnrm) st->status = kHalf;
}

// omega = (t . s) / (t . t)
__global__ void __launch_bounds__(256) k_omega(int64_t n, const double *__restrict__ t, const double *__restrict__ sv,
                                               double *part, KState *st) {
    if (st->status != kRun) return;
    double acc[2] = {0.0, 0.0}, tot[2];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double ti = t[i];
        acc[0] += ti * sv[i];
        acc[1] += ti * ti;
    }
    if (!finish_sums<2>(acc, part, st, tot) || threadIdx.x != 0) return;
    if (tot[1] == 0.0)
        st->status = kBreakdown;
    else
        st->omega = tot[0] / tot[1];
}

// x += alpha phat + omega shat, r = s - omega t; ||r||^2 and rhat . r. After a converged
// half step only x += alpha phat. The last launch of an iteration: it leaves the
// status in host memory.
__global__ void __launch_bounds__(256) k_step(int64_t n, const double *__restrict__ phat,
                                              const double *__restrict__ shat, const double *__restrict__ sv,
                                              const double *__restrict__ t, const double *__restrict__ rhat,
                                              double *__restrict__ x, double *__restrict__ r, double *part, KState *st,
                                              int32_t *host_status) {
    const int32_t status = st->status;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double acc[2] = {0.0, 0.0}, tot[2];
    if (status == kHalf) {
        const double alpha = st->alpha;
        for (int64_t i = i0; i < n; i += stride) x[i] = x[i] + alpha * phat[i];
        if (!finish_sums<2>(acc, part, st, tot) || threadIdx.x != 0) return;
        st->rr = st->ss;
        st->status = kConverged;
        __hip_atomic_store(host_status, (int32_t)kConverged, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    if (status != kRun) {
        if (i0 == 0) __hip_atomic_store(host_status, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    const double alpha = st->alpha, omega = st->omega;
    for (int64_t i = i0; i < n; i += stride) {
        x[i] = x[i] + alpha * phat[i] + omega * shat[i];
        const double ri = sv[i] - omega * t[i];
        r[i] = ri;
        acc[0] += ri * ri;
        acc[1] += rhat[i] * ri;
    }
    if (!finish_sums<2>(acc, part, st, tot) || threadIdx.x != 0) return;
    st->rr = tot[0];
    int32_t now = kRun;
    if (sqrt(tot[0]) <= st->rtol * st->bnrm) {
        now = kConverged;
    } else if (omega == 0.0) {
        now = kBreakdown;
    } else {
        const double rho_prev = st->rho, rho = tot[1];
        st->rho = rho;
        st->beta = (rho / rho_prev) * (alpha / omega);
        if (rho == 0.0 && st->it < st->maxiter) {  // found at the start of the next iteration
            st->it += 1;
            now = kBreakdown;
        }
    }
    if (now != kRun) {
        st->status = now;
        __hip_atomic_store(host_status, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

unsigned grid_dot(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b > kDotBlocks) b = kDotBlocks;
    return (unsigned)(b < 1 ? 1 : b);
}

// Status words in host memory that kernels write: a few are kept for later solves.
struct StatusWords {
    std::mutex mu;
    std::vector<int32_t *> idle;
};
StatusWords &status_words() {
    static StatusWords *w = new StatusWords();  // never destroyed: the driver may be gone at exit
    return *w;
}
hipError_t take_status(int32_t **p) {
    StatusWords &w = status_words();
    {
        std::lock_guard<std::mutex> lk(w.mu);
        if (!w.idle.empty()) {
            *p = w.idle.back();
            w.idle.pop_back();
            return hipSuccess;
        }
    }
    return hipHostMalloc((void **)p, 64, hipHostMallocPortable | hipHostMallocMapped);
}
void give_status(int32_t *p) {
    if (!p) return;
    StatusWords &w = status_words();
    {
        std::lock_guard<std::mutex> lk(w.mu);
        if (w.idle.size() < 8) {
            w.idle.push_back(p);
            return;
        }
    }
    (void)hipHostFree(p);
}

}  // namespace
}  // namespace mcmi

using namespace mcmi;

extern "C" mcmi_status mcmi_bicgstab(const mcmi_csr_in *B, const mcmi_csr_out *M, const double *b_dev, double *x_dev,
                                     double rtol, int32_t maxiter, mcmi_solve_stats *st, void *stream) {
    if (st) ::memset(st, 0, sizeof(*st));
    if (!B || !b_dev || !x_dev || !(rtol > 0.0) || maxiter < 1)
        return fail(MCMI_ERR_ARG, "mcmi_bicgstab: need B, b, x, rtol > 0 and maxiter >= 1");
    if (B->n <= 0 || !B->row_ptr_dev || !B->col_dev || !B->val_dev)
        return fail(MCMI_ERR_ARG, "mcmi_bicgstab: bad B");
    if (M && (M->n != B->n || !M->row_ptr_dev)) return fail(MCMI_ERR_ARG, "mcmi_bicgstab: M must be n x n");
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = B->n;
    hipEvent_t e0 = nullptr, e1 = nullptr, ev[kAhead + 1] = {};
    double *w = nullptr;
    int32_t *status = nullptr;
    const size_t vec = (size_t)n * sizeof(double);
    KState h;
    ::memset(&h, 0, sizeof(h));
    hipError_t err = hipSuccess;
    auto ok = [&err](hipError_t e) { return (err = e) == hipSuccess; };
    auto solve = [&]() -> bool {
        if (!ok(hipEventCreate(&e0)) || !ok(hipEventCreate(&e1))) return false;
        for (hipEvent_t &e : ev)
            if (!ok(hipEventCreateWithFlags(&e, hipEventDisableTiming))) return false;
        if (!ok(take_status(&status))) return false;
        *(volatile int32_t *)status = kRun;
        void *sdev = nullptr;
        if (!ok(hipHostGetDevicePointer(&sdev, status, 0))) return false;
        int32_t *status_dev = (int32_t *)sdev;
        if (!ok(dev_alloc((void **)&w, 8 * vec + 2 * kDotBlocks * sizeof(double) + sizeof(KState), s))) return false;
        double *r = w, *rhat = w + n, *p = w + 2 * n, *v = w + 3 * n, *sv = w + 5 * n, *t = w + 7 * n;
        // without M, phat = p and shat = s
        double *phat = M ? w + 4 * n : p, *shat = M ? w + 6 * n : sv;
        double *part = w + 8 * n;
        KState *st_dev = (KState *)(part + 2 * kDotBlocks);
        const int32_t *stop = &st_dev->status;
        const unsigned g = grid_dot(n);
        auto applyB = [&](const double *x, double *y) {
            return ok(spmv(n, B->nnz, B->row_ptr_dev, B->col_dev, B->val_dev, x, y, stop, s));
        };
        auto applyM = [&](const double *x, double *y) {
            return !M || ok(spmv(n, M->nnz, M->row_ptr_dev, M->col_dev, M->val_dev, x, y, stop, s));
        };
        if (!ok(hipEventRecord(e0, s))) return false;
        if (!ok(hipMemsetAsync(st_dev, 0, sizeof(KState), s))) return false;
        k_norm_b<<<g, 256, 0, s>>>(n, b_dev, rtol, maxiter, part, st_dev);
        if (!applyB(x_dev, v)) return false;
        k_residual<<<g, 256, 0, s>>>(n, b_dev, v, r, rhat, part, st_dev);
        for (int64_t it = 1; it <= maxiter; ++it) {
            k_dir<<<g, 256, 0, s>>>(n, r, v, p, x_dev, st_dev);
            if (!applyM(p, phat) || !applyB(phat, v)) return false;
            k_alpha<<<g, 256, 0, s>>>(n, rhat, v, part, st_dev);
            k_half<<<g, 256, 0, s>>>(n, r, v, sv, part, st_dev);
            if (!applyM(sv, shat) || !applyB(shat, t)) return false;
            k_omega<<<g, 256, 0, s>>>(n, t, sv, part, st_dev);
            k_step<<<g, 256, 0, s>>>(n, phat, shat, sv, t, rhat, x_dev, r, part, st_dev, status_dev);
            if (!ok(hipGetLastError())) return false;
            if (!ok(hipEventRecord(ev[it % (kAhead + 1)], s))) return false;
            if (it > kAhead && !ok(hipEventSynchronize(ev[(it - kAhead) % (kAhead + 1)]))) return false;
            if (*(volatile int32_t *)status != kRun) break;
        }
        if (!ok(hipEventRecord(e1, s))) return false;
        if (!ok(hipMemcpyAsync(&h, st_dev, sizeof(h), hipMemcpyDeviceToHost, s))) return false;
        return ok(hipStreamSynchronize(s));
    };
    const bool done = solve();
    float ms = 0.f;
    if (done)
        (void)hipEventElapsedTime(&ms, e0, e1);
    else
        (void)hipStreamSynchronize(s);  // nothing may still write the status word or the workspace
    if (w) dev_release(w, s);
    give_status(status);
    for (hipEvent_t e : {e0, e1, ev[0], ev[1], ev[2], ev[3]})
        if (e) (void)hipEventDestroy(e);
    if (!done) return fail(MCMI_ERR_HIP, std::string("mcmi_bicgstab: ") + hipGetErrorString(err));
    if (st) {
        st->iterations = h.it;
        st->rel_residual = h.bnrm > 0.0 ? sqrt(h.rr) / h.bnrm : 0.0;
        st->ms = ms;
        st->converged = h.status == kConverged || h.status == kZeroRhs;
    }
    return MCMI_OK;
}
