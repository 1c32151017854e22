// BiCGstab on the device around the sparse approximate inverse (gfx950).
//
// The paper uses M directly as a preconditioner of a Krylov solver (Section III-B,
// last paragraph; the solver experiments of Section VI). This is van der Vorst's
// BiCGstab with M applied on the right (solve B M y = b, x = M y): every step
// applies B and M once per half step (CSR SpMV), and each vector update also forms
// the workgroups' partial sums of the inner products that follow it. The kernel that needs
// such a product adds the partials itself, in every workgroup (in a fixed order: reruns
// give the same iterates) and forms the step's scalars from it, so an iteration is 7
// launches (9 with M) with no host round trip, and no workgroup waits for another;
// workgroup 0 keeps the scalars that later kernels read. Every kernel returns at once when
// the solve has ended. The host queues up to kAhead iterations ahead and reads the status and
// the iteration that launches leave in host memory. A 100 x 77 5-point grid (45 iterations)
// took 7.4 ms with two launches, a copy and a wait per inner product, 1.44 ms with the
// partials added by the last workgroup to arrive, and takes 1.27 to 1.4 ms so; a 64^3 27-point
// stencil with its M (1024 partials to a product) took 2.9 / 1.73 / 1.0 ms.
#include <math.h>
#include <string.h>

#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "common.hpp"

namespace mcmi {
hipError_t spmv(int64_t n, int64_t nnz, const int64_t *rp, const int32_t *ci, const double *v, const double *x,
                double *y, const int32_t *stop, hipStream_t s);

namespace {

constexpr int kDotBlocks = 1024;  // most workgroups of an inner product
constexpr int kAhead = 3;         // iterations queued past the last that has ended
// The host waits for the stream every kRetire iterations, and the runtime retires the launches
// so far; some hundred left to the end of the call slowed the caller's next 0.5 ms of host
// work by 0.3 ms. 100 x 77 grid, time of the solve and of that host work (0.47 ms by itself): an
// event per iteration 1.64 and 0.77 ms, host memory read instead 1.40 and 0.76, with a wait
// every 8 iterations 1.38 and 0.51, every 16 1.17 to 1.35 and 0.50 to 0.62.
constexpr int kRetire = 8;

// kHalf: converged in the half step of iteration half_it, whose last launch updates x
enum Status : int32_t { kRun = 0, kConverged = 1, kHalf = 2, kBreakdown = 3, kZeroRhs = 4 };

// Scalars of a solve (device memory), written by workgroup 0. A kernel reads none that it
// writes, but for the status, whose late readers only return early where all do: rho of
// an iteration is kept under its parity.
struct KState {
    int32_t status, pad;
    int64_t it, half_it;
    double bnrm, rr, alpha, omega, rho[2];
};

// Partial sums, kDotBlocks per inner product.
enum Part { kBB = 0, kRR = 1, kRhatR = 2, kRhatV = 3, kSS = 4, kTS = 5, kTT = 6, kParts = 7 };

struct Scalars {
    KState *st;
    double *part;
    int32_t *host_status;  // in host memory: the status, then the iteration that has begun
    double rtol;
};

// the workgroup's sum of acc into its place of product `which`
__device__ __forceinline__ void put_partial(const Scalars &c, int which, double acc) {
    __shared__ double red[4];
    acc = wave_sum(acc);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) c.part[which * kDotBlocks + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// the whole product, in every thread (all the solve's kernels have the same grid)
__device__ __forceinline__ double total(const Scalars &c, int which) {
    __shared__ double red[4];
    double a = 0.0;
    for (int i = threadIdx.x; i < (int)gridDim.x; i += 256) a += c.part[which * kDotBlocks + i];
    a = wave_sum(a);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

__device__ __forceinline__ bool first_thread() { return blockIdx.x == 0 && threadIdx.x == 0; }

// The status, the same in all of a workgroup's waves, for the kernels in which workgroup 0
// may end the solve: waves that read it one by one could return in part, and the others
// would then add up sums that the missing waves have not written.
__device__ __forceinline__ int32_t group_status(const Scalars &c) {
    __shared__ int32_t status;
    if (threadIdx.x == 0) status = c.st->status;
    __syncthreads();
    return status;
}

// (workgroup 0) the solve ends with `status` after `it` iterations
__device__ __forceinline__ void end_solve(const Scalars &c, int32_t status, int64_t it) {
    c.st->it = it;
    c.st->status = status;
    __hip_atomic_store(c.host_status, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// b . b
__global__ void __launch_bounds__(256) k_norm_b(int64_t n, const double *__restrict__ b, Scalars c) {
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) acc += b[i] * b[i];
    put_partial(c, kBB, acc);
}

// r = b - y, rhat = r; ||r||^2 (and rhat . r)
__global__ void __launch_bounds__(256) k_residual(int64_t n, const double *__restrict__ b,
                                                  const double *__restrict__ y, double *__restrict__ r,
                                                  double *__restrict__ rhat, Scalars c) {
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double v = b[i] - y[i];
        r[i] = v;
        rhat[i] = v;
        acc += v * v;
    }
    put_partial(c, kRR, acc);
    put_partial(c, kRhatR, acc);
}

// Iteration `it` begins: the state of the residual, then p = r + beta (p - omega v)
// (p = r in the first iteration); x = 0 when b = 0.
__global__ void __launch_bounds__(256) k_dir(int64_t n, int64_t it, const double *__restrict__ r,
                                             const double *__restrict__ v, double *__restrict__ p,
                                             double *__restrict__ x, Scalars c) {
    const int32_t status = group_status(c);
    if (status != kRun && status != kZeroRhs) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double bnrm = it == 1 ? sqrt(total(c, kBB)) : c.st->bnrm;
    if (bnrm == 0.0) {
        for (int64_t i = i0; i < n; i += stride) x[i] = 0.0;
        if (first_thread()) end_solve(c, kZeroRhs, 0);
        return;
    }
    const double rr = total(c, kRR), rho = total(c, kRhatR);
    const double omega = it == 1 ? 1.0 : c.st->omega;
    if (first_thread()) {
        c.st->bnrm = bnrm;
        c.st->rr = rr;
        c.st->rho[it & 1] = rho;
    }
    if (sqrt(rr) <= c.rtol * bnrm || omega == 0.0) {
        if (first_thread()) end_solve(c, sqrt(rr) <= c.rtol * bnrm ? kConverged : kBreakdown, it - 1);
        return;
    }
    if (rho == 0.0) {
        if (first_thread()) end_solve(c, kBreakdown, it);
        return;
    }
    if (it == 1) {
        for (int64_t i = i0; i < n; i += stride) p[i] = r[i] + 0.0;
    } else {
        const double beta = (rho / c.st->rho[(it - 1) & 1]) * (c.st->alpha / omega);
        for (int64_t i = i0; i < n; i += stride) p[i] = r[i] + beta * (p[i] - omega * v[i]);
    }
    if (first_thread()) {
        c.st->it = it;
        __hip_atomic_store(c.host_status + 1, (int32_t)it, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// rhat . v
__global__ void __launch_bounds__(256) k_rhat_v(int64_t n, const double *__restrict__ rhat,
                                                const double *__restrict__ v, Scalars c) {
    if (c.st->status != kRun) return;
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) acc += rhat[i] * v[i];
    put_partial(c, kRhatV, acc);
}

// alpha = rho / (rhat . v); s = r - alpha v; ||s||^2
__global__ void __launch_bounds__(256) k_half(int64_t n, int64_t it, const double *__restrict__ r,
                                              const double *__restrict__ v, double *__restrict__ sv, Scalars c) {
    if (group_status(c) != kRun) return;
    const double rv = total(c, kRhatV);
    if (rv == 0.0) {
        if (first_thread()) end_solve(c, kBreakdown, it);
        return;
    }
    const double alpha = c.st->rho[it & 1] / rv, a = -alpha;
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double s = r[i] + a * v[i];
        sv[i] = s;
        acc += s * s;
    }
    put_partial(c, kSS, acc);
    if (first_thread()) c.st->alpha = alpha;
}

// t . s and t . t, unless the half step has converged
__global__ void __launch_bounds__(256) k_t_dots(int64_t n, int64_t it, const double *__restrict__ t,
                                                const double *__restrict__ sv, Scalars c) {
    if (group_status(c) != kRun) return;
    const double ss = total(c, kSS);
    if (sqrt(ss) <= c.rtol * c.st->bnrm) {
        if (first_thread()) {
            c.st->rr = ss;
            c.st->half_it = it;
            end_solve(c, kHalf, it);
        }
        return;
    }
    double ts = 0.0, tt = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double ti = t[i];
        ts += ti * sv[i];
        tt += ti * ti;
    }
    put_partial(c, kTS, ts);
    put_partial(c, kTT, tt);
}

// omega = (t . s) / (t . t); x += alpha phat + omega shat, r = s - omega t; ||r||^2 and
// rhat . r. After a converged half step only x += alpha phat.
__global__ void __launch_bounds__(256) k_step(int64_t n, int64_t it, const double *__restrict__ phat,
                                              const double *__restrict__ shat, const double *__restrict__ sv,
                                              const double *__restrict__ t, const double *__restrict__ rhat,
                                              double *__restrict__ x, double *__restrict__ r, Scalars c) {
    const int32_t status = group_status(c);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (status == kHalf && c.st->half_it == it) {
        const double alpha = c.st->alpha;
        for (int64_t i = i0; i < n; i += stride) x[i] = x[i] + alpha * phat[i];
    }
    if (status != kRun) return;
    const double ts = total(c, kTS), tt = total(c, kTT);
    if (tt == 0.0) {
        if (first_thread()) end_solve(c, kBreakdown, it);
        return;
    }
    const double alpha = c.st->alpha, omega = ts / tt;
    double rr = 0.0, rho = 0.0;
    for (int64_t i = i0; i < n; i += stride) {
        x[i] = x[i] + alpha * phat[i] + omega * shat[i];
        const double ri = sv[i] - omega * t[i];
        r[i] = ri;
        rr += ri * ri;
        rho += rhat[i] * ri;
    }
    put_partial(c, kRR, rr);
    put_partial(c, kRhatR, rho);
    if (first_thread()) c.st->omega = omega;
}

// after the last iteration: its residual (same grid, one workgroup does the work)
__global__ void __launch_bounds__(256) k_last(Scalars c) {
    if (blockIdx.x != 0 || c.st->status != kRun) return;
    const double rr = total(c, kRR);
    if (threadIdx.x != 0) return;
    c.st->rr = rr;
    if (sqrt(rr) <= c.rtol * c.st->bnrm) c.st->status = kConverged;
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
    hipEvent_t e0 = nullptr, e1 = nullptr;
    double *w = nullptr;
    int32_t *status = nullptr;
    const size_t vec = (size_t)n * sizeof(double);
    KState h;
    ::memset(&h, 0, sizeof(h));
    hipError_t err = hipSuccess;
    auto ok = [&err](hipError_t e) { return (err = e) == hipSuccess; };
    auto solve = [&]() -> bool {
        if (!ok(hipEventCreate(&e0)) || !ok(hipEventCreate(&e1))) return false;
        if (!ok(take_status(&status))) return false;
        volatile int32_t *word = status;
        word[0] = kRun;
        word[1] = 0;
        void *sdev = nullptr;
        if (!ok(hipHostGetDevicePointer(&sdev, status, 0))) return false;
        if (!ok(dev_alloc((void **)&w, 8 * vec + kParts * kDotBlocks * sizeof(double) + sizeof(KState), s))) return false;
        double *r = w, *rhat = w + n, *p = w + 2 * n, *v = w + 3 * n, *sv = w + 5 * n, *t = w + 7 * n;
        // without M, phat = p and shat = s
        double *phat = M ? w + 4 * n : p, *shat = M ? w + 6 * n : sv;
        double *part = w + 8 * n;
        KState *st_dev = (KState *)(part + kParts * kDotBlocks);
        const int32_t *stop = &st_dev->status;
        const Scalars c{st_dev, part, (int32_t *)sdev, rtol};
        const unsigned g = grid_dot(n);
        auto applyB = [&](const double *x, double *y) {
            return ok(spmv(n, B->nnz, B->row_ptr_dev, B->col_dev, B->val_dev, x, y, stop, s));
        };
        auto applyM = [&](const double *x, double *y) {
            return !M || ok(spmv(n, M->nnz, M->row_ptr_dev, M->col_dev, M->val_dev, x, y, stop, s));
        };
        if (!ok(hipEventRecord(e0, s))) return false;
        if (!ok(hipMemsetAsync(st_dev, 0, sizeof(KState), s))) return false;
        k_norm_b<<<g, 256, 0, s>>>(n, b_dev, c);
        if (!applyB(x_dev, v)) return false;
        k_residual<<<g, 256, 0, s>>>(n, b_dev, v, r, rhat, c);
        for (int64_t it = 1; it <= maxiter; ++it) {
            k_dir<<<g, 256, 0, s>>>(n, it, r, v, p, x_dev, c);
            if (!applyM(p, phat) || !applyB(phat, v)) return false;
            k_rhat_v<<<g, 256, 0, s>>>(n, rhat, v, c);
            k_half<<<g, 256, 0, s>>>(n, it, r, v, sv, c);
            if (!applyM(sv, shat) || !applyB(shat, t)) return false;
            k_t_dots<<<g, 256, 0, s>>>(n, it, t, sv, c);
            k_step<<<g, 256, 0, s>>>(n, it, phat, shat, sv, t, rhat, x_dev, r, c);
            if (!ok(hipGetLastError())) return false;
            for (unsigned spins = 1; word[0] == kRun && word[1] <= it - kAhead; ++spins) {
                std::this_thread::yield();
                if (spins % 1024 != 0) continue;
                const hipError_t q = hipStreamQuery(s);  // an error that no kernel will report here
                if (q == hipSuccess) break;
                if (q != hipErrorNotReady) return ok(q);
                (void)hipGetLastError();
            }
            if (word[0] != kRun) break;
            if (it % kRetire == 0 && !ok(hipStreamSynchronize(s))) return false;
        }
        k_last<<<g, 256, 0, s>>>(c);
        if (!ok(hipGetLastError())) return false;
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
    for (hipEvent_t e : {e0, e1})
        if (e) (void)hipEventDestroy(e);
    if (!done) return fail(MCMI_ERR_HIP, std::string("mcmi_bicgstab: ") + hipGetErrorString(err));
    if (st) {
        st->iterations = h.it;
        st->rel_residual = h.bnrm > 0.0 ? sqrt(h.rr) / h.bnrm : 0.0;
        st->ms = ms;
        st->converged = h.status == kConverged || h.status == kHalf || h.status == kZeroRhs;
    }
    return MCMI_OK;
}
