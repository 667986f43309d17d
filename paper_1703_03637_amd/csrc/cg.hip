// Conjugate-gradient steps of the inverse iteration (Sec. 3.4): the scalars of
// the recurrence stay on the device, so iterations are enqueued ahead and the
// host looks at them only now and then.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hphi_internal.h"
#include "tail.h"

namespace hphi {
namespace {

__global__ void cg_init_kernel(CgScalars* c, const double* rr, double tol, int n_max) {
    c->rr = *rr;
    c->alpha = c->beta = 0.0;
    c->tol = tol;
    c->n_max = n_max;
    c->iters = 0;
    c->done = sqrt(*rr) <= tol ? 1 : 0;
    c->stop = c->done;
    c->pad = 0;
}

// x += alpha p, r -= alpha q and |r|^2 in one pass (bound by the six streams it
// moves); the last block takes beta and the stop test
__global__ __launch_bounds__(256) void cg_update_kernel(double* __restrict__ x, double* __restrict__ r,
                                                        const double* __restrict__ p, const double* __restrict__ q,
                                                        int64_t n, CgScalars* c, double* __restrict__ partials,
                                                        uint32_t* tickets) {
    if (c->stop) return;
    const double a = c->alpha;
    double s = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        x[i] += a * p[i];
        const double v = r[i] - a * q[i];
        r[i] = v;
        s += v * v;
    }
    __shared__ double sh[257];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) put_partial(partials + blockIdx.x, sh[0]);
    __syncthreads();
    if (!tail_last(tickets, int(blockIdx.x), int(gridDim.x), reinterpret_cast<int*>(sh + 256))) return;
    tail_sums(partials, int(gridDim.x), 1, sh);
    if (threadIdx.x == 0) {
        const double rn = sh[0];
        c->iters += 1;
        if (sqrt(rn) <= c->tol) c->done = c->stop = 1;
        else if (c->iters >= c->n_max) c->stop = 1;
        c->beta = rn / c->rr;
        c->rr = rn;
    }
}

// p = r + beta p
__global__ __launch_bounds__(256) void cg_direction_kernel(double* __restrict__ p, const double* __restrict__ r, int64_t n,
                                                           const CgScalars* c) {
    if (c->stop) return;
    const double b = c->beta;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) p[i] = r[i] + b * p[i];
}

int cg_grid(int64_t n) { return int(std::min<int64_t>(1024, std::max<int64_t>(1, (n + 1023) / 1024))); }

}  // namespace

int launch_cg_init(CgScalars* c, const double* rr, double tol, int n_max, hipStream_t st) {
    cg_init_kernel<<<1, 1, 0, st>>>(c, rr, tol, n_max);
    return check_hip(hipGetLastError(), "cg_init launch");
}

int launch_cg_update(double* x, double* r, double* p, const double* q, int64_t n, CgScalars* c, double* partials,
                     uint32_t* tickets, hipStream_t st) {
    const int grid = cg_grid(n);
    cg_update_kernel<<<grid, 256, 0, st>>>(x, r, p, q, n, c, partials, tickets);
    int rc = check_hip(hipGetLastError(), "cg_update launch");
    if (rc) return rc;
    cg_direction_kernel<<<grid, 256, 0, st>>>(p, r, n, c);
    return check_hip(hipGetLastError(), "cg_direction launch");
}

}  // namespace hphi
