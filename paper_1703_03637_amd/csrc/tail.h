// The end of a product or update kernel: the block that finishes last sums the
// block partials in a fixed order and takes the scalar step that reads the
// sums, so small problems pay no further launch for either.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "hphi_internal.h"

namespace hphi {
namespace {

// ---- scalar steps after the sums (also run by the separate launches)

// after the product: alpha_k and the update's coefficients
__device__ __forceinline__ void lz_after_hv_step(LzScalars* sc, const double* red, double* alpha, const double* evec) {
    const double a = red[1];          // Re<v_k|H v_k>, v_k = s_cur * X
    alpha[sc->k] = a;
    sc->c2 = -a * sc->s_cur;
    sc->ecoef = evec ? evec[sc->k] * sc->s_cur : 0.0;
}

// after the update: beta_{k+1}, the stop test and the next step's scales
__device__ __forceinline__ void lz_after_update_step(LzScalars* sc, const double* red, double* beta, const double* alpha) {
    const int k = sc->k;
    const double b = sqrt(red[0]);
    beta[k] = b;
    sc->n_done = k + 1;
    const double a = fabs(alpha[k]);
    double scale = a > sc->beta_k ? a : sc->beta_k;
    if (scale < 1.0) scale = 1.0;
    if (k + 1 >= sc->n_max || b <= sc->tol * scale) {
        sc->stop = 1;
        if (k + 1 < sc->n_max) sc->breakdown = 1;
        return;
    }
    sc->cy = -b * sc->s_cur;   // -beta_{k+1} times the scale of v_k (next step's v_{k-1})
    sc->s_cur = 1.0 / b;
    sc->beta_k = b;
    sc->k = k + 1;
}

// TPQ observables of vector b of a step with index k; returns 1 / |phi|
__device__ __forceinline__ double tpq_obs_step(const double* red, double* obs, int nvec, int b, double ns, double l, int k) {
    const double xx = red[0 * nvec + b], xh = red[1 * nvec + b], hh = red[2 * nvec + b], uu = red[3 * nvec + b];
    const double uk = xh / xx / ns;
    const double s = 1.0 / sqrt(uu);
    obs[0 * nvec + b] = uk;
    obs[1 * nvec + b] = hh / xx / (ns * ns);
    obs[2 * nvec + b] = (2.0 * double(k - 1) / ns) / (l - uk);
    obs[3 * nvec + b] = s;
    return s;
}

// <O> = Re<x|Ox> / <x|x> per vector, and <x|x>
__device__ __forceinline__ void expect_step(const double* red, double* out, int nvec, int b) {
    const double xx = red[0 * nvec + b], xo = red[1 * nvec + b];
    out[b] = xo / xx;
    out[nvec + b] = xx;
}

// after the product of a CG step: <p|A p>, A = H - l; zero or non-finite ends
// the solve with the current iterate
__device__ __forceinline__ void cg_after_hv_step(CgScalars* c, const double* red, double l) {
    const double pap = red[1] - l * red[0];
    if (!isfinite(pap) || pap == 0.0) c->stop = 1;
    else c->alpha = c->rr / pap;
}

// The scalar step of `T` on the sums red[q * nvec + b] (all threads of one block)
__device__ __forceinline__ void tail_step(const Tail& T, const double* red, int nvec) {
    const int t = int(threadIdx.x);
    if (T.mode == kTailLanczos) {
        if (t == 0) lz_after_hv_step(T.sc, red, T.alpha, T.evec);
    } else if (T.mode == kTailTpq) {
        if (t < nvec) tpq_obs_step(red, T.obs, nvec, t, T.ns, T.l, T.k);
    } else if (T.mode == kTailTpqRun) {
        // the step number lives on the device (graph replays advance it); the
        // scale of the produced state goes to the slot of this step's parity
        const int j = T.run->j, k = T.run->k;
        if (t < nvec) T.run->scale[j & 1][t] = tpq_obs_step(red, T.obs + size_t(j) * 4 * nvec, nvec, t, T.ns, T.l, k);
        __syncthreads();
        if (t == 0) {
            T.run->j = j + 1;
            T.run->k = k + 1;
        }
    } else if (T.mode == kTailCg) {
        if (t == 0) cg_after_hv_step(T.cg, red, T.l);
    } else if (T.mode == kTailExpect) {
        if (t < nvec) expect_step(red, T.obs, nvec, t);
    }
}

// A block partial, where every XCD sees it.  An exchange that returns the old
// value has been performed at the point where the device's atomics meet once
// the value is back, so a ticket taken after that cannot overtake it; the
// acknowledgement of a plain write-through store does not say as much.  (A
// release fence at device scope would do too, but writes the whole L2 back: 20
// to 30 us per launch of a few hundred blocks.)
__device__ __forceinline__ void put_partial(double* p, double x) {
    const unsigned long long old =
        __hip_atomic_exchange(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(__double_as_longlong(x)),
                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(old));   // the value is waited for
}

// the same for a kernel that may leave the sums to a later launch
__device__ __forceinline__ void put_partial(int32_t mode, double* p, double x) {
    if (mode == kTailNone) *p = x;
    else put_partial(p, x);
}

__device__ __forceinline__ double get_partial(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by every thread of every block (256 threads) after wave 0 of the block
// has stored its partials with put_partial.  True for the threads of the last
// block to arrive, which then reads the partials of all with get_partial.
// Two levels of tickets, 32 blocks to one, each in a line of its own: a single
// one serializes the atomics of all blocks (1,024 blocks: 15 to 20 us).
// `flag`: one word of LDS.
__device__ __forceinline__ bool tail_last(uint32_t* tickets, int blk, int n_blocks, int* flag) {
    if (threadIdx.x < 64) {
        // the wave's exchanges have returned before its ticket counts
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (threadIdx.x == 0) {
            const int g = blk >> 5, n_g = (n_blocks + 31) >> 5;
            const uint32_t size = uint32_t(g + 1 < n_g ? 32 : n_blocks - 32 * g);
            uint32_t* tg = tickets + size_t(1 + g) * kTicketStride;
            int last = 0;
            if (__hip_atomic_fetch_add(tg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == size - 1) {
                __hip_atomic_store(tg, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = __hip_atomic_fetch_add(tickets, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == uint32_t(n_g - 1);
                if (last) __hip_atomic_store(tickets, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            *flag = last;
        }
    }
    __syncthreads();
    return *flag != 0;
}

// Sums of partials[g * nq + q], g < n_parts, into lds[q]: the threads of a
// quantity take every (256 / nq)-th partial, then a fixed tree.  nq divides 256.
__device__ __forceinline__ void tail_sums(const double* partials, int n_parts, int nq, double* lds) {
    const int t = int(threadIdx.x), q = t % nq, s0 = t / nq, ns = 256 / nq;
    double s = 0.0;
    int g = s0;
    for (; g + 7 * ns < n_parts; g += 8 * ns) {
        double x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = get_partial(partials + size_t(g + j * ns) * nq + q);
#pragma unroll
        for (int j = 0; j < 8; ++j) s += x[j];
    }
    for (; g < n_parts; g += ns) s += get_partial(partials + size_t(g) * nq + q);
    lds[t] = s;
    __syncthreads();
    for (int w = ns / 2; w > 0; w >>= 1) {
        if (s0 < w) lds[t] += lds[t + w * nq];
        __syncthreads();
    }
}

// Where a kernel finds its Tail.  Read as an ordinary argument it is loaded when
// the kernel starts, and its 22 words stay in scalar registers beside the loop,
// which spills 16 to 37 of its own for them.  The address alone costs waves too: a
// SIMD holds 7 of a kernel of at most 96 scalar registers and 6 of more (the runtime's
// occupancy counts 7 for both, and the persistent grid then ends in a nearly empty
// wave: 3,312,400 rows of 2 FP64, per-tile kernel, 264 us at 96 registers, 417 at 100).
// So block-wide LDS keeps the address until the sums are due.
typedef const __attribute__((address_space(4))) Tail* TailAt;

// of a kernel whose first argument is an Args by value
template <typename Args>
__device__ __forceinline__ TailAt kernel_tail() {
    typedef const __attribute__((address_space(4))) char* Bytes;
    return (TailAt)((Bytes)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(Args, tail));
}

// What the end of a product kernel needs, in LDS: written when the kernel starts,
// read after a barrier
struct TailKeep {
    uint32_t at[2], partials[2];
    int32_t mode, n_blocks, blk, pad;

    __device__ __forceinline__ void put(TailAt a, double* p, int32_t m, int b, int nb) {
        if (threadIdx.x != 0) return;
        at[0] = uint32_t(uint64_t(a));
        at[1] = uint32_t(uint64_t(a) >> 32);
        partials[0] = uint32_t(uint64_t(p));
        partials[1] = uint32_t(uint64_t(p) >> 32);
        mode = m;
        n_blocks = nb;
        blk = b;
    }
    __device__ __forceinline__ static uint64_t wide(const uint32_t (&w)[2]) {
        const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int32_t(w[0])));
        const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int32_t(w[1])));
        return (uint64_t(hi) << 32) | lo;
    }
};

// The tail of a product over nvec vectors (not called with kTailNone).  `lds`:
// 257 doubles of LDS that no thread of the block reads any more.
__device__ __forceinline__ void product_tail(TailAt at, const double* partials, int blk, int n_blocks, int nvec, double* lds) {
    asm volatile("" : "+s"(at));   // its loads stay behind this point
    const Tail& T = *(const Tail*)at;
    if (!tail_last(T.tickets, blk, n_blocks, reinterpret_cast<int*>(lds + 256))) return;
    const int nq = kNQ * nvec, t = int(threadIdx.x);
    tail_sums(partials, n_blocks, nq, lds);
    if (t < nq) {
        if (T.out) T.out[t] = lds[t];
        if (T.flag && !isfinite(lds[t])) atomicOr(T.flag, HPHI_NONFINITE_PRODUCT);
    }
    tail_step(T, lds, nvec);
}

// The end of a product kernel: the block's sum s of quantity and vector
// threadIdx.x < kNQ * nvec, and the tail if it is taken along.  The block sums
// in `lds` are read after a barrier.
__device__ __forceinline__ void product_end(const TailKeep& keep, double s, int nvec, double* lds) {
    const int32_t mode = __builtin_amdgcn_readfirstlane(keep.mode), blk = __builtin_amdgcn_readfirstlane(keep.blk);
    double* const partials = reinterpret_cast<double*>(TailKeep::wide(keep.partials));
    if (int(threadIdx.x) < kNQ * nvec) {
        double* const p = partials + size_t(blk) * size_t(kNQ * nvec) + threadIdx.x;
        if (mode == kTailNone) *p = s;
        else put_partial(p, s);
    }
    if (mode == kTailNone) return;
    __syncthreads();   // the block sums are read
    product_tail(TailAt(TailKeep::wide(keep.at)), partials, blk, __builtin_amdgcn_readfirstlane(keep.n_blocks), nvec, lds);
}

// The tail of a Lanczos update: |y|^2, then beta and the next scales
__device__ __forceinline__ void update_tail(LzScalars* sc, uint32_t* tickets, const double* partials, int blk, int n_blocks, double* beta,
                                            const double* alpha, int32_t* flag, double* lds) {
    if (!tail_last(tickets, blk, n_blocks, reinterpret_cast<int*>(lds + 256))) return;
    tail_sums(partials, n_blocks, 1, lds);
    if (threadIdx.x == 0) {
        if (flag && !isfinite(lds[0])) atomicOr(flag, HPHI_NONFINITE_NORM);
        lz_after_update_step(sc, lds, beta, alpha);
    }
}

}  // namespace
}  // namespace hphi
