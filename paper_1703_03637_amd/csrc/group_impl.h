// The class-blocked sector product (group.h): kernels and launches for one
// storage scalar; each storage type is compiled in a file of its own.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "group.h"
#include "hphi_internal.h"
#include "lane.h"
#include "tail.h"

namespace hphi {
namespace {

template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T*;

// the lane's share of a row, from the lane's own chunk address p
template <typename S, int NE, int LPR>
__device__ __forceinline__ void load_at(const char* p, S (&out)[NE]) {
    using Ly = LaneLayout<S, NE, LPR>;
#pragma unroll
    for (int j = 0; j < Ly::NCH; ++j)
        copy_chunk<Ly::CB>(reinterpret_cast<char*>(out) + j * Ly::CB, p + j * LPR * Ly::CB);
}

// A table pointer that the compiler does not tie to earlier reads: values read
// through it live in scalar registers for one phase, not for the whole item
template <typename T>
__device__ __forceinline__ T phase(T p) {
    asm volatile("" : "+s"(p));
    return p;
}

// A row of zeros (the widest row: 16 complex128 values), read in place of the
// partners that pad a list: 0 * Inf of any other row would be NaN.  The choice of
// the address costs 0.5 to 1% (1.25e9 FP32 rows 34.8 -> 35.0 ms, 3.4e8 rows of four
// complex64 78.8 -> 79.3 ms); batches without padding in a loop of their own cost
// the same.
__device__ __align__(256) uint32_t kGroupZeroRow[64] = {};

// items of `size` bytes that fill `bytes`, between 1 and `most`
constexpr int group_batch(int bytes, int size, int most) { return size >= bytes ? 1 : bytes / size > most ? most : bytes / size; }

// One wavefront: a tile of 64 low halves of one class (LPR passes of 64 / LPR
// rows, a row shared by LPR lanes with NE scalars each) times K high halves.
// Complex vectors are 2 * nvec real columns: the coefficients are real, and the
// sums fold the column pairs at the end.
// SIGN: some operator with a bit in each half carries a low-half sign.
// Args: the kernel's arguments, or a problem's in constant memory.
template <typename S, int NS, int LPR, int K, bool SIGN, typename Args>
__device__ __forceinline__ void hvg_body(Args& A, const TailAt tail, const int blk, const int nblk) {
    constexpr int NE = NS / LPR;
    using Ly = LaneLayout<S, NE, LPR>;
    constexpr int RPW = 64 / LPR;
    constexpr int LOGL = Log2<LPR>::value;
    constexpr int LOGE = Log2<NE>::value;
    // Batches: EB list entries, OB cross operators and HB partner blocks of each
    // high half are gathered for the K blocks before any is accumulated, by
    // bytes per lane.  Narrow FP32 rows are bound by the L1's in-order returns
    // (its pending stalls take 60-70% of the cycles) and lose with more in
    // flight per wave: 1.25e9 FP32 rows, K = 8, LL/LH/HH = 32/16/64 36.2 ms,
    // 64/32/64 37.8, 128/64/64 60; lanes of 16 bytes and more are bound by
    // the traffic between L2 and the fabric (6.2 TB/s on four complex64
    // vectors) and want it full: 64/32/64 81.0 ms, 128/64/128 78.2.  One
    // complex128 vector, a 16-byte lane of two scalars, goes with them.
    constexpr int LL = Ly::LB >= 16 ? 128 : sizeof(S) == 4 ? 32 : 64;
    constexpr int LH = Ly::LB >= 16 ? 64 : sizeof(S) == 4 ? 16 : 32;
    constexpr int HH = Ly::LB >= 16 ? 128 : 64;
    constexpr int EB = group_batch(LL, K * Ly::LB, kGroupPad);
    constexpr int OB = group_batch(LH, K * Ly::LB, kGroupPad);
    constexpr int HB = group_batch(HH, K * Ly::LB, kGroupEnt);
    constexpr int LOGB = Log2<Ly::RB>::value;
    static_assert(kGroupPad % EB == 0 && kGroupPad % OB == 0 && kGroupEnt % HB == 0, "padding covers the batches");
    if (A.stop && *A.stop) return;

    const int lane = threadIdx.x & 63;
    const int sub = lane & (LPR - 1);
    const int rlane = lane >> LOGL;
    const int wave = wave_uniform(threadIdx.x >> 6);
    const char* const v = static_cast<const char*>(A.v);
    char* const u = static_cast<char*>(A.u);
    const char* const y = static_cast<const char*>(A.y);
    const ConstPtr<GGroup> groups = (ConstPtr<GGroup>)(A.grp.groups);
    const ConstPtr<GClass> cls = (ConstPtr<GClass>)(A.cls);
    const ConstPtr<uint32_t> cibit = (ConstPtr<uint32_t>)(A.plan.ci);
    const ConstPtr<GCross> lhops = (ConstPtr<GCross>)(A.plan.lh);
    const uint32_t n_low = A.plan.n_low, n_slot = A.plan.n_slot;

    __shared__ double coef[kGroupCoef];
    __shared__ double sh[kWavesPerBlock][kNQ][64];
    for (int i = int(threadIdx.x); i < A.plan.n_coef; i += kBlock) coef[i] = A.plan.coef[i];
    __syncthreads();

    // an XCD sweeps its own groups in order; the groups of the eight XCDs
    // advance together
    const int xcd = blk & 7;
    const uint32_t g_begin = A.grp.begin[xcd], g_last = A.grp.begin[xcd + 1] - 1;   // the last one only closes the range
    const uint32_t i_end = A.grp.items[xcd] * LPR;   // the LPR passes of a tile are neighbouring wavefronts
    const uint32_t i_step = uint32_t(nblk >> 3) * kWavesPerBlock;

    double wq[kNQ] = {0.0, 0.0, 0.0, 0.0};
    uint32_t gi = g_begin;
    for (uint32_t it = uint32_t(blk >> 3) * kWavesPerBlock + uint32_t(wave); it < i_end; it += i_step) {
        const uint32_t item = it / LPR;
        const int pass = int(it % LPR);
        if (item >= groups[gi + 1].item0) {
            // the last group that starts at or before the item
            uint32_t lo = gi + 1, hi_g = g_last - 1;
            while (lo < hi_g) {
                const uint32_t mid = (lo + hi_g + 1) >> 1;
                if (groups[mid].item0 <= item) lo = mid;
                else hi_g = mid - 1;
            }
            gi = lo;
        }
        const uint32_t p0 = groups[gi].p0, nk = groups[gi].n, ci = groups[gi].cls;
        const uint32_t tile = item - groups[gi].item0;
        const uint32_t n_l = cls[ci].n_l, l_off = cls[ci].l_off;
        {
            const uint32_t r = tile * 64u + uint32_t(pass * RPW + rlane);
            if (LPR > 1 && tile * 64u + uint32_t(pass * RPW) >= n_l) continue;
            const bool valid = r < n_l;
            const uint32_t rr = valid ? r : n_l - 1;
            const uint32_t li = l_off + rr;
            const uint32_t l = A.lows[li];
            const uint32_t own = rr * uint32_t(Ly::RB) + uint32_t(sub * Ly::CB);   // byte offset in a block

            double acc[K][NE];
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int e = 0; e < NE; ++e) acc[k][e] = 0.0;

            // ---- operators inside the low half: per operator the rank of
            // each row's partner and its element, one entry for the K
            // blocks.  Rows that the operator leaves alone skip the gathers.
            const uint32_t* const nb = A.plan.nbr + li;
            const int n_ll = A.plan.n_ll;
            uint32_t ent[EB];
#pragma unroll
            for (int j = 0; j < EB; ++j) ent[j] = nb[size_t(j) * n_low];
            const char* vb[K];
            {
                const ConstPtr<int64_t> r0 = phase((ConstPtr<int64_t>)(A.plan.row0) + p0);
#pragma unroll
                for (int k = 0; k < K; ++k) vb[k] = v + r0[k] * int64_t(Ly::RB);
            }
            for (int o = 0; o < n_ll; o += EB) {
                alignas(16) S g[EB][K][NE];
                double cl[EB];
                uint32_t off[EB];
                bool act[EB];
#pragma unroll
                for (int j = 0; j < EB; ++j) {
                    off[j] = (ent[j] & kGroupRank) * uint32_t(Ly::RB) + uint32_t(sub * Ly::CB);
                    act[j] = (ent[j] >> 24) != 0u;
                    cl[j] = coef[ent[j] >> 24];
                }
#pragma unroll
                for (int j = 0; j < EB; ++j)
                    if (act[j]) {
#pragma unroll
                        for (int k = 0; k < K; ++k)
                            load_at<S, NE, LPR>(vb[k] + off[j], g[j][k]);
                    }
#pragma unroll
                for (int j = 0; j < EB; ++j) ent[j] = nb[size_t(o + EB + j) * n_low];   // the list is padded
#pragma unroll
                for (int j = 0; j < EB; ++j)
                    if (act[j]) {
#pragma unroll
                        for (int k = 0; k < K; ++k)
#pragma unroll
                            for (int e = 0; e < NE; ++e) acc[k][e] += cl[j] * double(g[j][k][e]);
                    }
            }

            // ---- operators inside the high half: per high half a list of
            // partner blocks, read at the row's own rank.  The K lists run
            // together, HB entries of each at a time, to the end of the
            // longest; past its end a list has the zero element and reads
            // the row of zeros.  Without branches the scalar loads of a
            // batch go out together, and the elements arrive behind the
            // gathers.
            {
                const ConstPtr<uint32_t> np = (ConstPtr<uint32_t>)(A.plan.n_ent) + p0;
                uint32_t n = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) n = np[k] > n ? np[k] : n;
                const uint32_t stride = uint32_t(A.plan.hh_stride);
                const ConstPtr<uint64_t> he = (ConstPtr<uint64_t>)(A.plan.hh) + size_t(p0) * stride;
                const ConstPtr<double> hc = (ConstPtr<double>)(A.plan.coef);
                for (uint32_t e0 = 0; e0 < n; e0 += HB) {
                    alignas(16) S g[K][HB][NE];
                    double cf[K][HB];
#pragma unroll
                    for (int k = 0; k < K; ++k)
#pragma unroll
                        for (int j = 0; j < HB; ++j) {
                            const uint64_t t = he[size_t(k) * stride + e0 + j];
                            const bool pad = (t >> 48) == 0;
                            cf[k][j] = hc[uint32_t(t >> 48)];
                            const char* const blk0 = pad ? reinterpret_cast<const char*>(kGroupZeroRow)
                                                         : v + ((t << 16) >> (16 - LOGB));
                            load_at<S, NE, LPR>(phase(blk0) + (own & (pad ? uint32_t(Ly::RB - 1) : ~0u)), g[k][j]);
                        }
#pragma unroll
                    for (int k = 0; k < K; ++k)
#pragma unroll
                        for (int j = 0; j < HB; ++j)
#pragma unroll
                            for (int e = 0; e < NE; ++e) acc[k][e] += cf[k][j] * double(g[k][j][e]);
                }
            }

            // ---- operators with one bit in each half: the partner's rank
            // from the low half (one column per low bit), its block and
            // the element from the high half; live where the bits differ
            const uint32_t* const xb = A.plan.xnb + li;
            const int n_lh = A.plan.n_lh;
            uint32_t hv[K];
            {
                const ConstPtr<uint32_t> hp = phase((ConstPtr<uint32_t>)(A.plan.hval) + p0);
#pragma unroll
                for (int k = 0; k < K; ++k) hv[k] = hp[k];
            }
            uint32_t ex[OB];
#pragma unroll
            for (int j = 0; j < OB; ++j) ex[j] = xb[size_t(lhops[j].col) * n_low];
            for (int o = 0; o < n_lh; o += OB) {
                // lanes of rows that are not live keep zeros, so only the
                // loads are predicated
                alignas(16) S g[OB][K][NE];
                uint32_t neg[OB][K];
#pragma unroll
                for (int j = 0; j < OB; ++j) {
                    const int hj = lhops[o + j].j;
                    const ConstPtr<int64_t> le = (ConstPtr<int64_t>)(A.plan.lhe) + size_t(o + j) * n_slot + p0;
                    const uint32_t off = (ex[j] & kGroupRank) * uint32_t(Ly::RB) + uint32_t(sub * Ly::CB);
                    const bool bi = int32_t(ex[j]) < 0;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const int64_t t = le[k];
                        if (SIGN) neg[j][k] = uint32_t(uint64_t(t) >> 32) & 0x80000000u;
#pragma unroll
                        for (int e = 0; e < NE; ++e) g[j][k][e] = S(0);
                        if (bi != (((hv[k] >> hj) & 1u) != 0))
                            load_at<S, NE, LPR>(v + (SIGN ? t & INT64_MAX : t) * int64_t(Ly::RB) + off, g[j][k]);
                    }
                }
                uint32_t sg[OB];
#pragma unroll
                for (int j = 0; j < OB; ++j) sg[j] = SIGN ? (ex[j] << 1) & 0x80000000u : 0u;
#pragma unroll
                for (int j = 0; j < OB; ++j) ex[j] = xb[size_t(lhops[o + OB + j].col) * n_low];   // padded
#pragma unroll
                for (int j = 0; j < OB; ++j) {
                    const double c = lhops[o + j].c;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const double ck = SIGN ? __hiloint2double(__double2hiint(c) ^ int(sg[j] ^ neg[j][k]), __double2loint(c)) : c;
#pragma unroll
                        for (int e = 0; e < NE; ++e) acc[k][e] += ck * double(g[j][k][e]);
                    }
                }
            }

            // ---- diagonal: the parts of the low and the high half, and the
            // terms that need a bit of each, per low bit
            double dd[K];
            {
                const double dl = A.plan.dlo[li];
#pragma unroll
                for (int k = 0; k < K; ++k) dd[k] = dl + ((ConstPtr<double>)(A.plan.dhi))[p0 + k];
                for (int i = 0; i < A.plan.n_ci; ++i) {
                    const uint32_t bit = cibit[i];
                    const ConstPtr<double> wp = (ConstPtr<double>)(A.plan.w) + size_t(i) * n_slot + p0;
                    const double b = (l >> (bit & 31u)) & 1u ? 1.0 : ((bit & 32u) ? -1.0 : 0.0);
#pragma unroll
                    for (int k = 0; k < K; ++k) dd[k] += b * wp[k];
                }
            }

            // ---- epilogue: w = a H x + b x + cy y with x = sx v, and the sums
            const ConstPtr<int64_t> r0 = phase((ConstPtr<int64_t>)(A.plan.row0) + p0);
            double q[kNQ][NE];
#pragma unroll
            for (int qi = 0; qi < kNQ; ++qi)
#pragma unroll
                for (int e = 0; e < NE; ++e) q[qi][e] = 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                __builtin_amdgcn_sched_barrier(0);   // one block's values at a time in registers
                if (uint32_t(k) >= nk || !valid) continue;
                const int64_t row0 = r0[k];
                alignas(16) S xv[NE], yv[NE], us[NE];
                load_at<S, NE, LPR>(v + row0 * int64_t(Ly::RB) + own, xv);
                if (y) load_at<S, NE, LPR>(y + row0 * int64_t(Ly::RB) + own, yv);
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    const int vec = (((e / Ly::CPS) * LPR + sub) * Ly::CPS + e % Ly::CPS) >> A.cshift;
                    const double sc = A.sx ? A.sx[vec] : 1.0;
                    const double vv = double(xv[e]);
                    const double x = sc * vv;
                    const double h = sc * (acc[k][e] + dd[k] * vv);
                    double w = (y && A.cy) ? A.cy[vec] * double(yv[e]) : 0.0;
                    w += A.a * h + A.b * x;
                    us[e] = S(w);
                    q[0][e] += x * x;
                    q[1][e] += x * h;
                    q[2][e] += h * h;
                    q[3][e] += w * w;
                }
                if (u) {
#pragma unroll
                    for (int j = 0; j < Ly::NCH; ++j)
                        put_chunk<Ly::CB>(u + row0 * int64_t(Ly::RB) + own + j * LPR * Ly::CB,
                                          reinterpret_cast<const char*>(us) + j * Ly::CB);
                }
            }
#pragma unroll
            for (int qi = 0; qi < kNQ; ++qi) wq[qi] += wave_reduce_rows<double, NE, LPR>(q[qi], lane);
        }
    }

    // block sums, then the columns of each vector
#pragma unroll
    for (int qi = 0; qi < kNQ; ++qi) sh[wave][qi][lane] = wq[qi];
    __syncthreads();
    const int nc = 1 << A.cshift, B = NS >> A.cshift;
    if (int(threadIdx.x) < kNQ * B) {
        const int qi = int(threadIdx.x) / B, b = int(threadIdx.x) % B;
        double s = 0.0;
        for (int cc = 0; cc < nc; ++cc) {
            const int col = b * nc + cc;
            const int chunk = col / Ly::CPS;
            const int L = (((chunk / LPR) * Ly::CPS + col % Ly::CPS) << (6 - LOGE)) | (chunk % LPR);
#pragma unroll
            for (int w = 0; w < kWavesPerBlock; ++w) s += sh[w][qi][L];
        }
        put_partial(A.tail.mode, &A.partials[size_t(blk) * size_t(kNQ * B) + threadIdx.x], s);
    }
    if (A.tail.mode != kTailNone) {
        __syncthreads();   // the block sums are read
        product_tail(tail, A.partials, blk, nblk, B, &sh[0][0][0]);
    }
}

template <typename S, int NS, int LPR, int K, bool SIGN>
__global__ __launch_bounds__(kBlock) void hvg_kernel(HvgArgs A) {
    hvg_body<S, NS, LPR, K, SIGN>(A, kernel_tail<HvgArgs>(), int(blockIdx.x), int(gridDim.x));
}

typedef const __attribute__((address_space(4))) HvgArgs ConstArgs;

// several problems in one launch: problem p owns the blocks begin[p] ..
// begin[p+1]-1 (multiples of 8) and its own partials
template <typename S, int NS, int K, bool SIGN>
__global__ __launch_bounds__(kBlock) void hvg_multi_kernel(const HvgArgs* __restrict__ probs,
                                                           const int* __restrict__ begin, int n_probs) {
    int p = 0;
    for (int q = 1; q < n_probs; ++q)
        if (int(blockIdx.x) >= begin[q]) p = q;
    p = wave_uniform(p);
    ConstArgs& A = ((ConstArgs*)(probs))[p];
    hvg_body<S, NS, 1, K, SIGN>(A, &A.tail, int(blockIdx.x) - begin[p], begin[p + 1] - begin[p]);
}

template <typename Kernel>
int group_occupancy(Kernel k) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, kBlock, 0) != hipSuccess || nb < 1) nb = 1;
    return std::min(nb, kScalarBlocks);
}

template <typename S, int NS, int LPR, int K, bool SIGN>
int launch_hvg_k(HvgArgs& A, const HvLaunch& L, int per_cu_cap, int cus, hipStream_t st, int* grid_out) {
    static const int occ = group_occupancy(hvg_kernel<S, NS, LPR, K, SIGN>);
    const int per_cu = per_cu_cap > 0 && per_cu_cap < occ ? per_cu_cap : occ;
    int64_t g = 0;
    for (int x = 0; x < 8; ++x) g = std::max<int64_t>(g, (int64_t(A.grp.items[x]) * LPR + kWavesPerBlock - 1) / kWavesPerBlock);
    g = std::min<int64_t>(std::max<int64_t>(g, 1) * 8, int64_t(per_cu) * cus / 8 * 8);
    g = std::min<int64_t>(g, kMaxGrid);
    A.tail = product_tail_of(L, int(g), group_sums_max(int(g)));
    hvg_kernel<S, NS, LPR, K, SIGN><<<int(g), kBlock, 0, st>>>(A);
    *grid_out = int(g);
    return check_hip(hipGetLastError(), "hvg_kernel launch");
}

// `lanes` per row: group_lanes, or twice as many for FP64 rows of 8 or 16
// scalars with four high halves (group_shape)
template <typename S, int NS, bool SIGN>
int launch_hvg_ns(HvgArgs& A, const HvLaunch& L, int k, int lanes, int cap, int cus, hipStream_t st, int* grid) {
    constexpr int LPR = group_lanes(NS);
    if constexpr (sizeof(S) == 8 && (NS == 8 || NS == 16))
        if (lanes == 2 * LPR && k == 4) return launch_hvg_k<S, NS, 2 * LPR, 4, SIGN>(A, L, cap, cus, st, grid);
    switch (k) {
        case 1: return launch_hvg_k<S, NS, LPR, 1, SIGN>(A, L, cap, cus, st, grid);
        case 2: return launch_hvg_k<S, NS, LPR, 2, SIGN>(A, L, cap, cus, st, grid);
        case 4: return launch_hvg_k<S, NS, LPR, 4, SIGN>(A, L, cap, cus, st, grid);
        case 8:
            if constexpr (NS / LPR <= 2) return launch_hvg_k<S, NS, LPR, 8, SIGN>(A, L, cap, cus, st, grid);
            break;
    }
    return set_error(HPHI_EINVAL, "class-blocked product: bad group size %d", k);
}

template <typename S, bool SIGN>
int launch_hvg_s(HvgArgs& A, const HvLaunch& L, int ns, int k, int lanes, int cap, int cus, hipStream_t st, int* grid) {
    switch (ns) {
        case 1: return launch_hvg_ns<S, 1, SIGN>(A, L, k, lanes, cap, cus, st, grid);
        case 2: return launch_hvg_ns<S, 2, SIGN>(A, L, k, lanes, cap, cus, st, grid);
        case 4: return launch_hvg_ns<S, 4, SIGN>(A, L, k, lanes, cap, cus, st, grid);
        case 8: return launch_hvg_ns<S, 8, SIGN>(A, L, k, lanes, cap, cus, st, grid);
        case 16: return launch_hvg_ns<S, 16, SIGN>(A, L, k, lanes, cap, cus, st, grid);
        case 32: return launch_hvg_ns<S, 32, SIGN>(A, L, k, lanes, cap, cus, st, grid);
    }
    return set_error(HPHI_EINVAL, "class-blocked product: bad row of %d scalars", ns);
}

template <typename S, int NS, int K, bool SIGN>
int launch_hvg_multi_k(const HvgArgs* d_args, const int* d_begin, int n, int grid, int* occ, hipStream_t st) {
    static const int o = group_occupancy(hvg_multi_kernel<S, NS, K, SIGN>);
    if (occ) {   // resident blocks per CU only
        *occ = o;
        return HPHI_OK;
    }
    hvg_multi_kernel<S, NS, K, SIGN><<<grid, kBlock, 0, st>>>(d_args, d_begin, n);
    return check_hip(hipGetLastError(), "hvg_multi_kernel launch");
}

template <typename S, bool SIGN>
int launch_hvg_multi_s(const HvgArgs* d_args, const int* d_begin, int n, int ns, int k, int grid, int* occ, hipStream_t st) {
    if (ns == 1) return k <= 2 ? launch_hvg_multi_k<S, 1, 2, SIGN>(d_args, d_begin, n, grid, occ, st)
                      : k == 4 ? launch_hvg_multi_k<S, 1, 4, SIGN>(d_args, d_begin, n, grid, occ, st)
                               : launch_hvg_multi_k<S, 1, 8, SIGN>(d_args, d_begin, n, grid, occ, st);
    return k <= 2 ? launch_hvg_multi_k<S, 2, 2, SIGN>(d_args, d_begin, n, grid, occ, st)
         : k == 4 ? launch_hvg_multi_k<S, 2, 4, SIGN>(d_args, d_begin, n, grid, occ, st)
                  : launch_hvg_multi_k<S, 2, 8, SIGN>(d_args, d_begin, n, grid, occ, st);
}

}  // namespace

#define HVG_INSTANTIATE(S, NAME, MULTI)                                                                                \
    int NAME(HvgArgs& A, const HvLaunch& L, int ns, int k, int lanes, bool sign, int cap, int cus, hipStream_t st,      \
             int* g) {                                                                                                 \
        return sign ? launch_hvg_s<S, true>(A, L, ns, k, lanes, cap, cus, st, g)                                        \
                    : launch_hvg_s<S, false>(A, L, ns, k, lanes, cap, cus, st, g);                                      \
    }                                                                                                                  \
    int MULTI(const HvgArgs* d_args, const int* d_begin, int n, int ns, int k, bool sign, int grid, int* occ,           \
              hipStream_t st) {                                                                                        \
        return sign ? launch_hvg_multi_s<S, true>(d_args, d_begin, n, ns, k, grid, occ, st)                             \
                    : launch_hvg_multi_s<S, false>(d_args, d_begin, n, ns, k, grid, occ, st);                           \
    }

}  // namespace hphi
