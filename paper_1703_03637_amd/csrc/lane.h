// Device helpers shared by the product kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "hphi_internal.h"

namespace hphi {
namespace {

constexpr int ilog2(int b) { return b <= 1 ? 0 : 1 + ilog2(b / 2); }

template <int B>
struct Log2 {
    static_assert(B > 0 && (B & (B - 1)) == 0, "power of two");
    static constexpr int value = ilog2(B);
};

__device__ __forceinline__ int wave_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// ---- lane share of an interleaved row.  A row of nvec vectors is split
// over LPR lanes in chunks of CB = min(16, lane bytes) bytes, dealt
// round-robin: lane `sub` owns chunks sub, sub + LPR, sub + 2 LPR, ...  One
// 16-byte load instruction of the LPR lanes of a row therefore reads
// LPR * 16 contiguous bytes of it (a whole 128-byte line at LPR = 8), so
// no line is requested by several instructions.
template <typename S, int NE, int LPR>
struct LaneLayout {
    static constexpr int LB = NE * int(sizeof(S));     // bytes per lane per row
    static constexpr int CB = LB >= 16 ? 16 : LB;      // chunk bytes
    static constexpr int NCH = LB / CB;                // chunks per lane
    static constexpr int CPS = CB / int(sizeof(S));    // scalars per chunk
    static constexpr int RB = LB * LPR;                // row bytes
};

template <int CB>
__device__ __forceinline__ void copy_chunk(char* dst, const char* src) {
    if constexpr (CB == 16) {
        const uint4 w = *reinterpret_cast<const uint4*>(src);
        __builtin_memcpy(dst, &w, 16);
    } else if constexpr (CB == 8) {
        const uint2 w = *reinterpret_cast<const uint2*>(src);
        __builtin_memcpy(dst, &w, 8);
    } else {
        static_assert(CB == 4, "chunk of 4, 8 or 16 bytes");
        const uint32_t w = *reinterpret_cast<const uint32_t*>(src);
        __builtin_memcpy(dst, &w, 4);
    }
}

template <int CB>
__device__ __forceinline__ void put_chunk(char* dst, const char* src) {
    if constexpr (CB == 16) {
        uint4 w;
        __builtin_memcpy(&w, src, 16);
        *reinterpret_cast<uint4*>(dst) = w;
    } else if constexpr (CB == 8) {
        uint2 w;
        __builtin_memcpy(&w, src, 8);
        *reinterpret_cast<uint2*>(dst) = w;
    } else {
        uint32_t w;
        __builtin_memcpy(&w, src, 4);
        *reinterpret_cast<uint32_t*>(dst) = w;
    }
}

// streaming variants: non-temporal hint (data not reused, should not evict
// the L2 window of the gathers)
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

template <int CB>
__device__ __forceinline__ void copy_chunk_nt(char* dst, const char* src) {
    if constexpr (CB == 16) {
        const u32x4_t w = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(src));
        __builtin_memcpy(dst, &w, 16);
    } else if constexpr (CB == 8) {
        const u32x2_t w = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(src));
        __builtin_memcpy(dst, &w, 8);
    } else {
        const uint32_t w = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(src));
        __builtin_memcpy(dst, &w, 4);
    }
}

template <int CB>
__device__ __forceinline__ void put_chunk_nt(char* dst, const char* src) {
    if constexpr (CB == 16) {
        u32x4_t w;
        __builtin_memcpy(&w, src, 16);
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4_t*>(dst));
    } else if constexpr (CB == 8) {
        u32x2_t w;
        __builtin_memcpy(&w, src, 8);
        __builtin_nontemporal_store(w, reinterpret_cast<u32x2_t*>(dst));
    } else {
        uint32_t w;
        __builtin_memcpy(&w, src, 4);
        __builtin_nontemporal_store(w, reinterpret_cast<uint32_t*>(dst));
    }
}

template <typename S, int NE, int LPR>
__device__ __forceinline__ void load_lane(const S* __restrict__ base, int64_t row, int sub, S (&out)[NE]) {
    using Ly = LaneLayout<S, NE, LPR>;
    const char* p = reinterpret_cast<const char*>(base) + row * Ly::RB + sub * Ly::CB;
#pragma unroll
    for (int j = 0; j < Ly::NCH; ++j)
        copy_chunk<Ly::CB>(reinterpret_cast<char*>(out) + j * Ly::CB, p + j * LPR * Ly::CB);
}

template <typename S, int NE, int LPR>
__device__ __forceinline__ void store_lane(S* __restrict__ base, int64_t row, int sub, const S (&in)[NE]) {
    using Ly = LaneLayout<S, NE, LPR>;
    char* p = reinterpret_cast<char*>(base) + row * Ly::RB + sub * Ly::CB;
#pragma unroll
    for (int j = 0; j < Ly::NCH; ++j)
        put_chunk<Ly::CB>(p + j * LPR * Ly::CB, reinterpret_cast<const char*>(in) + j * Ly::CB);
}

// the lane's share of the row at byte address rowp
template <typename S, int NE, int LPR>
__device__ __forceinline__ void load_lane_at(const char* rowp, int sub, S (&out)[NE]) {
    using Ly = LaneLayout<S, NE, LPR>;
    const char* p = rowp + sub * Ly::CB;
#pragma unroll
    for (int j = 0; j < Ly::NCH; ++j)
        copy_chunk<Ly::CB>(reinterpret_cast<char*>(out) + j * Ly::CB, p + j * LPR * Ly::CB);
}

// branch-free choice between two values by a lane mask (all ones / zero):
// a bitwise select, so no register array is ever indexed per lane
__device__ __forceinline__ double pick(uint32_t m, double a, double b) {
    const uint64_t mm = (uint64_t(m) << 32) | m;
    const uint64_t ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    return __longlong_as_double(static_cast<long long>((ua & mm) | (ub & ~mm)));
}

// Reduce one quantity over the rows held by a wavefront.  Each lane holds
// VPL per-row values (its share of the vectors); afterwards lane L holds the
// wave sum for the local vector L >> (6 - log2 VPL) of share L & (LPR-1)
// (vec_lane maps a vector to its share and local index).  Every step is
// FP64.
template <typename R, int VPL, int LPR>
__device__ __forceinline__ double wave_reduce_rows(R (&x)[VPL], int lane) {
    constexpr int LOGV = Log2<VPL>::value;
#pragma unroll
    for (int j = 0; j < LOGV; ++j) {
        const int half = (VPL >> j) >> 1, off = 32 >> j;
        const uint32_t up = (lane & off) ? 0xffffffffu : 0u;
#pragma unroll
        for (int i = 0; i < half; ++i) {
            const R lo = x[i], hi = x[i + half];
            const R send = pick(up, lo, hi);
            const R keep = pick(up, hi, lo);
            x[i] = keep + __shfl_xor(send, off, 64);
        }
    }
    double r = double(x[0]);
#pragma unroll
    for (int off = 32 >> LOGV; off >= LPR; off >>= 1) r += __shfl_xor(r, off, 64);
    return r;
}

}  // namespace
}  // namespace hphi
