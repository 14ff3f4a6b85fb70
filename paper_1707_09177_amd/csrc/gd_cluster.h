// gd_cluster.h -- sums over the workgroups that share one field.
//
// A workgroup publishes its sums as 64-bit words of 32 payload bits and the
// 32-bit number of the reduction, so a word is valid by itself: no fence, no
// counter, one store and one load per word.  Two slot sets alternate: a
// workgroup can only be one reduction ahead of the slowest, which has then
// left the set before the last.  Sums are taken in workgroup order: the same
// result in every workgroup and every run.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gd_kernels.h"

namespace gdcl {

constexpr int kMaxW = 256;  // workgroups per field
constexpr int kWords = 6;   // words of a workgroup in a slot set: three sums

template <int WAVES>
struct Shared {
    double red[2][3][WAVES];
    double tot[2][3];
    int abort;
};

// v summed over groups of 2, 4, ... LANES lanes (16 or 64), in every lane, by
// DPP and half-exchanges: a step costs a few clocks where one through the LDS
// crossbar costs about 100
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int LANES>
__device__ __forceinline__ double lane_sum(double v) {
    v = dpp_add<0xB1>(v);   // quad_perm 1 0 3 2
    v = dpp_add<0x4E>(v);   // quad_perm 2 3 0 1
    v = dpp_add<0x141>(v);  // row_half_mirror: the other quad of 8
    v = dpp_add<0x140>(v);  // row_mirror: the other 8 of 16
    if constexpr (LANES == 64) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        auto halves = [&](auto swap) {
            const uint64_t x = __builtin_bit_cast(uint64_t, v);
            const u32x2 lo = swap((uint32_t)x), hi = swap((uint32_t)(x >> 32));
            const double a = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]);
            const double b = __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
            v = a + b;
        };
        halves([](uint32_t w) { return __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(w, w, false, false)); });
        halves([](uint32_t w) { return __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(w, w, false, false)); });
    }
    return v;
}

// One field's cluster of W workgroups.
struct Cluster {
    uint64_t *slot;    // [2][W][kWords], zero before the first reduction
    uint32_t *abort;   // set when a wait exceeded its bound
    int64_t wait_ticks;
    int W, wg;
    uint32_t seq;      // reductions done
};

// v, which is the same in every lane, in scalar registers
__device__ __forceinline__ double uniform(double v) {
    return __builtin_bit_cast(double, gd::wave_uniform(__builtin_bit_cast(int64_t, v)));
}

// v[k] summed over the cluster (the same value in every thread); false when
// the run was aborted.  WAVES: waves of the workgroup, at most 16.
template <int N, int WAVES>
__device__ __forceinline__ bool all_sum(Cluster &c, Shared<WAVES> &sh, double (&v)[N]) {
    static_assert(WAVES <= 16, "one row of lanes sums the waves");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int par = c.seq & 1;
    ++c.seq;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double s = lane_sum<64>(v[k]);
        if (lane == 0) sh.red[par][k][wave] = s;
    }
    __syncthreads();
    auto waves = [&](int k) {  // every row of 16 lanes sums the waves
        const int w = lane & 15;
        const double s = sh.red[par][k][w < WAVES ? w : 0];
        return lane_sum<16>(w < WAVES ? s : 0.0);
    };
    if (c.W == 1) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = uniform(waves(k));
        return true;
    }
    // the first wave publishes and collects
    if (wave == 0) {
        uint64_t *slot = c.slot + (int64_t)par * c.W * kWords;
        const uint64_t tag = (uint64_t)c.seq << 32;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const uint64_t bits = __builtin_bit_cast(uint64_t, waves(k));
            if (lane < 2)
                __hip_atomic_store(slot + (int64_t)c.wg * kWords + 2 * k + lane,
                                   tag | (lane == 0 ? bits & 0xffffffffull : bits >> 32), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        double s[N];
#pragma unroll
        for (int k = 0; k < N; ++k) s[k] = 0.0;
        const int64_t t0 = wall_clock64();
        for (int w = lane; w < c.W; w += 64) {
            uint64_t *p = slot + (int64_t)w * kWords;
            uint64_t x[2 * N];
            for (;;) {
                bool all = true;
#pragma unroll
                for (int k = 0; k < 2 * N; ++k) {
                    x[k] = __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    all = all && (uint32_t)(x[k] >> 32) == c.seq;
                }
                if (all) break;
                if (__hip_atomic_load(c.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
                    wall_clock64() - t0 > c.wait_ticks) {
                    __hip_atomic_store(c.abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    sh.abort = 1;
                    break;
                }
            }
#pragma unroll
            for (int k = 0; k < N; ++k)
                s[k] += __builtin_bit_cast(double, x[2 * k + 1] << 32 | (x[2 * k] & 0xffffffffull));
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double t = lane_sum<64>(s[k]);
            if (lane == 0) sh.tot[par][k] = t;
        }
    }
    __syncthreads();
    if (sh.abort) return false;
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = uniform(sh.tot[par][k]);
    return true;
}

}  // namespace gdcl
