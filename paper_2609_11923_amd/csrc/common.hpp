// common.hpp -- device helpers shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

namespace cfrx {

constexpr int BLOCK = 256;

[[maybe_unused]] static inline unsigned grid_for(int64_t n) { return (unsigned)((n + BLOCK - 1) / BLOCK); }

__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float max_t(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double max_t(double a, double b) { return fmax(a, b); }

// child a of node n: explicit layouts list children, the breadth-first layout numbers them
template <bool EXPLICIT>
__device__ __forceinline__ int32_t child_of(const int32_t *__restrict__ kid, int32_t edge) {
    if constexpr (EXPLICIT) return kid[edge];
    else return edge;
}

// XCD-aware tile order.  The dispatcher hands the workgroups of a launch to the 8 XCDs in turn
// (workgroup b to XCD b mod 8) and each XCD has its own L2, so neighbouring tiles -- which share
// cache lines: the child values of interleaved information sets, the strategy rows of one set --
// would be fetched once per XCD.  Tiles are dealt out instead in runs of XCD_RUN consecutive tiles
// per XCD: workgroup b = 8 i + x runs tile (i / R) 8R + x R + (i mod R), R = XCD_RUN, a bijection
// of [0, M) with M the largest multiple of 8R not above n; tiles from M on keep their index.  Runs
// (rather than one contiguous eighth of the level per XCD) keep the XCDs' shares of a level
// alike where the work per tile drifts along it.  Measured: on the 256-subgame batch the update
// levels took 13 % less time than with the plain order, the large game was 1 % faster; one
// contiguous eighth per XCD was as fast on the batch but 3-7 % slower on the large game.
constexpr int32_t XCD_RUN = 16;
__device__ __forceinline__ int32_t xcd_tile(int32_t b, int32_t n) {
    const int32_t M = n / (8 * XCD_RUN) * (8 * XCD_RUN);
    if (b >= M) return b;
    const int32_t x = b & 7, i = b >> 3;
    return i / XCD_RUN * (8 * XCD_RUN) + x * XCD_RUN + i % XCD_RUN;
}

// Calls f with the smallest action bound of {2, 3, MAXA} (MAXA = 4) or {4, MAXA} (wider
// instantiations) that is at least n, as a compile-time constant, so a pass over sets or members
// that need fewer actions issues fewer loads (large game: FP64 state 5 % faster, FP32 unchanged; a
// 16-action instantiation would otherwise load 16 children per member of a 2-action set).  n must
// be uniform over the wave (or the block).
template <int MAXA, typename F>
__device__ __forceinline__ void with_action_bound(int32_t n, F &&f) {
    if constexpr (MAXA <= 4) {
        if (n <= 2) f(std::integral_constant<int, 2>{});
        else if (n <= 3) f(std::integral_constant<int, 3>{});
        else f(std::integral_constant<int, MAXA>{});
    } else {
        if (n <= 4) f(std::integral_constant<int, 4>{});
        else f(std::integral_constant<int, MAXA>{});
    }
}

}  // namespace cfrx
