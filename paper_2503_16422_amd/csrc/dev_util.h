// Device helpers shared by the integer kernels: wave64 and block scans.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fdgs {

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

// XCD-aware item of block b in a grid of n blocks.  Workgroups go to the
// eight XCDs (each with its own L2) round-robin by block index; here the
// blocks of one XCD take one contiguous range of items, so that neighbouring
// items -- which share cache lines of column-major histograms and of the runs
// a radix pass scatters -- are handled under one L2 and their partial-line
// writes merge there instead of reaching HBM separately.  A bijection of
// [0, n): XCD x takes n / 8 items, one more when x < n % 8.
__device__ __forceinline__ int64_t xcd_item(int64_t b, int64_t n) {
    constexpr int64_t kXcds = 8;
    const int64_t q = n / kXcds, r = n % kXcds, x = b % kXcds;
    return x * q + min(x, r) + b / kXcds;
}

// Inclusive sum over the 64 lanes of a wavefront: shifts by 1, 2, 4 and 8
// within each row of 16 lanes, then row broadcasts 15 and 31, all as DPP
// operands (six dependent additions; six shuffles through LDS took ten times
// as long, and nearly every front-end kernel waits for a few of these).  A lane
// whose source lies outside its row adds 0.  Compiled for the host (the
// kernels' emulation in the tests), it is the shuffle form.
#if defined(__AMDGCN__)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_from(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint64_t dpp_from(uint64_t v) {
    return (uint64_t)dpp_from<CTRL, ROW_MASK>((uint32_t)(v >> 32)) << 32 | dpp_from<CTRL, ROW_MASK>((uint32_t)v);
}
template <typename T>
__device__ __forceinline__ T wave_inclusive_sum(T v) {
    v += dpp_from<0x111, 0xf>(v);    // row_shr:1
    v += dpp_from<0x112, 0xf>(v);    // row_shr:2
    v += dpp_from<0x114, 0xf>(v);    // row_shr:4
    v += dpp_from<0x118, 0xf>(v);    // row_shr:8
    v += dpp_from<0x142, 0xa>(v);    // row_bcast:15 into rows 1 and 3
    v += dpp_from<0x143, 0xc>(v);    // row_bcast:31 into rows 2 and 3
    return v;
}
#else
template <typename T>
__device__ __forceinline__ T wave_inclusive_sum(T v) {
    const int lane = lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T o = __shfl_up(v, off, 64);
        if (lane >= off) v += o;
    }
    return v;
}
#endif

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sums with DPP row operations (no LDS traffic).  Steps: xor-1 and xor-2 inside
// quads, half-row mirror, row mirror (every lane then holds its 16-lane row
// sum); the row broadcast 15 folds rows 0 and 2 into rows 1 and 3.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_add_c(float v) {
    const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, true);
    return v + __builtin_bit_cast(float, o);
}
// Sum over each row of 16 lanes, valid in every lane of the row.
__device__ __forceinline__ float row_sum16(float v) {
    v = dpp_add_c<0xB1>(v);          // quad_perm(1,0,3,2)
    v = dpp_add_c<0x4E>(v);          // quad_perm(2,3,0,1)
    v = dpp_add_c<0x141>(v);         // row_half_mirror
    v = dpp_add_c<0x140>(v);         // row_mirror
    return v;
}
// Sum over each half of the wavefront (32 lanes), valid in lanes 31 and 63.
__device__ __forceinline__ float half_sum32(float v) {
    v = row_sum16(v);
    v = dpp_add_c<0x142, 0xa>(v);    // row_bcast:15 into rows 1 and 3
    return v;
}
// Exclusive sum over a block of NT threads (NT a multiple of 64, <= 1024).
// `tmp` must hold NT/64 elements of shared memory.  Returns the thread's
// exclusive prefix; *total receives the block total.  Every thread adds up the
// wavefronts' totals itself (broadcast reads).  Contains barriers.
template <int NT, typename T>
__device__ __forceinline__ T block_exclusive_sum(T v, T *tmp, T *total) {
    constexpr int NW = NT / 64;
    const T inc = wave_inclusive_sum(v);
    if (lane_id() == 63) tmp[wave_id()] = inc;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const T x = tmp[w];
        if (w < wave_id()) before += x;
        all += x;
    }
    *total = all;
    __syncthreads();
    return before + inc - v;
}

}  // namespace fdgs
