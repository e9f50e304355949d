// Wavefront and workgroup helpers shared by the kernels: loops over compile-time
// indices, lane moves and sums in registers, the block order of the XCDs.
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

namespace nh {

// Workgroups are handed to the 8 XCDs round robin (b mod 8), and each XCD has
// its own L2.  Give XCD x the contiguous range [x q + min(x, r), ...)
// (q = n / 8, r = n mod 8): blocks that run at the same time on one XCD are
// neighbours whose x/y halos overlap, so halo re-reads hit that L2.
__device__ __forceinline__ int xcd_block(int b, int n)
{
    const int q = n >> 3, r = n & 7, x = b & 7, j = b >> 3;
    return x * q + (x < r ? x : r) + j;
}

template <class F, int... J>
__device__ __forceinline__ void static_for_impl(F &f, std::integer_sequence<int, J...>)
{
    (f(std::integral_constant<int, J>{}), ...);
}
// f(integral_constant<int, j>) for j = 0 .. n-1, in order
template <int n, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, n>{});
}

__device__ __forceinline__ double join_d(unsigned lo, unsigned hi)
{
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// DPP lane move; lanes without a source read 0.
template <int CTRL>
__device__ __forceinline__ double lane_move(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return join_d((unsigned)lo, (unsigned)hi);
}
constexpr int kSwapPair = 0xB1;     // quad_perm [1,0,3,2]: lane i <-> lane i ^ 1
constexpr int kSwapTwo = 0x4E;      // quad_perm [2,3,0,1]
constexpr int kHalfMirror = 0x141;  // lane i of a half of a 16-lane row <- lane 7 - i of it
constexpr int kRowMirror = 0x140;   // lane i of a row <- lane 15 - i

// every lane of each 16-lane row <- the sum over its row
__device__ __forceinline__ double row_sum(double v)
{
    v += lane_move<kSwapPair>(v);
    v += lane_move<kSwapTwo>(v);
    v += lane_move<kHalfMirror>(v);
    v += lane_move<kRowMirror>(v);
    return v;
}

// gfx950 exchanges between two registers (one 16-lane row is a "row"):
// swap32: a <- [a lanes 0-31, b lanes 0-31], b <- [a lanes 32-63, b lanes 32-63]
// swap16: a <- [a row 0, b row 0, a row 2, b row 2], b <- [a row 1, b row 1, a row 3, b row 3]
__device__ __forceinline__ void swap32(double &a, double &b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    a = join_d(lo[0], hi[0]);
    b = join_d(lo[1], hi[1]);
}

__device__ __forceinline__ void swap16(double &a, double &b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    a = join_d(lo[0], hi[0]);
    b = join_d(lo[1], hi[1]);
}

// orders the wave's own LDS accesses
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

}  // namespace nh
