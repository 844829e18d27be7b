// Reductions shared by the Schwarz kernels: wavefront sums by DPP row
// operations (no LDS crossbar) and workgroup sums through LDS.
#pragma once

#include "tm_device.h"

namespace tmsap {

// DPP move of one 32-bit word / of a value (rows outside ROW_MASK read 0).
template <int CTRL, int ROW_MASK>
__device__ inline int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, true);
}
template <int CTRL, int ROW_MASK>
__device__ inline float dpp_v(float v) {
    return __builtin_bit_cast(float, dpp_i<CTRL, ROW_MASK>(__builtin_bit_cast(int, v)));
}
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_v(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)dpp_i<CTRL, ROW_MASK>((int)(unsigned)b);
    const unsigned hi = (unsigned)dpp_i<CTRL, ROW_MASK>((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ inline float lane63(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ inline double lane63(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Wavefront sum: quad and row reductions, then row broadcasts; the total ends
// in lane 63.  Every lane of the wavefront must be active.
template <class R>
__device__ inline R wave_sum(R v) {
    v += dpp_v<0xb1, 0xf>(v);   // quad_perm [1,0,3,2]
    v += dpp_v<0x4e, 0xf>(v);   // quad_perm [2,3,0,1]
    v += dpp_v<0x114, 0xf>(v);  // row_shr:4
    v += dpp_v<0x118, 0xf>(v);  // row_shr:8
    v += dpp_v<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_v<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return lane63(v);
}

// Smallest normal number.  An MR step is taken only when <q,q> is at least
// this: a block whose residual has (nearly) vanished keeps e, and neither the
// hardware reciprocal nor a flushed division meets a subnormal divisor
// (which would turn the step length into inf or NaN).
template <class R>
__device__ constexpr R min_normal() {
    return sizeof(R) == 8 ? (R)2.2250738585072014e-308 : (R)1.17549435e-38f;
}

// The same by lane exchanges, for the FP64 kernel on blocks of up to 256 sites other than 4^4, which is 2 to 4 %
// faster with it (2^4 blocks on 16x12^3, 6 systems: 1195 us against 1240; the other FP64 kernels, on 8x4^3 blocks, are
// 10 to 18 % slower).
template <class R>
__device__ inline R wave_sum_xor(R v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sum of three values over the workgroup; every thread gets the result.
template <bool XOR = false, class R>
__device__ inline void block_sum3(R* red, R& a, R& b, R& c) {
    a = XOR ? wave_sum_xor(a) : wave_sum(a);
    b = XOR ? wave_sum_xor(b) : wave_sum(b);
    c = XOR ? wave_sum_xor(c) : wave_sum(c);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    if (lane == 0) {
        red[4 * w] = a;
        red[4 * w + 1] = b;
        red[4 * w + 2] = c;
    }
    __syncthreads();
    a = b = c = (R)0;
    for (int i = 0; i < nw; ++i) {
        a += red[4 * i];
        b += red[4 * i + 1];
        c += red[4 * i + 2];
    }
}

}  // namespace tmsap
