// Lane exchanges inside a wave on the vector ALU (DPP) and the byte transposition shared by the
// integer-matrix-core kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace specache {
namespace {

// lane exchange patterns inside a row of 16 lanes
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppRowRor8 = 0x128;              // lane i <-> lane i ^ 8 inside a row of 16

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t max_u32(uint32_t a, uint32_t b) { return a > b ? a : b; }
// largest value of a wave; floats that are not negative order as their bits do
__device__ __forceinline__ uint32_t wave_max_bits(uint32_t v) {
    v = max_u32(v, dpp_move_u32<kDppXor1>(v));
    v = max_u32(v, dpp_move_u32<kDppXor2>(v));
    v = max_u32(v, dpp_move_u32<kDppHalfMirror>(v));
    v = max_u32(v, dpp_move_u32<kDppMirror>(v));
    const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return max_u32(max_u32(a, b), max_u32(c, d));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// bytes p = 0..3 of four 32-bit words, gathered per byte position: out[p] = (y0.p, y1.p, y2.p, y3.p)
__device__ __forceinline__ void byte_planes(uint32_t y0, uint32_t y1, uint32_t y2, uint32_t y3, uint32_t out[4]) {
    const uint32_t a_lo = __builtin_amdgcn_perm(y1, y0, 0x05010400u), a_hi = __builtin_amdgcn_perm(y1, y0, 0x07030602u);
    const uint32_t b_lo = __builtin_amdgcn_perm(y3, y2, 0x05010400u), b_hi = __builtin_amdgcn_perm(y3, y2, 0x07030602u);
    out[0] = __builtin_amdgcn_perm(b_lo, a_lo, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(b_lo, a_lo, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(b_hi, a_hi, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(b_hi, a_hi, 0x07060302u);
}

// 32-bit numbers below 2^30 in magnitude as four signed bytes each (the top one as it is), byte by byte as above: adding 0x80 to the
// low three bytes carries into the next one what a signed byte cannot hold, and flips its sign, which is flipped back behind the transposition
__device__ __forceinline__ void signed_byte_planes(const uint32_t y[4], uint32_t out[4]) {
    byte_planes(y[0] + 0x00808080u, y[1] + 0x00808080u, y[2] + 0x00808080u, y[3] + 0x00808080u, out);
    out[0] ^= 0x80808080u;
    out[1] ^= 0x80808080u;
    out[2] ^= 0x80808080u;
}
// the sum of products from those of the four byte planes (each below 2^18 in magnitude): two exact integer steps, one rounding of
// either half and one of their sum
__device__ __forceinline__ float of_byte_planes(int s0, int s1, int s2, int s3) {
    return __builtin_fmaf((float)(s2 + (s3 << 8)), 65536.0f, (float)(s0 + (s1 << 8)));
}

// The lanes of a wave run in lockstep and LDS serves one wave's accesses in order: a wave-level
// fence is all an exchange through a wave-private LDS area needs.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace
}  // namespace specache
