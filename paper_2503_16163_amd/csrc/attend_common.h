// Pieces of the mixed attention of Eq. 1 (Section 3.3) shared by the attention kernels: wave reductions and the
// stores of a chunk's partial results (the 16-bit candidates: extra_wave.h).
#pragma once
#include "kernels.h"
#include "layout.h"
#include "rows_args.h"
#include "wave_ops.h"

namespace specache {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kExtraChunk = 128;

template <int B>
__device__ __forceinline__ float cvt_ubyte(uint32_t w) {
    float f;
    if constexpr (B == 0) asm("v_cvt_f32_ubyte0 %0, %1" : "=v"(f) : "v"(w));
    if constexpr (B == 1) asm("v_cvt_f32_ubyte1 %0, %1" : "=v"(f) : "v"(w));
    if constexpr (B == 2) asm("v_cvt_f32_ubyte2 %0, %1" : "=v"(f) : "v"(w));
    if constexpr (B == 3) asm("v_cvt_f32_ubyte3 %0, %1" : "=v"(f) : "v"(w));
    return f;
}

__device__ __forceinline__ uint32_t comp(const uint4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// Operands of v_mfma_f32_16x16x32_f16: lane l holds A[l % 16][8 (l / 16) .. + 7] and
// B[8 (l / 16) .. + 7][l % 16] as eight f16, and C[4 (l / 16) .. + 3][l % 16] as four floats.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

// Wave-wide reductions on the VALU: four DPP steps leave every lane with its 16-lane row's
// result, the four row results are then read as scalars.  (A butterfly of ds_bpermute
// shuffles costs an LDS round trip per step.)
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_move<kDppXor1>(v));
    v = fmaxf(v, dpp_move<kDppXor2>(v));
    v = fmaxf(v, dpp_move<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_move<kDppMirror>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_move<kDppXor1>(v);
    v += dpp_move<kDppXor2>(v);
    v += dpp_move<kDppHalfMirror>(v);
    v += dpp_move<kDppMirror>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Partials that another workgroup of the same launch merges (finish_row.h) are stored past the L2.
constexpr int kAgentScope = 16;   // cache policy bit sc1 of a buffer load or store: device scope, where the L2 caches meet

__device__ __forceinline__ auto buffer_of(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00027000);
}
// a chunk's partials: output e of [NR][128], outputs 4 e to 4 e + 3, and the maximum and sum of row r
template <typename Buffer>
__device__ __forceinline__ void store_partial(Buffer po, int e, float v, bool past_l2) {
    if (past_l2) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), po, e * 4, 0, kAgentScope);
    else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), po, e * 4, 0, 0);
}
template <typename Buffer>
__device__ __forceinline__ void store_partials(Buffer po, int e, float4v v, bool past_l2) {
    if (past_l2) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, v), po, e * 16, 0, kAgentScope);
    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, v), po, e * 16, 0, 0);
}
template <typename Buffer>
__device__ __forceinline__ void store_max_sum(Buffer pml, int r, float m, float sum, bool past_l2) {
    typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
    const uint2v v = {__float_as_uint(m), __float_as_uint(sum)};
    if (past_l2) __builtin_amdgcn_raw_buffer_store_b64(v, pml, r * 8, 0, kAgentScope);
    else __builtin_amdgcn_raw_buffer_store_b64(v, pml, r * 8, 0, 0);
}

}  // namespace
}  // namespace specache
