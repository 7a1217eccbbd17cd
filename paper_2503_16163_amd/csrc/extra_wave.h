// One wave's share of the 16-bit candidates of the mixed attention of Eq. 1 (staged pairs, residual, the speculative
// token's transient pair): 32 of them, the keys times the queries on the matrix cores in the cache's own type, the values on
// the vector ALUs.  The chain of dependent loads, not the arithmetic, is what this chunk of a launch takes: the index list, the
// keys (the first 16 bytes of either tile are waited for by themselves, being loads behind a condition), then the values
// (AHEAD of them with the keys).  The addresses come from several buffers, so that keys and values are flat loads, which
// also hold back the reads of the queries from LDS.  A workgroup of 128 candidates
// that went from barrier to barrier, its values requested in batches of 8 behind the softmax, took 10.8 us alone
// with two query rows and was the last to end in a launch over 32 rows x 16384 positions (16.0 of 16.6 us); a wave each
// takes 4.6 us alone (that kernel over 1 x 4096 positions: 10.8 -> 5.4 us) and 11.2 there.  In the kernels of attention alone, us a
// pass: non-speculative 32 x 8192 444 -> 425, 4 heads on 2, 2000 positions 257 -> 211, one layer of 32 x 16000 56 -> 49.
#pragma once
#include "attend_common.h"

namespace specache {
namespace {

typedef __bf16 bfloat8 __attribute__((ext_vector_type(8)));

constexpr int kRowsOStride = kD + 4;           // floats between the columns of a wave's merged outputs
constexpr float kLog2e = 1.44269504088896340736f;

// lane exchange across the 16-lane rows of a wave: result pairs of lanes 16 (32) apart
__device__ __forceinline__ float xor16_max(float v) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ float xor32_max(float v) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ float xor16_sum(float v) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float xor32_sum(float v) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float quarters_max(float v) { return xor32_max(xor16_max(v)); }
__device__ __forceinline__ float quarters_sum(float v) { return xor32_sum(xor16_sum(v)); }

__device__ __forceinline__ float4v mfma16(uint4v a, uint4v b, float4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}
// the product of 16-bit inputs of the cache's own type: exact products, fp32 accumulation
template <bool BF16>
__device__ __forceinline__ float4v mfma_native(uint4v a, uint4v b, float4v c) {
    if constexpr (BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bfloat8, a), __builtin_bit_cast(bfloat8, b), c, 0, 0, 0);
    else return mfma16(a, b, c);
}

__device__ __forceinline__ float exp2_of(float x) { return __builtin_amdgcn_exp2f(x); }

// what the waves hand to the merge, per column (r, s): softmax maximum and sum; the merge turns the maximum into the weight
struct RowsOut {
    float m[kWaves][16], l[kWaves][16], w[kWaves][16];
};

// ---- one wave's 32 candidates in 16 bits: staged pairs, residual, the speculative pair ---------------------------
// The staged positions of a lane's two candidates (x0 + 2 (lane % 16), + 1), requested ahead of everything else: where they lead decides
// what the rest of the chunk reads (behind the queries' exchange: 24 x 5003 with 8 query rows 266 us a pass, now 262).  Beyond the
// list: 0, and the candidate is another kind.
__device__ __forceinline__ int2 staged_positions(const LayerView& L, const AttendArgs& A, int row, int x0, int lane) {
    const auto list = buffer_of(A.slot_idx ? A.slot_idx + (size_t)row * L.topk : nullptr, A.slot_idx ? (uint32_t)L.topk * 4u : 0u);
    const int at = (x0 + 2 * (lane & 15)) * 4;
    return make_int2((int)__builtin_amdgcn_raw_buffer_load_b32(list, at, 0, 0), (int)__builtin_amdgcn_raw_buffer_load_b32(list, at + 4, 0, 0));
}

// staged: staged_positions of the wave; weights: [32][NR] of the wave; o_lds: [kWaves][O_ROWS][kRowsOStride], may lie over the query rows and the weights.
// AHEAD: values requested with the keys (32: all of them), the others once the keys are used up, which takes fewer registers.
template <int NR, bool BF16, int O_ROWS = 16, int AHEAD = 32>
__device__ __forceinline__ void rows_extra_wave(const LayerView& L, const AttendArgs& A, int n_rows, int row, int x0, int2 staged, int lane, int wave,
                                                const uint16_t* qraw, int q_stride, float* weights, float* o_lds, RowsOut& out) {
    const int ic = lane & 15, kq = lane >> 4, r = ic % NR, s = ic / NR;
    const int ks = A.slot_idx ? L.topk : 0, n_res = A.N - A.Nq, n_ex = ks + n_res + (A.k_spec ? 1 : 0);
    // A rows: tile mt, row ic is candidate x0 + 2 ic + mt
    const uint16_t* kp[2];
    const uint16_t* vp[2];
    bool spec[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const int x = x0 + 2 * ic + mt;
        kp[mt] = nullptr;
        spec[mt] = false;
        if (x < ks) {
            const int t = mt ? staged.y : staged.x;
            if (t >= 0 && t < A.Nq) kp[mt] = A.slot + ((size_t)row * L.topk + x) * 256;
        } else if (x < ks + n_res) {
            const int t = A.Nq + (x - ks);
            kp[mt] = L.ring + ((size_t)row * L.R + (t % L.R)) * 256;
        } else {
            spec[mt] = x < n_ex;
        }
        vp[mt] = kp[mt] ? kp[mt] + kD : nullptr;
        // a token that this very launch appends (its copy into the ring may not have landed yet) is read from the
        // caller's buffers, and so is the speculative pair
        if (L.tail_k != nullptr && x >= ks && x < ks + n_res && A.Nq + (x - ks) == L.tail_N0) {
            kp[mt] = L.tail_k + (size_t)row * kD;
            vp[mt] = L.tail_v + (size_t)row * kD;
        }
        if (spec[mt]) {
            kp[mt] = A.k_spec + (size_t)row * kD;
            vp[mt] = A.v_spec + (size_t)row * kD;
        }
    }
    // one or two rows look at the weights before the values: where there is no pair any 256 bytes do, and the loads need no branches
    if constexpr (NR <= 2)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) vp[mt] = vp[mt] ? vp[mt] : A.q + (size_t)row * NR * kD;
    uint4v kb[2][4];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int kc = 0; kc < 4; ++kc)
            kb[mt][kc] = kp[mt] ? *reinterpret_cast<const uint4v*>(kp[mt] + 32 * kc + 8 * kq) : uint4v{0u, 0u, 0u, 0u};
    // value rows: lane = channel pair, one 256-byte row per candidate (lane 2 ic + mt / 2 of the wave knows where)
    uint32_t vw[32];
    auto load_value = [&](int i) {
        const uint64_t p = (uint64_t)(uintptr_t)vp[i & 1];
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)p, i >> 1), hi = __builtin_amdgcn_readlane((uint32_t)(p >> 32), i >> 1);
        const uint16_t* v = reinterpret_cast<const uint16_t*>((uintptr_t)(((uint64_t)hi << 32) | lo));
        if constexpr (NR <= 2) vw[i] = *reinterpret_cast<const uint32_t*>(v + 2 * lane);
        else vw[i] = v ? *reinterpret_cast<const uint32_t*>(v + 2 * lane) : 0u;
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load_value(i);
    if constexpr (AHEAD < 32) __builtin_amdgcn_sched_barrier(0);
    float4v acc[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) {
        const uint4v b = *reinterpret_cast<const uint4v*>(qraw + r * q_stride + 32 * kc + 8 * kq);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) acc[mt] = mfma_native<BF16>(kb[mt][kc], b, acc[mt]);
    }
    if constexpr (AHEAD < 32) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = AHEAD; i < 32; ++i) load_value(i);
    // C row 4 kq + v of tile mt is candidate x0 + 8 kq + 2 v + mt.  Which of them exist, and which is the speculative
    // pair: one bit per candidate, from the lanes of the first quarter
    const unsigned long long have0 = __ballot(kp[0] != nullptr) & 0xFFFFull, have1 = __ballot(kp[1] != nullptr) & 0xFFFFull;
    const unsigned long long spec0 = __ballot(spec[0]) & 0xFFFFull, spec1 = __ballot(spec[1]) & 0xFFFFull;
    const bool last = r % n_rows == n_rows - 1;
    float l[8], m = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const int i = 4 * kq + v;
            const bool sees = s == 0 && (((mt ? have1 : have0) >> i) & 1) && (last || !(((mt ? spec1 : spec0) >> i) & 1));
            l[2 * v + mt] = sees ? acc[mt][v] * A.sm_scale : -INFINITY;
            m = fmaxf(m, l[2 * v + mt]);
        }
    m = quarters_max(m);
    const float ms = m == -INFINITY ? 0.0f : m;
    float sum = 0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float p = exp2_of((l[t] - ms) * kLog2e);
        sum += p;
        if (s == 0) weights[(8 * kq + t) * NR + r] = p;
    }
    sum = quarters_sum(sum);
    if (kq == 0) {
        out.m[wave][ic] = m;
        out.l[wave][ic] = sum;
    }
    wave_sync();
    float o[NR][2];
#pragma unroll
    for (int rr = 0; rr < NR; ++rr) o[rr][0] = o[rr][1] = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const float v0 = widen16<BF16>(vw[i] & 0xFFFFu), v1 = widen16<BF16>(vw[i] >> 16);
        if constexpr (NR == 1) {
            const float p = weights[i];
            const bool use = p != 0.0f;
            o[0][0] = __builtin_fmaf(p, use ? v0 : 0.0f, o[0][0]);
            o[0][1] = __builtin_fmaf(p, use ? v1 : 0.0f, o[0][1]);
        }
        if constexpr (NR == 2) {
            const float2 p = *reinterpret_cast<const float2*>(weights + i * 2);
            const bool use = p.x != 0.0f || p.y != 0.0f;      // a value that nobody weighs may be infinite
            const float u0 = use ? v0 : 0.0f, u1 = use ? v1 : 0.0f;
            o[0][0] = __builtin_fmaf(p.x, u0, o[0][0]);
            o[0][1] = __builtin_fmaf(p.x, u1, o[0][1]);
            o[1][0] = __builtin_fmaf(p.y, u0, o[1][0]);
            o[1][1] = __builtin_fmaf(p.y, u1, o[1][1]);
        }
#pragma unroll
        for (int r4 = 0; r4 < NR / 4; ++r4) {
            const float4 p = *reinterpret_cast<const float4*>(weights + i * NR + 4 * r4);
            const float pv[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[4 * r4 + e][0] = __builtin_fmaf(pv[e], v0, o[4 * r4 + e][0]);
                o[4 * r4 + e][1] = __builtin_fmaf(pv[e], v1, o[4 * r4 + e][1]);
            }
        }
    }
    __syncthreads();   // every wave is done with its weights and with the query rows: the outputs take their place
#pragma unroll
    for (int rr = 0; rr < NR; ++rr)
        *reinterpret_cast<float2*>(o_lds + ((size_t)wave * O_ROWS + rr) * kRowsOStride + 2 * lane) = make_float2(o[rr][0], o[rr][1]);
}

// A workgroup's chunk of up to 128 16-bit candidates for one or two query rows: a wave each per 32, merged into the chunk's partials.
// smem: extra_chunk_floats(NR) floats, 16-byte aligned.
constexpr int kExtraQStride = kD + 8;                                      // halves between the query rows
__host__ __device__ constexpr int extra_chunk_floats(int NR) {
    return NR * kExtraQStride / 2 + kWaves * 32 * NR > kWaves * NR * kRowsOStride ? NR * kExtraQStride / 2 + kWaves * 32 * NR : kWaves * NR * kRowsOStride;
}
template <int NR, int NROWS, bool BF16, int AHEAD, typename Buffer>
__device__ __forceinline__ void extra_chunk(const LayerView& L, const AttendArgs& A, int row, int chunk, float* smem, RowsOut& out, Buffer po,
                                            Buffer pml, bool past_l2) {
    static_assert(NR <= 2 && (NR * kExtraQStride / 2) % 4 == 0, "a thread per output");
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    uint16_t* qraw = reinterpret_cast<uint16_t*>(smem);
    const int x0 = ((chunk - A.n_main) * kWaves + wave) * 32;
    const int2 staged = staged_positions(L, A, row, x0, lane);
    if (wave < NR) reinterpret_cast<uint32_t*>(qraw + wave * kExtraQStride)[lane] = reinterpret_cast<const uint32_t*>(A.q + ((size_t)row * NR + wave) * kD)[lane];
    __syncthreads();
    rows_extra_wave<NR, BF16, NR, AHEAD>(L, A, NROWS, row, x0, staged, lane, wave, qraw, kExtraQStride, smem + NR * kExtraQStride / 2 + wave * 32 * NR,
                                         smem, out);
    __syncthreads();
    const int r = tid >> 7, c = tid & 127;
    if (r < NR) {
        float mx = -INFINITY, o = 0.0f, sum = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, out.m[w][r]);
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float e = out.m[w][r] == -INFINITY ? 0.0f : exp2_of((out.m[w][r] - mx) * kLog2e);
            if (e != 0.0f) o = __builtin_fmaf(e, smem[(w * NR + r) * kRowsOStride + c], o);
            sum = __builtin_fmaf(e, out.l[w][r], sum);
        }
        store_partial(po, r * kD + c, o, past_l2);
        if (c == 0) store_max_sum(pml, r, mx, sum, past_l2);
    }
}

}  // namespace
}  // namespace specache
