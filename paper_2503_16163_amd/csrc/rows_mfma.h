// Scoring and mixed attention for several query rows per KV head (grouped-query attention: 4, 8 or 16 rows; 1 to 16 on 4-bit codes)
// on the f16 matrix cores: the low-bit scoring of Appendix A "Decoding" (A = Q K^T on C'), the mixed attention of
// Eq. 1, or both in one pass over the packed cache (the logits then never leave the chip).
//
// Both contractions have the packed codes as their A operand, read as f16 subnormals straight from the packed
// bytes: a dword is two 16-bit halves of 2-bit (1-, 4-bit) fields, and a shift and a mask leave one field of either
// half at bits 8 and 9 (4-bit codes: 6 to 9), as high as a subnormal goes (see rows_normal_operands).  0.94 vector
// instructions per 2-bit code.
//   scoring  logit[r][i] = sum_c code[i][c] (sm q[r][c] s[j][c]) + sm sum_c q[r][c] z[j][c],  j = i / g
//            B = the multipliers of (row, token group) as hi + lo f16: to 2^-23 of a multiplier down to 2^-3, to 2^-25 below;
//   values   o[r][c] = sum_i code[i][c] (p[r][i] s[i][m]) + sum_i p[r][i] z[i][m],  m = c / g
//            B = p s as hi + lo f16, the scale factor of each value group following the scales of the unit's tokens.
// Building the operands is what bounds these shapes (vector-instruction issue: at 8 rows, g = 64 400 vector instructions
// per 32 tokens, each of a SIMD's three waves issuing 29 % of its life), so no lane does it twice: the 16 columns are
// (row r, sub-group s) with 16 / NR sub-groups of 32 tokens in flight.  For 8 rows the two lanes of a row then exchange
// halves, so that the columns of a product are (r, hi | lo) and every column of it is used (the matrix cores are not
// free: 16 clocks each), and hi and lo add up in sums of their own;
// with 16 rows the columns are the rows.
// A lane (column (r, s), quarter kq) ends the scoring with the logits of row r for 8 consecutive tokens, which is the
// order in which the value side wants its B operand: no logit is exchanged between lanes.
//
// A wave walks units of 32 * 16 / NR tokens with a running softmax maximum per row (moved only when a logit exceeds it
// by 4, so that the accumulators are rescaled rarely); the loads of the next unit travel while the other half of the
// current one is worked on.  The four waves of a workgroup merge once, at the end.  The 16-bit candidates are a wave
// each per 32: the keys times the queries on the matrix cores in their own type, the values on the vector ALUs.
//
// Measured on MI355X (scoring + attention as two launches of the kernels before it -> as one launch; then with the first
// loads requested together and a merge of the waves that reads 16 bytes at a time, 0.8 us instead of 2.5 to 2.8): 32 KV rows x 32768 tokens, 8 query rows, 2 bits, g = 64: 27.5 +
// 37.9 -> 37.2 -> 33.5 us; 8 x 131072, 1 bit, g = 32: 33.1 + 43.9 -> 43.2 -> 39.6 us; 24 x 5003, 2 bits, g = 32: 8.5 + 24.8 -> 13.0
// at best -> 10.3 at best, 12.3 beside the gathers; 16 x 8192, 16 query rows, g = 128: 10.8 + 40.2 -> 17.0 -> 13.6 us.  4-bit codes,
// two launches, 32 x 16384, 2 query rows as 8 columns' worth, g = 32: scoring 13.9, attention with its merge 18.9 us at best, 16.0 and 21.4 beside
// the gathers (the 84 MB they read need 14 us at the rate of a plain read); a decode step of a layer 70.7 -> 51 us against
// vector-ALU kernels.  (The figures are the kernel's without the merge of a row's chunks, which the launch does as well where they are at most
// 128: 4.4 us of a launch of its own before, 3.6 of this one's 37.1 and 4.6 of 44.5 now, beside the fetches and a profiler.)
// Up to 168 registers, three workgroups per compute unit; held to four it spills (as it is, both passes in groups of 32 with 8 columns' worth of
// rows spill two registers with 2 bits, one with 1 bit where rows are missing).
#pragma once
#include "attend_common.h"
#include "extra_wave.h"
#include "finish_row.h"
#include "rows_args.h"

namespace specache {
namespace {

constexpr float kLazyMax = 4.0f;               // a column's maximum moves when a logit exceeds it by more than this
// The f16 operands are hi + lo (23 bits of a product's multiplier as long as hi is at least 2^-3, an absolute 2^-25 below
// that), so the scales that go into them are kept near the top of the range: times a power of two, 2^3 to 2^9 for the value
// scales (p < 2^6), 2^4 to 2^8 for the key scales (|q'| < 2^7), moved where a unit's largest one leaves these bounds.
constexpr float kValueScaleMost = 512.0f, kValueScaleLeast = 8.0f, kKeyScaleMost = 256.0f, kKeyScaleLeast = 16.0f;
constexpr int kScaleSet = 7;

// hi halves of the lanes of sub-group 0 beside lo halves of sub-group 1's lanes, or the other way round: with the two lanes of a
// row (8 apart) holding (hi, lo) of sub-groups 0 and 1, columns (r, hi | lo) of sub-group 0 and of sub-group 1
__device__ __forceinline__ void hi_lo_columns(const uint4v& hi, const uint4v& lo, uint4v& sub0, uint4v& sub1) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        sub0[d] = (uint32_t)__builtin_amdgcn_update_dpp((int)hi[d], (int)lo[d], kDppRowRor8, 0xf, 0xc, false);
        sub1[d] = (uint32_t)__builtin_amdgcn_update_dpp((int)lo[d], (int)hi[d], kDppRowRor8, 0xf, 0x3, false);
    }
}
__device__ __forceinline__ float times_pow2(float x, int e) { return __builtin_amdgcn_ldexpf(x, e); }

// Codes as normal numbers instead of subnormals, at half a vector instruction more per code.  The matrix cores align products
// by their operands' exponents, so that a subnormal code gives up the low end of the other products of a step by as many bits as
// it has leading zeros.  Outputs' distance from 64 bits (rms; value scales even | 4096 apart from token to token), in units of
// 1e-7: 4-bit codes at bits 6 to 9 9.8 | 17, normal 6.4 | 7.9, in binary32 on the vector ALUs 6.9 | 7.6; 2-bit codes at bits 8
// and 9 7.0 | 13, binary32 8.5 | 7.3.  With 8 and 16 rows the f16 operands took the place of kernels with 47 | 80.
constexpr bool rows_normal_operands(int bits, bool padded) { return bits == 4 || padded; }
constexpr int kNormalBits = 14;

// Key codes.  Dword W of a token holds 32 / BITS channels, channel 4 h + b of it at bit 8 b + BITS h.  A lane quarter kq
// reads the dwords W = kq + 4 i; step kc of the contraction takes two fields h, i.e. 8 consecutive channels from
// key_channel(kc, kq) on, in the pair order (0, 2) (1, 3) (4, 6) (5, 7) that the halves of a dword have.
template <int BITS>
__device__ __forceinline__ constexpr int key_channel(int kc, int kq) {
    return BITS == 2 ? 16 * (kq + 4 * (kc >> 1)) + 8 * (kc & 1) : BITS == 1 ? 32 * kq + 8 * kc : 32 * kc + 8 * kq;
}
template <int BITS>
__device__ __forceinline__ constexpr int key_load(int kc) { return BITS == 2 ? kc >> 1 : BITS == 1 ? 0 : kc; }
template <int BITS>
__device__ __forceinline__ uint4v key_fields(uint32_t w, int kc) {
    if constexpr (BITS == 2) {
        constexpr uint32_t m = 0x03000300u;
        return (kc & 1) == 0 ? uint4v{(w << 8) & m, w & m, (w << 6) & m, (w >> 2) & m} : uint4v{(w << 4) & m, (w >> 4) & m, (w << 2) & m, (w >> 6) & m};
    } else if constexpr (BITS == 1) {
        switch (kc) {
            case 0: return uint4v{(w << 8) & 0x01000100u, w & 0x01000100u, (w << 8) & 0x02000200u, w & 0x02000200u};
            case 1: return uint4v{(w << 6) & 0x01000100u, (w >> 2) & 0x01000100u, (w << 6) & 0x02000200u, (w >> 2) & 0x02000200u};
            case 2: return uint4v{(w << 4) & 0x01000100u, (w >> 4) & 0x01000100u, (w << 4) & 0x02000200u, (w >> 4) & 0x02000200u};
            default: return uint4v{(w << 2) & 0x01000100u, (w >> 6) & 0x01000100u, (w << 2) & 0x02000200u, (w >> 6) & 0x02000200u};
        }
    } else {
        return uint4v{(w << 6) & 0x03C003C0u, (w >> 2) & 0x03C003C0u, (w << 2) & 0x03C003C0u, (w >> 6) & 0x03C003C0u};
    }
}
template <bool NORMAL>
__device__ __forceinline__ uint4v normal(uint4v a) {
    return NORMAL ? __builtin_bit_cast(uint4v, __builtin_bit_cast(half8, a) * (_Float16)(1 << kNormalBits)) : a;
}
template <int BITS, bool NORMAL>
__device__ __forceinline__ uint4v key_operand(uint32_t w, int kc) { return normal<NORMAL>(key_fields<BITS>(w, kc)); }
// the fields arrive at different bits: the multiplier of channel c carries the factor that makes every product
// code * 2^kKeyPos * 2^-24
template <int BITS>
__device__ __forceinline__ float key_factor(int c) {
    return BITS == 1 && !((c >> 2) & 1) ? 2.0f : 1.0f;
}
template <int BITS, bool NORMAL>
__device__ __forceinline__ constexpr int key_pos() { return (BITS == 2 ? 8 : BITS == 1 ? 9 : 6) + (NORMAL ? kNormalBits : 0); }
constexpr int key_q_bits(int bits) { return bits == 1 ? 6 : 7; }   // |q'| < 2^this: q' factor s' < 2^15 with s' < 2^8

// Value codes.  Byte t of a 16-byte piece is a token, its fields are channels.  A channel tile (mb, jj) is 16 channels of
// the 32-channel block mb, so that it lies in one value group whatever g is: A row i is channel value_channel(mb, jj, i).
// Even tokens of a dword sit in the low byte of its halves, odd ones in the high byte; a lane's shift brings the two
// fields its row may want to bits 6 to 9 (8 and 9 with 1-bit codes).
template <int BITS>
__device__ __forceinline__ int value_lane(int mb, int ic) { return BITS == 2 ? 8 * mb + (ic & 7) : BITS == 1 ? 4 * mb + (ic & 3) : 16 * mb + ic; }
template <int BITS>
__device__ __forceinline__ int value_channel(int mb, int jj, int i) {
    return BITS == 2 ? 4 * (8 * mb + (i & 7)) + 2 * (i >> 3) + jj : BITS == 1 ? 8 * (4 * mb + (i & 3)) + 2 * (i >> 2) + jj : 2 * (16 * mb + i) + jj;
}
template <int BITS, bool NORMAL>
__device__ __forceinline__ constexpr int value_pos(int jj) { return (BITS == 2 ? 8 : BITS == 1 ? 8 + jj : 6) + (NORMAL ? kNormalBits : 0); }
struct ValueShift { uint32_t left, right; };   // of the lane's A row (2- and 1-bit codes)
template <int BITS>
__device__ __forceinline__ ValueShift value_shift(int ic) {
    if constexpr (BITS == 2) return {6u - 4u * (ic >> 3), 2u + 4u * (ic >> 3)};
    return {8u - 2u * (ic >> 2), 2u * (ic >> 2)};
}
// both channel tiles of a block from the 8 tokens of a lane
template <int BITS, bool NORMAL>
__device__ __forceinline__ void value_operands(uint2 w, ValueShift sh, uint4v a[2]) {
    if constexpr (BITS == 4) {
        a[0] = uint4v{(w.x << 6) & 0x03C003C0u, (w.x >> 2) & 0x03C003C0u, (w.y << 6) & 0x03C003C0u, (w.y >> 2) & 0x03C003C0u};
        a[1] = uint4v{(w.x << 2) & 0x03C003C0u, (w.x >> 6) & 0x03C003C0u, (w.y << 2) & 0x03C003C0u, (w.y >> 6) & 0x03C003C0u};
    } else {
        constexpr uint32_t m0 = BITS == 2 ? 0x03000300u : 0x01000100u, m1 = BITS == 2 ? 0x03000300u : 0x02000200u;
        constexpr int up = BITS == 2 ? 2 : 0;
        const uint32_t e0 = w.x << sh.left, o0 = w.x >> sh.right, e1 = w.y << sh.left, o1 = w.y >> sh.right;
        a[0] = uint4v{(e0 << up) & m0, (o0 << up) & m0, (e1 << up) & m0, (o1 << up) & m0};
        a[1] = uint4v{e0 & m1, o0 & m1, e1 & m1, o1 & m1};
    }
    a[0] = normal<NORMAL>(a[0]);
    a[1] = normal<NORMAL>(a[1]);
}

// x as hi + lo f16, both rounded to nearest (to 2^-23 of x), packed in the pair order of the A operands
typedef float float2v __attribute__((ext_vector_type(2)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split8(const float x[8], uint4v& hi, uint4v& lo) {
    constexpr int kFirst[4] = {0, 1, 4, 5};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const float2v a = {x[kFirst[d]], x[kFirst[d] + 2]};
        const half2v h = __builtin_convertvector(a, half2v);
        const float2v rest = {a.x - (float)h.x, a.y - (float)h.y};
        hi[d] = __builtin_bit_cast(uint32_t, h);
        lo[d] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, half2v));
    }
}

template <int BITS, int GROUP, int NR>
struct RowsShape {
    static constexpr int SUBS = 16 / NR;                                     // sub-groups of 32 tokens in flight
    static constexpr int UNIT = 32 * SUBS;                                   // tokens of a unit
    static constexpr int SG = UNIT > GROUP ? UNIT / GROUP : 1;               // token groups of a unit
    static constexpr int M = kD / GROUP;
    static constexpr int kSStride = kD + 4;                                  // floats between the token groups' scale rows
    static constexpr int kZStride = kD + 8;                                  // halves between the token groups' (min), (max) rows
    static constexpr int kQStride = kD + 4;
    static constexpr int kKeyStride = UNIT + 4;
    // LDS: query rows scaled (floats) and as they are (halves), then per wave the tables; later the waves' outputs
    static constexpr int kQBytes = NR * kQStride * 4 + NR * kZStride * 2 + NR * 8;
    static constexpr int kKeyTab = SG * kSStride * 4 + SG * kZStride * 2 * (BITS == 1 ? 2 : 1);
    static constexpr int kValTab = 2 * M * UNIT * 4;
    static constexpr int kLogitTab = NR * kKeyStride * 4;
    static constexpr int kWaveBytes = (kKeyTab + kValTab + kLogitTab + 15) / 16 * 16;
    static constexpr int kMainBytes = (kQBytes + 15) / 16 * 16 + kWaves * kWaveBytes;
    // a workgroup of 16-bit candidates: per wave its weights [32][NR]
    static constexpr int kExtraBytes = (kQBytes + 15) / 16 * 16 + kWaves * 32 * NR * 4;
    static constexpr int kMergeBytes = kWaves * 16 * kRowsOStride * 4;
    static constexpr int kBytes = kMainBytes > kMergeBytes ? (kMainBytes > kExtraBytes ? kMainBytes : kExtraBytes)
                                                           : (kMergeBytes > kExtraBytes ? kMergeBytes : kExtraBytes);
};

// sum_c code[i][c] q'[c] s'[c] of the eight tokens of a lane in binary32
template <int BITS>
__device__ __forceinline__ void scaled_logits(const uint8_t* kc_row, int sub, int kq, const float* q, const float* s, float o[8]) {
    const uint8_t* base = kc_row + (size_t)(sub / 16) * k_tile_bytes(BITS) + (size_t)(4 * (sub % 16) + kq) * 16;
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = 0.0f;
#pragma unroll 1
    for (int W = 0; W < 4 * BITS; ++W) {
        const uint4 a = *reinterpret_cast<const uint4*>(base + (size_t)W * 2048), b = *reinterpret_cast<const uint4*>(base + (size_t)W * 2048 + 1024);
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll 1
        for (int j = 0; j < 32 / BITS; ++j) {
            const int c = W * (32 / BITS) + j, bit = 8 * (j & 3) + BITS * (j >> 2);
            const float x = q[c] / key_factor<BITS>(c) * s[c];
#pragma unroll
            for (int t = 0; t < 8; ++t) o[t] = __builtin_fmaf((float)((w[t] >> bit) & ((1u << BITS) - 1u)), x, o[t]);
        }
    }
}

template <int BITS, int GROUP, int NR, bool PADDED, bool BF16, int MODE>
__global__ __launch_bounds__(kThreads, 3) void rows_kernel(LayerView L, RowsArgs R) {
    using S = RowsShape<BITS, GROUP, NR>;
    constexpr int SUBS = S::SUBS, UNIT = S::UNIT, SG = S::SG, M = S::M;
    constexpr bool NORMAL = rows_normal_operands(BITS, PADDED);
    __shared__ __attribute__((aligned(16))) uint8_t smem[S::kBytes];
    __shared__ uint32_t maskbits[MODE == kRowsScore ? 1 : kRowsMaxChunk / 32];
    __shared__ RowsOut out;
    __shared__ FinishShared fin_shared;
    static_assert(MODE == kRowsScore || S::kBytes >= kFinishLdsBytes, "the merge of a row in the same region");
    const AttendArgs& A = R.at;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int ic = lane & 15, kq = lane >> 4, r = ic % NR, s = ic / NR;
    // fewer than 8 rows: the columns of rows that do not exist carry zero queries and nothing of them is written
    const int nq = PADDED ? L.G * R.n_rows : NR;

    // ---- which (row, chunk): workgroups that append the step's token first, then the 16-bit chunks, then the
    // others, then those that only merge
    const int n_tail = L.tail_k ? L.rows : 0;
    if ((int)blockIdx.x < n_tail) {
        const int rw = blockIdx.x;
        if (tid < 32) {
            const uint4 v = reinterpret_cast<const uint4*>(tid < 16 ? L.tail_k : L.tail_v)[(size_t)rw * 16 + (tid & 15)];
            reinterpret_cast<uint4*>(L.host)[((size_t)rw * L.max_seq + L.tail_N0) * 32 + tid] = v;
            reinterpret_cast<uint4*>(L.ring)[((size_t)rw * L.R + (L.tail_N0 % L.R)) * 32 + tid] = v;
        }
        return;
    }
    int row, chunk = 0;
    uint32_t shares = 0;
    const int bid = (int)blockIdx.x - n_tail, n_extra = A.n_chunks - A.n_main, id = bid - L.rows * n_extra, merger = bid - L.rows * A.n_chunks;
    if (id < 0) {
        row = bid / n_extra;
        chunk = A.n_main + bid % n_extra;
    } else if (MODE == kRowsScore || merger < 0) {
        row = id / A.n_main;
        chunk = id % A.n_main;
    } else {
        row = merger / A.fin.shares;
        shares = row_complete(A, row, merger % A.fin.shares, fin_shared);
    }
    if (MODE == kRowsScore || merger < 0) {
        // ---- the query rows: scaled by a power of two and by the channels' factors, and as they are
        float* qs = reinterpret_cast<float*>(smem);                                    // [NR][kQStride]
        uint16_t* qraw = reinterpret_cast<uint16_t*>(smem + NR * S::kQStride * 4);      // [NR][kZStride]
        int* q_unscale = reinterpret_cast<int*>(smem + NR * S::kQStride * 4 + NR * S::kZStride * 2);   // [NR], exponents
        // requested here and worked on when the first unit's loads are under way, too.  One behind the other (the queries, then the unit, then
        // the index list) the three round trips made a step of 16 x 8192 with 16 query rows 35.9 us a layer, now 32.0; 24 x 5003 with 8 rows 30.7
        // and 28.1, 32 x 32768 53.9 and 50.9.
        static_assert(NR % kWaves == 0, "every wave takes as many rows");
        uint32_t qw[NR / kWaves];
        {
            const auto q_buf = buffer_of(A.q + (size_t)row * nq * kD, (uint32_t)(nq * kD) * 2u);   // rows beyond: 0
#pragma unroll
            for (int i = 0; i < NR / kWaves; ++i) qw[i] = __builtin_amdgcn_raw_buffer_load_b32(q_buf, ((wave + i * kWaves) * (kD / 2) + lane) * 4, 0, 0);
        }
        auto prepare_queries = [&]() {
#pragma unroll
            for (int i = 0; i < NR / kWaves; ++i) {
                const int rr = wave + i * kWaves;
                const uint32_t w = qw[i];
                reinterpret_cast<uint32_t*>(qraw + rr * S::kZStride)[lane] = w;
                if constexpr (MODE == kRowsBoth)
                    if (A.q_out && chunk == 0 && rr < nq) reinterpret_cast<uint32_t*>(A.q_out + ((size_t)row * nq + rr) * kD)[lane] = w;
                if constexpr (MODE != kRowsAttend) {
                    const float a = widen16<BF16>(w & 0xFFFFu) * A.sm_scale, b = widen16<BF16>(w >> 16) * A.sm_scale;
                    const float top = wave_max(fmaxf(fabsf(a), fabsf(b)));
                    int f = 253 + key_q_bits(BITS) - (int)((__float_as_uint(top) >> 23) & 0xFFu);   // top < 2^(E - 126): field of 2^(kbits - E + 126)
                    f = f > 254 ? 254 : f;
                    const float sc = __uint_as_float((uint32_t)f << 23);
                    const int c = 2 * lane;
                    *reinterpret_cast<float2*>(qs + rr * S::kQStride + c) = make_float2(a * sc * key_factor<BITS>(c), b * sc * key_factor<BITS>(c + 1));
                    if (lane == 0) q_unscale[rr] = 127 - f;
                }
            }
        };

        float* o_lds = reinterpret_cast<float*>(smem);                                  // [kWaves][16][kRowsOStride], at the end
        if (MODE != kRowsScore && chunk >= A.n_main) {
            const int x0 = ((chunk - A.n_main) * kWaves + wave) * 32;
            const int2 staged = staged_positions(L, A, row, x0, lane);
            prepare_queries();
            __syncthreads();
            float* weights = reinterpret_cast<float*>(smem + (S::kQBytes + 15) / 16 * 16) + wave * 32 * NR;
            rows_extra_wave<NR, BF16>(L, A, R.n_rows, row, x0, staged, lane, wave, qraw, S::kZStride, weights,
                                      o_lds, out);
        } else {
            const int chunk_tokens = kWaves * R.wave_units * UNIT, c0 = chunk * chunk_tokens;
            const int w0 = c0 + wave * R.wave_units * UNIT;                             // the wave's first token
            const int n_sub = A.Nq / kBlockTokens;
            const uint8_t* kc_row = L.kc + (size_t)row * L.kc_stride;
            const uint8_t* vc_row = L.vc + (size_t)row * L.vc_stride;
            const uint32_t* km_row = L.km + (size_t)row * L.km_stride;
            const uint32_t* vm_row = L.vm + (size_t)row * L.vm_stride;
            uint8_t* area = smem + (S::kQBytes + 15) / 16 * 16 + wave * S::kWaveBytes;
            float* s_tab = reinterpret_cast<float*>(area);                              // [SG][kSStride]
            uint16_t* z_tab = reinterpret_cast<uint16_t*>(area + SG * S::kSStride * 4);  // [1 or 2][SG][kZStride]
            float* vs_tab = reinterpret_cast<float*>(area + S::kKeyTab);                 // [M][UNIT]
            float* vz_tab = vs_tab + M * UNIT;
            float* l_tab = vz_tab + M * UNIT;                                            // [heads][kKeyStride]

            // ---- loads of one unit
            constexpr int kVm = UNIT * M / 64 > 0 ? UNIT * M / 64 : 1;                   // value metadata words per lane
            uint2 kcw[SUBS][BITS], kmw[SG], vcw[SUBS][4];
            uint32_t vmw[kVm];
            int vexp[M], kexp[SG];    // the same for the whole wave: acc of value group m is scaled by 2^vexp[m]
            // the lanes whose word e is of value group m
            auto group_lanes = [](int m, int e) constexpr {
                unsigned long long lanes = 0;
                for (int i = 0; i < 64; ++i) lanes |= (unsigned long long)((i * kVm + e) % M == m && i * kVm + e < UNIT * M) << i;
                return lanes;
            };
            auto group_exp = [&](int m) {
                int x = vexp[0];
#pragma unroll
                for (int mm = 1; mm < M; ++mm) x += m == mm ? vexp[mm] - vexp[0] : 0;     // (no choice between array elements: it stays in registers)
                return x;
            };
            auto sub_of = [&](int t0, int x) {
                const int sub = t0 / kBlockTokens + x;
                return sub < n_sub ? sub : n_sub - 1;                                    // past the end: a valid sub-group again
            };
            // a wave's position is the same for its lanes: addresses are a scalar base plus a lane's offset
            const uint32_t km_lane = 8u * lane, kc_lane = (uint32_t)(((ic % 4) / 2) * 1024 + (ic / 4) * 16 + 8 * (ic % 2) + kq * 2048);
            const uint32_t vc_lane = (uint32_t)((kq >> 1) * (256 * BITS) + 8 * (kq & 1) + value_lane<BITS>(0, ic) * 16);
            // (where the launch announces its scores, the keys have to be past the L2 by then: finish_row.h)
            const auto keys_row = buffer_of(R.keys + (size_t)row * R.key_stride, (uint32_t)A.Nq * 4u);
            const size_t row_logits = (size_t)row * nq * A.logit_stride;
            const uint32_t logit_lane = (uint32_t)(r * A.logit_stride + 32 * s + 8 * kq);
            auto load_keys = [&](int t_wave) {
                if constexpr (MODE != kRowsAttend) {
                    const int t0 = __builtin_amdgcn_readfirstlane(t_wave);
#pragma unroll
                    for (int gi = 0; gi < SG; ++gi) {
                        int grp = t0 / GROUP + gi;
                        const int n_grp = A.Nq / GROUP;
                        grp = grp < n_grp ? grp : n_grp - 1;
                        kmw[gi] = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(km_row + (size_t)grp * kD) + km_lane);
                    }
#pragma unroll
                    for (int x = 0; x < SUBS; ++x) {
                        const int sub = sub_of(t0, x);
                        // row ic is tokens 2 ic and 2 ic + 1: half (ic % 4) / 2 of layout lane 4 (sub % 16) + ic / 4
                        const uint8_t* base = kc_row + (size_t)(sub / 16) * k_tile_bytes(BITS) + (size_t)(sub % 16) * 64;
#pragma unroll
                        for (int i = 0; i < BITS; ++i) kcw[x][i] = *reinterpret_cast<const uint2*>(base + 4 * i * 2048 + kc_lane);
                    }
                }
            };
            auto load_values = [&](int t_wave) {
                if constexpr (MODE != kRowsScore) {
                    const int t0 = __builtin_amdgcn_readfirstlane(t_wave);
                    // metadata words of the unit in memory order: word lane * kVm + e
                    const int word = lane * kVm;
                    const int last = A.Nq * M - kVm;
                    int at = t0 * M + word;
                    at = at < last ? at : last;
                    if constexpr (kVm % 4 == 0) {
#pragma unroll
                        for (int e = 0; e < kVm; e += 4) {
                            const uint4 v = *reinterpret_cast<const uint4*>(vm_row + (uint32_t)(at + e));
                            vmw[e] = v.x; vmw[e + 1] = v.y; vmw[e + 2] = v.z; vmw[e + 3] = v.w;
                        }
                    } else if constexpr (kVm == 2) {
                        const uint2 v = *reinterpret_cast<const uint2*>(vm_row + (uint32_t)at);
                        vmw[0] = v.x; vmw[1] = v.y;
                    } else {
                        vmw[0] = vm_row[(uint32_t)at];
                    }
#pragma unroll
                    for (int x = 0; x < SUBS; ++x) {
                        const uint8_t* base = vc_row + (size_t)sub_of(t0, x) * code_block_bytes(BITS);
#pragma unroll
                        for (int mb = 0; mb < 4; ++mb) vcw[x][mb] = *reinterpret_cast<const uint2*>(base + value_lane<BITS>(mb, 0) * 16 + vc_lane);
                    }
                }
            };
            // the first entries of the index list travel with them
            const int n_idx = MODE != kRowsScore && A.slot_idx ? L.topk : 0;
            const int first_idx = (int)__builtin_amdgcn_raw_buffer_load_b32(buffer_of(n_idx ? A.slot_idx + (size_t)row * L.topk : nullptr, (uint32_t)n_idx * 4u), tid * 4, 0, 0);
            load_keys(w0 < A.Nq ? w0 : 0);
            load_values(w0 < A.Nq ? w0 : 0);
            __builtin_amdgcn_sched_barrier(0);
            prepare_queries();

            // ---- bitmap of the chunk's staged positions (they enter through the 16-bit chunks)
            if constexpr (MODE != kRowsScore) {
                const int words = chunk_tokens / 32;
                for (int i = tid; i < words; i += kThreads) maskbits[i] = 0u;
                __syncthreads();
                for (int j = tid; j < n_idx; j += kThreads) {
                    const int t = (j == tid ? first_idx : A.slot_idx[(size_t)row * L.topk + j]) - c0;
                    if (t >= 0 && t < chunk_tokens) atomicOr(&maskbits[t >> 5], 1u << (t & 31));
                }
            }
            __syncthreads();

            const ValueShift vsh = value_shift<BITS>(ic);
            const int my_group = SG > 1 ? s * kBlockTokens / GROUP : 0;                   // the column's token group inside the unit
            float4v acc[4][2];
            float m_used = -INFINITY, lsum = 0.0f, zacc[M];
#pragma unroll
            for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) acc[mb][jj] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < M; ++m) {
                zacc[m] = 0.0f;
                vexp[m] = 0;
            }
#pragma unroll
            for (int gi = 0; gi < SG; ++gi) kexp[gi] = 0;
            // Two sub-groups in flight: columns (r, hi | lo).  Where they are one token group the two lanes of a row work out
            // half of its multipliers each, for all the units it has; else each those of its own group, step by step.
            constexpr bool kHiLo = SUBS == 2, kHalves = kHiLo && SG == 1;
            constexpr bool kKeepB = MODE != kRowsAttend && UNIT < GROUP;                  // a token group's multipliers serve several units
            uint4v bhi[kKeepB || kHalves ? 4 : 1], blo[kKeepB && !kHiLo ? 4 : 1];
            auto multipliers = [&](int kc, uint4v& hi, uint4v& lo) {
                const int c = key_channel<BITS>(kc, kq);
                float x[8];
#pragma unroll
                for (int e4 = 0; e4 < 2; ++e4) {
                    const float4 qv = *reinterpret_cast<const float4*>(qs + r * S::kQStride + c + 4 * e4);
                    const float4 sv4 = *reinterpret_cast<const float4*>(s_tab + my_group * S::kSStride + c + 4 * e4);
                    x[4 * e4] = qv.x * sv4.x;
                    x[4 * e4 + 1] = qv.y * sv4.y;
                    x[4 * e4 + 2] = qv.z * sv4.z;
                    x[4 * e4 + 3] = qv.w * sv4.w;
                }
                split8(x, hi, lo);
            };
            float unscale = 0.0f;
            int unscale_more = 0, group_done = -1;
            const bool q_some = MODE != kRowsAttend && q_unscale[r] > -127;             // a query that is not zero
            float qz = 0.0f;

            for (int u = 0; u < R.wave_units; ++u) {
                const int t0 = w0 + u * UNIT;
                if (t0 >= A.Nq) break;                                                    // uniform over the wave
                const bool active = t0 / kBlockTokens + s < n_sub && (!PADDED || r < nq);
                float l[8];
                if constexpr (MODE != kRowsAttend) {
                    // ---- multipliers of the unit's token groups (a group longer than a unit is worked out once)
                    const int grp0 = t0 / GROUP;
                    if (grp0 != group_done) {
                        group_done = grp0;
                        wave_sync();
                        int es = 0;
#pragma unroll
                        for (int gi = 0; gi < SG; ++gi) {
                            const uint32_t wd[2] = {kmw[gi].x, kmw[gi].y};
                            // words 2 lane, 2 lane + 1 are channels c and c + 4
                            const int c = 4 * ((2 * lane) & 31) + (lane >> 4);
                            float sv[2];
#pragma unroll
                            for (int e = 0; e < 2; ++e) {
                                float z;
                                derive_scale_zero<BITS>(widen16<BF16>(wd[e] & 0xFFFFu), widen16<BF16>(wd[e] >> 16), L.one_bit_plain, sv[e], z);
                                z_tab[gi * S::kZStride + c + 4 * e] = (uint16_t)wd[e];
                                if constexpr (BITS == 1) z_tab[(SG + gi) * S::kZStride + c + 4 * e] = (uint16_t)(wd[e] >> 16);
                            }
                            float sc[2] = {times_pow2(sv[0], kexp[gi]), times_pow2(sv[1], kexp[gi])};
                            const float top = fmaxf(sc[0], sc[1]);
                            if (__builtin_expect(__any(top > kKeyScaleMost) || !__any(top > kKeyScaleLeast), 0)) {
                                const uint32_t E = wave_max_bits(__float_as_uint(fmaxf(sv[0], sv[1]))) >> 23;      // s < 2^(E - 126)
                                kexp[gi] = 126 + kScaleSet - (int)(E & 0xFFu);
                                sc[0] = times_pow2(sv[0], kexp[gi]);
                                sc[1] = times_pow2(sv[1], kexp[gi]);
                            }
                            s_tab[gi * S::kSStride + c] = sc[0];
                            s_tab[gi * S::kSStride + c + 4] = sc[1];
                            es = my_group == gi ? kexp[gi] : es;
                        }
                        wave_sync();
                        {
                            const int e = q_unscale[r] - es + 24 - key_pos<BITS, NORMAL>(), u = e > 127 ? 127 : e < -126 ? -126 : e;
                            unscale = __uint_as_float((uint32_t)(127 + u) << 23);
                            unscale_more = e - u;                                          // beyond binary32's powers of two
                        }
                        // zero-point term: z is the stored 16-bit minimum (Eq. 3: a quarter of three minima and a maximum),
                        // q the 16-bit query, so the products are exact.  A row i is token group i & (SG - 1).
                        const int zg = SG > 1 ? (ic & (SG - 1)) : 0;
                        float4v zc = {0.f, 0.f, 0.f, 0.f}, xc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int kc = 0; kc < 4; ++kc) {
                            const uint4v b = *reinterpret_cast<const uint4v*>(qraw + r * S::kZStride + 32 * kc + 8 * kq);
                            const uint4v a = *reinterpret_cast<const uint4v*>(z_tab + zg * S::kZStride + 32 * kc + 8 * kq);
                            zc = mfma_native<BF16>(a, b, zc);
                            if constexpr (BITS == 1) {
                                const uint4v a2 = *reinterpret_cast<const uint4v*>(z_tab + (SG + zg) * S::kZStride + 32 * kc + 8 * kq);
                                xc = mfma_native<BF16>(a2, b, xc);
                            }
                        }
                        float zq = zc[0], xq = xc[0];
#pragma unroll
                        for (int gi = 1; gi < SG; ++gi) {
                            zq = my_group == gi ? zc[gi] : zq;
                            xq = my_group == gi ? xc[gi] : xq;
                        }
                        if constexpr (BITS == 1) zq = L.one_bit_plain ? zq : __builtin_fmaf(zq, 3.0f, xq) * 0.25f;
                        qz = zq * A.sm_scale;
                        if constexpr (kHalves) {
#pragma unroll
                            for (int i = 0; i < 2; ++i) {
                                uint4v hi, lo;
                                multipliers(i + 2 * s, hi, lo);
                                hi_lo_columns(hi, lo, bhi[i], bhi[i + 2]);
                            }
                        } else if constexpr (kKeepB) {
#pragma unroll
                            for (int kc = 0; kc < 4; ++kc) multipliers(kc, bhi[kc], blo[kc]);
                        }
                    }
                    float o[8];
                    {
                        // ---- products: four channel steps x sub-groups x two tiles (even and odd tokens), hi and lo in sums of their
                        // own: added to the larger one step by step the small sum would lose its low end each time
                        float4v c[2][2];
#pragma unroll
                        for (int x = 0; x < 2; ++x) c[x][0] = c[x][1] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int kc = 0; kc < 4; ++kc) {
                            uint4v b[2];     // kHiLo: of either sub-group; else hi and lo
                            if constexpr (kHalves) {
                                b[0] = b[1] = bhi[kc];
                            } else if constexpr (kKeepB) {
                                b[0] = bhi[kc];
                                b[1] = blo[kc];
                            } else {
                                uint4v hi, lo;
                                multipliers(kc, hi, lo);
                                if constexpr (kHiLo) {
                                    hi_lo_columns(hi, lo, b[0], b[1]);
                                } else {
                                    b[0] = hi;
                                    b[1] = lo;
                                }
                            }
#pragma unroll
                            for (int mt = 0; mt < 2; ++mt) {
                                uint4v a;
#pragma unroll
                                for (int x = 0; x < 2; ++x) {
                                    if (x < SUBS) {
                                        const uint2 w = kcw[x][key_load<BITS>(kc)];
                                        a = key_operand<BITS, NORMAL>(mt == 0 ? w.x : w.y, kc);
                                    }
                                    c[x][mt] = mfma16(a, b[x], c[x][mt]);
                                }
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v)
#pragma unroll
                            for (int mt = 0; mt < 2; ++mt) {
                                if constexpr (kHiLo) {     // the lane's sub-group: its own column plus the other one's
                                    const float other = s ? c[0][mt][v] : c[1][mt][v];
                                    o[2 * v + mt] = (s ? c[1][mt][v] : c[0][mt][v]) + dpp_move<kDppRowRor8>(other);
                                } else {
                                    o[2 * v + mt] = c[0][mt][v] + c[1][mt][v];
                                }
                            }
                    }
                    // Tokens of a row all next to nothing: its query is small where the channels' scales are large.  What is
                    // left of the multipliers then lies in the f16 subnormals, and the lanes work in binary32 instead.
                    const float most = fmaxf(fmaxf(fabsf(o[0]), fabsf(o[2])), fmaxf(fabsf(o[5]), fabsf(o[7])));
                    const bool faint = most < times_pow2(4.0f, key_pos<BITS, NORMAL>() - 24) && q_some && (!PADDED || r < nq);
                    if (__builtin_expect(__any(faint || unscale_more != 0), 0)) {
                        if (__any(faint)) {
                            scaled_logits<BITS>(kc_row, sub_of(t0, s), kq, qs + r * S::kQStride, s_tab + my_group * S::kSStride, o);
#pragma unroll
                            for (int t = 0; t < 8; ++t) o[t] = times_pow2(o[t], key_pos<BITS, NORMAL>() - 24);
                        }
#pragma unroll
                        for (int t = 0; t < 8; ++t) o[t] = times_pow2(o[t], unscale_more);
                    }
                    if (u + 1 < R.wave_units) load_keys(t0 + UNIT < A.Nq ? t0 + UNIT : t0);
#pragma unroll
                    for (int t = 0; t < 8; ++t) l[t] = __builtin_fmaf(o[t], unscale, qz);
                    // ---- selection keys: the largest logit of the heads' last rows
                    {
                        const int G = nq / R.n_rows;
                        if (r % R.n_rows == R.n_rows - 1 && (!PADDED || r < nq)) {
                            float4* d = reinterpret_cast<float4*>(l_tab + (r / R.n_rows) * S::kKeyStride + 32 * s + 8 * kq);
                            d[0] = make_float4(l[0], l[1], l[2], l[3]);
                            d[1] = make_float4(l[4], l[5], l[6], l[7]);
                        }
                        wave_sync();
#pragma unroll
                        for (int i = 0; i < (UNIT + 63) / 64; ++i) {
                            const int t = UNIT >= 64 ? 64 * i + lane : lane & (UNIT - 1);
                            float b = -INFINITY;
                            if constexpr (UNIT >= 64) {
                                for (int h = 0; h < G; ++h) b = fmaxf(b, l_tab[h * S::kKeyStride + t]);
                            } else {       // two lanes per token, half of the heads each
                                for (int h = 0; h < G / 2; ++h) b = fmaxf(b, l_tab[((lane >> 5) * (G / 2) + h) * S::kKeyStride + t]);
                                b = xor32_max(b);
                            }
                            if (UNIT >= 64 || lane < 32) {   // (positions beyond the quantised ones lie beyond the buffer's range)
                                if (MODE == kRowsBoth && A.fin.word) __builtin_amdgcn_raw_buffer_store_b32(float_to_key(b), keys_row, (t0 + t) * 4, 0, kAgentScope);
                                else __builtin_amdgcn_raw_buffer_store_b32(float_to_key(b), keys_row, (t0 + t) * 4, 0, 0);
                            }
                        }
                        wave_sync();
                    }
                    if (A.logits_out && active) {
                        float4* d = reinterpret_cast<float4*>(A.logits_out + row_logits + (logit_lane + (uint32_t)t0));
                        d[0] = make_float4(l[0], l[1], l[2], l[3]);
                        d[1] = make_float4(l[4], l[5], l[6], l[7]);
                    }
                } else {
                    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
                    if (active) {
                        const float4* d = reinterpret_cast<const float4*>(A.logits + row_logits + (logit_lane + (uint32_t)t0));
                        a = d[0];
                        b = d[1];
                    }
                    l[0] = a.x; l[1] = a.y; l[2] = a.z; l[3] = a.w; l[4] = b.x; l[5] = b.y; l[6] = b.z; l[7] = b.w;
                }

                if constexpr (MODE != kRowsScore) {
                    // ---- scales and zero-points of the unit's tokens
                    wave_sync();
                    float vs[kVm], vsc[kVm];
#pragma unroll
                    for (int e = 0; e < kVm; ++e) {
                        const int word = lane * kVm + e, tok = word / M, m = word % M;
                        float z;
                        derive_scale_zero<BITS>(widen16<BF16>(vmw[e] & 0xFFFFu), widen16<BF16>(vmw[e] >> 16), L.one_bit_plain, vs[e], z);
                        if (UNIT * M >= 64 || word < UNIT * M) vz_tab[m * UNIT + tok] = z;
                        vsc[e] = times_pow2(vs[e], group_exp(m));
                    }
                    // does every group's largest scale lie within the bounds?  (which lanes hold a group's words is fixed)
                    bool moved = false;
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        unsigned long long over = 0, some = 0;
#pragma unroll
                        for (int e = 0; e < kVm; ++e) {
                            const unsigned long long lanes = group_lanes(m, e);
                            if (lanes == 0) continue;
                            over |= __ballot(vsc[e] > kValueScaleMost) & lanes;
                            some |= __ballot(vsc[e] > kValueScaleLeast) & lanes;
                        }
                        moved = moved || over != 0 || some == 0;
                    }
                    if (__builtin_expect(moved, 0)) {
#pragma unroll
                        for (int m = 0; m < M; ++m) {
                            uint32_t top = 0;
#pragma unroll
                            for (int e = 0; e < kVm; ++e) {
                                const int word = lane * kVm + e;
                                const uint32_t b = word % M == m && word < UNIT * M ? __float_as_uint(vs[e]) : 0u;
                                top = top > b ? top : b;
                            }
                            top = wave_max_bits(top);
                            float sum = 0.0f;
#pragma unroll
                            for (int mb = m * (GROUP / 32); mb < (m + 1) * (GROUP / 32); ++mb)
#pragma unroll
                                for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                                    for (int i = 0; i < 4; ++i) sum = fmaxf(sum, fabsf(acc[mb][jj][i]));
                            // s < 2^(E - 126): to below 2^kScaleSet, but no sum so far beyond 2^100
                            const int room = 226 - (int)(wave_max_bits(__float_as_uint(sum)) >> 23);
                            int e = 126 + kScaleSet - (int)((top >> 23) & 0xFFu);
                            e = top == 0 ? vexp[m] : e < vexp[m] + room ? e : vexp[m] + room;
#pragma unroll
                            for (int mb = m * (GROUP / 32); mb < (m + 1) * (GROUP / 32); ++mb)
#pragma unroll
                                for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                                    for (int i = 0; i < 4; ++i) acc[mb][jj][i] = times_pow2(acc[mb][jj][i], e - vexp[m]);
                            vexp[m] = e;
                        }
#pragma unroll
                        for (int e = 0; e < kVm; ++e) vsc[e] = times_pow2(vs[e], group_exp((lane * kVm + e) % M));
                    }
#pragma unroll
                    for (int e = 0; e < kVm; ++e) {
                        const int word = lane * kVm + e, tok = word / M, m = word % M;
                        if (UNIT * M >= 64 || word < UNIT * M) vs_tab[m * UNIT + tok] = vsc[e];
                    }
                    wave_sync();
                    // ---- softmax numerators
                    const uint32_t mask = (maskbits[(t0 - c0) / 32 + s] >> (8 * kq)) & 0xFFu;
                    float mx = -INFINITY;
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        l[t] = active && !((mask >> t) & 1u) ? l[t] : -INFINITY;
                        mx = fmaxf(mx, l[t]);
                    }
                    mx = quarters_max(mx);
                    if constexpr (SUBS == 2) mx = fmaxf(mx, dpp_move<kDppRowRor8>(mx));   // both columns of a row share the maximum
                    if (__any(mx > m_used + kLazyMax)) {
                        const float m_new = fmaxf(m_used, mx);
                        const float a = m_new == -INFINITY ? 1.0f : exp2_of((m_used - m_new) * kLog2e);
#pragma unroll
                        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[mb][jj][e] *= a;
#pragma unroll
                        for (int m = 0; m < M; ++m) zacc[m] *= a;
                        lsum *= a;
                        m_used = m_new;
                    }
                    const float ms = m_used == -INFINITY ? 0.0f : m_used;
                    float p[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        p[t] = exp2_of((l[t] - ms) * kLog2e);
                        lsum += p[t];
                    }
                    // ---- per value group: B operand and zero-point sums; per sub-group and 32-channel block of the
                    // ---- group two channel tiles x (hi, lo)
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        uint4v phi, plo;
                        {
                            const float4* sp = reinterpret_cast<const float4*>(vs_tab + m * UNIT + 32 * s + 8 * kq);
                            const float4* zp = reinterpret_cast<const float4*>(vz_tab + m * UNIT + 32 * s + 8 * kq);
                            const float4 s0 = sp[0], s1 = sp[1], z0 = zp[0], z1 = zp[1];
                            const float sv[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
                            const float zv[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
                            float x[8];
#pragma unroll
                            for (int t = 0; t < 8; ++t) {
                                x[t] = p[t] * sv[t];
                                zacc[m] = __builtin_fmaf(p[t], zv[t], zacc[m]);
                            }
                            split8(x, phi, plo);
                        }
                        if constexpr (SUBS == 2) {
                            uint4v b[2];     // columns (r, hi | lo) of either sub-group
                            hi_lo_columns(phi, plo, b[0], b[1]);
#pragma unroll
                            for (int x = 0; x < 2; ++x)
#pragma unroll
                                for (int mb = m * (GROUP / 32); mb < (m + 1) * (GROUP / 32); ++mb) {
                                    uint4v a[2];
                                    value_operands<BITS, NORMAL>(vcw[x][mb], vsh, a);
#pragma unroll
                                    for (int jj = 0; jj < 2; ++jj) acc[mb][jj] = mfma16(a[jj], b[x], acc[mb][jj]);
                                }
                        } else {
#pragma unroll
                            for (int mb = m * (GROUP / 32); mb < (m + 1) * (GROUP / 32); ++mb) {
                                uint4v a[2];
                                value_operands<BITS, NORMAL>(vcw[0][mb], vsh, a);
#pragma unroll
                                for (int jj = 0; jj < 2; ++jj) {
                                    acc[mb][jj] = mfma16(a[jj], phi, acc[mb][jj]);
                                    acc[mb][jj] = mfma16(a[jj], plo, acc[mb][jj]);
                                }
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (u + 1 < R.wave_units) load_values(t0 + UNIT < A.Nq ? t0 + UNIT : t0);
                }
            }
            if constexpr (MODE == kRowsScore) return;
            // ---- the wave's outputs per column, for the merge
            lsum = quarters_sum(lsum);
#pragma unroll
            for (int m = 0; m < M; ++m) zacc[m] = quarters_sum(zacc[m]);
            if (kq == 0) {
                out.m[wave][ic] = m_used;
                out.l[wave][ic] = lsum;
            }
            __syncthreads();   // every wave is done with its tables: the outputs take their place
#pragma unroll
            for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        // C row 4 kq + e of the tile
                        const int c = value_channel<BITS>(mb, jj, 4 * kq + e);
                        const int m = mb * 32 / GROUP;
                        o_lds[((size_t)wave * 16 + ic) * kRowsOStride + c] =
                            times_pow2(acc[mb][jj][e], 24 - value_pos<BITS, NORMAL>(jj) - vexp[m]) + zacc[m];
                    }
        }
        if constexpr (MODE == kRowsScore) return;
        __syncthreads();
        // ---- merge: the columns of a row over the waves and sub-groups
        if (tid < kWaves * 16) {
            const int w = tid >> 4, col = tid & 15, rr = col % NR;
            float mx = -INFINITY;
            for (int ww = 0; ww < kWaves; ++ww)
#pragma unroll
                for (int ss = 0; ss < SUBS; ++ss) mx = fmaxf(mx, out.m[ww][ss * NR + rr]);
            const float mv = out.m[w][col];
            out.w[w][col] = mv == -INFINITY ? 0.0f : exp2_of((mv - mx) * kLog2e);
        }
        __syncthreads();
        const auto po = buffer_of(A.part_o + (((size_t)row * A.max_chunks + chunk) * nq) * kD, (uint32_t)(nq * kD) * 4u);
        const auto pml = buffer_of(A.part_ml + (((size_t)row * A.max_chunks + chunk) * nq) * 2, (uint32_t)nq * 8u);
        // four outputs of a thread at a time, read 16 bytes at once and without a branch on the weight (one by one and behind it the waves'
        // outputs took 2.5 to 2.8 us of a kernel of 12 to 14, now 0.8)
        for (int e = tid; e < nq * (kD / 4); e += kThreads) {
            const int rr = e / (kD / 4), c = 4 * (e % (kD / 4));
            float4v v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
#pragma unroll
                for (int ss = 0; ss < SUBS; ++ss) {
                    const float wt = out.w[w][ss * NR + rr];
                    const float4v o = *reinterpret_cast<const float4v*>(o_lds + ((size_t)w * 16 + ss * NR + rr) * kRowsOStride + c);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = wt != 0.0f ? __builtin_fmaf(wt, o[i], v[i]) : v[i];
                }
            store_partials(po, e, v, A.fin.arrived != nullptr);
        }
        if (tid < nq) {
            float mx = -INFINITY, sum = 0.0f;
            for (int w = 0; w < kWaves; ++w)
#pragma unroll
                for (int ss = 0; ss < SUBS; ++ss) {
                    mx = fmaxf(mx, out.m[w][ss * NR + tid]);
                    sum = __builtin_fmaf(out.w[w][ss * NR + tid], out.l[w][ss * NR + tid], sum);
                }
            store_max_sum(pml, tid, mx, sum, A.fin.arrived != nullptr);
        }
        if (A.fin.arrived == nullptr) return;
        shares = row_arrival(A, row, fin_shared);
    }
    merge_shares<16>(A, row, nq, shares, reinterpret_cast<float*>(smem));
}

// launch of one mode for codes of BITS bits; at: everything but the chunking
template <int BITS, int MODE>
hipError_t launch_rows_mode(const LayerView& L, const RowsArgs& R, int NR, hipStream_t stream) {
    const dim3 grid((R.at.n_chunks + (R.at.fin.mergers ? R.at.fin.shares : 0)) * L.rows + (L.tail_k ? L.rows : 0)), block(kThreads);
    const bool padded = L.G * R.n_rows < NR;
#define SPC_ROWS(G_, N_, P_)                                                                            \
    if (L.group == G_ && NR == N_ && padded == P_) {                                                    \
        if (L.bf16) SPC_LAUNCH((rows_kernel<BITS, G_, N_, P_, true, MODE>), grid, block, stream, L, R); \
        else SPC_LAUNCH((rows_kernel<BITS, G_, N_, P_, false, MODE>), grid, block, stream, L, R);       \
        return hipGetLastError();                                                                       \
    }
    SPC_ROWS(32, 8, false) SPC_ROWS(64, 8, false) SPC_ROWS(128, 8, false)
    SPC_ROWS(32, 8, true) SPC_ROWS(64, 8, true) SPC_ROWS(128, 8, true)
    SPC_ROWS(32, 16, false) SPC_ROWS(64, 16, false) SPC_ROWS(128, 16, false)
#undef SPC_ROWS
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace specache
