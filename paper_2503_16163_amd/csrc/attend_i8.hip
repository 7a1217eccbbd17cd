// Mixed attention of Eq. 1 (Section 3.3) for one query head per KV head and the two query rows
// of a decode step, 1- or 2-bit values: the value side on the integer matrix cores, alone
// (attend_i8_kernel, after a scoring pass that left the logits in memory) or in one pass with the
// low-bit scoring of Appendix A "Decoding" (the same kernel with the scoring pass in front: the logits never leave the chip).
//
// Values are quantised per token over g channels (Section 2.1 / 4.1), so over the quantised
// positions of a chunk
//   sum_i p[r][i] V'[i][c] = sum_i (p[r][i] s[i][m]) code[i][c]  +  sum_i p[r][i] z[i][m],   m = c / g.
// The first sum is a contraction over tokens.  On the vector ALUs it costs a conversion per code
// and a multiply-accumulate per code and row, and that instruction count bounds the kernel (three
// times the time its bytes need).  Here it runs as v_mfma_i32_16x16x64_i8:
//   A = codes.  The packed layout gives a lane 16 consecutive tokens of four channels in 16 bytes;
//       masking with 0x03030303 or 0x0C0C0C0C (after a shift by 4 for the upper two channels) leaves
//       the 16 int8 operands of one channel as they stand, code or 4 x code: five vector
//       instructions per 64 codes.  The 16 rows of an MFMA are 16 channels four apart: one half
//       ("set") of the head's channels, two value groups at g = 32;
//   B = p s as 32-bit fixed point relative to the largest scale of the wave's tokens (p <= 1), cut
//       into four byte planes, the low three re-centred to signed: column (row r, group, plane).
//       With two rows, two groups and four planes the 16 columns are exactly full; of every result
//       the half whose column group matches the row's channel group is used;
//   C = int32, exact.  The planes are recombined in fp32 when the workgroup merges its waves.
// With 1-bit codes a byte holds 8 channels of a token and 16 code lanes are all 128 channels: the masks are
// 0x01010101 << j on the word and on the word shifted by 4 (operands code x 1, 2, 4, 8), eight products per
// token step, each run against the columns of either channel half; of a product's 16 rows the 8 code lanes
// of that half are kept.
// The zero-point term and the row sums stay on the vector ALUs (one multiply-add per token, group
// and row).
//
// A workgroup takes a chunk of 512 quantised positions (or, as in the vector-ALU kernel, 128 16-bit
// candidates: extra_chunk); its four waves are independent, each with 128 tokens and its own
// softmax maximum, and meet once, at the end, to merge their (max, sum, sum p V) into the chunk's
// partial result.  Lane = (32-token sub-group, h, token quad): it holds the logits of four
// consecutive tokens of row h (the layout in which the scoring wave finishes them), exchanges the
// numerators with the lane that holds the other row (one DPP rotation), and prepares p s of both
// rows for the value groups of channel set h.
#include "attend_common.h"
#include "extra_wave.h"
#include "finish_row.h"
#include "score_i8_wave.h"

namespace specache {
namespace {

constexpr int kI8Chunk = 512;                   // quantised tokens per workgroup
constexpr int kWaveTok = kI8Chunk / kWaves;     // 128
constexpr int kColStride = kWaveTok + 16;       // bytes between the B columns of a wave (pad: banks)
constexpr int kSetBytes = 16 * kColStride;      // the 16 columns (row, group of the set, plane) of a channel set
constexpr int kWaveArea = 2 * kSetBytes;        // bytes per wave; a set's results [2][4][4][16] int32 replace its columns
constexpr int kResPlane = 64 + 4;               // dwords between the results of (row, plane) of a set (pad: banks)
static_assert(kSetBytes >= 2 * 4 * kResPlane * 4, "a set's results reuse the set's operand columns");
static_assert(kWaveDwords * 4 >= kWaveArea, "the value phase reuses the scoring wave's exchange area");
constexpr int kWaveBitmapTopk = 256;            // up to here every wave builds the bitmap of its own tokens

// sum / max over the 8 lanes that share (sub-group, h): lanes differ in their low three bits
__device__ __forceinline__ float sum8(float v) {
    v += dpp_move<kDppXor1>(v);
    v += dpp_move<kDppXor2>(v);
    return v + dpp_move<kDppHalfMirror>(v);
}
__device__ __forceinline__ float max8(float v) {
    v = fmaxf(v, dpp_move<kDppXor1>(v));
    v = fmaxf(v, dpp_move<kDppXor2>(v));
    return fmaxf(v, dpp_move<kDppHalfMirror>(v));
}

// what the waves of a workgroup hand to the merge
struct WaveOut {
    float m[kWaves][2];            // softmax maximum of the wave's tokens, per row
    float unscale[kWaves];         // 1 / fixed-point scale of the wave's B operands
    float part[kWaves][4][2][5];   // per (wave, sub-group, h): zero-point sums [rows x groups of the lane], cell 4: sum of row h
};

// The lane's share of a wave's value-side loads: packed codes of 16 tokens x 4 channels for two token steps
// and two channel sets, and (min, max) words.  The metadata is stored per token ([token][group]); every lane
// requests consecutive 16 bytes of it (so that a load instruction covers whole cache lines) and the wave
// then hands the words through its LDS area to the lanes that use them: the groups of channel set h for
// the lane's four tokens (value_meta_exchange).
template <int GROUP, int BITS>
struct ValueLoads {
    static constexpr int M = kD / GROUP, MPL = M >= 2 ? M / 2 : 1;
    uint4 vw[2][BITS];           // [token step][channel set] with 2 bits; one word per token step holds all channels with 1
    uint4 raw[M == 4 ? 2 : 1];
    uint32_t mw[4][MPL];
};

template <int GROUP, int BITS>
__device__ __forceinline__ void value_loads(const LayerView& L, int Nq, int row, int c0, int w0, int nw, int lane, ValueLoads<GROUP, BITS>& v) {
    constexpr int M = kD / GROUP;
    const int sg = lane >> 4, l16 = lane & 15;
    const size_t tok = (size_t)c0 + w0 + 32 * sg;                      // the sub-group's first token
    const uint32_t* vm_row = L.vm + (size_t)row * L.vm_stride;
    // (positions beyond the quantised ones lie beyond the buffer's range: 0.  Loads behind a condition went through scratch memory in
    // groups of 64 and 128)
    const auto vm = buffer_of(vm_row, (uint32_t)Nq * M * 4u);
    auto load = [&](size_t t) { return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(vm, (int)(t * M * 4), 0, 0)); };
    if constexpr (M == 4) {            // 16 bytes per token: lane l16 takes tokens l16 and 16 + l16
        v.raw[0] = load(tok + l16);
        v.raw[1] = load(tok + 16 + l16);
    } else if constexpr (M == 2) {     // 8 bytes per token: tokens 2 l16 and 2 l16 + 1
        v.raw[0] = load(tok + 2 * l16);
    } else {                           // 4 bytes per token: the lane's own four tokens
        v.raw[0] = load(tok + 4 * (lane & 7));
    }
    // codes: lane (il = lane % 16, tg = lane / 16) reads, for token step ks and channel set s, the 16 tokens
    // 64 ks + 16 tg .. + 15 of code lane 16 s + il (channels 4 (16 s + il) .. + 3); with 1-bit codes of code
    // lane il (channels 8 il .. + 7)
    const int il = lane & 15, tg = lane >> 4;
    const uint8_t* vc_row = L.vc + (size_t)row * L.vc_stride;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int tw = 64 * ks + 16 * tg;                                  // inside the wave
        const size_t t16 = tw < nw ? (size_t)c0 + w0 + tw : (size_t)c0;    // past the end: the chunk's first tokens (p = 0 there)
        const uint8_t* base = vc_row + (t16 / kBlockTokens) * code_block_bytes(BITS) + ((t16 / 16) & 1) * (256 * BITS);
#pragma unroll
        for (int s = 0; s < BITS; ++s) v.vw[ks][s] = *reinterpret_cast<const uint4*>(base + (16 * s + il) * 16);
    }
}

// Metadata words from the lanes that loaded them to the lanes that use them, through the wave's LDS area
// (free at that point): [h][128 tokens] cells of the groups of channel set h, written per token, read as the
// lane's four consecutive tokens.
template <int GROUP, int BITS>
__device__ __forceinline__ void value_meta_exchange(ValueLoads<GROUP, BITS>& v, int lane, uint8_t* area) {
    constexpr int M = kD / GROUP;
    const int sg = lane >> 4, l16 = lane & 15, h = (lane >> 3) & 1, t0 = 32 * sg + 4 * (lane & 7);
    if constexpr (M == 4) {
        uint2* cells = reinterpret_cast<uint2*>(area);                 // [2][128] x 8 bytes
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int t = 32 * sg + 16 * e + l16;
            cells[t] = make_uint2(v.raw[e].x, v.raw[e].y);
            cells[128 + t] = make_uint2(v.raw[e].z, v.raw[e].w);
        }
        wave_sync();
        const uint4 a = *reinterpret_cast<const uint4*>(cells + 128 * h + t0), b = *reinterpret_cast<const uint4*>(cells + 128 * h + t0 + 2);
        v.mw[0][0] = a.x; v.mw[0][1] = a.y; v.mw[1][0] = a.z; v.mw[1][1] = a.w;
        v.mw[2][0] = b.x; v.mw[2][1] = b.y; v.mw[3][0] = b.z; v.mw[3][1] = b.w;
        wave_sync();
    } else if constexpr (M == 2) {
        uint32_t* cells = reinterpret_cast<uint32_t*>(area);           // [2][128] x 4 bytes
        const int t = 32 * sg + 2 * l16;
        cells[t] = v.raw[0].x;
        cells[128 + t] = v.raw[0].y;
        cells[t + 1] = v.raw[0].z;
        cells[128 + t + 1] = v.raw[0].w;
        wave_sync();
        const uint4 a = *reinterpret_cast<const uint4*>(cells + 128 * h + t0);
        v.mw[0][0] = a.x; v.mw[1][0] = a.y; v.mw[2][0] = a.z; v.mw[3][0] = a.w;
        wave_sync();
    } else {
        v.mw[0][0] = v.raw[0].x; v.mw[1][0] = v.raw[0].y; v.mw[2][0] = v.raw[0].z; v.mw[3][0] = v.raw[0].w;
    }
}

// Bits of the wave's 128 tokens that the staged index list names (they enter through the 16-bit chunks),
// built by the wave alone from an index list of at most 256 entries: the lane's four entries are requested
// with wave_bitmap_loads and turned into wbits[4] by wave_bitmap_apply, once other loads are under way.  (Requested under a
// condition and made relative at once, they were up to four loads one behind the other, each waited for before the wave asked for
// its keys: a step of 32 x 16384, k = 64, 38.5 us a layer against 37.6.)
__device__ __forceinline__ void wave_bitmap_loads(const int32_t* __restrict__ idx_row, int topk, int lane, int t[4]) {
    const auto list = buffer_of(idx_row, idx_row ? (uint32_t)topk * 4u : 0u);   // beyond the list: 0, and no lane looks at it
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (u > 0 && 64 * u >= topk) break;     // uniform
        t[u] = (int)__builtin_amdgcn_raw_buffer_load_b32(list, (64 * u + lane) * 4, 0, 0);
    }
}
__device__ __forceinline__ void wave_bitmap_apply(const int t[4], int n_idx, int first, int nw, int lane, uint32_t* wbits) {
    if (lane < 4) wbits[lane] = 0u;
    wave_sync();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (u > 0 && 64 * u >= n_idx) break;
        const uint32_t p = (uint32_t)(t[u] - first);       // (an empty place of the list, -1, lies before the first position, too)
        if (64 * u + lane < n_idx && p < (uint32_t)nw) atomicOr(&wbits[p >> 5], 1u << (p & 31));
    }
    wave_sync();
}

// The value side of one wave: softmax numerators relative to the wave's maximum, B operands, zero-point and
// row sums, the contraction, and the results left in the wave's area for the merge.  lgv: the logits of the
// lane's four tokens of row h (-inf where not a candidate).  nw > 0.
template <int GROUP, int BITS, bool BF16>
__device__ __forceinline__ void value_wave(const ValueLoads<GROUP, BITS>& v, float lgv[4], bool one_bit_plain, int wave, int lane,
                                           uint8_t* area, WaveOut& out) {
    constexpr int M = kD / GROUP;                 // value groups per token: 4, 2, 1
    constexpr int MPL = M >= 2 ? M / 2 : 1;       // groups a lane prepares
    constexpr int RPL = M >= 2 ? 2 : 1;           // rows a lane prepares (one group only: each lane its own row)
    const int sg = lane >> 4, h = (lane >> 3) & 1, tg = lane >> 4;
    const int t0 = 32 * sg + 4 * (lane & 7);

    const float m_own = quarters_max(max8(fmaxf(fmaxf(lgv[0], lgv[1]), fmaxf(lgv[2], lgv[3]))));   // of row h
    const float ms = m_own == -INFINITY ? 0.0f : m_own;
    float p[4], psum = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        p[j] = __expf(lgv[j] - ms);
        psum += p[j];
    }
    // numerators of the lane's tokens: of row h and, from the lane that holds it, of the other row
    float pr[RPL][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        pr[0][j] = p[j];
        if constexpr (RPL == 2) pr[1][j] = dpp_move<kDppRowRor8>(p[j]);
    }

    // scale and zero-point of the lane's (token, group) pairs; the wave's largest scale
    float sc[4][MPL], zp[4][MPL], smax = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int ml = 0; ml < MPL; ++ml) {
            derive_scale_zero<BITS>(widen16<BF16>(v.mw[j][ml] & 0xFFFFu), widen16<BF16>(v.mw[j][ml] >> 16), one_bit_plain, sc[j][ml], zp[j][ml]);
            smax = fmaxf(smax, sc[j][ml]);
        }
    // s < 2^(E - 126) with E the largest one's exponent field, p <= 1: p s 2^(156 - E) stays below 2^30
    uint32_t E = wave_max_bits(__float_as_uint(smax)) >> 23;
    E = E < 30u ? 30u : (E > 254u ? 254u : E);
    const float up = __uint_as_float((283u - E) << 23);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int ml = 0; ml < MPL; ++ml) sc[j][ml] *= up;

    // B columns: byte planes of p s, four tokens per dword; zero-point sums.  Column (set, row, group of the
    // set, plane); with one value group per token each lane fills its own row's columns of both sets.
    float zacc[RPL][MPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const int rr = r == 0 ? h : 1 - h;
        uint8_t* column = area + (M >= 2 ? h * kSetBytes : 0) + rr * (8 * kColStride) + t0;
#pragma unroll
        for (int ml = 0; ml < MPL; ++ml) {
            uint32_t y[4], planes[4];
            float za = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                y[j] = (uint32_t)(int)(pr[r][j] * sc[j][ml]);
                za = __builtin_fmaf(pr[r][j], zp[j][ml], za);
            }
            zacc[r][ml] = za;
            signed_byte_planes(y, planes);
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                *reinterpret_cast<uint32_t*>(column + (ml * 4 + pp) * kColStride) = planes[pp];
                if constexpr (M < 2) *reinterpret_cast<uint32_t*>(column + kSetBytes + pp * kColStride) = planes[pp];
            }
        }
    }
    // partial sums of the 8 lanes that share (sub-group, h); the merge adds them up
    psum = sum8(psum);
#pragma unroll
    for (int r = 0; r < RPL; ++r)
#pragma unroll
        for (int ml = 0; ml < MPL; ++ml) zacc[r][ml] = sum8(zacc[r][ml]);
    if ((lane & 7) == 0) {
        float* dst = out.part[wave][sg][h];
#pragma unroll
        for (int r = 0; r < RPL; ++r)
#pragma unroll
            for (int ml = 0; ml < MPL; ++ml) dst[(RPL == 1 ? 0 : r == 0 ? h : 1 - h) * MPL + ml] = zacc[r][ml];
        dst[4] = psum;
        if (sg == 0) out.m[wave][h] = m_own;
    }
    if (lane == 0) {
        out.unscale[wave] = __uint_as_float((E - 29u) << 23);   // 2^(E - 156) = 1 / up
    }
    wave_sync();

    // the contraction, one channel set at a time: per token step one B operand and the masks of the code bytes
    const int bn = lane & 15;
    const int brow = bn >> 3, bml = (bn >> 2) & 1, bpp = bn & 3;
    if constexpr (BITS == 2) {
        // Result register e of lane (column bn, quarter tg) is MFMA row 4 tg + e: code lane 16 s + 4 tg + e, i.e.
        // channel 64 s + 16 tg + 4 e + j, whose value group is 2 s + tg / 2 (g = 32), s (g = 64) or 0.  The columns
        // of that group are kept: [row][plane][j][16 rows] int32 per set.
        const bool keep = M == 4 ? bml == (tg >> 1) : bml == 0;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            v4i acc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = (v4i){0, 0, 0, 0};
            uint8_t* set = area + s * kSetBytes;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const v4i b = *reinterpret_cast<const v4i*>(set + ((brow * 2 + (M == 4 ? bml : 0)) * 4 + bpp) * kColStride + 64 * ks + 16 * tg);
                const uint4 w = v.vw[ks][s];
                const uint4 t = make_uint4(w.x >> 4, w.y >> 4, w.z >> 4, w.w >> 4);
                const v4i a0 = {(int)(w.x & 0x03030303u), (int)(w.y & 0x03030303u), (int)(w.z & 0x03030303u), (int)(w.w & 0x03030303u)};
                const v4i a1 = {(int)(w.x & 0x0C0C0C0Cu), (int)(w.y & 0x0C0C0C0Cu), (int)(w.z & 0x0C0C0C0Cu), (int)(w.w & 0x0C0C0C0Cu)};
                const v4i a2 = {(int)(t.x & 0x03030303u), (int)(t.y & 0x03030303u), (int)(t.z & 0x03030303u), (int)(t.w & 0x03030303u)};
                const v4i a3 = {(int)(t.x & 0x0C0C0C0Cu), (int)(t.y & 0x0C0C0C0Cu), (int)(t.z & 0x0C0C0C0Cu), (int)(t.w & 0x0C0C0C0Cu)};
                acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, b, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, b, acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a2, b, acc[2], 0, 0, 0);
                acc[3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a3, b, acc[3], 0, 0, 0);
            }
            wave_sync();   // every lane has read the set's B operands: its columns are free for the results
            if (keep) {
                int* res = reinterpret_cast<int*>(set);
#pragma unroll
                for (int j = 0; j < 4; ++j) *reinterpret_cast<v4i*>(res + (brow * 4 + bpp) * kResPlane + j * 16 + 4 * tg) = acc[j];
            }
        }
    } else {
        // MFMA row 4 tg + e is code lane 4 tg + e, channels 8 (4 tg + e) .. + 7: channel half (set) tg / 2, value
        // group tg (g = 32), tg / 2 (g = 64) or 0.  Each set's columns run against all 16 code lanes and the 8 of
        // the set are kept: [row][plane][j = 0..7][8 code lanes] int32 per set, the size of the 2-bit results.
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            uint8_t* set = area + s * kSetBytes;
            v4i b[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                b[ks] = *reinterpret_cast<const v4i*>(set + ((brow * 2 + (M == 4 ? bml : 0)) * 4 + bpp) * kColStride + 64 * ks + 16 * tg);
            wave_sync();   // every lane holds the set's B operands: its columns are free for the results
            const bool keep = (tg >> 1) == s && (M == 4 ? bml == (tg & 1) : bml == 0);
#pragma unroll
            for (int jh = 0; jh < 2; ++jh) {
                v4i acc[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[j] = (v4i){0, 0, 0, 0};
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    uint4 w = v.vw[ks][0];
                    if (jh) w = make_uint4(w.x >> 4, w.y >> 4, w.z >> 4, w.w >> 4);
                    const v4i a0 = {(int)(w.x & 0x01010101u), (int)(w.y & 0x01010101u), (int)(w.z & 0x01010101u), (int)(w.w & 0x01010101u)};
                    const v4i a1 = {(int)(w.x & 0x02020202u), (int)(w.y & 0x02020202u), (int)(w.z & 0x02020202u), (int)(w.w & 0x02020202u)};
                    const v4i a2 = {(int)(w.x & 0x04040404u), (int)(w.y & 0x04040404u), (int)(w.z & 0x04040404u), (int)(w.w & 0x04040404u)};
                    const v4i a3 = {(int)(w.x & 0x08080808u), (int)(w.y & 0x08080808u), (int)(w.z & 0x08080808u), (int)(w.w & 0x08080808u)};
                    acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, b[ks], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, b[ks], acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a2, b[ks], acc[2], 0, 0, 0);
                    acc[3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a3, b[ks], acc[3], 0, 0, 0);
                }
                if (keep) {
                    int* res = reinterpret_cast<int*>(set);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        *reinterpret_cast<v4i*>(res + (brow * 4 + bpp) * kResPlane + (4 * jh + j) * 8 + 4 * (tg & 1)) = acc[j];
                }
            }
        }
    }
}

// a wave without tokens contributes nothing, in finite numbers
__device__ __forceinline__ void empty_wave(int wave, int lane, WaveOut& out) {
    if (lane < 40) (&out.part[wave][0][0][0])[lane] = 0.0f;
    if (lane == 0) {
        out.m[wave][0] = -INFINITY;
        out.m[wave][1] = -INFINITY;
        out.unscale[wave] = 0.0f;
    }
}

// Merge of the four waves of a chunk (after a workgroup barrier): thread = (row r, channel c).
template <int GROUP, int BITS, typename Buffer>
__device__ __forceinline__ void merge_waves(const uint8_t* areas, int area_stride, const WaveOut& out, int tid, Buffer po,
                                            Buffer pml, bool past_l2) {
    constexpr int M = kD / GROUP, MPL = M >= 2 ? M / 2 : 1;
    const int r = tid >> 7, c = tid & 127;
    // where the channel's sums sit in its set's results: 2 bits [row][plane][j = c % 4][code lane (c / 4) % 16],
    // 1 bit [row][plane][j = c % 8][code lane (c / 8) % 8]
    const int s = c >> 6, i = BITS == 2 ? (c >> 2) & 15 : (c >> 3) & 7, j = BITS == 2 ? c & 3 : c & 7;
    constexpr int NI = BITS == 2 ? 16 : 8;
    const int m = c / GROUP;
    const int hh = M >= 2 ? m / MPL : r, zi = M >= 2 ? r * MPL + m % MPL : 0;   // where the zero-point sum of (r, m) sits
    float mmax = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mmax = fmaxf(mmax, out.m[w][r]);
    float o = 0.0f, lsum = 0.0f;
    // the masks leave a code where it sits in its nibble: 4 x code for odd channels (2 bits), 2^(c % 4) x code (1 bit)
    const float jscale = BITS == 2 ? ((j & 1) ? 0.25f : 1.0f) : __uint_as_float((uint32_t)(127 - (j & 3)) << 23);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const float mwv = out.m[w][r];
        const float e = mwv == -INFINITY ? 0.0f : __expf(mwv - mmax);
        const int* res = reinterpret_cast<const int*>(areas + w * area_stride + s * kSetBytes);
        int f[4];
#pragma unroll
        for (int pp = 0; pp < 4; ++pp) f[pp] = res[(r * 4 + pp) * kResPlane + j * NI + i];
        const float t = of_byte_planes(f[0], f[1], f[2], f[3]);
        float zs = 0.0f, ls = 0.0f;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            zs += out.part[w][g4][hh][zi];
            ls += out.part[w][g4][r][4];
        }
        // a wave without tokens left its area as it was: whatever integers sit there are finite and weigh 0
        const float val = __builtin_fmaf(t, out.unscale[w] * jscale, zs);
        o = __builtin_fmaf(e, val, o);
        lsum = __builtin_fmaf(e, ls, lsum);
    }
    store_partial(po, r * kD + c, o, past_l2);
    if (c == 0) store_max_sum(pml, r, mmax, lsum, past_l2);
}

// Workgroup-wide bitmap of the chunk's staged positions, for index lists too long for every wave to walk
__device__ __forceinline__ void chunk_bitmap(const AttendArgs& A, int topk, int row, int c0, int n, int tid, uint32_t* maskbits) {
    if (tid < kI8Chunk / 32) maskbits[tid] = 0u;
    __syncthreads();
    if (A.slot_idx)
        for (int j = tid; j < topk; j += kThreads) {
            const int t = A.slot_idx[(size_t)row * topk + j] - c0;
            if (t >= 0 && t < n) atomicOr(&maskbits[t >> 5], 1u << (t & 31));
        }
    __syncthreads();
}

// One chunk of a row: its partial results and, FUSED, its positions' logits and selection keys.
template <bool FUSED>
struct I8Shape {
    static constexpr int kAreaBytes = FUSED ? kWaveDwords * 4 : kWaveArea;        // per wave
    static constexpr int kRegion = (kWaves * kAreaBytes) / 4;
};
template <int GROUP, int BITS, bool BF16, bool FUSED, typename Buffer>
__device__ __forceinline__ void attend_i8_chunk(const LayerView& L, const AttendArgs& A, float sm_scale, uint32_t* __restrict__ keys, size_t key_stride, int row, int chunk,
                                                float* smem, uint32_t* maskbits, float2 (*fin)[4][2], WaveOut& wout, Buffer po, Buffer pml) {
    constexpr int NR = 2, kAreaBytes = I8Shape<FUSED>::kAreaBytes;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c0 = chunk * kI8Chunk;
    const int n = (A.Nq - c0) < kI8Chunk ? (A.Nq - c0) : kI8Chunk;   // multiple of 32, >= 32
    const int w0 = kWaveTok * wave;                                    // first token of the wave inside the chunk
    int nw = n - w0;                                                   // its valid tokens
    nw = nw < 0 ? 0 : (nw > kWaveTok ? kWaveTok : nw);
    const int sg = lane >> 4, h = (lane >> 3) & 1;
    const int t0 = 32 * sg + 4 * (lane & 7);                           // first of the lane's four tokens inside the wave
    const bool live = t0 < nw;
    uint8_t* area = reinterpret_cast<uint8_t*>(smem) + wave * kAreaBytes;
    const bool wave_maps = L.topk <= kWaveBitmapTopk;                  // uniform over the launch
    if (!wave_maps) chunk_bitmap(A, L.topk, row, c0, n, tid, maskbits);

    if (nw > 0) {   // wave-uniform
        ValueLoads<GROUP, BITS> v;
        float lgv[4];
        // everything this wave reads from global memory is requested before the first wait on any of it
        int ti[4];
        const int n_idx = A.slot_idx ? L.topk : 0;
        if (wave_maps) wave_bitmap_loads(n_idx ? A.slot_idx + (size_t)row * L.topk : nullptr, L.topk, lane, ti);
        if constexpr (!FUSED) {
            float4 lg4 = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (live) lg4 = *reinterpret_cast<const float4*>(A.logits + ((size_t)row * NR + h) * A.logit_stride + c0 + w0 + t0);
            value_loads<GROUP, BITS>(L, A.Nq, row, c0, w0, nw, lane, v);
            if (wave_maps) wave_bitmap_apply(ti, n_idx, c0 + w0, nw, lane, maskbits + 4 * wave);
            lgv[0] = lg4.x; lgv[1] = lg4.y; lgv[2] = lg4.z; lgv[3] = lg4.w;
        } else {
            // the low-bit logits of the wave's tokens (Appendix A "Decoding": A = Q K^T on C'); the value-side loads
            // are requested once the scoring operands are built and travel while the scoring contraction runs
            score_i8_wave<BITS, GROUP, BF16>(L, A.q, row, chunk, wave, lane, A.Nq / kBlockTokens, sm_scale, reinterpret_cast<uint32_t*>(area),
                                   fin[wave], lgv,
                                   [&]() { if (wave_maps) wave_bitmap_apply(ti, n_idx, c0 + w0, nw, lane, maskbits + 4 * wave); },
                                   [&]() { value_loads<GROUP, BITS>(L, A.Nq, row, c0, w0, nw, lane, v); });
            if (live) {
                if (h == 1) {   // the speculative row ranks the positions
                    const uint4v k4 = {float_to_key(lgv[0]), float_to_key(lgv[1]), float_to_key(lgv[2]), float_to_key(lgv[3])};
                    const auto keys_row = buffer_of(keys + (size_t)row * key_stride, (uint32_t)A.Nq * 4u);
                    // past the L2 where the launch announces them before it ends (finish_row.h)
                    if (A.fin.word) __builtin_amdgcn_raw_buffer_store_b128(k4, keys_row, (c0 + w0 + t0) * 4, 0, kAgentScope);
                    else __builtin_amdgcn_raw_buffer_store_b128(k4, keys_row, (c0 + w0 + t0) * 4, 0, 0);
                }
                if (A.logits_out)   // kept only when the caller asked for them (parity hook)
                    *reinterpret_cast<float4*>(A.logits_out + ((size_t)row * NR + h) * A.logit_stride + c0 + w0 + t0) =
                        make_float4(lgv[0], lgv[1], lgv[2], lgv[3]);
            }
            wave_sync();   // the scoring exchange is over: the area now serves the value side
        }
        value_meta_exchange<GROUP, BITS>(v, lane, area);
        const uint32_t mbits = maskbits[4 * wave + sg] >> (4 * (lane & 7));
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (!live || ((mbits >> j) & 1u)) lgv[j] = -INFINITY;
        value_wave<GROUP, BITS, BF16>(v, lgv, L.one_bit_plain, wave, lane, area, wout);
    } else {
        empty_wave(wave, lane, wout);
    }
    __syncthreads();
    merge_waves<GROUP, BITS>(reinterpret_cast<const uint8_t*>(smem), kAreaBytes, wout, tid, po, pml, A.fin.arrived != nullptr);
}

// Registers: the pass that also scores needs 84 to 90 (five waves per SIMD); compiled for six or eight it
// spills and runs slower (measured at the 7B shape: 28.6 us, 32 with two registers spilled, 58 with 34).  Attention alone takes 64 with 2-bit
// codes (eight waves; its 16-bit chunk asks for the values when the keys are used up: with 16 of them ahead it takes 72, 1 % of a
// step of 128 rows x 30000), and up to 91 with 1-bit codes (held to 80 it spills: 64 -> 82 us for 32 x 32000, one layer).
// What the waves of a full chip wait for is issue slots, of the vector ALUs and of LDS (a wave of 128 tokens: 1136 vector instructions, 1012 since;
// with 1 bit LDS was busy for 58 % of the launch, two fifths of that with bank conflicts).  So maxima are of bits, signs are set behind the transpositions, results
// lie where neither their writers nor their readers share banks, and the metadata's loads have no conditions: a pass of 4 layers
// of 32 x 32768, 1 bit, g = 64 121 -> 115 us, 2 bits, g = 32 132 -> 128, of 8 of 32 x 16384 208 -> 205.5 (sharing the fetch's queue 182 -> 173, 196 ->
// 192, 321 -> 316).
template <int GROUP, int BITS, bool BF16, bool FUSED>
__global__ __launch_bounds__(kThreads, FUSED || BITS == 1 ? 5 : 7) void attend_i8_kernel(LayerView L, AttendArgs A, float sm_scale, uint32_t* __restrict__ keys,
                                                             size_t key_stride) {
    constexpr int NR = 2;
    constexpr int kLoads = FUSED ? 12 : BITS == 2 ? 4 : 8;                // of a thread that merges: no more registers than the rest needs
    constexpr int kRegion = I8Shape<FUSED>::kRegion;
    static_assert(kRegion >= extra_chunk_floats(NR), "a 16-bit chunk in the same region");
    __shared__ __attribute__((aligned(16))) float smem[kRegion];
    __shared__ RowsOut xout;
    __shared__ uint32_t maskbits[kI8Chunk / 32];
    __shared__ __attribute__((aligned(8))) float2 fin[FUSED ? kWaves : 1][4][2];
    __shared__ WaveOut wout;
    __shared__ FinishShared fin_shared;
    static_assert(kRegion * 4 >= kFinishLdsBytes, "the merge of a row in the same region");

    // which (row, chunk): workgroups that append the step's token first, then the 16-bit chunks (chains of dependent loads), then the quantised
    // positions, then the workgroups that only merge
    const int tid = threadIdx.x, n_tail = L.tail_k ? L.rows : 0, bid = (int)blockIdx.x - n_tail, n_extra = A.n_chunks - A.n_main;
    if (bid < 0) {
        // a launch that also appends the step's new token (Appendix A "Decoding": Offload of the new pair to the
        // CPU copy; it also joins the 16-bit residual): one more workgroup per row, 32 lanes x 16 bytes.  They are
        // dispatched first: the store to host memory crosses a link the prefetch keeps busy, and the launch
        // ends only when it has landed.
        const int r = blockIdx.x;
        if (tid < 32) {
            const uint4 v = reinterpret_cast<const uint4*>(tid < 16 ? L.tail_k : L.tail_v)[(size_t)r * 16 + (tid & 15)];
            reinterpret_cast<uint4*>(L.host)[((size_t)r * L.max_seq + L.tail_N0) * 32 + tid] = v;
            reinterpret_cast<uint4*>(L.ring)[((size_t)r * L.R + (L.tail_N0 % L.R)) * 32 + tid] = v;
        }
        return;
    }
    int row, chunk = 0;
    const int main_id = bid - L.rows * n_extra, merger = bid - L.rows * A.n_chunks;
    if (main_id < 0) {
        row = bid / n_extra;
        chunk = A.n_main + bid % n_extra;
    } else if (merger < 0) {
        row = main_id / A.n_main;
        chunk = main_id % A.n_main;
    } else {
        row = merger / A.fin.shares;
    }
    uint32_t shares;
    if (merger < 0) {
        const auto po = buffer_of(A.part_o + (((size_t)row * A.max_chunks + chunk) * NR) * kD, NR * kD * 4);
        const auto pml = buffer_of(A.part_ml + (((size_t)row * A.max_chunks + chunk) * NR) * 2, NR * 8);
        if (chunk >= A.n_main)
            extra_chunk<NR, 2, BF16, FUSED ? 32 : BITS == 1 ? 16 : 0>(L, A, row, chunk, smem, xout, po, pml, A.fin.arrived != nullptr);
        else
            attend_i8_chunk<GROUP, BITS, BF16, FUSED>(L, A, sm_scale, keys, key_stride, row, chunk, smem, maskbits, fin, wout, po, pml);
        if (A.fin.arrived == nullptr) return;
        shares = row_arrival(A, row, fin_shared);
    } else {
        shares = row_complete(A, row, merger % A.fin.shares, fin_shared);
    }
    merge_shares<kLoads>(A, row, NR, shares, smem);
}

}  // namespace

// Both passes in one launch leave the merge to a launch of its own, where they are more workgroups than the chip holds at a time and the step
// fetches more than a pair for so many keys.  The selections on the side streams, each a workgroup that needs most of a compute unit, find one between the
// launches; behind launches of several rounds that follow each other at once they come late, the fetches of the side streams fall into step, and the
// link idles meanwhile.  us a layer, merged inside / so (32 layers, free running): 32 x 32768, k = 256 74.3 to 79.4, up to 70 % of the steps
// slow / 74.0, k = 128 45.2 / 41.3, k = 112 40.1 / 39.5, 1 bit, k = 96 35.5 / 33.0, k = 128 42.4 / 38.4, 32 x 49152, k = 160 59.8 / 59.1 (where link and kernels
// are far from even it is 1 % the other way: k = 192 55.7 / 56.0).  Fewer pairs: k = 96 36.6 / 37.4, k = 80 33.7 / 34.3, k = 64 31.4 / 32.0, 1 bit
// 27.7 / 28.0, 32 x 24576, k = 48 26.5 / 27.2.  One round: 32 x 16384, k = 128 38.2 / 39.5, k = 64 25.3 / 26.5.
constexpr int kRoundChunks = 5 * 256, kMergeKeysPerPair = 384;

bool attend_uses_int8_matrix_cores(const LayerView& L, int n_rows) { return L.G == 1 && n_rows == 2 && (L.bits == 2 || L.bits == 1); }

// keys != null: the scoring pass runs inside the launch (logits are not read; they are written to logits_out if set)
hipError_t launch_attend_i8_partial(const LayerView& L, const void* q, int N, int Nq, float sm_scale, const float* logits,
                                    size_t logit_stride, const uint16_t* slot, const int32_t* slot_idx, const void* k_spec,
                                    const void* v_spec, const AttendScratch& scratch, uint32_t* keys, size_t key_stride,
                                    float* logits_out, const Finish& finish, bool* merged, hipStream_t stream) {
    if (!attend_uses_int8_matrix_cores(L, 2) || Nq % kBlockTokens) return hipErrorInvalidValue;
    AttendArgs A;
    A.q = (const uint16_t*)q;
    A.logits = logits;
    A.logits_out = logits_out;
    A.logit_stride = logit_stride;
    A.slot = slot;
    A.slot_idx = slot_idx;
    A.k_spec = (const uint16_t*)k_spec;
    A.v_spec = (const uint16_t*)v_spec;
    A.part_o = scratch.part_o;
    A.part_ml = scratch.part_ml;
    A.max_chunks = scratch.max_chunks;
    A.N = N;
    A.Nq = Nq;
    A.sm_scale = sm_scale;
    const int n_ex = (slot_idx ? L.topk : 0) + (N - Nq) + (k_spec ? 1 : 0);
    A.n_main = (Nq + kI8Chunk - 1) / kI8Chunk;
    A.n_chunks = A.n_main + (n_ex + kExtraChunk - 1) / kExtraChunk;
    if (A.n_chunks > A.max_chunks || A.n_chunks < 1) return hipErrorInvalidValue;
    A.fin = finish;
    if (keys && slot_idx && L.rows * A.n_chunks > kRoundChunks && Nq < kMergeKeysPerPair * L.topk) A.fin.arrived = nullptr;
    *merged = plan_merge(A.fin, L.rows, A.n_chunks, 2, !keys || L.rows <= kFinishFewRows);
    const dim3 grid((A.n_chunks + (A.fin.mergers ? A.fin.shares : 0)) * L.rows + (L.tail_k ? L.rows : 0)), block(kThreads);
#define SPC_AI8_B(G_, B_, F_)                                                                                              \
    do {                                                                                                                   \
        if (keys) SPC_LAUNCH((attend_i8_kernel<G_, B_, F_, true>), grid, block, stream, L, A, sm_scale, keys, key_stride); \
        else SPC_LAUNCH((attend_i8_kernel<G_, B_, F_, false>), grid, block, stream, L, A, sm_scale, keys, key_stride);     \
    } while (0)
#define SPC_AI8(G_, F_)                    \
    do {                                   \
        if (L.bits == 2) SPC_AI8_B(G_, 2, F_); \
        else SPC_AI8_B(G_, 1, F_);         \
    } while (0)
    if (L.group == 32) { if (L.bf16) SPC_AI8(32, true); else SPC_AI8(32, false); }
    else if (L.group == 64) { if (L.bf16) SPC_AI8(64, true); else SPC_AI8(64, false); }
    else if (L.group == 128) { if (L.bf16) SPC_AI8(128, true); else SPC_AI8(128, false); }
    else return hipErrorInvalidValue;
#undef SPC_AI8_B
#undef SPC_AI8
    return hipGetLastError();
}

}  // namespace specache
