// Mixed attention of Eq. 1 (Section 3.3): Attn([T_t, T'_{t+1}], C' u C_K).
//
// Candidates of a query row: quantised positions i < Nq (the prefetched 16-bit
// pair where i is in the slot's index list, the dequantised low-bit pair
// elsewhere), the 16-bit residual positions, and for the speculative row its own
// transient pair.  The low-bit logits were kept by the scoring pass.
//
// Split over the sequence: "main" workgroups take chunks of quantised positions,
// "extra" workgroups take the 16-bit candidates (staged pairs, residual, transient
// pair); each writes an un-normalised partial (max, sum, sum p*V), merged with the usual
// log-sum-exp rescaling inside the launch (finish_row.h) or by a kernel of its own
// (attend_merge_kernel; attend_combine_kernel for rows of very many chunks).  Prefetched positions
// are removed from the main chunks by setting their logit to -inf in LDS; the
// staged pair then enters through the extra chunks, which is Eq. 1's "replace".
//
// Values are quantised per token over g channels, so for the main chunks
//   sum_i p_i V'[i][c] = sum_i (p_i s[i][m]) code[i][c] + sum_i p_i z[i][m],  m = c / g.
// The first sum runs on the vector ALUs: a lane owns 8/BITS channels and reads 16 tokens of them as one 16-byte load;
// p_i s[i][m] comes from LDS (computed once per token by the softmax phase).  With 4, 8 or 16 query rows per KV head the
// matrix cores take the contraction (rows_mfma.h).
#include "attend_common.h"
#include "extra_wave.h"
#include "finish_row.h"

namespace specache {
namespace {

constexpr int kMainChunk = 512;   // quantised positions per workgroup

// MERGES: rows short enough for the merge inside the launch (last_chunk_merges), where few workgroups wait for the 16-bit chunk's chain of
// loads: it asks for 14 values with the keys (with 16, one instance spills a register) and the kernel takes 72 registers.  Longer rows fill the
// chip and are bound by vector issue: eight waves per SIMD (64 registers), no code and no arguments of the merge, the 16-bit chunks last.
// Attention with one query row, us (the kernel before the merge was there, one kernel of 72 registers for both with scalar ones spilled, now):
// 1 bit, g = 128, 16 x 60000 11.7, 13.1, 11.5; 16 x 65000 12.4, 13.4, 12.9; 8 x 131000 12.0, 13.8, 12.8; g = 32, 32 x 32300 14.0, 16.2, 14.6; 2
// bits, 16 x 65000 13.5, 15.1, 13.9.
template <int BITS, int GROUP, int G, int NROWS, bool BF16, bool MERGES>
__global__ __launch_bounds__(kThreads, MERGES ? 7 : 8) void attend_partial_kernel(LayerView L, AttendArgs A) {
    constexpr int NR = G * NROWS;
    constexpr int CH = kMainChunk;
    constexpr int M = kD / GROUP;            // value groups per token
    constexpr int CPB = 8 / BITS;            // channels per code byte (per lane)
    constexpr int LPB = 32 * BITS;           // lanes per 32-token block
    constexpr uint32_t MASK = ((1u << BITS) - 1u) * 0x01010101u;
    constexpr int TPT = (CH + kThreads - 1) / kThreads;   // chunk tokens per thread
    // One LDS region serves, in turn: for main chunks ps[M][CH][NR]; for extra chunks the areas of
    // extra_chunk; at the end o_lds[kWaves][NR][128].
    // ps is stored in cells [16-token half block][value group m] of 16*NR floats plus one
    // 16-byte pad: the lanes of one LDS read differ only in (half block, m), i.e. in
    // consecutive cells, and the pad spreads those over distinct banks.
    constexpr int kCell = 16 * NR + 4;
    constexpr int kPs = (CH / 16) * M * kCell, kOl = kWaves * NR * kD;
    // a workgroup is either a main or an extra chunk (16-bit candidates, extra_chunk): both use
    // the one region, and LDS per workgroup decides how many chunks are resident per compute unit
    constexpr int kExtra = extra_chunk_floats(NR);
    constexpr int kMax1 = kExtra > kPs ? kExtra : kPs;
    constexpr int kMax2 = kMax1 > kOl ? kMax1 : kOl;
    constexpr int kRegion = !MERGES || kMax2 * 4 > kFinishLdsBytes ? kMax2 : kFinishLdsBytes / 4;
    __shared__ __attribute__((aligned(16))) float smem[kRegion];
    __shared__ float red[kWaves * NR * (1 + M)];
    __shared__ float red_sum[kWaves * NR];
    __shared__ float red_z[kWaves * NR * M];
    __shared__ uint32_t maskbits[CH / 32];
    __shared__ FinishShared fin_shared;
    __shared__ RowsOut xout;

    float* ps = smem;                        // [CH/16][M] cells
    float* o_lds = smem;                     // [kWaves][NR][128]

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // The 16-bit chunks are chains of dependent loads.  Where the whole launch is resident at once (MERGES) they are dispatched first (all
    // rows).  Where it is not they go last: first, the many rows' chunks wait together while the chip has nothing else to do (one query row,
    // 2 bits, g = 32, scoring and attention: 512 x 2000 37.1 us, last 35.6; 256 x 4000 34.9 / 33.8; 16 x 60000 31.8 / 31.2).
    const int n_extra = A.n_chunks - A.n_main, rows = L.rows;
    const int id = blockIdx.x, n_first = rows * (MERGES ? n_extra : A.n_main);
    int row, chunk;
    if ((id < n_first) == MERGES) {
        const int x = MERGES ? id : id - n_first;
        row = x / n_extra;
        chunk = A.n_main + x % n_extra;
    } else {
        const int m = MERGES ? id - n_first : id;
        row = m / A.n_main;
        chunk = m % A.n_main;
    }
    float m_row[NR], l_row[NR];
    // (built where they are used: held from here on they took scalar registers that the main chunk's arguments were spilled for)
    auto part_o = [&]() { return buffer_of(A.part_o + (((size_t)row * A.max_chunks + chunk) * NR) * kD, NR * kD * 4); };
    auto part_ml = [&]() { return buffer_of(A.part_ml + (((size_t)row * A.max_chunks + chunk) * NR) * 2, NR * 8); };

    if (chunk < A.n_main) {
        // ------------------------------------------------------------ quantised positions
        const int c0 = chunk * CH;
        const int n = (A.Nq - c0) < CH ? (A.Nq - c0) : CH;   // multiple of 32
        const uint8_t* vc_row = L.vc + (size_t)row * L.vc_stride + (size_t)(c0 / kBlockTokens) * code_block_bytes(BITS);
        const uint32_t* vm_row = L.vm + (size_t)row * L.vm_stride;
        const int units = (n / kBlockTokens) * LPB;
        const int within = lane % LPB;                       // position inside a block
        const int Lc = within % (16 * BITS);                 // code lane: channels Lc*CPB .. +CPB-1
        const int mgrp = (Lc * CPB) / GROUP;
        const uint8_t* vc_lane = vc_row + within * 16;

        // every global read this thread needs before the value loop is issued up front
        float lgr[TPT][NR];
        uint32_t meta[TPT][M];
#pragma unroll
        for (int tt = 0; tt < TPT; ++tt) {
            const int i = tid + tt * kThreads;
            const bool valid = i < n;
#pragma unroll
            for (int r = 0; r < NR; ++r)
                lgr[tt][r] = valid ? A.logits[((size_t)row * NR + r) * A.logit_stride + c0 + i] : -INFINITY;
            if constexpr (M == 4) {
                const uint4 t4 = valid ? *reinterpret_cast<const uint4*>(vm_row + (size_t)(c0 + i) * 4) : make_uint4(0, 0, 0, 0);
                meta[tt][0] = t4.x; meta[tt][1] = t4.y; meta[tt][2] = t4.z; meta[tt][3] = t4.w;
            } else if constexpr (M == 2) {
                const uint2 t2 = valid ? *reinterpret_cast<const uint2*>(vm_row + (size_t)(c0 + i) * 2) : make_uint2(0, 0);
                meta[tt][0] = t2.x; meta[tt][1] = t2.y;
            } else {
                meta[tt][0] = valid ? vm_row[c0 + i] : 0u;
            }
        }
        // the first value codes of this thread, needed only after the softmax phase
        uint4 w4_first = make_uint4(0, 0, 0, 0);
        if (tid < units) w4_first = *reinterpret_cast<const uint4*>(vc_lane + (size_t)(tid / LPB) * code_block_bytes(BITS));
        // prefetched positions of this chunk, as a bitmap (the first entries of the index list
        // are requested with the other loads)
        constexpr int kIdxUpfront = 2;
        int sidx[kIdxUpfront];
#pragma unroll
        for (int u = 0; u < kIdxUpfront; ++u) {
            const int j = tid + u * kThreads;
            sidx[u] = (A.slot_idx && j < L.topk) ? A.slot_idx[(size_t)row * L.topk + j] : -1;
        }
        if (tid < CH / 32) maskbits[tid] = 0u;
        __syncthreads();
        if (A.slot_idx) {
#pragma unroll
            for (int u = 0; u < kIdxUpfront; ++u) {
                const int t = sidx[u] - c0;
                if (sidx[u] >= 0 && t >= 0 && t < n) atomicOr(&maskbits[t >> 5], 1u << (t & 31));
            }
            for (int j = tid + kIdxUpfront * kThreads; j < L.topk; j += kThreads) {
                const int t = A.slot_idx[(size_t)row * L.topk + j] - c0;
                if (t >= 0 && t < n) atomicOr(&maskbits[t >> 5], 1u << (t & 31));
            }
        }
        __syncthreads();

        float mloc[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) mloc[r] = -INFINITY;
#pragma unroll
        for (int tt = 0; tt < TPT; ++tt) {
            const int i = tid + tt * kThreads;
            const bool masked = i < n && ((maskbits[i >> 5] >> (i & 31)) & 1u);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                if (masked) lgr[tt][r] = -INFINITY;
                mloc[r] = fmaxf(mloc[r], lgr[tt][r]);
            }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const float v = wave_max(mloc[r]);
            if (lane == 0) red[wave * NR + r] = v;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            float v = red[r];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) v = fmaxf(v, red[w * NR + r]);
            m_row[r] = v;
        }

        // p = exp(l - m); p * s per (token, value group); the zero-point term sum_i p_i z[i][m] and
        // the row sums sum_i p_i: every thread adds up its own tokens and the waves reduce those sums
        float zacc[NR][M], sloc[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            sloc[r] = 0.0f;
#pragma unroll
            for (int m = 0; m < M; ++m) zacc[r][m] = 0.0f;
        }
#pragma unroll
        for (int tt = 0; tt < TPT; ++tt) {
            const int i = tid + tt * kThreads;
            if (i < n) {
                float p[NR];
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const float ms = m_row[r] == -INFINITY ? 0.0f : m_row[r];
                    p[r] = __expf(lgr[tt][r] - ms);
                    sloc[r] += p[r];
                }
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    float sc, z;
                    derive_scale_zero<BITS>(widen16<BF16>(meta[tt][m] & 0xFFFFu), widen16<BF16>(meta[tt][m] >> 16), L.one_bit_plain, sc, z);
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        ps[((i >> 4) * M + m) * kCell + (i & 15) * NR + r] = p[r] * sc;
                        zacc[r][m] = __builtin_fmaf(p[r], z, zacc[r][m]);
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const float v = wave_sum(sloc[r]);
            if (lane == 0) red_sum[wave * NR + r] = v;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const float zv = wave_sum(zacc[r][m]);
                if (lane == 0) red_z[(wave * NR + r) * M + m] = zv;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            float v = red_sum[r];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) v += red_sum[w * NR + r];
            l_row[r] = v;
        }

        // sum_i (p_i s_i) code[i][c] for this lane's CPB channels
        float acc[CPB][NR];
#pragma unroll
        for (int j = 0; j < CPB; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[j][r] = 0.0f;
        uint4 w4 = w4_first;
        for (int u = tid; u < units; u += kThreads) {
            const int blk = u / LPB;
            uint4 w4n = make_uint4(0, 0, 0, 0);   // next iteration's codes, in flight during this one's arithmetic
            if (u + kThreads < units)
                w4n = *reinterpret_cast<const uint4*>(vc_lane + (size_t)((u + kThreads) / LPB) * code_block_bytes(BITS));
            const int hb = blk * 2 + within / (16 * BITS);   // 16-token half block inside the chunk
            const float* psb = ps + (hb * M + mgrp) * kCell;
#pragma unroll
            for (int dq = 0; dq < 4; ++dq) {
                const uint32_t w = comp(w4, dq);
                float pv[4][NR];
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < NR; ++r) pv[b][r] = psb[(dq * 4 + b) * NR + r];
#pragma unroll
                for (int j = 0; j < CPB; ++j) {
                    const uint32_t mk = w & (MASK << (BITS * j));
                    const float f0 = cvt_ubyte<0>(mk), f1 = cvt_ubyte<1>(mk), f2 = cvt_ubyte<2>(mk), f3 = cvt_ubyte<3>(mk);
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        acc[j][r] = __builtin_fmaf(f0, pv[0][r], acc[j][r]);
                        acc[j][r] = __builtin_fmaf(f1, pv[1][r], acc[j][r]);
                        acc[j][r] = __builtin_fmaf(f2, pv[2][r], acc[j][r]);
                        acc[j][r] = __builtin_fmaf(f3, pv[3][r], acc[j][r]);
                    }
                }
            }
            w4 = w4n;
        }
        // codes arrived scaled by 2^(BITS*j); lanes with equal Lc hold the same channels
#pragma unroll
        for (int j = 0; j < CPB; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                float v = acc[j][r] * __uint_as_float((uint32_t)(127 - BITS * j) << 23);
#pragma unroll
                for (int mask = 32; mask >= 16 * BITS; mask >>= 1) v += __shfl_xor(v, mask, 64);
                acc[j][r] = v;
            }
        __syncthreads();   // o_lds shares the region with ps: everyone is done with ps
        if (lane < 16 * BITS) {
#pragma unroll
            for (int j = 0; j < CPB; ++j)
#pragma unroll
                for (int r = 0; r < NR; ++r) o_lds[((size_t)wave * NR + r) * kD + Lc * CPB + j] = acc[j][r];
        }
        __syncthreads();
        const auto po = part_o();
        for (int e = tid; e < NR * kD; e += kThreads) {
            const int r = e / kD, c = e % kD;
            float v = 0.0f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v += o_lds[((size_t)w * NR + r) * kD + c] + red_z[(w * NR + r) * M + c / GROUP];
            store_partial(po, e, v, MERGES);
        }
        if (tid < NR) {
            float mv = 0.f, lv = 0.f;
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (r == tid) { mv = m_row[r]; lv = l_row[r]; }
            store_max_sum(part_ml(), tid, mv, lv, MERGES);
        }
    } else {
        extra_chunk<NR, NROWS, BF16, MERGES ? 14 : 0>(L, A, row, chunk, smem, xout, part_o(), part_ml(), MERGES);
    }
    if constexpr (MERGES) merge_shares<8>(A, row, NR, row_arrival(A, row, fin_shared), smem);
}

// The merge of merge_rows (finish_row.h) in a launch of its own, a workgroup per share: for calls that bring scratch memory of their own
// (the sums are then those of the merge inside a launch, bit by bit) and what last_chunk_merges (kernels.h) leaves.
__global__ __launch_bounds__(kThreads) void attend_merge_kernel(AttendArgs A, int NR, Announce announce) {
    if (announce.word && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(announce.word, announce.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __shared__ __attribute__((aligned(16))) float lds[kFinishLdsBytes / 4];
    merge_rows<16>(A, blockIdx.x / A.fin.shares, NR, blockIdx.x % A.fin.shares, __builtin_ctz(NR / A.fin.shares), lds);
}

// Merge the chunk partials of one (KV head, query row): o = sum_c o_c e^(m_c - m) / sum_c l_c e^(m_c - m).
// 1024 threads = 16 slices of the chunk list x 64 channel pairs; the chunk weights are
// computed once into LDS so that the partial-output loads are independent of each other.
// Takes the rows of more than kFinishChunks chunks (kernels.h).
constexpr int kCombineMaxChunks = 1280;
constexpr int kCombineThreads = 1024, kCombineSlices = kCombineThreads / 64;
__global__ __launch_bounds__(kCombineThreads) void attend_combine_kernel(const float* __restrict__ part_o,
                                                                         const float* __restrict__ part_ml,
                                                                         int max_chunks, int n_chunks, int NR,
                                                                         float* __restrict__ out, Announce announce) {
    // The kernel boundary in front of this kernel has made everything the earlier launch wrote visible, so a plain store is
    // all another stream's wait needs.
    if (announce.word && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(announce.word, announce.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __shared__ float wgt[kCombineMaxChunks];
    __shared__ float red[2 * kCombineSlices];
    __shared__ float2 osum[kCombineSlices][64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int row = blockIdx.x / NR, r = blockIdx.x % NR;
    const float* ml = part_ml + ((size_t)row * max_chunks * NR + r) * 2;
    const size_t ml_stride = (size_t)NR * 2;
    // the first batch of partial outputs is requested before anything depends on the maxima
    const int cp = lane, slice = wave;
    const float2* po = reinterpret_cast<const float2*>(part_o + ((size_t)row * max_chunks * NR + r) * kD) + cp;
    const size_t po_stride = (size_t)NR * kD / 2;
    float2 v0[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int ch = slice + kCombineSlices * u;
        v0[u] = ch < n_chunks ? po[ch * po_stride] : make_float2(0.f, 0.f);
    }
    // (max, sum) of this thread's chunks: one 8-byte load each, all requested at once
    constexpr int kMlPerThread = (kCombineMaxChunks + kCombineThreads - 1) / kCombineThreads;
    float2 mlv[kMlPerThread];
#pragma unroll
    for (int u = 0; u < kMlPerThread; ++u) {
        const int ch = tid + u * kCombineThreads;
        mlv[u] = ch < n_chunks ? *reinterpret_cast<const float2*>(ml + ch * ml_stride) : make_float2(-INFINITY, 0.0f);
    }
    float mloc = -INFINITY;
#pragma unroll
    for (int u = 0; u < kMlPerThread; ++u) mloc = fmaxf(mloc, mlv[u].x);
    mloc = wave_max(mloc);
    if (lane == 0) red[wave] = mloc;
    __syncthreads();
    float mmax = red[0];
#pragma unroll
    for (int w = 1; w < kCombineSlices; ++w) mmax = fmaxf(mmax, red[w]);
    float dloc = 0.0f;
#pragma unroll
    for (int u = 0; u < kMlPerThread; ++u) {
        const int ch = tid + u * kCombineThreads;
        if (ch < n_chunks) {
            const float w = mlv[u].x == -INFINITY ? 0.0f : __expf(mlv[u].x - mmax);
            wgt[ch] = w;
            dloc = __builtin_fmaf(mlv[u].y, w, dloc);
        }
    }
    dloc = wave_sum(dloc);
    if (lane == 0) red[kCombineSlices + wave] = dloc;
    __syncthreads();
    float den = 0.0f;
#pragma unroll
    for (int w = 0; w < kCombineSlices; ++w) den += red[kCombineSlices + w];
    float2 o = make_float2(0.f, 0.f);
    for (int c0 = slice; c0 < n_chunks; c0 += kCombineSlices * 8) {
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int ch = c0 + kCombineSlices * u;
            if (c0 == slice) v[u] = v0[u];
            else v[u] = ch < n_chunks ? po[ch * po_stride] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int ch = c0 + kCombineSlices * u;
            const float w = ch < n_chunks ? wgt[ch] : 0.0f;
            if (w != 0.0f) {   // a chunk without candidates may hold anything
                o.x = __builtin_fmaf(v[u].x, w, o.x);
                o.y = __builtin_fmaf(v[u].y, w, o.y);
            }
        }
    }
    osum[slice][cp] = o;
    __syncthreads();
    if (tid < 64) {
        float2 res = make_float2(0.f, 0.f);
#pragma unroll
        for (int w = 0; w < kCombineSlices; ++w) {
            res.x += osum[w][tid].x;
            res.y += osum[w][tid].y;
        }
        res.x /= den;
        res.y /= den;
        reinterpret_cast<float2*>(out + ((size_t)row * NR + r) * kD)[tid] = res;
    }
}

// the merge that no launch has done
hipError_t launch_merge(const LayerView& L, AttendArgs A, int NR, float* out, Announce announce, hipStream_t stream) {
    if (A.n_chunks > kFinishChunks) {
        SPC_LAUNCH(attend_combine_kernel, dim3(L.rows * NR), dim3(kCombineThreads), stream, A.part_o, A.part_ml, A.max_chunks, A.n_chunks, NR, out, announce);
    } else {
        A.fin = Finish{};
        A.fin.out = out;
        A.fin.shares = merge_shares_of(A.n_chunks, NR);
        SPC_LAUNCH(attend_merge_kernel, dim3(L.rows * A.fin.shares), dim3(kThreads), stream, A, NR, announce);
    }
    return hipGetLastError();
}

template <int BITS, int GROUP, int G, int NROWS>
hipError_t launch3(const LayerView& L, const AttendArgs& A, int n_extra, float* out, int phases, Announce announce, hipStream_t stream) {
    constexpr int NR = G * NROWS;
    if (A.n_main + n_extra > kCombineMaxChunks) return hipErrorInvalidValue;
    if (phases & kAttendPartial) {
        const dim3 grid((A.n_main + n_extra) * L.rows), block(kThreads);
        if (L.bf16 && A.fin.arrived)
            SPC_LAUNCH((attend_partial_kernel<BITS, GROUP, G, NROWS, true, true>), grid, block, stream, L, A);
        else if (L.bf16)
            SPC_LAUNCH((attend_partial_kernel<BITS, GROUP, G, NROWS, true, false>), grid, block, stream, L, A);
        else if (A.fin.arrived)
            SPC_LAUNCH((attend_partial_kernel<BITS, GROUP, G, NROWS, false, true>), grid, block, stream, L, A);
        else
            SPC_LAUNCH((attend_partial_kernel<BITS, GROUP, G, NROWS, false, false>), grid, block, stream, L, A);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if ((phases & kAttendCombine) && !A.fin.arrived) return launch_merge(L, A, NR, out, announce, stream);
    return hipSuccess;
}

template <int BITS, int GROUP>
hipError_t launch2(const LayerView& L, AttendArgs& A, int n_rows, int n_ex, float* out, int phases, Announce announce, hipStream_t stream) {
#define SPC_CASE(g_, n_)                                                        \
    if (L.G == g_ && n_rows == n_) {                                            \
        A.n_main = (A.Nq + kMainChunk - 1) / kMainChunk;                        \
        const int n_extra = (n_ex + kExtraChunk - 1) / kExtraChunk;             \
        A.n_chunks = A.n_main + n_extra;                                        \
        if (A.n_main + n_extra > A.max_chunks) return hipErrorInvalidValue;     \
        const bool i8 = attend_uses_int8_matrix_cores(L, n_rows) && !(kernel_choice() & kChoiceAttendValu); \
        if (!(i8 ? plan_merge(A.fin, L.rows, A.n_chunks, g_ * n_, false) : last_chunk_merges(L.rows, A.n_chunks, g_ * n_))) A.fin = Finish{}; \
        return launch3<BITS, GROUP, g_, n_>(L, A, n_extra, out, phases, announce, stream); \
    }
    SPC_CASE(1, 1) SPC_CASE(1, 2) SPC_CASE(2, 1)
#undef SPC_CASE
    return hipErrorInvalidValue;
}

}  // namespace

// What the limits of specache_create and specache_attend_static are stated in: the chunks above, half as long with 16 rows
// (rows_kernel splits a row as the room allows).
int attend_main_chunk_tokens(int NR) { return NR <= 8 ? kMainChunk : kMainChunk / 2; }
int attend_chunks(int NR, int Nq, int n_16bit) {
    const int chunk = attend_main_chunk_tokens(NR);
    return (Nq + chunk - 1) / chunk + (n_16bit + kExtraChunk - 1) / kExtraChunk;
}
int attend_extra_chunk_tokens() { return kExtraChunk; }
int attend_max_chunks() { return kCombineMaxChunks; }

hipError_t launch_attend(const LayerView& L, const void* q, int n_rows, int N, int Nq, float sm_scale,
                         const float* logits, size_t logit_stride, const uint16_t* slot, const int32_t* slot_idx,
                         const void* k_spec, const void* v_spec, const AttendScratch& scratch, float* out,
                         int phases, uint32_t* arrived, hipStream_t stream, Announce announce) {
    AttendArgs A;
    A.q = (const uint16_t*)q;
    A.logits = logits;
    A.logits_out = nullptr;
    A.q_out = nullptr;
    A.logit_stride = logit_stride;
    A.slot = slot;
    A.slot_idx = slot_idx;
    A.k_spec = (const uint16_t*)k_spec;
    A.v_spec = (const uint16_t*)v_spec;
    A.part_o = scratch.part_o;
    A.part_ml = scratch.part_ml;
    A.max_chunks = scratch.max_chunks;
    A.n_main = 0;
    A.n_chunks = 0;
    A.N = N;
    A.Nq = Nq;
    A.sm_scale = sm_scale;
    A.fin.arrived = arrived;
    A.fin.out = out;
    A.fin.rows = L.rows;
    const int n_ex = (slot_idx ? L.topk : 0) + (N - Nq) + (k_spec ? 1 : 0);
    // 4, 8 or 16 query rows per KV head, and 4-bit codes: a partial pass of their own (rows_mfma.h), with its own chunking
    if (rows_uses_matrix_cores(L, n_rows)) {
        const int n_chunks = rows_chunks(L, n_rows, Nq, n_ex, A.max_chunks);
        const bool merged = plan_merge(A.fin, L.rows, n_chunks, L.G * n_rows, true);
        if (phases & kAttendPartial) {
            RowsArgs R{A, nullptr, 0, n_rows, 0};
            hipError_t e = launch_rows(L, R, kRowsAttend, nullptr, stream);
            if (e != hipSuccess) return e;
        }
        A.n_chunks = n_chunks;
        if ((phases & kAttendCombine) && !merged) return launch_merge(L, A, L.G * n_rows, out, announce, stream);
        return hipSuccess;
    }
    // one query head per KV head, two rows, 2-bit values: the partial pass with the value side on the
    // integer matrix cores (same chunking, same partial-result format, same merge kernel)
    if ((phases & kAttendPartial) && attend_uses_int8_matrix_cores(L, n_rows) && !(kernel_choice() & kChoiceAttendValu)) {
        bool merged = false;
        hipError_t e = launch_attend_i8_partial(L, q, N, Nq, sm_scale, logits, logit_stride, slot, slot_idx, k_spec, v_spec,
                                                scratch, nullptr, 0, nullptr, A.fin, &merged, stream);
        if (e != hipSuccess) return e;
        phases &= ~kAttendPartial;
        if (!phases) return hipSuccess;
    }
    if (L.bits == 2 && L.group == 32) return launch2<2, 32>(L, A, n_rows, n_ex, out, phases, announce, stream);
    if (L.bits == 2 && L.group == 64) return launch2<2, 64>(L, A, n_rows, n_ex, out, phases, announce, stream);
    if (L.bits == 1 && L.group == 32) return launch2<1, 32>(L, A, n_rows, n_ex, out, phases, announce, stream);
    if (L.bits == 1 && L.group == 64) return launch2<1, 64>(L, A, n_rows, n_ex, out, phases, announce, stream);
    if (L.bits == 2 && L.group == 128) return launch2<2, 128>(L, A, n_rows, n_ex, out, phases, announce, stream);
    if (L.bits == 1 && L.group == 128) return launch2<1, 128>(L, A, n_rows, n_ex, out, phases, announce, stream);
    return hipErrorInvalidValue;
}

}  // namespace specache
