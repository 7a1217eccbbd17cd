// Merge of a row's chunk partials inside the launch that makes them: the (max, sum, sum p V) of a (batch, KV head) row's chunks are combined
// with the usual log-sum-exp rescaling by workgroups that only merge, or by the workgroup that completes the row, and the
// one that completes the last row announces the scores (Announce).  A kernel boundary costs the stream 2.5 us, and 6 beside a prefetch (the
// command processor reads packets over the link that the prefetch keeps busy; a chain of empty kernels), the merge kernel 2 to 6 us,
// and its launch 3 us of the issuing thread.  What the merge takes here is a chain of memory round trips: the last stores, the
// counter, the partials.  Measured at plan_merge (kernels.h), the rule for it.
//
// What the other workgroups wrote has to be visible across the XCDs' L2 caches without a fence: a device-scope release writes the
// XCD's whole L2 back, and in every workgroup it made the kernel eight times slower.  So the partials (and the selection keys, where
// the word announces them) are stored past the L2 (kAgentScope), each thread waits until its stores have arrived, the workgroup
// counts itself at device scope, and whoever finds the count complete loads the partials past its L2 as well.
#pragma once
#include "attend_common.h"
#include "extra_wave.h"

namespace specache {
namespace {

// LDS besides the region
struct FinishShared {
    uint32_t shares;
};
constexpr int kFinishPairs = kFinishChunks / 32;                    // (max, sum) pairs of a lane
constexpr int kFinishLoads = 16;                                    // partials of a lane under way, at most
constexpr int kFinishWeights = kFinishChunks + kFinishLoads;        // of a half wave
constexpr int kFinishLdsBytes = 8 * kFinishWeights * 4 + kThreads * 16;   // the chunks' weights of every half wave, then the slices' sums

__device__ __forceinline__ float half_wave_max(float v) {
    v = fmaxf(v, dpp_move<kDppXor1>(v));
    v = fmaxf(v, dpp_move<kDppXor2>(v));
    v = fmaxf(v, dpp_move<kDppHalfMirror>(v));
    return xor16_max(fmaxf(v, dpp_move<kDppMirror>(v)));
}
__device__ __forceinline__ float half_wave_sum(float v) {
    v += dpp_move<kDppXor1>(v);
    v += dpp_move<kDppXor2>(v);
    v += dpp_move<kDppHalfMirror>(v);
    return xor16_sum(v + dpp_move<kDppMirror>(v));
}

// Merges share `share` of a row whose partials have all arrived: query rows nr share to nr share + nr - 1 (nr = 2^log_nr <= 8).  Half a
// wave takes one query row and every (8 / nr)-th chunk, a lane four outputs; its first LOADS partials and the (max, sum) pairs are
// requested together.  lds: kFinishLdsBytes, 16-byte aligned, free once every thread has arrived here.
template <int LOADS>
__device__ __forceinline__ void merge_rows(const AttendArgs& A, int row, int nq, int share, int log_nr, float* lds) {
    typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
    static_assert(LOADS % 4 == 0 && LOADS <= kFinishLoads, "weights are read by fours, and as far as the loads go");
    const int tid = threadIdx.x, l = tid & 31, n = A.n_chunks, nr = 1 << log_nr, log_slices = 3 - log_nr;
    int half = tid >> 5;
    asm volatile("" : "+v"(half));                                     // (addresses of one share are not kept for the next: they would be spilled)
    const int r = nr * share + (half & (nr - 1)), slice = half >> log_nr;
    // beyond the row's chunks a load returns 0
    const auto po = buffer_of(A.part_o + (size_t)row * A.max_chunks * nq * kD, (uint32_t)(n * nq * kD * 4));
    const auto pml = buffer_of(A.part_ml + (size_t)row * A.max_chunks * nq * 2, (uint32_t)(n * nq * 8));
    float* wgt = lds + half * kFinishWeights;                          // of the half wave's chunks, side by side
    float4v* part = reinterpret_cast<float4v*>(lds + 8 * kFinishWeights);
    const int step = (nq * kD * 4) << log_slices;                      // bytes between them
    int at = ((slice * nq + r) * kD + 4 * l) * 4;
    float4v v[LOADS];
    auto load = [&](int left) {                                        // left: chunks from here on; four of a slice's at a time
#pragma unroll
        for (int u4 = 0; u4 < LOADS; u4 += 4) {
            if (u4 > 0 && u4 << log_slices >= left) break;             // uniform
#pragma unroll
            for (int u = u4; u < u4 + 4; ++u) v[u] = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(po, at, u * step, kAgentScope));
        }
    };
    uint2v pair[kFinishPairs];
#pragma unroll
    for (int j = 0; j < kFinishPairs; ++j) {
        if (j > 0 && 32 * j >= n) break;                               // uniform
        pair[j] = __builtin_amdgcn_raw_buffer_load_b64(pml, (l * nq + r) * 8, j * nq * 256, kAgentScope);
    }
    load(n);
    float m = -INFINITY, den = 0.0f;
#pragma unroll
    for (int j = 0; j < kFinishPairs; ++j) m = fmaxf(m, 32 * j + l < n ? __uint_as_float(pair[j].x) : -INFINITY);
    m = half_wave_max(m);
#pragma unroll
    for (int j = 0; j < kFinishPairs; ++j) {
        if (j > 0 && 32 * j >= n) break;
        const int ch = 32 * j + l;
        const float pm = __uint_as_float(pair[j].x);
        const float w = ch >= n || pm == -INFINITY ? 0.0f : __expf(pm - m);
        if ((ch & ((1 << log_slices) - 1)) == slice) wgt[ch >> log_slices] = w;
        den = __builtin_fmaf(__uint_as_float(pair[j].y), w, den);
    }
    if (l < LOADS) wgt[((n + 31) >> 5 << 5 >> log_slices) + l] = 0.0f;   // the last batch may reach beyond
    den = half_wave_sum(den);
    wave_sync();
    float4v o = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](int left) {
#pragma unroll
        for (int u4 = 0; u4 < LOADS; u4 += 4) {
            if (u4 > 0 && u4 << log_slices >= left) break;
            const float4v w = *reinterpret_cast<const float4v*>(wgt + u4);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = w[u] != 0.0f ? __builtin_fmaf(v[u4 + u][e], w[u], o[e]) : o[e];   // a chunk without candidates may hold anything
        }
    };
    add(n);
#pragma unroll 1
    for (int c0 = LOADS << log_slices; c0 < n; c0 += LOADS << log_slices) {
        at += LOADS * step;
        wgt += LOADS;
        load(n - c0);
        add(n - c0);
    }
    if (nr < 8) {
        part[tid] = o;
        __syncthreads();
#pragma unroll 1
        for (int s = 32 * nr; s < kThreads; s += 32 * nr) o += part[(tid & (32 * nr - 1)) + s];
    }
    if (slice == 0) *reinterpret_cast<float4*>(A.fin.out + ((size_t)row * nq + r) * kD + 4 * l) = make_float4(o[0] / den, o[1] / den, o[2] / den, o[3] / den);
}

// What a workgroup merges of its row, as bits of shares: nothing, mostly.  Uniform over the workgroup.
//
// A workgroup that has stored its chunk's partials, all of its kThreads threads: everything if it is the last of the row, or
// what the mergers left to it.
__device__ __forceinline__ uint32_t row_arrival(const AttendArgs& A, int row, FinishShared& fs) {
    const Finish& F = A.fin;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have arrived
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t* at = F.arrived + row * kFinishStride;
        const uint32_t before = __hip_atomic_fetch_add(at, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool last = (before & 0xFFFFu) == (uint32_t)(A.n_chunks - 1);
        if (last && !F.mergers) __hip_atomic_store(at, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
        fs.shares = !last ? 0u : F.mergers ? before >> 16 : (1u << F.shares) - 1u;
        if (last && F.word) {
            // every key of the row is stored: the scores are complete when all rows are
            uint32_t* all = F.arrived + F.rows * kFinishStride;
            if (__hip_atomic_fetch_add(all, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(F.rows - 1)) {
                __hip_atomic_store(all, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(F.word, F.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(fs.shares);
}
// A workgroup that only merges: its share, once all of the row's chunks have arrived.  It does not wait for them for ever (they may not
// even have been dispatched): after F.polls looks it leaves its share to the last workgroup that arrives.  Either the mark is there
// when that one counts itself, or the count was complete when the mark was set.
__device__ __forceinline__ uint32_t row_complete(const AttendArgs& A, int row, int share, FinishShared& fs) {
    const Finish& F = A.fin;
    if (threadIdx.x == 0) {
        uint32_t* at = F.arrived + row * kFinishStride;
        const uint32_t n = (uint32_t)A.n_chunks;
        bool complete = false;
#pragma unroll 1
        for (int i = 0; i < F.polls && !complete; ++i) {
            const uint32_t missing = n - (__hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xFFFFu);
            complete = missing == 0;
            // Looks and additions to the one line wait for each other, so many mergers of many chunks look seldom until the end is near
            // (always after 0.2 us: 16 query rows over 8 x 32768 27.7 us, so 26.0; always after 1.3 us: 16 x 8192 16.7 -> 17.3)
            if (!complete && missing * F.shares > 128u) __builtin_amdgcn_s_sleep(48);
            else if (!complete) __builtin_amdgcn_s_sleep(8);
        }
        if (!complete)
            complete = (__hip_atomic_fetch_or(at, 0x10000u << share, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xFFFFu) == n;
        fs.shares = complete ? 1u << share : 0u;
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(fs.shares);
}

template <int LOADS>
__device__ __forceinline__ void merge_shares(const AttendArgs& A, int row, int nq, uint32_t shares, float* lds) {
    const Finish& F = A.fin;
    const int log_nr = __builtin_ctz(nq / F.shares);
#pragma unroll 1
    for (; shares; shares &= shares - 1) {
        merge_rows<LOADS>(A, row, nq, __builtin_ctz(shares), log_nr, lds);
        __syncthreads();
        // the last share leaves the counters as the next launch wants them
        uint32_t* at = F.arrived + row * kFinishStride;
        if (threadIdx.x == 0 && F.mergers && __hip_atomic_fetch_add(at + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(F.shares - 1)) {
            __hip_atomic_store(at, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(at + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace
}  // namespace specache
