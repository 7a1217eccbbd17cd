// Merge of a row's chunk partials inside the launch that makes them: the workgroup that completes a (batch, KV head) row
// combines its (max, sum, sum p V) with the usual log-sum-exp rescaling, and the one that completes the last row announces
// the scores (Announce).  A kernel boundary costs the stream 2 to 5 us beside a prefetch (the command processor reads packets and
// arguments over the link that the prefetch keeps busy), the merge kernel 2 to 6 us, and its launch 3 us of the
// issuing thread.  Measured at merges_in_launch (kernels.h), the rule for it.
//
// What the other workgroups wrote has to be visible across the XCDs' L2 caches without a fence: a device-scope release writes the
// XCD's whole L2 back, and in every workgroup it made the kernel eight times slower.  So the partials (and the selection keys, where
// the word announces them) are stored past the L2 (kAgentScope), each thread waits until its stores have arrived, the workgroup
// counts itself at device scope, and the one that finds it is the last loads the partials past its L2 as well.
#pragma once
#include "attend_common.h"

namespace specache {
namespace {

// LDS of finish_row besides the region: who is last, and the rows' sums
struct FinishShared {
    float den[16];
    int last;
};
constexpr int kFinishLdsBytes = kThreads * 16 + kFinishMost * 4;   // (max, sum) pairs, then the slices' sums; weights
static_assert(kFinishMost <= 64, "one wave reads the pairs, and a thread's share of the chunks is at most kFinishLoads");
constexpr int kFinishLoads = 8;                                     // chunks x rows / (threads / (32 quads of outputs)) at most

// Called by all of a workgroup's kThreads threads when they have stored the chunk's partials.  lds: kFinishLdsBytes, 16-byte
// aligned, free once every thread has arrived here.
__device__ __forceinline__ void finish_row(const AttendArgs& A, int row, int nq, float* lds, FinishShared& fs) {
    const Finish& F = A.fin;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = A.n_chunks;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have arrived
    __syncthreads();
    if (tid == 0) {
        const bool last = __hip_atomic_fetch_add(F.arrived + row * kFinishStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(n - 1);
        if (last) __hip_atomic_store(F.arrived + row * kFinishStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
        fs.last = last;
    }
    __syncthreads();
    if (!fs.last) return;
    float2* ml = reinterpret_cast<float2*>(lds);
    float* wgt = lds + kThreads * 4;
    // everything this thread reads, requested together.  Beyond the row's chunks a load returns 0.
    const auto po = buffer_of(A.part_o + (size_t)row * A.max_chunks * nq * kD, (uint32_t)(n * nq * kD * 4));
    const auto pml = buffer_of(A.part_ml + (size_t)row * A.max_chunks * nq * 2, (uint32_t)(n * nq * 8));
    typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
    uint2v pair = {0u, 0u};
    if (wave == 0) pair = __builtin_amdgcn_raw_buffer_load_b64(pml, lane * 8, 0, kAgentScope);
    const int quads = nq * (kD / 4);                               // a power of two: four outputs each
    const int slices = quads < kThreads ? kThreads / quads : 1;     // of the chunks, where there are threads to spare
    const int q0 = tid & (quads < kThreads ? quads - 1 : kThreads - 1), slice = quads < kThreads ? tid / quads : 0;
    float4v v[kFinishLoads];
    auto load = [&](int q) {
#pragma unroll
        for (int u = 0; u < kFinishLoads; ++u)
            v[u] = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(po, (slice * quads + q) * 16, u * slices * quads * 16, kAgentScope));
    };
    load(q0);
    if (tid == 0 && F.word) {
        // every key of the row is stored: the scores are complete when all rows are
        if (__hip_atomic_fetch_add(F.arrived + F.rows * kFinishStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(F.rows - 1)) {
            __hip_atomic_store(F.arrived + F.rows * kFinishStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(F.word, F.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    if (tid < n * nq) ml[tid] = make_float2(__uint_as_float(pair.x), __uint_as_float(pair.y));
    __syncthreads();
#pragma unroll 1
    for (int r = wave; r < nq; r += kWaves) {
        const float2 p = lane < n ? ml[lane * nq + r] : make_float2(-INFINITY, 0.0f);
        const float m = wave_max(p.x), w = p.x == -INFINITY ? 0.0f : __expf(p.x - m);
        if (lane < n) wgt[lane * nq + r] = w;
        const float den = wave_sum(p.y * w);
        if (lane == 0) fs.den[r] = den;
    }
    __syncthreads();
#pragma unroll 1
    for (int q = q0; q < quads; q += kThreads) {
        const int r = q / (kD / 4);
        if (q != q0) load(q);
        float4v o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < kFinishLoads; ++u) {
            const int ch = u * slices + slice;
            const float w = ch < n ? wgt[ch * nq + r] : 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = w != 0.0f ? __builtin_fmaf(v[u][e], w, o[e]) : o[e];   // a chunk without candidates may hold anything
        }
        if (slices > 1) {            // then every thread has one quad
            float4v* part = reinterpret_cast<float4v*>(lds);
            part[tid] = o;
            __syncthreads();
            if (slice != 0) return;
#pragma unroll 1
            for (int s = 1; s < slices; ++s) o += part[s * quads + q];
        }
        const float den = fs.den[r];
        *reinterpret_cast<float4*>(F.out + ((size_t)row * nq + r) * kD + 4 * (q % (kD / 4))) = make_float4(o[0] / den, o[1] / den, o[2] / den, o[3] / den);
    }
}

}  // namespace
}  // namespace specache
