// ArgTopK of the speculative row (Appendix A "Decoding": K_{t+1} = ArgTopK(A_{1,:});
// "Pre-decoding" for the single-row case), alone or with Pre-fetch(C_K) of the selected pairs
// behind it in the same launch.  Softmax is monotone, so the selection runs on the logits'
// order-preserving integer keys.
//
// One workgroup per (batch, KV head), its keys in registers (longer rows in two launches, see
// topk_parts).  What bounds the kernel is neither arithmetic nor the 4 bytes per key but the chain of
// barrier-separated phases and, in each of them, the instructions of a pass over the registers
// (unrolled, and fetched once per compute unit).  So two passes see all the keys and the rest works on a few hundred:
//   1. floor: every thread's largest key is a distinct element of the row (every four registers', where k is not
//      small beside the number of threads), so tau, the k-th largest key, is at least the k-th largest of those maxima.  A
//      512-bin histogram of the maxima over the four binades below the row's largest gives a floor F <= tau; every wave reads
//      it for itself, which saves a barrier;
//   2. the keys >= F (1.2 to 1.5 k of them where k is a quarter to a half of the maxima) are collected in LDS, and a second
//      histogram, of those, finds the bin that holds tau and tau's rank inside it;
//   3. the handful of keys in that bin are ranked by one wave (larger key first, then lower position), which decides for
//      each of them at once, ties included; the selected positions are bits of a bitmap, whose order is the output's.
// Larger k has room for more candidates and takes maxima of two (many_candidates); where k is a quarter of the row or more a
// floor would leave too few keys out, and the histograms are of all keys; so they are of short rows where k asks for most of the
// maxima (no_floor).
// Where the boundary bin is crowded (many equal or almost equal scores) the candidates go on by themselves, with histograms
// inside the range left; a row with more candidates than there is room for does so with all its keys.  Both leave two
// bitmaps, the keys above tau and those equal to it, which one ordered pass writes out.
//
// Measured on MI355X, us, one launch alone (first: a histogram of the maxima's leading bits, one of the keys, 64
// readlanes to rank, a counting and an emitting pass over all registers): rows x keys, k = 64 unless stated: 1 x 4096 10.6 -> 5.2,
// 32 x 8192 13.8 -> 6.2, 32 x 16384 12.0 -> 5.3, 32 x 32768 15.2 -> 6.7 (k = 256: 16.7 -> 8.4), 32 x 16384 with k = 1024 14.0 ->
// 8.3, with k = 3000 16.5 -> 11.3; in two launches 8 x 131072 with k = 256 27.2 -> 15.3, with k = 1024 32.3 -> 20.3, with k = 4096
// 54.4 -> 41.  Large k with room for 2048 candidates only, its keys read from memory again in every pass: 32 x 16384, k = 3000 19.0; 32 x
// 8192, k = 4096 16.0, now 9.9 (first 12.1); 32 x 32768, k = 4096 30.2, now 14.7 (23.8).  64 values in a row, each many times over: 32 x
// 32768 40.3, now 12.0 to 15.6 (19.3), k = 4096 42.7, now 17.1 (23.0); a single value 80.6, now 47 (68).
#include <cmath>

#include "kernels.h"
#include "layout.h"

namespace specache {
namespace {

constexpr int kCandidates = 2048;      // keys the short way has room for,
constexpr int kCandidatesMost = 8192;  // and where k asks for more of them (many_candidates)
constexpr int kSmall = 64;             // keys one wave ranks directly
constexpr int kMaxTopk = 4096;
constexpr int kMapWords = 65536 / 32;

template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}
// sum over this lane and the lanes below it
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) {
    v += dpp_or_zero<0x111>(v);          // row_shr 1, 2, 4, 8: inside rows of 16 lanes
    v += dpp_or_zero<0x112>(v);
    v += dpp_or_zero<0x114>(v);
    v += dpp_or_zero<0x118>(v);
    v += dpp_or_zero<0x142, 0xa>(v);     // row_bcast 15: a row's sum to the odd row behind it
    v += dpp_or_zero<0x143, 0xc>(v);     // row_bcast 31: the first two rows' sum to the last two
    return v;
}
__device__ __forceinline__ uint32_t wave_largest(uint32_t v) {
    auto step = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    v = step(v, dpp_or_zero<0xB1>(v));   // lanes 1 and 2 apart, the other half and the mirror of the row of 16
    v = step(v, dpp_or_zero<0x4E>(v));
    v = step(v, dpp_or_zero<0x141>(v));
    v = step(v, dpp_or_zero<0x140>(v));
    const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return step(step(a, b), step(c, d));
}
// The bin that holds the need-th largest counted key (larger bin = larger keys) and that key's rank in the bin (from
// 1, largest first), worked out by every wave for itself; bin = BINS if fewer than `need` keys were counted.
struct BinRank { uint32_t bin, rank; };
template <int BINS>
__device__ __forceinline__ BinRank find_bin(const uint32_t* hist, uint32_t need) {
    constexpr int kChunk = BINS < 512 ? BINS : 512, kChunks = BINS / kChunk;   // bins read at a time, from the top; a lane's 8 side by side
    const int lane = threadIdx.x & 63;
    uint32_t passed = 0;
#pragma unroll 1
    for (int ch = kChunks - 1; ch >= 0; --ch) {
        const uint4* at = reinterpret_cast<const uint4*>(hist + kChunk * ch) + 2 * (63 - lane);
        const uint4 lo = at[0], hi = at[1];
        const uint32_t h[8] = {hi.w, hi.z, hi.y, hi.x, lo.w, lo.z, lo.y, lo.x};   // bins 8 (63 - lane) + 7 downwards
        uint32_t mine = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) mine += h[j];
        const uint32_t upto = passed + wave_prefix(mine);
        const unsigned long long reached = __ballot(upto >= need);
        if (reached == 0) {
            passed = __builtin_amdgcn_readlane(upto, 63);
            continue;
        }
        uint32_t above = upto - mine, bin = 0, rank = 0;
        bool found = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool here = !found && above + h[j] >= need;
            bin = here ? 8 * (63 - lane) + 7 - j : bin;
            rank = here ? need - above : rank;
            found = found || here;
            above += h[j];
        }
        const int first = __builtin_ctzll(reached);
        return {(uint32_t)(kChunk * ch) + __builtin_amdgcn_readlane(bin, first), (uint32_t)__builtin_amdgcn_readlane(rank, first)};
    }
    return {(uint32_t)BINS, 0};
}

// A row may be split into `parts` ranges of part_len keys, one workgroup each, that write
// their selections (position in the row, and the key if key_out is set) side by side; a
// second launch then selects among those candidates and translates its positions through
// `map`.  parts == 1, map == key_out == null is the plain single-launch selection.
struct TopkIo {
    int nq_total, parts, part_len;
    const int32_t* map;      // [rows][map_stride] or null
    size_t map_stride;
    uint32_t* key_out;       // [rows * parts][k] or null
    bool all_keys = false;   // no_floor; for the launch to set
};

// Pre-fetch(C_K) behind the selection (GATHER): the row's pairs from the pinned host store into the staging slot.
struct GatherIo {
    const uint4* host;       // [rows][max_seq][32]
    uint4* slot;             // [rows][k][32]
    int32_t* slot_idx;       // [rows][k]
    int max_seq, waves, reads;   // waves of a workgroup that fetch, host reads of a lane in flight
};

template <int READS>
__device__ __forceinline__ void fetch_pairs(const GatherIo& g, int row, int k, const int32_t* list) {
    const int part = threadIdx.x & 31, group = threadIdx.x >> 5, groups = 2 * g.waves;
    const uint4* host = g.host + (size_t)row * g.max_seq * 32 + part;
    uint4* slot = g.slot + (size_t)row * k * 32 + part;
    for (int j0 = group; j0 < k; j0 += groups * READS) {
        int src[READS];
        uint4 v[READS];
#pragma unroll
        for (int u = 0; u < READS; ++u) {
            const int j = j0 + u * groups;
            src[u] = j < k ? list[j] : -1;
        }
#pragma unroll
        for (int u = 0; u < READS; ++u) v[u] = src[u] >= 0 ? host[(size_t)src[u] * 32] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < READS; ++u)
            if (src[u] >= 0) slot[(size_t)(j0 + u * groups) * 32] = v[u];
    }
}

// THREADS: 1024 for long rows; 256 for rows of up to 8192 keys, so that several rows share a
// compute unit and hide each other's barrier latency.  CAND: candidates the short way has room for.
template <int THREADS, int KPT, bool GATHER, int CAND>
__global__ __launch_bounds__(THREADS) void topk_kernel(TopkIo io, int k, const uint32_t* __restrict__ keys,
                                                       size_t key_stride, int32_t* __restrict__ idx_out, GatherIo g) {
    constexpr int kWavesHere = THREADS / 64;
    constexpr int kMapHere = THREADS * KPT / 32;      // words of the bitmap
    constexpr int kSub = CAND > kCandidates ? 2 : 4;  // registers of a finer maximum
    static_assert(kMapHere <= kMapWords, "a row's positions");
    // Where k is a large part of the row, tau lies among small scores of either sign, and keys there are binades apart: few bins then
    // hold all keys, whose atomics wait for each other
    constexpr int kBins = CAND > kCandidates ? 2048 : 512, kBinBits = CAND > kCandidates ? 11 : 9;
    __shared__ __attribute__((aligned(16))) uint32_t bins[2][kBins];
    __shared__ __attribute__((aligned(16))) uint2 cand[CAND];   // key, position
    __shared__ __attribute__((aligned(8))) uint32_t bitmap[kMapHere];
    __shared__ uint32_t wave_red[kWavesHere], result[2];
    __shared__ uint2 small_keys[kSmall];
    __shared__ uint32_t n_cand, n_small;

    static_assert(sizeof(cand) >= kMapHere * 4, "a crowded row's second bitmap takes the candidates' place");
    uint32_t* eq_map = reinterpret_cast<uint32_t*>(cand);
    static_assert(sizeof(cand) >= kMaxTopk * 4, "and so does the list of the selected positions, when both are done with");
    int32_t* list = reinterpret_cast<int32_t*>(cand);

    const int row = blockIdx.x / io.parts, part = blockIdx.x % io.parts;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;   // (scalar: the loads' descriptor is)
    const int base = part * io.part_len;
    const int left = io.nq_total - base;
    const int Nq = left < 0 ? 0 : (left < io.part_len ? left : io.part_len);   // keys of this range
    const uint32_t* kr = keys + (size_t)row * key_stride + base;
    int32_t* out = idx_out + (size_t)blockIdx.x * k;
    uint32_t* kout = io.key_out ? io.key_out + (size_t)blockIdx.x * k : nullptr;
    const int32_t* map = io.map ? io.map + (size_t)row * io.map_stride : nullptr;
    const int keff = k < Nq ? k : Nq;
    // output slot `pos` receives local position i, whose key is kv
    auto emit = [&](uint32_t pos, int i, uint32_t kv) {
        const int at = map ? map[i] : base + i;
        if constexpr (GATHER) list[pos] = at;
        else out[pos] = at;
        if (kout) kout[pos] = kv;
    };
    auto none = [&](int j) {
        if constexpr (GATHER) list[j] = -1;
        else out[j] = -1;
        if (kout) kout[j] = 0u;     // below every key: never selected by the second launch
    };

    // wave w owns the contiguous index range [w*seg, (w+1)*seg), seg a multiple of 64
    const int seg = ((Nq + kWavesHere * 64 - 1) / (kWavesHere * 64)) * 64;
    const int lo = wave * seg, hi = (lo + seg < Nq) ? lo + seg : Nq;

    auto select = [&]() {
        // Key slots with index >= hi are padding and hold key 0 (what a load beyond the descriptor's range returns); every
        // range tested below starts at 1 or above, so padding never matches and no pass needs an index test.  (Key 0
        // itself is the one NaN pattern 0xFFFFFFFF; it is treated as below every other score.)
        uint32_t key[KPT];
        auto load_keys = [&]() {
            int at = (lo + lane) * 4;
            asm volatile("" : "+v"(at));           // (each call's addresses are its own: kept from one to the next they would be spilled)
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(kr), 0, hi > lo ? hi * 4 : 0, 0x00027000);
#pragma unroll
            for (int it = 0; it < KPT; ++it) key[it] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, at + it * 256, 0, 0);
        };
        load_keys();
        // while they travel
        for (int b = tid; b < 2 * kBins; b += THREADS) bins[0][b] = 0;
        for (int b = tid; b < kMapHere; b += THREADS) bitmap[b] = 0;
        if (tid == 0) n_cand = n_small = 0;
        // ---- the maxima, of the thread or of every kSub registers
        const bool fine = 2 * keff > THREADS;     // uniform
        uint32_t sub[KPT / kSub], tmax = 0;
#pragma unroll
        for (int s = 0; s < KPT / kSub; ++s) {
            sub[s] = 0;
#pragma unroll
            for (int it = s * kSub; it < (s + 1) * kSub; ++it) sub[s] = key[it] > sub[s] ? key[it] : sub[s];
            tmax = sub[s] > tmax ? sub[s] : tmax;
        }
        {
            const uint32_t wm = wave_largest(tmax);
            if (lane == 0) wave_red[wave] = wm;
        }
        __syncthreads();
        uint32_t row_max = wave_red[0];
#pragma unroll
        for (int w = 1; w < kWavesHere; ++w) row_max = wave_red[w] > row_max ? wave_red[w] : row_max;
        // ---- floor: the maxima among the top four binades, else all of them by binade
        constexpr uint32_t kTopSpan = 1u << 25;
        constexpr int kTopShift = 25 - kBinBits, kAllShift = 32 - kBinBits;
        const uint32_t top_lo = row_max >= kTopSpan ? row_max - (kTopSpan - 1) : 0u;
        auto count_maxima = [&](uint32_t* hist, uint32_t from, int shift) {
            if (fine) {
#pragma unroll
                for (int s = 0; s < KPT / kSub; ++s)
                    if (sub[s] >= from && sub[s] != 0) atomicAdd(&hist[(sub[s] - from) >> shift], 1u);
            } else if (tmax >= from && tmax != 0) {
                atomicAdd(&hist[(tmax - from) >> shift], 1u);
            }
        };
        uint32_t floor_key = 1u;                   // fewer maxima than keff: no floor
        uint32_t n = 0xFFFFFFFFu;                  // candidates; uniform, as everything that decides on the way is
        // (us with a floor against all keys: 32 x 4096, k = 2048 16.9 / 8.6; 32 x 8192, k = 2048 9.9 / 11.8, k = 3000 13.2 / 12.0, k = 4096
        // 20 / 9.9; 32 x 16384, k = 4096 12.4 / 13.4, but with 64 values in the row 17.5 / 14.)
        // (fewer candidates: no_floor)
        const bool all_keys = CAND > kCandidates ? 4 * keff >= Nq : KPT <= 16 && io.all_keys;
        if (!all_keys) {
            count_maxima(bins[0], top_lo, kTopShift);
            __syncthreads();
            const BinRank br = find_bin<kBins>(bins[0], (uint32_t)keff);
            if (br.bin < kBins) {
                floor_key = top_lo + (br.bin << kTopShift);
            } else {                               // uniform over the workgroup
                __syncthreads();
                for (int b = tid; b < kBins; b += THREADS) bins[0][b] = 0;
                __syncthreads();
                count_maxima(bins[0], 0u, kAllShift);
                __syncthreads();
                const BinRank all = find_bin<kBins>(bins[0], (uint32_t)keff);
                if (all.bin < kBins) floor_key = all.bin << kAllShift;
            }
            floor_key = floor_key < 1u ? 1u : floor_key;
            // ---- the keys from the floor on
#pragma unroll
            for (int it = 0; it < KPT; ++it)
                if (key[it] >= floor_key) {
                    const uint32_t at = atomicAdd(&n_cand, 1u);
                    if (at < CAND) cand[at] = make_uint2(key[it], (uint32_t)(lo + it * 64 + lane));
                }
            __syncthreads();
            n = n_cand;
        }
        constexpr int kWords = (kMapHere + THREADS - 1) / THREADS;   // of the bitmap, of a thread
        uint32_t need = (uint32_t)keff;
        if (n < need && n <= CAND) need = n;       // keys that are NaN are below everything and stay unselected
        // a wave finds the rank-th largest of up to kSmall keys and how many keys equal to it are wanted
        auto rank_small = [&](uint32_t rank) {
            const uint32_t m = n_small;
            const uint32_t mine = lane < (int)m ? small_keys[lane].x : 0u;
            uint32_t greater = 0, equal = 0;
#pragma unroll 2
            for (uint32_t j = 0; j < m; ++j) {
                const uint32_t kj = small_keys[j].x;
                greater += kj > mine;
                equal += kj == mine;
            }
            if (lane < (int)m && greater < rank && rank <= greater + equal) {
                result[0] = mine;
                result[1] = rank - greater;
            }
        };
        // Crowded: tau, the need-th largest of the keys in [range_lo, range_hi], by histograms inside a range that becomes kBins times
        // narrower each time, and narrower still by the least and the largest key found in it: equal scores end it there.
        // need becomes the number of keys equal to tau that are wanted.  for_each(f): f(key) for this thread's keys.
        auto narrow = [&](auto&& for_each, uint32_t range_lo, uint32_t range_hi) {
            for (int round = 0; round < 4 && range_lo != range_hi; ++round) {
                const uint32_t span = range_hi - range_lo;
                const int shift = span < (uint32_t)kBins ? 0 : 32 - __builtin_clz(span) - kBinBits;
                __syncthreads();
                for (int b = tid; b < kBins; b += THREADS) bins[0][b] = 0;
                if (tid == 0) {
                    n_small = 0;
                    result[0] = 0xFFFFFFFFu;
                    result[1] = 0u;
                }
                __syncthreads();
                for_each([&](uint32_t kv) {
                    const uint32_t off = kv - range_lo;
                    if (off <= span) atomicAdd(&bins[0][off >> shift], 1u);   // one unsigned test for range_lo <= kv <= range_hi
                });
                __syncthreads();
                const BinRank br = find_bin<kBins>(bins[0], need);
                if (br.bin >= kBins) {             // fewer keys than wanted (the others are NaN): all of them
                    need = 0xFFFFFFFFu;
                    break;
                }
                const uint32_t in_bin = bins[0][br.bin];
                range_lo += br.bin << shift;
                range_hi = range_lo + ((1u << shift) - 1u);
                need = br.rank;
                if (shift == 0) break;             // the bin is a single key value
                if (in_bin <= (uint32_t)kSmall) {
                    for_each([&](uint32_t kv) {
                        if (kv - range_lo <= range_hi - range_lo) small_keys[atomicAdd(&n_small, 1u)].x = kv;
                    });
                    __syncthreads();
                    if (wave == 0) rank_small(br.rank);
                    __syncthreads();
                    range_lo = result[0];
                    need = result[1];
                    break;
                }
                uint32_t least = 0xFFFFFFFFu, largest = 0u;
                for_each([&](uint32_t kv) {
                    if (kv - range_lo <= range_hi - range_lo) {
                        least = kv < least ? kv : least;
                        largest = kv > largest ? kv : largest;
                    }
                });
                least = ~wave_largest(~least);
                largest = wave_largest(largest);
                if (lane == 0) {
                    atomicMin(&result[0], least);
                    atomicMax(&result[1], largest);
                }
                __syncthreads();
                range_lo = result[0];
                range_hi = result[1];
            }
            return range_lo;                       // tau
        };
        bool crowded = n > CAND;
        if (!crowded) {
            // ---- the bin of tau
            const uint32_t span = row_max - floor_key;
            const int shift = span < (uint32_t)kBins ? 0 : 32 - __builtin_clz(span) - kBinBits;
            for (uint32_t c = tid; c < n; c += THREADS) atomicAdd(&bins[1][(cand[c].x - floor_key) >> shift], 1u);
            __syncthreads();
            const BinRank br = find_bin<kBins>(bins[1], need);
            crowded = bins[1][br.bin < kBins ? br.bin : 0] > kSmall;
            if (!crowded) {
                for (uint32_t c = tid; c < n; c += THREADS) {
                    const uint2 kv = cand[c];
                    const uint32_t b = (kv.x - floor_key) >> shift;
                    if (b > br.bin) atomicOr(&bitmap[kv.y >> 5], 1u << (kv.y & 31));
                    if (b == br.bin) small_keys[atomicAdd(&n_small, 1u)] = kv;
                }
                __syncthreads();
                // ---- the boundary bin's keys: larger first, then lower position
                if (wave == 0) {
                    const uint32_t m = n_small;
                    const uint2 mine = lane < (int)m ? small_keys[lane] : make_uint2(0u, 0u);
                    uint32_t before = 0;
#pragma unroll 2
                    for (uint32_t j = 0; j < m; ++j) {
                        const uint2 o = small_keys[j];
                        before += o.x > mine.x || (o.x == mine.x && o.y < mine.y);
                    }
                    if (lane < (int)m && before < br.rank) atomicOr(&bitmap[mine.y >> 5], 1u << (mine.y & 31));
                }
                __syncthreads();
                // ---- the bits in order: this thread's words, behind those of the threads and waves before it
                uint32_t w[kWords], mine = 0;
#pragma unroll
                for (int u = 0; u < kWords; ++u) {
                    w[u] = tid * kWords + u < kMapHere ? bitmap[tid * kWords + u] : 0u;
                    mine += __popc(w[u]);
                }
                const uint32_t upto = wave_prefix(mine);
                if (lane == 63) wave_red[wave] = upto;
                __syncthreads();
                uint32_t pos = upto - mine;
#pragma unroll 1
                for (int v = 0; v < wave; ++v) pos += wave_red[v];
#pragma unroll
                for (int u = 0; u < kWords; ++u)
                    while (w[u]) {
                        const int i = 32 * (tid * kWords + u) + __builtin_ctz(w[u]);
                        w[u] &= w[u] - 1;
                        emit(pos++, i, kout ? kr[i] : 0u);
                    }
                for (int j = (int)need + tid; j < k; j += THREADS) none(j);
                return;
            }
            // ---- crowded boundary: the candidates narrow it down among themselves, out of registers, and their place takes
            // the bitmap of the keys equal to tau
            constexpr int kMine = CAND / THREADS;
            uint2 c[kMine];
#pragma unroll
            for (int u = 0; u < kMine; ++u) c[u] = tid + u * THREADS < (int)n ? cand[tid + u * THREADS] : make_uint2(0u, 0u);
            const uint32_t bin_lo = floor_key + (br.bin << shift);
            need = br.rank;
            const uint32_t tau = narrow([&](auto&& f) {
#pragma unroll
                for (int u = 0; u < kMine; ++u) f(c[u].x);
            }, bin_lo, shift == 0 ? bin_lo : bin_lo + ((1u << shift) - 1u));
            __syncthreads();
            for (int b = tid; b < kMapHere; b += THREADS) eq_map[b] = 0;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kMine; ++u) {
                if (c[u].x > tau) atomicOr(&bitmap[c[u].y >> 5], 1u << (c[u].y & 31));
                else if (c[u].x == tau) atomicOr(&eq_map[c[u].y >> 5], 1u << (c[u].y & 31));
            }
        } else {
            // ---- more candidates than there is room for: all keys, loaded once more (registers that held them since the floor
            // would be spilled).  A lane's keys are 64 apart, so a ballot is two words of a bitmap.
            if (!all_keys) load_keys();
            const uint32_t tau = narrow([&](auto&& f) {
#pragma unroll
                for (int it = 0; it < KPT; ++it) f(key[it]);
            }, floor_key, row_max);
            __syncthreads();
            for (int b = tid; b < kMapHere; b += THREADS) eq_map[b] = 0;
            __syncthreads();
#pragma unroll
            for (int it = 0; it < KPT; ++it) {
                const unsigned long long gt = __ballot(key[it] > tau), eq = __ballot(key[it] == tau);
                if (it * 64 < seg && lane < 2)
                    reinterpret_cast<unsigned long long*>(lane ? eq_map : bitmap)[(lo >> 6) + it] = lane ? eq : gt;
            }
        }
        __syncthreads();
        // ---- both bitmaps in order, a thread as many bits as it has keys (where k is most of the row it has as many to write).  Fewer
        // than k keys are above tau, so both counts fit one word.
        static_assert(kMaxTopk < 1 << 13 && THREADS * KPT <= 1 << 18, "the counts of a row");
        const int n_bits = seg >> 6, first = tid * n_bits;
        auto bits_of = [&](const uint32_t* map_words) {
            const int at = first >> 5, by = first & 31;
            auto word = [&](int i) { return i < kMapHere ? (uint64_t)map_words[i] : 0ull; };
            uint64_t v = (word(at) | word(at + 1) << 32) >> by;
            if (by > 0) v |= word(at + 2) << (64 - by);
            return n_bits < 64 ? v & ((1ull << n_bits) - 1) : v;
        };
        const uint64_t gt = bits_of(bitmap), eq = bits_of(eq_map);
        const uint32_t mine = __popcll(gt) + (__popcll(eq) << 13);
        const uint32_t upto = wave_prefix(mine);
        if (lane == 63) wave_red[wave] = upto;
        __syncthreads();
        uint32_t before = upto - mine, total = 0;
#pragma unroll 1
        for (int v = 0; v < kWavesHere; ++v) {
            before += v < wave ? wave_red[v] : 0u;
            total += wave_red[v];
        }
        uint32_t gt_before = before & 0x1FFFu, eq_before = before >> 13;
        for (uint64_t either = gt | eq; either; either &= either - 1) {
            const int bit = __builtin_ctzll(either);
            const uint32_t pos = gt_before + (eq_before < need ? eq_before : need);
            if (gt >> bit & 1) ++gt_before;
            else if (eq_before++ >= need) continue;
            emit(pos, first + bit, kout ? kr[first + bit] : 0u);
        }
        const uint32_t eq_all = total >> 13;
        for (int j = (int)((total & 0x1FFFu) + (eq_all < need ? eq_all : need)) + tid; j < k; j += THREADS) none(j);
    };

    if (keff == Nq) {   // everything is selected
        for (int j = tid; j < k; j += THREADS) {
            if (j < Nq) emit(j, j, kr[j]);
            else none(j);
        }
    } else {
        select();
    }

    if constexpr (GATHER) {
        __syncthreads();
        for (int j = tid; j < k; j += THREADS) {
            const int i = list[j];
            out[j] = i;
            g.slot_idx[(size_t)row * k + j] = i < g.max_seq ? i : -1;
        }
        if (wave >= g.waves) return;
        __builtin_amdgcn_s_setprio(3);   // a wave's issue priority inside its SIMD, not a stream priority
        switch (g.reads) {
            case 1: fetch_pairs<1>(g, row, k, list); break;
            case 2: fetch_pairs<2>(g, row, k, list); break;
            case 4: fetch_pairs<4>(g, row, k, list); break;
            default: fetch_pairs<8>(g, row, k, list); break;
        }
    }
}

// Whether the short way of ArgTopK should have room for kCandidatesMost candidates.  It collects the keys above the k-th largest of
// the maxima of four: of n keys in no particular order the share x with 1 - (1 - x)^4 = 4 k / n (to which the floor's bins add up
// to a tenth).  Room for more costs a workgroup 60 KB of LDS and twice as many maxima; too little room a pass over the keys for
// nothing and the way of the crowded rows (32 x 32768, k = 2000: 30.0 us, now 12.7).
bool many_candidates(int n, int k) {
    if (k <= kCandidates / 4) return false;
    const double p = 4.0 * k / n;
    return n * (p < 1.0 ? 1.0 - std::sqrt(std::sqrt(1.0 - p)) : 1.0) > 0.85 * kCandidates;
}

// Where the short way of few candidates is no use.  A floor needs more than k maxima above zero, and one of `per` scores of either sign is with a
// chance of 1 - 2^-per; short of that it lies among small scores, binades wide, and its pass over the keys is for nothing.  us with a floor /
// with all keys: 32 x 256, k = 104 5.6 / 4.8, k = 156 9.6 / 4.8, k = 234 11.6 / 5.3; 32 x 640, k = 171 5.6 / 6.3, k = 198 10.8 / 6.3; 32 x 960, k = 220 6.0 / 5.8,
// k = 249 11.3 / 5.8, k = 384 7.5 / 9.2, k = 576 13.2 / 9.2; 32 x 1440, k = 438 7.0 / 9.4, k = 584 13.6 / 9.4.
bool no_floor(int n, int k, int threads) {
    const int of_a_thread = (n + threads - 1) / threads, most = 2 * k > threads ? 4 : 31;
    const int per = of_a_thread < most ? of_a_thread : most;
    return 16.0 * per * k > 15.0 * (n - (n >> per));
}

// one launch over `rows * io.parts` ranges of at most n keys each; gather: and the fetch behind it (gather_kb: KB of a row's pairs
// under way at a time)
hipError_t launch_ranges(int rows, int n, TopkIo io, int k, const uint32_t* keys, size_t key_stride,
                         int32_t* idx_out, hipStream_t stream, const GatherIo* gather = nullptr, int gather_kb = 0) {
    const int per_lane_256 = (n + 255) / 256, per_lane = (n + 1023) / 1024;   // keys per lane held in registers
    GatherIo g = gather ? *gather : GatherIo{};
    // the floor needs more maxima than k to bite: small workgroups only for small k; nor can one with few waves keep the reads of a
    // launch over few rows under way (2 rows, k = 200: 188 us a pass with 256 threads, 182 with 1024; the others level)
    const bool small_wg = k <= 256 && per_lane_256 <= 32 && (!gather || gather_kb <= 4);
    if (gather) {
        const int most = (small_wg ? 256 : 1024) / 64;
        g.waves = gather_kb < most ? gather_kb : most;   // a wave's read is 1 KB
        const int reads = gather_kb / g.waves;
        g.reads = reads >= 8 ? 8 : reads >= 4 ? 4 : reads >= 2 ? 2 : 1;
    }
    const bool many = many_candidates(n, k);
    io.all_keys = no_floor(n, k, small_wg ? 256 : 1024);
#define SPC_TOPK_AT(T, K, C) SPC_LAUNCH((topk_kernel<T, K, false, C>), dim3(rows * io.parts), dim3(T), stream, io, k, keys, key_stride, idx_out, g)
#define SPC_TOPK_LONG(K)                                    \
    do {                                                    \
        if (many) SPC_TOPK_AT(1024, K, kCandidatesMost);    \
        else SPC_TOPK_AT(1024, K, kCandidates);             \
    } while (0)
#define SPC_TOPK_GATHER(T, K, SELECT)                                                                                                    \
    do {                                                                                                                         \
        if (gather) SPC_LAUNCH((topk_kernel<T, K, true, kCandidates>), dim3(rows), dim3(T), stream, io, k, keys, key_stride, idx_out, g);     \
        else SELECT;                                                                                                             \
    } while (0)
    if (small_wg && per_lane_256 <= 8) SPC_TOPK_GATHER(256, 8, SPC_TOPK_AT(256, 8, kCandidates));
    else if (small_wg && per_lane_256 <= 16) SPC_TOPK_GATHER(256, 16, SPC_TOPK_AT(256, 16, kCandidates));
    else if (small_wg) SPC_TOPK_GATHER(256, 32, SPC_TOPK_AT(256, 32, kCandidates));
    else if (per_lane <= 16) SPC_TOPK_GATHER(1024, 16, SPC_TOPK_LONG(16));
    else if (per_lane <= 24) SPC_TOPK_GATHER(1024, 24, SPC_TOPK_LONG(24));
    else if (per_lane <= 32) SPC_TOPK_GATHER(1024, 32, SPC_TOPK_LONG(32));
    else if (per_lane <= 40) SPC_TOPK_GATHER(1024, 40, SPC_TOPK_LONG(40));
    else if (per_lane <= 48) SPC_TOPK_GATHER(1024, 48, SPC_TOPK_LONG(48));
    else if (gather) return hipErrorInvalidValue;     // selects_and_gathers: rows of one launch
    else if (per_lane <= 64) SPC_TOPK_LONG(64);
    else return hipErrorInvalidValue;                // launch_topk splits such a row
#undef SPC_TOPK_AT
#undef SPC_TOPK_LONG
#undef SPC_TOPK_GATHER
    return hipGetLastError();
}

}  // namespace

// One workgroup's registers hold 65536 keys, but with more than 48 a thread they are spilled, so rows beyond kTopkSingleLaunchKeys
// are split into ranges of about kTopkPartKeys keys, as many as keep the candidate list of the second launch within
// one workgroup's registers.  us, one launch / two: 32 x 45000, k = 64 7.6 / 13.7, 32 x 49152, k = 256 9.7 / 16.5, but 32 x 59008
// 16.8 / 13.5 and 18.3 / 16.0.
constexpr int kTopkRegisterKeys = 65536, kTopkPartKeys = 16384, kTopkSingleLaunchKeys = 49152;

int topk_parts(int Nq, int k) {
    if (Nq <= kTopkSingleLaunchKeys || k <= 0) return 1;
    int parts = (Nq + kTopkPartKeys - 1) / kTopkPartKeys;
    const int most = kTopkRegisterKeys / k;
    parts = parts < most ? parts : most;
    return parts < 2 ? 1 : parts;
}

hipError_t launch_topk(int rows, int Nq, int k, const uint32_t* keys, size_t key_stride, int32_t* idx_out,
                       const TopkScratch& scratch, hipStream_t stream) {
    const int parts = topk_parts(Nq, k);
    if (parts > 1 && parts <= scratch.max_parts && scratch.cand_keys && scratch.cand_idx) {
        if (pending_launch_events().stop) pending_launch_events().launches = 2;   // a timing pair spans both launches
        const int part_len = (((Nq + parts - 1) / parts) + 63) / 64 * 64;
        TopkIo first{Nq, parts, part_len, nullptr, 0, scratch.cand_keys};
        hipError_t e = launch_ranges(rows, part_len, first, k, keys, key_stride, scratch.cand_idx, stream);
        if (e != hipSuccess) return e;
        TopkIo second{parts * k, 1, parts * k, scratch.cand_idx, (size_t)parts * k, nullptr};
        return launch_ranges(rows, parts * k, second, k, scratch.cand_keys, (size_t)parts * k, idx_out, stream);
    }
    TopkIo io{Nq, 1, Nq, nullptr, 0, nullptr};
    return launch_ranges(rows, Nq, io, k, keys, key_stride, idx_out, stream);
}

// In one launch the selection's 4-byte list does not go through memory to a kernel of its own, which costs a boundary (2.4 us on a
// side stream), a launch of the issuing thread (3 us) and the list's latency.  us a pass, two launches against one: 1 x 4096, 16 layers 280 /
// 158 to 230 (bound by the issuing thread), 32 x 16k 337 / 308, 32 x 32k with k = 256 372 / 360, 1 bit 196 / 176, 24 x 5003 with 8 rows 255 / 246.
// Not where a row takes two launches to select (8 x 131072: 387 / 394) or the larger room for candidates, nor with many rows: a row's workgroup keeps its place on a
// compute unit for as long as it fetches, and more reads are under way than the link wants: 128 rows 207 / 182, 160 rows 215 / 206, 192 rows
// 296 / 290, but 256 rows 172 / 193 and 512 rows 176 / 223.  Nor many pairs of few rows: a compute unit by itself brings 13 GB/s of the
// link's 57.  A step of layers over 16384 positions, us a layer, two launches against one: 1 row, k = 192 18.1 / 14.7, k = 512 23.5 / 29.2, k = 1024 28.7 / 40.5; 2 rows,
// k = 256 22.4 / 24.4, k = 512 28.2 / 33.6; 3 rows, k = 256 24.7 / 26.3, k = 768 26.3 / 31.7; 4 rows, k = 384 21.0 / 22.3, k = 768 31.8 / 34.7; 6
// rows, k = 1024 66.0 / 64.9.  The fetch alone: 1 row, k = 128 14.0 / 12.3, k = 192 14.9 / 14.5, k = 256 15.6 / 16.9.
bool selects_and_gathers(int rows, int Nq, int k) {
    return rows <= 128 && (rows >= 6 || k <= 192 || k <= 64 * (rows + 1)) && topk_parts(Nq, k) == 1 && !many_candidates(Nq, k);
}

hipError_t launch_select_gather(const LayerView& L, int Nq, const uint32_t* keys, size_t key_stride, int32_t* idx_out,
                                uint16_t* slot, int32_t* slot_idx, bool link_shared, hipStream_t stream) {
    if (!selects_and_gathers(L.rows, Nq, L.topk)) return hipErrorInvalidValue;
    // How much of the host store is under way at a time: as much as the link needs, and no more, since every read in flight slows the
    // attention kernels beside the fetch.  Steps of several layers, us a pass with 32, 64, 96, 128, 256 KB (two fetches
    // sharing the link): 32 rows x 16k, k = 64: 267, 241, 230, 241, 275; 32 x 32k, k = 256: 451, 387, 370, 367, 400; 32 x 32k, 1
    // bit: 191, 166, 162, 166, 172; 32 x 32k, 8 query rows: 137, 119, 119, 122, 128.  A caller with one fetch at a time gets what
    // gather_kernel (gather.hip) gives it: more the fewer keys are scored for a fetched pair.  (launch_ranges rounds a lane's reads down to a
    // power of two: 96 KB are 64 for 1, 2 and 4 rows.)
    const double keys_per_pair = (double)L.G * Nq / L.topk;
    const int total_kb = link_shared ? 96 : keys_per_pair >= 384.0 ? 128 : keys_per_pair >= 192.0 ? 192 : 256;
    const GatherIo g{(const uint4*)L.host, (uint4*)slot, slot_idx, L.max_seq, 0, 0};
    const TopkIo io{Nq, 1, Nq, nullptr, 0, nullptr};
    return launch_ranges(L.rows, Nq, io, L.topk, keys, key_stride, idx_out, stream, &g, total_kb > L.rows ? total_kb / L.rows : 1);
}

}  // namespace specache
