// Internal launch interface between the C-ABI host code (specache.hip) and the
// kernel translation units.  Every launcher only enqueues on `stream` and
// returns the hipGetLastError() of its launches.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

namespace specache {

// Geometry and device pointers of one layer, as the kernels see them.
struct LayerView {
    int rows;          // B * Hkv
    int G;             // query heads per KV head
    int bits, group, R, max_seq, topk;
    bool bf16;
    bool one_bit_plain;   // bits == 1: Eq. 2 with B = 1 instead of Eq. 3
    uint8_t* kc;       // K codes   [rows][kc_stride bytes]
    uint32_t* km;      // K meta    [rows][km_stride dwords]  ([group j][128])
    uint8_t* vc;       // V codes   [rows][vc_stride bytes]
    uint32_t* vm;      // V meta    [rows][vm_stride dwords]  ([token][128/g])
    uint16_t* ring;    // residual  [rows][R][256] 16-bit
    uint16_t* host;    // pinned C  [rows][max_seq][256] 16-bit (device-visible address)
    size_t kc_stride, km_stride, vc_stride, vm_stride;
    // Set for one scoring launch only (specache_append_score): the new token's (K, V) pair, which one
    // extra workgroup per row copies to the host store and the residual ring as token tail_N0.
    const uint16_t* tail_k = nullptr;   // [rows][128] 16-bit, null: nothing to append
    const uint16_t* tail_v = nullptr;
    int tail_N0 = 0;
};

// quantize_append: flush `n_flush` groups starting at token Nq0, whose sources are
// the ring (tokens < N0) or k_new/v_new (tokens >= N0, index t - N0 of n_new).
// copy_from >= 0: launch_append_copy (with that as ring_from) in the same launch, where the ring's tokens that are quantised and those that
// are written do not share places
hipError_t launch_flush(const LayerView& L, const void* k_new, const void* v_new, int n_new, int N0,
                        int Nq0, int n_flush, int copy_from, hipStream_t stream);
// copy the n_new tokens to the host store (all) and to the ring (tokens >= ring_from)
hipError_t launch_append_copy(const LayerView& L, const void* k_new, const void* v_new, int n_new, int N0,
                              int ring_from, hipStream_t stream);

// Per-kernel timing of the scoring pass and of ArgTopK: a pair of events that the next kernel launched through
// SPC_LAUNCH on this thread carries on its own dispatch packet (start and stop of that kernel, as a
// profiler sees them) instead of event records around the launch, which would add the stream's
// marker packets and the launch gap to the figure.
struct LaunchEvents {
    hipEvent_t start = nullptr, stop = nullptr;
    int launches = 1;   // kernels the pair spans: the first carries start, the last stop
};
LaunchEvents& pending_launch_events();
#define SPC_LAUNCH(kernel, grid, block, stream, ...)                                                          \
    do {                                                                                                      \
        specache::LaunchEvents& le_ = specache::pending_launch_events();                                      \
        if (le_.stop) {                                                                                       \
            const bool last_ = le_.launches <= 1;                                                             \
            hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, le_.start, last_ ? le_.stop : nullptr, 0,   \
                                  __VA_ARGS__);                                                               \
            if (last_) le_ = specache::LaunchEvents{};                                                        \
            else { le_.start = nullptr; --le_.launches; }                                                     \
        } else {                                                                                              \
            hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);                                  \
        }                                                                                                     \
    } while (0)

// score: logits [rows*G*n_rows][logit_stride] fp32 and keys [rows][key_stride] u32 for i < Nq
hipError_t launch_score(const LayerView& L, const void* q, int n_rows, int Nq, float sm_scale, float* logits,
                        size_t logit_stride, uint32_t* keys, size_t key_stride, hipStream_t stream);

// selection keys from the heads' log-probabilities (after launch_score); scratch of
// select_logprob_scratch_floats(rows, G, max_seq) floats
size_t select_logprob_scratch_floats(int rows, int G, int max_seq);
hipError_t launch_select_logprob(const LayerView& L, int n_rows, int Nq, const float* logits, size_t logit_stride,
                                 float* scratch, uint32_t* keys, size_t key_stride, hipStream_t stream);
// after launch_score: logits and keys of the staged positions from their 16-bit keys (selection on the mixed cache)
hipError_t launch_patch_staged(const LayerView& L, const void* q, int n_rows, int Nq, float sm_scale, const uint16_t* slot,
                               const int32_t* slot_idx, float* logits, size_t logit_stride, uint32_t* keys,
                               size_t key_stride, hipStream_t stream);
// one query head per KV head, two rows: integer matrix cores (q must be 16-byte aligned)
bool score_uses_int8_matrix_cores(int G, int n_rows);
hipError_t launch_score_i8(const LayerView& L, const void* q, int Nq, float sm_scale, float* logits,
                           size_t logit_stride, uint32_t* keys, size_t key_stride, hipStream_t stream);

// top-k over keys[row][0..Nq): idx_out [rows][k], ascending, -1 padded.  Rows too long for one
// workgroup's registers are selected in two launches through the candidate buffers.
struct TopkScratch {
    uint32_t* cand_keys;   // [rows][max_parts][k]
    int32_t* cand_idx;     // [rows][max_parts][k]
    int max_parts;
};
int topk_parts(int Nq, int k);   // ranges a row of Nq keys is split into (1 = single launch)
hipError_t launch_topk(int rows, int Nq, int k, const uint32_t* keys, size_t key_stride, int32_t* idx_out,
                       const TopkScratch& scratch, hipStream_t stream);

// gather rows idx[row][j] of the host store into slot [rows][k][256] and slot_idx [rows][k];
// Nq (quantised positions of the layer), link_shared (another gather runs beside this one) and alone (on the stream that scored: nothing of this
// context runs beside it) only pace the transfer
hipError_t launch_gather(const LayerView& L, int Nq, const int32_t* idx, uint16_t* slot, int32_t* slot_idx,
                         bool link_shared, bool alone, hipStream_t stream);

// both in one launch: a row's pairs are fetched by the workgroup that selected them
bool selects_and_gathers(int rows, int Nq, int k);   // where that is the better way
hipError_t launch_select_gather(const LayerView& L, int Nq, const uint32_t* keys, size_t key_stride, int32_t* idx_out,
                                uint16_t* slot, int32_t* slot_idx, bool link_shared, hipStream_t stream);

// attend: partial pass + combine.  slot/slot_idx may be null (nothing prefetched).
struct AttendScratch {
    float* part_o;   // [rows][max_chunks][NR][128]
    float* part_ml;  // [rows][max_chunks][NR][2]  (max, sum)
    int max_chunks;
};
enum { kAttendPartial = 1, kAttendCombine = 2 };   // which of the two launches launch_attend issues
// A 64-bit word that other streams wait on (hipStreamWaitValue64).  The merge kernel stores value there as it starts, i.e. when
// the launch in front of it on its stream has completed.  finish_row stores it from inside the launch that scores: by then
// the selection keys of every row are stored and its chunks have read all they read, but the outputs and the pair that the launch
// appends need not have landed, and what reads those goes behind the launch by an event.  word == null: nothing to announce.
struct Announce {
    uint64_t* word = nullptr;
    uint64_t value = 0;
};
// The merge inside the launch that makes the partials (finish_row.h).  arrived: rows + 1 counters, zero between launches, each in a
// cache line of its own (all of a launch's workgroups count at about the same time, and the additions to one line wait for each
// other: attention alone over 16 x 31000 with one query row 19.4 us with the counters side by side, 10.9 so; 32 x 15800
// 17.2 / 11.3; both passes over 32 x 15500 20.5 / 16.5); null: a launch of its own merges.
constexpr int kFinishStride = 32;
struct Finish {
    uint32_t* arrived = nullptr;
    float* out = nullptr;        // [rows][NR][128]
    uint64_t* word = nullptr;    // announced when every row's keys are stored (null: nothing to announce)
    uint64_t value = 0;
    int rows = 0;
    int shares = 1;              // a share is up to 8 of the row's query rows
    bool mergers = false;        // a workgroup for each share that does nothing else; else the last of the row's chunks to arrive merges them all
    int polls = 0;               // of such a workgroup, before it leaves its share to the last chunk
};
// Where a launch of rows_kernel or attend_i8_kernel merges, by workgroups of its own: up to kFinishChunks chunks per row, in shares that one
// workgroup's loads cover at once (chunks x query rows of a share <= kFinishShare) where that leaves at least one query row.  us, a launch
// of its own (the last chunk of a row where that was better: 1) / mergers.  The launches alone: both passes over 1 x 4096 9.2 (1) / 9.0, 32 x
// 8000, 1 bit 13.3 (1) / 12.9, 16 x 16384 13.8 / 12.3, 32 x 32768 30.4 / 29.9, 512 x 1000 24.5 / 21.3; 8 query rows over 64 x 1000 12.6 (1) / 12.1, 24 x
// 5003 14.9 / 14.2, 32 x 8192 18.3 / 17.0, 8 x 131072, 1 bit (99 chunks) 43.4 / 42.7; 16 over 16 x 8192 17.3 / 16.3, 8 x 32768 (98) 25.6 / 26.0; but
// 1 x 60000 (119) 10.4 / 11.0.  A pass of steps with their fetches: 8 layers of 32 x 16384 223 / 211, of 24 x 5003, 8 query rows 279 / 269, of 16 x
// 8192, 16 rows 163 / 158, of 64 x 1000 198 (1) / 180, of 1 x 60000 151 / 134, of 8 x 32768, 16 rows 302 / 302.  The last chunk as the only one to
// merge where the partials are many: 8 x 131072 59.8 and 16 rows over 8 x 32768 67.8 (one workgroup reads them all).  (Launches of attend_i8_kernel that
// take several rounds of workgroups: kRoundChunks, attend_i8.hip.  rows_kernel splits its rows so that they are one.)
constexpr int kFinishChunks = 128, kFinishShare = 128;
constexpr int kMergerPolls = 2000;   // two to five milliseconds
int& merger_polls();                 // that, unless specache_debug_merger_polls says otherwise
inline int merge_shares_of(int n_chunks, int NR) {
    int nr = NR > 8 ? 8 : NR;
    while (nr > 1 && n_chunks * nr > kFinishShare) nr /= 2;
    return NR / nr;
}
// attend_partial_kernel, and rows_kernel where it only attends, leave the merge to the last chunk to arrive where the launch is no more than
// one round of workgroups and the partials are few.  us, a launch of its own / so: one query row over 1 x 31000 9.5 / 7.4, 32 x 15800 12.5 /
// 11.3; mergers / so: 4 bits (scoring with it), 16 x 4000 15.6 / 15.4, 32 x 6000 22.2 / 21.9.  So does attend_i8_kernel where it only attends (1 x 2000
// 8.5 / 7.6, 1 x 9000 8.7 / 7.8, 8 x 3000 8.3 / 7.7, 32 x 7000 10.1 / 9.5, 16 x 14000 10.5 / 9.7), and, scoring as well, for up to kFinishFewRows rows: a pass
// of 16 layers with their fetches on the queue of the main stream, 1 x 1000 238 / 233, 1 x 2000 242 / 233, 1 x 9000 245 / 242, of 8 layers, 2 x 6000 129 / 126, but 8 x
// 3000 154 / 155, 32 x 2000 251 / 254 (on queues of their own within 1 % up to 8 x 3000, 32 x 2000 168 / 171).
constexpr int kFinishMost = 64, kFinishFewRows = 4;
inline bool last_chunk_merges(int rows, int n_chunks, int NR) { return rows * n_chunks <= 1024 && n_chunks * NR <= kFinishMost; }
// last_chunk: it may be left to that one
inline bool plan_merge(Finish& fin, int rows, int n_chunks, int NR, bool last_chunk) {
    if (!fin.arrived || n_chunks > kFinishChunks) {
        fin = Finish{};
        return false;
    }
    fin.shares = merge_shares_of(n_chunks, NR);
    fin.mergers = !(last_chunk && last_chunk_merges(rows, n_chunks, NR));
    fin.polls = merger_polls();
    return true;
}

int attend_main_chunk_tokens(int NR);   // for the limits of specache_create and specache_attend_static
// the chunks that such a limit allows for NR query rows per KV head, Nq quantised and n_16bit 16-bit candidates
int attend_chunks(int NR, int Nq, int n_16bit);
int attend_extra_chunk_tokens();
int attend_max_chunks();   // chunks per row the merge kernel handles
hipError_t launch_attend(const LayerView& L, const void* q, int n_rows, int N, int Nq, float sm_scale,
                         const float* logits, size_t logit_stride, const uint16_t* slot,
                         const int32_t* slot_idx, const void* k_spec, const void* v_spec,
                         const AttendScratch& scratch, float* out, int phases, uint32_t* arrived, hipStream_t stream,
                         Announce announce = Announce());

// the same partial pass for one query head per KV head, two rows, 2-bit values: value side on the integer matrix cores
bool attend_uses_int8_matrix_cores(const LayerView& L, int n_rows);
// keys != null: the low-bit scoring runs inside the same launch (logits are not read; the speculative row's
// selection keys go to keys, and the logits to logits_out if that is set)
hipError_t launch_attend_i8_partial(const LayerView& L, const void* q, int N, int Nq, float sm_scale, const float* logits,
                                    size_t logit_stride, const uint16_t* slot, const int32_t* slot_idx, const void* k_spec,
                                    const void* v_spec, const AttendScratch& scratch, uint32_t* keys, size_t key_stride,
                                    float* logits_out, const Finish& finish, bool* merged, hipStream_t stream);

// Process-wide choice of kernels, for A/B measurements of one formulation against the other
// (specache_debug_kernel_choice): bits set here send the shapes that the matrix-core kernels
// would take to the vector-ALU kernels instead.
enum { kChoiceScoreValu = 1, kChoiceAttendValu = 2, kChoiceKeepLogits = 4 };
int& kernel_choice();

// export: canonical unpacked view of rows' quantised prefix into device buffers
hipError_t launch_export(const LayerView& L, int Nq, uint8_t* k_codes, uint16_t* k_mnmx, float* k_sz,
                         uint8_t* v_codes, uint16_t* v_mnmx, float* v_sz, hipStream_t stream);

}  // namespace specache
