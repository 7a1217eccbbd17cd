// Launch arguments of the attention kernels.
#pragma once
#include "kernels.h"

namespace specache {

struct AttendArgs {
    const uint16_t* q;         // [rows*NR][128]
    const float* logits;       // [rows*NR][logit_stride]
    float* logits_out;         // only the kernel that scores and attends in one pass: where to leave the logits, or null
    uint16_t* q_out;           // that kernel, for several rows per KV head: where to leave a copy of q instead, or null
    size_t logit_stride;
    const uint16_t* slot;      // [rows][k][256] or null
    const int32_t* slot_idx;   // [rows][k] or null
    const uint16_t* k_spec;    // [rows][128] or null
    const uint16_t* v_spec;
    float* part_o;             // [rows][max_chunks][NR][128]
    float* part_ml;            // [rows][max_chunks][NR][2]
    int max_chunks, n_main, n_chunks, N, Nq;
    float sm_scale;
    Finish fin;
};

// rows_kernel (rows_mfma.h): scoring and attention of 4, 8 or 16 query rows per KV head, and of any number on 4-bit codes
enum { kRowsBoth = 0, kRowsScore = 1, kRowsAttend = 2 };
struct RowsArgs {
    AttendArgs at;       // n_main, n_chunks: filled in by launch_rows
    uint32_t* keys;
    size_t key_stride;
    int n_rows;          // query rows per query head (1 or 2); the last one ranks the positions
    int wave_units;      // units of a wave (filled in by launch_rows)
};
constexpr int kRowsMaxChunk = 16384;   // tokens of a workgroup's chunk, at most (its bitmap of staged positions)

bool rows_uses_matrix_cores(const LayerView& L, int n_rows);
bool rows_in_one_launch(const LayerView& L, int n_rows);                       // scoring and attention together (kRowsBoth)
int rows_max_main_chunks(int rows, int max_seq);                               // most chunks of quantised positions per row
// chunks launch_rows splits a row into: at most max_chunks, where chunks of kRowsMaxChunk tokens allow that
int rows_chunks(const LayerView& L, int n_rows, int Nq, int n_16bit, int max_chunks);
// merged: whether the launch merges its partials itself (R.at.fin)
hipError_t launch_rows(const LayerView& L, RowsArgs R, int mode, bool* merged, hipStream_t stream);

}  // namespace specache
