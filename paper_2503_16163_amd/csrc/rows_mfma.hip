// Chunking and dispatch of rows_kernel (rows_mfma.h).
#include "kernels.h"
#include "layout.h"
#include "rows_args.h"

namespace specache {

hipError_t launch_rows_b1(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream);
hipError_t launch_rows_b2(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream);
hipError_t launch_rows_b4(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream);

namespace {

// Workgroups that a launch aims at: three are resident per compute unit (registers), and with at most that many of
// equal length the launch has no second, emptier round.
constexpr int kRowsTarget = 768;

// rows of the kernel's columns: fewer than 8 run as 8, of which some do not exist
int padded_rows(const LayerView& L, int n_rows) { return L.G * n_rows < 8 ? 8 : L.G * n_rows; }

// units of 32 * 16 / NR tokens that each of a workgroup's four waves takes, and the chunks of a row
void rows_split(int rows, int NR, int Nq, int max_main, int& wave_units, int& n_main) {
    const int unit = 32 * (16 / NR), units = (Nq + unit - 1) / unit, most = kRowsMaxChunk / (4 * unit);
    int w = (int)(((long)rows * units + 4 * kRowsTarget - 1) / (4 * kRowsTarget));
    // scratch memory for fewer chunks (specache_attend_static): longer ones
    const int at_least = max_main > 0 ? (units + 4 * max_main - 1) / (4 * max_main) : 1;
    w = w < at_least ? at_least : w;
    w = w < 1 ? 1 : (w > most ? most : w);
    n_main = (units + 4 * w - 1) / (4 * w);
    wave_units = n_main > 0 ? (units + 4 * n_main - 1) / (4 * n_main) : 1;   // chunks of equal length
}

}  // namespace

bool rows_uses_matrix_cores(const LayerView& L, int n_rows) {
    // Four rows leave half of the columns empty and are still faster than a conversion and four multiply-accumulates per code
    // on the vector ALUs in two launches: a decode step of a layer, 16 x 16384, 2 bits 45.5 -> 28 us, 32 x 32768 85.3 -> 61,
    // 8 x 131072, 1 bit 79.5 -> 59.5; one row of each of four heads, 8 x 32768, 62.7 -> 57.
    // Fewer rows leave more of them empty.  1- and 2-bit codes have kernels made for them (two rows: scoring and attention in one
    // launch on the int8 matrix cores, 17.8 us for 32 x 16384 positions); with 4-bit codes the alternative was a conversion and
    // a multiply-accumulate per code on the vector ALUs: 45 + 54 us for 32 x 32768, two rows, against 27.1 + 33.1.
    const int NR = L.G * n_rows;
    return NR >= 4 || L.bits == 4;
}

// 4-bit codes keep two launches because no instance of the one launch is built for them: a step's arrangement scores and
// attends in two calls there.
bool rows_in_one_launch(const LayerView& L, int n_rows) { return L.bits != 4 && rows_uses_matrix_cores(L, n_rows); }

int rows_max_main_chunks(int rows, int max_seq) {
    const int by_length = max_seq / kRowsMaxChunk + 2, by_target = kRowsTarget / rows + 2;
    return by_length > by_target ? by_length : by_target;
}

int rows_chunks(const LayerView& L, int n_rows, int Nq, int n_16bit, int max_chunks) {
    int wave_units, n_main;
    const int n_extra = (n_16bit + 127) / 128;
    rows_split(L.rows, padded_rows(L, n_rows), Nq, max_chunks - n_extra, wave_units, n_main);
    return n_main + n_extra;
}

hipError_t launch_rows(const LayerView& L, RowsArgs R, int mode, bool* merged, hipStream_t stream) {
    const int NR = padded_rows(L, R.n_rows);
    if (!rows_uses_matrix_cores(L, R.n_rows) || R.at.Nq % kBlockTokens || R.at.Nq % L.group) return hipErrorInvalidValue;
    const int n_ex = mode == kRowsScore ? 0 : (R.at.slot_idx ? L.topk : 0) + (R.at.N - R.at.Nq) + (R.at.k_spec ? 1 : 0);
    const int n_extra = (n_ex + 127) / 128;
    rows_split(L.rows, NR, R.at.Nq, mode == kRowsScore ? R.at.Nq : R.at.max_chunks - n_extra, R.wave_units, R.at.n_main);
    R.at.n_chunks = R.at.n_main + n_extra;
    if (R.at.n_chunks < 1) return hipErrorInvalidValue;
    if (mode != kRowsScore && R.at.n_chunks > R.at.max_chunks) return hipErrorInvalidValue;
    const bool merges = mode != kRowsScore && plan_merge(R.at.fin, L.rows, R.at.n_chunks, L.G * R.n_rows, mode == kRowsAttend);
    if (merged) *merged = merges;
    return L.bits == 1   ? launch_rows_b1(L, R, NR, mode, stream)
           : L.bits == 2 ? launch_rows_b2(L, R, NR, mode, stream)
                         : launch_rows_b4(L, R, NR, mode, stream);
}

}  // namespace specache
