// Chunking and dispatch of rows_kernel (rows_mfma.h): 4, 8 or 16 query rows per KV head.
#include "kernels.h"
#include "layout.h"
#include "rows_args.h"

namespace specache {

hipError_t launch_rows_b1(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream);
hipError_t launch_rows_b2(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream);

namespace {

// Workgroups that a launch aims at: three are resident per compute unit (registers), and with at most that many of
// equal length the launch has no second, emptier round.
constexpr int kRowsTarget = 768;

// units of 32 * 16 / NR tokens that each of a workgroup's four waves takes, and the chunks of a row
void rows_split(int rows, int NR, int Nq, int& wave_units, int& n_main) {
    const int unit = 32 * (16 / NR), units = (Nq + unit - 1) / unit, most = kRowsMaxChunk / (4 * unit);
    int w = (int)(((long)rows * units + 4 * kRowsTarget - 1) / (4 * kRowsTarget));
    w = w < 1 ? 1 : (w > most ? most : w);
    n_main = (units + 4 * w - 1) / (4 * w);
    wave_units = n_main > 0 ? (units + 4 * n_main - 1) / (4 * n_main) : 1;   // chunks of equal length
}

}  // namespace

bool rows_uses_matrix_cores(const LayerView& L, int n_rows) {
    const int NR = L.G * n_rows;
    return (NR == 8 || NR == 16) && (L.bits == 1 || L.bits == 2);
}

int rows_max_main_chunks(int rows, int max_seq) {
    const int by_length = max_seq / kRowsMaxChunk + 2, by_target = kRowsTarget / rows + 2;
    return by_length > by_target ? by_length : by_target;
}

int rows_chunks(const LayerView& L, int n_rows, int Nq, int n_16bit) {
    int wave_units, n_main;
    rows_split(L.rows, L.G * n_rows, Nq, wave_units, n_main);
    return n_main + (n_16bit + 127) / 128;
}

hipError_t launch_rows(const LayerView& L, RowsArgs R, int mode, hipStream_t stream) {
    const int NR = L.G * R.n_rows;
    if (!rows_uses_matrix_cores(L, R.n_rows) || R.at.Nq % kBlockTokens || R.at.Nq % L.group) return hipErrorInvalidValue;
    rows_split(L.rows, NR, R.at.Nq, R.wave_units, R.at.n_main);
    const int n_ex = mode == kRowsScore ? 0 : (R.at.slot_idx ? L.topk : 0) + (R.at.N - R.at.Nq) + (R.at.k_spec ? 1 : 0);
    R.at.n_chunks = R.at.n_main + (n_ex + 127) / 128;
    if (R.at.n_chunks < 1) return hipErrorInvalidValue;
    if (mode != kRowsScore && R.at.n_chunks > R.at.max_chunks) return hipErrorInvalidValue;
    return L.bits == 1 ? launch_rows_b1(L, R, NR, mode, stream) : launch_rows_b2(L, R, NR, mode, stream);
}

}  // namespace specache
