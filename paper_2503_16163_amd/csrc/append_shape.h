// Which workgroup does what where an append quantises and copies in one launch (flush_copy_kernel, quant.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace specache {

constexpr int kAppendThreads = 256;
constexpr int kCopyTokens = kAppendThreads / 32;   // tokens that a workgroup copies, 32 lanes each

inline __host__ __device__ int append_copy_blocks(int n_new) { return (n_new + kCopyTokens - 1) / kCopyTokens; }

// A row's workgroups side by side, the rows in the second dimension: all in one, they would be more threads than a dimension of a launch
// holds (2^32 - 1) from 107 million (row, token) pairs on, 55 GB of host store, in groups of 32.
inline dim3 append_grid(int n_flush, int n_new, int rows) { return dim3(n_flush + append_copy_blocks(n_new), rows); }

// The workgroups that quantise are spread evenly among those that copy.  nth: of the row's groups or of its pieces of kCopyTokens tokens.
struct AppendJob {
    bool quantise;
    int nth;
};
inline __host__ __device__ AppendJob append_job(int id, int n_flush, int n_copy) {
    const int every = (n_flush + n_copy) / n_flush, nth = id / every;
    if (id % every == 0 && nth < n_flush) return {true, nth};
    return {false, id - (nth + 1 < n_flush ? nth + 1 : n_flush)};
}

}  // namespace specache
