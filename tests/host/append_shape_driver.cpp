// Driver of csrc/append_shape.h (run by tests/test_boundary.py on the CPU): the workgroups of the launch that quantises and copies.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2503_16163_amd/csrc/append_shape.h"

using namespace specache;

#define REQUIRE(cond)                                                                     \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "append_shape_driver: %s failed at line %d\n", #cond, __LINE__); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

int main() {
    // a dimension of a launch holds 2^32 - 1 threads: the longest cache there is, many rows, and both
    for (int rows : {1, 32, 512, 1024, 60000})
        for (int n_new : {32, 210000, 650000})
            for (int g : {32, 64, 128}) {
                const dim3 grid = append_grid(n_new / g, n_new, rows);
                REQUIRE((uint64_t)grid.x * kAppendThreads < (uint64_t)1 << 32);
                REQUIRE(grid.y < 65536 && grid.z == 1);
                REQUIRE((uint64_t)grid.x * grid.y == (uint64_t)(n_new / g + append_copy_blocks(n_new)) * rows);
            }
    // every group is quantised and every piece of the new tokens copied once, whatever their numbers (one token may complete a group, a
    // prompt need not complete any but its first)
    for (int n_flush : {1, 2, 3, 7, 64, 1000})
        for (int n_new : {1, 7, 8, 9, 31, 64, 100, 2048, 2051, 32000, 65000}) {
            const int n_copy = append_copy_blocks(n_new);
            REQUIRE(n_copy * kCopyTokens >= n_new && (n_copy - 1) * kCopyTokens < n_new);
            std::vector<int> groups(n_flush, 0), pieces(n_copy, 0);
            for (int id = 0; id < (int)append_grid(n_flush, n_new, 1).x; ++id) {
                const AppendJob job = append_job(id, n_flush, n_copy);
                REQUIRE(job.nth >= 0 && job.nth < (job.quantise ? n_flush : n_copy));
                ++(job.quantise ? groups : pieces)[job.nth];
            }
            for (int n : groups) REQUIRE(n == 1);
            for (int n : pieces) REQUIRE(n == 1);
        }
    std::printf("append_shape_driver ok\n");
    return 0;
}
