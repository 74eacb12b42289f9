// Where the labels of a graph's cells lie (kernels_sparse.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace alpa {

constexpr int GRAPH_CELLS = 1536;              // of one graph, the end included

// A stage's second word: the byte of its cell's label, and in the upper half the byte of that of the cell behind it.
__host__ __device__ __forceinline__ int32_t graph_label_bytes(int cell, int behind) { return 8 * cell | 8 * behind << 16; }

// The byte of the label behind that a lane reads.  A lane that has no stage holds what lies behind the graph, another
// graph's stage or memory that nobody has written: it reads the end's label.
__host__ __device__ __forceinline__ uint32_t graph_label_behind(int32_t bytes, bool has_stage)
{
    return has_stage ? (uint32_t)bytes >> 16 : 0;
}

}  // namespace alpa
