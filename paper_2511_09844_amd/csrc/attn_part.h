// Where the spans of an attention launch leave their partial sums (see arrive_last).  The workgroup
// that merges a group reads with ordinary loads, so no 128-byte line may hold values of two groups:
// the merge of one would bring the line into its XCD's L2 before the other group's values are
// written, and a later merge on that XCD would read the stale copy.
#pragma once
#include <stddef.h>

#ifdef __HIPCC__
#define SD2_PART_FN __host__ __device__ inline
#else
#define SD2_PART_FN inline
#endif

namespace sd2 {

constexpr int kPartLine = 32;  // floats of a 128-byte line

// The un-normalised outputs of a query vector (activation row, head) over span sp: hd floats, whole
// lines ...
SD2_PART_FN size_t part_out(size_t row, int H, int h, int nspan, int sp, int hd) {
    return ((row * H + h) * nspan + sp) * hd;
}
// ... and behind those of all rows the (max, sum) pairs, a line for the 16 query vectors of a block
// (which lie in one group) and a span: pair i of block `block`.
SD2_PART_FN size_t part_ml(size_t rows, int H, int hd, size_t block, int nspan, int sp, int i) {
    return rows * H * nspan * hd + (block * nspan + sp) * kPartLine + 2 * i;
}
// Floats per span.
SD2_PART_FN size_t part_floats(size_t rows, int H, int hd, size_t blocks) { return rows * H * hd + blocks * kPartLine; }

// Persistent kernel: floats of an activation row's head, nsplit records of hd + 4 (outputs, max, sum)
// padded to whole lines (a row's head lies in one group).
SD2_PART_FN size_t part_row(int nsplit, int hd) {
    return ((size_t)nsplit * (hd + 4) + kPartLine - 1) / kPartLine * kPartLine;
}

}  // namespace sd2
