// Many-row projections on the matrix cores (see pgemm.hip).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace sd2 {

constexpr int kPgBlk = 64;            // columns of one block of the activation planes
constexpr int kPgBlkWords = 2 * kPgBlk;  // its bf16 words per row: 64 hi, then 64 lo
// bytes read past the last row of the planes by the last row block (never used)
constexpr size_t kPgSlack = 128 * kPgBlkWords * 2;

// Shape of a launch: 16 MG rows by 64 NG weight rows per workgroup, K in S ranges.
struct PgPlan {
    int MG, NG, S, nblk_m, nblk_n;
    size_t part;  // floats of split-K partials (0 without a split)
    size_t cnt;   // arrival counters
};
// N: weight rows, counting gate and up together.
PgPlan pg_plan(int M, int N, int K);

inline int pg_rows(int M) { return (M + 15) / 16 * 16; }
// bytes of the planes of M rows and K columns
inline size_t pg_plane_bytes(int M, int K) { return (size_t)pg_rows(M) * K * 4 + kPgSlack; }

}  // namespace sd2
