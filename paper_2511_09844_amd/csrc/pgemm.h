// Projections on activation planes (see pgemm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace sd2 {

constexpr int kPgBlk = 64;            // columns of one block of the activation planes
constexpr int kPgBlkWords = 2 * kPgBlk;  // its bf16 words per row: 64 hi, then 64 lo
// The last row block reads up to 112 rows (28 KB) past the end of the planes, never used: the
// workspace holds more than that behind every plane buffer.

// Shape of a launch: 16 MG rows by 64 NG weight rows per workgroup, K in S ranges.
struct PgPlan {
    int MG, NG, S, nblk_m, nblk_n, grid;
    bool skinny;  // k_sgemm takes it (nothing else is set)
    int units;    // block partials the workspace has room for
    size_t part;  // floats of split-K partials (0 without a split)
};
// Arrival counters: one per block of a split launch, of which two ranges each come to kPgUnits at most.
constexpr int kPgUnits = 512, kPgCounters = kPgUnits / 2;
// K ranges for a number of blocks: up to two workgroups per CU (one with up to 32 rows, 16 MG), and
// no more block partials than `units`.
__host__ __device__ inline int pg_ranges(int blocks, int MG, int K, int units) {
    const int want = MG <= 2 ? kPgUnits / 2 : kPgUnits, min_k = MG <= 2 ? 256 : 512;
    const int target = want < units ? want : units;
    const int s = target / blocks < K / min_k ? target / blocks : K / min_k;
    return s > 1 ? s : 1;
}
// N: weight rows, counting gate and up together.  packed: the rows that hold data may be fewer
// than M; the kernel then takes blocks and ranges for those (any number may occur).  room: floats of
// partials that the workspace holds.
PgPlan pg_plan(int M, int N, int K, bool packed = false, size_t room = SIZE_MAX);

inline int pg_rows(int M) { return (M + 15) / 16 * 16; }
// bytes of the planes of M rows and K columns
inline size_t pg_plane_bytes(int M, int K) { return (size_t)pg_rows(M) * K * 4; }

#ifdef __HIPCC__
typedef __bf16 pg_bf2 __attribute__((ext_vector_type(2)));
typedef float pg_f2 __attribute__((ext_vector_type(2)));

// hi/lo bf16 split of two fp32 values, packed (hi = x rounded to nearest even, lo = (x - hi)
// rounded likewise)
__device__ __forceinline__ void pg_split2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
    const pg_f2 v = {x0, x1};
    const pg_bf2 h = __builtin_convertvector(v, pg_bf2);
    const pg_bf2 l = __builtin_convertvector(v - __builtin_convertvector(h, pg_f2), pg_bf2);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}
// Columns c .. c + 3 (c a multiple of 4), or column c, of a row into planes of Mp rows.
__device__ __forceinline__ void pg_put4(uint16_t* planes, int Mp, size_t row, int c, float4 v) {
    uint2 h, l;
    pg_split2(v.x, v.y, h.x, l.x);
    pg_split2(v.z, v.w, h.y, l.y);
    uint16_t* p = planes + ((size_t)(c / kPgBlk) * Mp + row) * kPgBlkWords + c % kPgBlk;
    *(uint2*)p = h;
    *(uint2*)(p + kPgBlk) = l;
}
__device__ __forceinline__ void pg_put1(uint16_t* planes, int Mp, size_t row, int c, float v) {
    uint32_t h, l;
    pg_split2(v, 0.f, h, l);
    uint16_t* p = planes + ((size_t)(c / kPgBlk) * Mp + row) * kPgBlkWords + c % kPgBlk;
    p[0] = (uint16_t)h;
    p[kPgBlk] = (uint16_t)l;
}
#endif

}  // namespace sd2
