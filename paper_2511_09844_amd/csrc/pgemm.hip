// Projections with bf16 weights outside the persistent kernel, on any number of activation rows
// (drafter steps and verify passes of batches, prefill chunks, the training-objective forward):
//
//   Y[m][n] (op)= sum_k W[n][k] * xn[m][k],   xn = x (optionally RMS-normalised and scaled by gamma)
//
// The activations enter as "planes": whoever produces a value (times the gain of the norm that
// reads it) splits it once into a bf16 hi/lo pair and stores it as [K / 64][row][64 hi | 64 lo],
// the order in which a workgroup stages it, so staging is a linear copy (16-byte loads, 16-byte
// LDS stores) with no arithmetic.  1/rms of the rows is applied by the epilogue.
//
// A workgroup of four waves owns 16 MG rows and 64 NG weight rows: each wave holds 16 NG weight
// rows of its own, whose fragments it loads straight into registers (a weight is read by one wave
// only, so LDS would add traffic), against all the rows, whose planes all four waves read from
// LDS.  K goes in steps of KB blocks of 64 columns with two LDS buffers; step i requests the planes of
// step i + 1 and each weight fragment of a later step (WD steps on).  As compiled these loads stand at
// the end of the step, among its last products: the planes are waited for there, and with WD 1 the
// weights at the start of the next step, so a step shows a good part of a memory round trip that only
// the CU's other workgroup covers.  A row of a block is 256 bytes in LDS, its sixteen 16-byte chunks
// permuted by chunk ^ (row & 15), so that the sixteen rows of an operand read fall into different
// banks.
//
// The weights are the A operand of v_mfma_f32_16x16x32_bf16 and the activations the B operand, so
// a lane ends with four consecutive output columns of one row: the epilogues (store, residual add
// with the next norm's sums of squares, SwiGLU, Q|K|V with RoPE and the cache append) run on
// registers with 16-byte accesses.  Weight rows are dealt in pairs of 16-row sub-tiles so that
// what an epilogue combines sits in one lane: gate and up of the same features, or the two
// rotate-half partners of a head.
//
// Bound: the weight bytes up to about 64 rows, the matrix cores from about 256.  Gate|up of the 8B
// verifier (28672 x 4096): 8 rows 50 to 52 us (4.6 TB/s), 36 rows 63, 128 rows 92, 512 rows 209 (354
// with the kernel before, which split fp32 rows in every workgroup and read them from LDS for half as
// many weight rows), 2048 rows 758 to 790 (1.25 PFLOP/s of bf16 products).
#include <hip/hip_ext.h>

#include <algorithm>

#include "device_common.h"
#include "engine.h"
#include "pgemm.h"

namespace sd2 {

typedef __bf16 pg_bf8 __attribute__((ext_vector_type(8)));
typedef float pg_f4 __attribute__((ext_vector_type(4)));
typedef unsigned int pg_u4 __attribute__((ext_vector_type(4)));

// Planes of rows that no producer stored as planes (steering projections, the training objective).
struct PlaneArgs {
    const float* X;
    const int32_t* in_map;  // source row of each row (negative: zeros), or null
    int Mp, K;              // rows of the planes, columns
    const uint16_t* gamma;  // bf16 gain, or null
    uint16_t* planes;
};

constexpr int kPlaneCols = 1024;  // columns per workgroup: one float4 per thread

__global__ __launch_bounds__(256) void k_planes(PlaneArgs a) {
    const int row = blockIdx.x, c = blockIdx.y * kPlaneCols + 4 * threadIdx.x;
    const int src = a.in_map ? a.in_map[row] : row;
    if (c >= a.K) return;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (src >= 0) v = *(const float4*)(a.X + (size_t)src * a.K + c);
    if (a.gamma) {
        const uint2 w = *(const uint2*)(a.gamma + c);
        v.x *= bf16_lo(w.x); v.y *= bf16_hi(w.x); v.z *= bf16_lo(w.y); v.w *= bf16_hi(w.y);
    }
    pg_put4(a.planes, a.Mp, row, c, v);
}

struct PgArgs {
    const uint16_t* planes;
    // RMSNorm input (ss not null): the outputs of a row are scaled by 1/rms, from the nss partial
    // sums of squares of its source row
    const float* ss;
    const int32_t* in_map;
    int nss;
    float eps;
    const int32_t* m_live;  // rows that hold data, of M (null: all)
    int M, Mp, K, S, nblk_m, nblk_n, nbs, units;
    const uint16_t* W[3];
    int pairs;          // pairs of 16-row sub-tiles
    int tiles;          // 16-column tiles of the output (store, add, SwiGLU)
    int seg_pairs[2];   // Q|K|V: pairs of Q and of K
    float* Y;
    int ldy;
    const int32_t* out_map;
    float* ss_out;
    uint16_t* yplanes;       // SwiGLU: planes of the output, in place of Y; add: planes of the new
    const uint16_t* ygamma;  // residual times this gain, beside Y; or null
    float* part;
    int32_t* cnt;
    int H, Hkv, hd;
    const int32_t *row_pos, *row_seq;
    const float *rcos, *rsin;
    float *qout, *kc, *vc;
    int cap, max_batch, layer;
    const float* ubias;
    int ub_ld;
};

// Segment (Q, K or V) of pair P, which becomes the pair's number within it.
__device__ __forceinline__ int pg_seg(const PgArgs& a, int& P) {
    int seg = 0;
    if (P >= a.seg_pairs[0]) { P -= a.seg_pairs[0]; seg = 1; }
    if (seg == 1 && P >= a.seg_pairs[1]) { P -= a.seg_pairs[1]; seg = 2; }
    return seg;
}

// Weight row of lane row n in sub-tile `sub` of pair P (P uniform, so that all but n stays scalar).
template <int MODE>
__device__ __forceinline__ const uint16_t* pg_row(const PgArgs& a, int P, int sub, int n) {
    if constexpr (MODE == kEpiSwiglu) {
        return (sub ? a.W[1] : a.W[0]) + (size_t)(P * 16 + n) * a.K;
    } else if constexpr (MODE == kEpiQkv) {
        const int seg = pg_seg(a, P);
        const int per = a.hd / 32, h = P / per, p = P % per;
        return (seg == 0 ? a.W[0] : seg == 1 ? a.W[1] : a.W[2]) + (size_t)(h * a.hd + sub * (a.hd / 2) + 16 * p + n) * a.K;
    } else {
        // an odd number of tiles leaves the last pair half empty: its second sub-tile re-reads the first
        return a.W[0] + (size_t)(min(2 * P + sub, a.tiles - 1) * 16 + n) * a.K;
    }
}

__device__ __forceinline__ pg_f4 pg_ld4(const float* p) { return *(const pg_f4*)p; }

__device__ __forceinline__ void pg_put_gain(const PgArgs& a, int row, int c, pg_f4 v) {
    const uint2 w = *(const uint2*)(a.ygamma + c);
    pg_put4(a.yplanes, a.Mp, row, c,
            make_float4(v.x * bf16_lo(w.x), v.y * bf16_hi(w.x), v.z * bf16_lo(w.y), v.w * bf16_hi(w.y)));
}

// What an epilogue reads of one pair and row: the residual (add) or the rotation (Q|K|V).
struct PgPre {
    pg_f4 a, b;
};
template <int MODE>
__device__ __forceinline__ PgPre pg_pre(const PgArgs& a, int P, int row, int pos, int q) {
    PgPre r = {};
    if constexpr (MODE == kEpiAdd) {
        const float* y = a.Y + (size_t)row * a.ldy + 32 * P + 4 * q;
        r.a = pg_ld4(y);
        r.b = pg_ld4(2 * P + 1 < a.tiles ? y + 16 : y);
    } else if constexpr (MODE == kEpiQkv) {
        pg_seg(a, P);  // (V pairs read factors they do not use)
        const size_t o = (size_t)max(pos, 0) * (a.hd / 2) + 16 * (P % (a.hd / 32)) + 4 * q;
        r.a = pg_ld4(a.rcos + o);
        r.b = pg_ld4(a.rsin + o);
    }
    return r;
}

// Epilogue of pair P for one row (at position pos): lane (n, q) holds columns 4q .. 4q + 3 of both
// sub-tiles.  Executed by all lanes (`valid`: the row exists), since the add mode reduces across
// lanes.
template <int MODE>
__device__ __forceinline__ void pg_epilogue(const PgArgs& a, int P, int row, bool valid, int pos, int q, pg_f4 v0,
                                            pg_f4 v1, const PgPre& pre) {
    if constexpr (MODE == kEpiStore) {
        if (!valid) return;
        const int orow = a.out_map ? a.out_map[row] : row;
        if (orow < 0) return;
        float* y = a.Y + (size_t)orow * a.ldy + 32 * P + 4 * q;
        *(pg_f4*)y = v0;
        if (2 * P + 1 < a.tiles) *(pg_f4*)(y + 16) = v1;
    } else if constexpr (MODE == kEpiAdd) {
        const bool two = 2 * P + 1 < a.tiles;
        float s0 = 0.f, s1 = 0.f;
        if (valid) {
            float* y = a.Y + (size_t)row * a.ldy + 32 * P + 4 * q;
            pg_f4 r0 = pre.a + v0, r1 = pre.b + v1;
            if (a.ubias) {
                const float* ub = a.ubias + (size_t)a.row_seq[row] * a.ub_ld + 32 * P + 4 * q;
                r0 += pg_ld4(ub);
                if (two) r1 += pg_ld4(ub + 16);
            }
            *(pg_f4*)y = r0;
            if (two) *(pg_f4*)(y + 16) = r1;
            if (a.yplanes) {
                pg_put_gain(a, row, 32 * P + 4 * q, r0);
                if (two) pg_put_gain(a, row, 32 * P + 16 + 4 * q, r1);
            }
            s0 = (r0.x * r0.x + r0.y * r0.y) + (r0.z * r0.z + r0.w * r0.w);
            s1 = (r1.x * r1.x + r1.y * r1.y) + (r1.z * r1.z + r1.w * r1.w);
        }
        s0 += __shfl_xor(s0, 16, 64);
        s1 += __shfl_xor(s1, 16, 64);
        s0 += __shfl_xor(s0, 32, 64);
        s1 += __shfl_xor(s1, 32, 64);
        if (valid && q == 0) {
            a.ss_out[(size_t)row * a.tiles + 2 * P] = s0;
            if (two) a.ss_out[(size_t)row * a.tiles + 2 * P + 1] = s1;
        }
    } else if constexpr (MODE == kEpiSwiglu) {
        if (!valid) return;
        if (a.ubias) v1 += pg_ld4(a.ubias + (size_t)a.row_seq[row] * a.ub_ld + 16 * P + 4 * q);
        pg_f4 o = {silu(v0.x) * v1.x, silu(v0.y) * v1.y, silu(v0.z) * v1.z, silu(v0.w) * v1.w};
        if (a.yplanes) pg_put4(a.yplanes, a.Mp, row, 16 * P + 4 * q, make_float4(o.x, o.y, o.z, o.w));
        else *(pg_f4*)(a.Y + (size_t)row * a.ldy + 16 * P + 4 * q) = o;
    } else {
        if (!valid) return;
        const int seg = pg_seg(a, P);
        const int per = a.hd / 32, h = P / per, i = 16 * (P % per) + 4 * q, half = a.hd / 2;
        if (seg < 2) {
            const pg_f4 x = v0;
            v0 = x * pre.a - v1 * pre.b;
            v1 = v1 * pre.a + x * pre.b;
        }
        float* y;
        if (seg == 0) {
            y = a.qout + (size_t)row * a.H * a.hd + h * a.hd + i;
        } else {
            if (pos < 0) return;
            y = (seg == 1 ? a.kc : a.vc) +
                ((((size_t)a.layer * a.max_batch + a.row_seq[row]) * a.Hkv + h) * a.cap + pos) * a.hd + i;
        }
        *(pg_f4*)y = v0;
        *(pg_f4*)(y + half) = v1;
    }
}

template <int MG, int NG, int KB, int WD, int MODE>
__global__ __launch_bounds__(256, 2) void k_pgemm(PgArgs a) {
    static_assert(NG % 2 == 0, "sub-tiles come in pairs");
    constexpr int kBlkB = 16 * MG * kPgBlkWords * 2;    // bytes of one 64-column block in LDS
    constexpr int kStageB = KB * kBlkB;
    constexpr int NA = kStageB / (256 * 16);            // 16-byte words per thread and step
    static_assert(NA >= 1, "stage");
    __shared__ __attribute__((aligned(16))) char sm[2 * kStageB];
    __shared__ float inv_s[16 * MG];
    __shared__ int last_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, q = lane >> 4;
    // workgroups are dealt to the 8 XCDs in turn, so blocks b, b + 8, ... share an XCD: they take
    // the row blocks of one weight block, whose weights then come from that XCD's L2
    // with packed rows, blocks and ranges are those of the rows that hold data
    int M = a.M, nblk_m = a.nblk_m, nbs = a.nbs, S = a.S;
    if (a.m_live) {
        M = *a.m_live;
        if (M == 0) return;
        nblk_m = (M + 16 * MG - 1) / (16 * MG);
        nbs = 8 * nblk_m * ((a.nblk_n + 7) / 8);
        S = S > 1 ? pg_ranges(nblk_m * a.nblk_n, MG, a.K, a.units) : 1;
    }
    const int s = blockIdx.x / nbs, bb = blockIdx.x % nbs;
    if (s >= S) return;
    const int r = bb >> 3, mb = r % nblk_m, nb = (bb & 7) + 8 * (r / nblk_m);
    if (nb >= a.nblk_n) return;  // grid padding (uniform per workgroup)
    const int m0 = mb * 16 * MG;
    const int P0 = nb * 2 * NG + wave * (NG / 2);       // first pair of this wave
    const uint16_t* wp[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) wp[j] = pg_row<MODE>(a, min(P0 + j / 2, a.pairs - 1), j & 1, n) + 16 * q;
    // this range's steps of 64 KB columns
    const int nst = a.K / (kPgBlk * KB);
    const int b0 = nst * s / S, b1 = nst * (s + 1) / S;

    pg_u4 w[WD][KB][2][NG];
    pg_u4 xa[NA];
    auto load_w = [&](int step, int d, int kb, int h) {
#pragma unroll
        for (int j = 0; j < NG; ++j) w[d][kb][h][j] = *(const pg_u4*)(wp[j] + (size_t)(step * KB + kb) * kPgBlk + 8 * h);
    };
    // planes: block kb of a step is one run of 16 MG rows of 256 bytes
    const char* const xbase = (const char*)a.planes + (size_t)m0 * kPgBlkWords * 2 + tid * 16;
    const size_t xstep = (size_t)a.Mp * kPgBlkWords * 2;
    auto load_x = [&](int step) {
#pragma unroll
        for (int e = 0; e < NA; ++e) {
            constexpr int per = kBlkB / 4096;
            xa[e] = *(const pg_u4*)(xbase + (size_t)(step * KB + e / per) * xstep + (e % per) * 4096);
        }
    };
    const int srow = tid >> 4, schunk = tid & 15;
    char* const sbase = sm + srow * 256 + ((schunk ^ srow) << 4);
    auto stage = [&](int buf) {
#pragma unroll
        for (int e = 0; e < NA; ++e) *(pg_u4*)(sbase + buf * kStageB + e * 4096) = xa[e];
    };
    // Prologue.  Loads return in the order of their issue: positions, then with few rows the row
    // statistics (4 MG rows of partial sums of squares per wave, all in flight together), the planes
    // and the weights of the first step, and what the epilogue reads; the sums are added while the
    // weights are on their way.  With more rows the statistics would fill the registers: they follow
    // the weights, eight rows in flight, and the epilogue reads its inputs itself, in a round trip or
    // more for each row group and pair.
    constexpr bool kFew = MG <= 2;
    constexpr int RW = 4 * MG, RU = RW < 8 ? RW : 8;
    int pos[MG];
#pragma unroll
    for (int g = 0; g < MG; ++g)
        pos[g] = MODE == kEpiQkv && kFew ? a.row_pos[min(m0 + 16 * g + n, M - 1)] : 0;
    const bool stats = MODE != kEpiAdd && a.ss;
    const int n4s = a.nss / 4;
    pg_f4 sv[RU];
    auto load_ss = [&](int r0, int f0) {
        int src[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) src[u] = min(m0 + wave * RW + r0 + u, M - 1);
        if (a.in_map)
#pragma unroll
            for (int u = 0; u < RU; ++u) src[u] = max(a.in_map[src[u]], 0);
        const int f = 4 * min(f0 + lane, n4s - 1);
#pragma unroll
        for (int u = 0; u < RU; ++u) sv[u] = *(const pg_f4*)(a.ss + (size_t)src[u] * a.nss + f);
    };
    auto sum_ss = [&](int r0) {
        float sm[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) sm[u] = lane < n4s ? (sv[u].x + sv[u].y) + (sv[u].z + sv[u].w) : 0.f;
        for (int f0 = 64; f0 < n4s; f0 += 64) {
            load_ss(r0, f0);
#pragma unroll
            for (int u = 0; u < RU; ++u)
                sm[u] += f0 + lane < n4s ? (sv[u].x + sv[u].y) + (sv[u].z + sv[u].w) : 0.f;
        }
        // lane u keeps row u's sum
        float mine = 0.f;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const float x = wave_sum_dpp(sm[u]);
            mine = lane == u ? x : mine;
        }
        if (lane < RU) inv_s[wave * RW + r0 + lane] = rsqrtf(mine / (float)a.K + a.eps);
    };
    if (kFew && stats) load_ss(0, 0);
    load_x(b0);
#pragma unroll
    for (int d = 0; d < WD; ++d)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            load_w(min(b0 + d, b1 - 1), d, kb, 0);
            load_w(min(b0 + d, b1 - 1), d, kb, 1);
        }
    PgPre pre[kFew ? MG : 1][NG / 2];
    if constexpr (kFew)
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int p = 0; p < NG / 2; ++p)
                pre[g][p] = pg_pre<MODE>(a, min(P0 + p, a.pairs - 1), min(m0 + 16 * g + n, M - 1), pos[g], q);
    if (stats) {
        if constexpr (kFew) {
            sum_ss(0);
        } else {
#pragma unroll 1
            for (int r0 = 0; r0 < RW; r0 += RU) {
                load_ss(r0, 0);
                sum_ss(r0);
            }
        }
    } else if (tid < 16 * MG) {
        inv_s[tid] = 1.0f;
    }
    pg_f4 acc[MG][NG];
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int j = 0; j < NG; ++j) acc[g][j] = pg_f4{0.f, 0.f, 0.f, 0.f};
    stage(0);
    __syncthreads();
    auto run = [&](int step, int d) {
        const int buf = (step - b0) & 1;
        load_x(min(step + 1, b1 - 1));
        const char* const lb = sm + buf * kStageB + n * 256;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int ch = 2 * q + h;
                const char* const ph = lb + kb * kBlkB + ((ch ^ n) << 4);
                const char* const pl = lb + kb * kBlkB + (((8 + ch) ^ n) << 4);
#pragma unroll
                for (int g = 0; g < MG; ++g) {
                    const pg_bf8 xh = __builtin_bit_cast(pg_bf8, *(const pg_u4*)(ph + g * 4096));
                    const pg_bf8 xl = __builtin_bit_cast(pg_bf8, *(const pg_u4*)(pl + g * 4096));
#pragma unroll
                    for (int j = 0; j < NG; ++j)
                        acc[g][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(pg_bf8, w[d][kb][h][j]), xh,
                                                                           acc[g][j], 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < NG; ++j)
                        acc[g][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(pg_bf8, w[d][kb][h][j]), xl,
                                                                           acc[g][j], 0, 0, 0);
                }
                load_w(min(step + WD, b1 - 1), d, kb, h);
            }
        stage(buf ^ 1);
        __syncthreads();
    };
    if constexpr (WD == 1) {
        for (int step = b0; step < b1; ++step) run(step, 0);
    } else {
        for (int step = b0; step < b1; step += WD) {
#pragma unroll
            for (int d = 0; d < WD; ++d)
                if (step + d < b1) run(step + d, d);
        }
    }

    if (S > 1) {
        // every range writes its sums through, lane by lane; the last to arrive adds them in range
        // order (see arrive_last)
        const size_t tile = (size_t)nb * nblk_m + mb;
        constexpr int kTile = MG * NG * 4 * 256;  // floats
        float* pt = a.part + tile * S * kTile + (size_t)wave * MG * NG * 256 + lane * 4;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(pt + (size_t)s * kTile - lane * 4, 0, MG * NG * 1024, 0x00027000);
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int j = 0; j < NG; ++j)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(pg_u4, acc[g][j]), rs,
                                                       (g * NG + j) * 1024 + lane * 16, 0, 16 /* sc1 */);
        if (!arrive_last(a.cnt + tile, S, &last_s)) return;
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int j = 0; j < NG; ++j) acc[g][j] = pg_f4{0.f, 0.f, 0.f, 0.f};
        // several ranges' sums per round trip, as many as fit 128 registers (loads past S re-read
        // the last range and are not added)
        constexpr int TB = 32 / (MG * NG);
        for (int t0 = 0; t0 < S; t0 += TB) {
            pg_f4 pv[TB][MG][NG];
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int g = 0; g < MG; ++g)
#pragma unroll
                    for (int j = 0; j < NG; ++j)
                        pv[t][g][j] = pg_ld4(pt + (size_t)min(t0 + t, S - 1) * kTile + (g * NG + j) * 256);
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int g = 0; g < MG; ++g)
#pragma unroll
                    for (int j = 0; j < NG; ++j) acc[g][j] += t0 + t < S ? pv[t][g][j] : pg_f4{0.f, 0.f, 0.f, 0.f};
        }
    }
#pragma unroll
    for (int g = 0; g < MG; ++g) {
        const int row = m0 + 16 * g + n;
        const bool valid = row < M;
        const int rr = min(row, M - 1);
        const float sc = inv_s[16 * g + n];
#pragma unroll
        for (int p = 0; p < NG / 2; ++p)
            if (P0 + p < a.pairs) {
                if constexpr (kFew) {
                    pg_epilogue<MODE>(a, P0 + p, rr, valid, pos[g], q, acc[g][2 * p] * sc, acc[g][2 * p + 1] * sc, pre[g][p]);
                } else {
                    const int ps = MODE == kEpiQkv ? a.row_pos[rr] : 0;
                    pg_epilogue<MODE>(a, P0 + p, rr, valid, ps, q, acc[g][2 * p] * sc, acc[g][2 * p + 1] * sc,
                                      pg_pre<MODE>(a, P0 + p, rr, ps, q));
                }
            }
    }
}

// The same projection for up to 16 rows onto few weight rows and short K: a workgroup owns one pair of
// sub-tiles (32 weight rows) and its four waves take K ranges of it, each streaming weights and
// planes straight into registers, D blocks of 64 columns ahead, with no LDS and no barrier until
// the waves' sums meet in LDS.  Against k_pgemm, whose 128-row blocks need K split over workgroups to
// fill the chip at these sizes, it saves the staging and the hand-off through memory, which are
// most of a launch this short.
template <int MODE>
__global__ __launch_bounds__(256, 2) void k_sgemm(PgArgs a) {
    constexpr int D = 4, WK = 4;
    __shared__ __attribute__((aligned(16))) pg_f4 red[WK][2][64];
    __shared__ float inv_s[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, q = lane >> 4;
    const int P = blockIdx.x;
    const uint16_t* const w0 = pg_row<MODE>(a, P, 0, n) + 16 * q;
    const uint16_t* const w1 = pg_row<MODE>(a, P, 1, n) + 16 * q;
    const int nkb = a.K / kPgBlk, b0 = nkb * wave / WK, b1 = nkb * (wave + 1) / WK;
    const uint16_t* const xp = a.planes + n * kPgBlkWords + 16 * q;
    const size_t xstep = (size_t)a.Mp * kPgBlkWords;
    // statistics first (see k_pgemm): wave w takes rows w, w + WK, ...
    constexpr int RU = 16 / WK;
    const bool stats = MODE != kEpiAdd && a.ss;
    const int n4s = a.nss / 4;
    pg_f4 sv[RU];
    const int row = min(n, a.M - 1);
    const int pos = MODE == kEpiQkv && wave == 0 ? a.row_pos[row] : 0;
    auto load_ss = [&](int f0) {
        const int f = 4 * min(f0 + lane, n4s - 1);
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int r = min(wave + WK * u, a.M - 1);
            const int src = a.in_map ? max(a.in_map[r], 0) : r;
            sv[u] = *(const pg_f4*)(a.ss + (size_t)src * a.nss + f);
        }
    };
    if (stats) load_ss(0);
    pg_u4 w[D][2][2], x[D][2][2];
    auto load = [&](int kb, int d) {
        kb = max(min(kb, b1 - 1), 0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            w[d][h][0] = *(const pg_u4*)(w0 + (size_t)kb * kPgBlk + 8 * h);
            w[d][h][1] = *(const pg_u4*)(w1 + (size_t)kb * kPgBlk + 8 * h);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int p = 0; p < 2; ++p) x[d][h][p] = *(const pg_u4*)(xp + kb * xstep + 8 * h + p * kPgBlk);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(b0 + d, d);
    PgPre pre = {};
    if (wave == 0) pre = pg_pre<MODE>(a, P, row, pos, q);
    if (stats) {
        float sm[RU], mine = 0.f;
#pragma unroll
        for (int u = 0; u < RU; ++u) sm[u] = lane < n4s ? (sv[u].x + sv[u].y) + (sv[u].z + sv[u].w) : 0.f;
        for (int f0 = 64; f0 < n4s; f0 += 64) {
            load_ss(f0);
#pragma unroll
            for (int u = 0; u < RU; ++u)
                sm[u] += f0 + lane < n4s ? (sv[u].x + sv[u].y) + (sv[u].z + sv[u].w) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const float v = wave_sum_dpp(sm[u]);
            mine = lane == u ? v : mine;
        }
        if (lane < RU) inv_s[wave + WK * lane] = rsqrtf(mine / (float)a.K + a.eps);
    } else if (tid < 16) {
        inv_s[tid] = 1.0f;
    }
    pg_f4 acc[2];
    acc[0] = acc[1] = pg_f4{0.f, 0.f, 0.f, 0.f};
    for (int kb = b0; kb < b1; kb += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (kb + d < b1) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(pg_bf8, w[d][h][j]),
                                                                            __builtin_bit_cast(pg_bf8, x[d][h][p]),
                                                                            acc[j], 0, 0, 0);
            }
            if (kb + D < b1) load(kb + D + d, d);
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) red[wave][j][lane] = acc[j];
    __syncthreads();
    if (wave != 0) return;
    pg_f4 v[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) v[j] = (red[0][j][lane] + red[1][j][lane]) + (red[2][j][lane] + red[3][j][lane]);
    const float sc = inv_s[n];
    pg_epilogue<MODE>(a, P, row, n < a.M, pos, q, v[0] * sc, v[1] * sc, pre);
}

// Shapes from a sweep of tiles and splits over 8 to 2048 rows at the 8B, 70B and drafter widths
// (weights cycled through more than the last-level cache; loads as compiled, see above).  MG: the fewest row groups that hold
// the rows, up to 128 rows, so that the weights are read once.  NG 4 (128 x 256) halves the LDS
// reads per product and wins wherever its grid fills the chip (512 rows of gate|up 8B: 209 us
// against 269 with NG 2), or K is long enough to split (1024 rows of down: 225 against 252);
// below that its few blocks and their large partials lose (512 rows of down: 176 against 135).
// 64-row blocks take short K with few columns, where even split 128-row blocks leave workgroups
// idle (128 rows of O 8B: 28 against 34 us); with up to 64 rows they take NG 4 where that leaves
// enough blocks (36 rows of gate|up 8B: 63 against 70 us, 70B 208 against 226, of a vocabulary 392
// against 478).  S: up to two workgroups per CU, one with up to 32
// rows (24 rows of gate|up: 55 us unsplit, 60 with S 2; of Q|K|V: 19 with S 4, 23 with S 8).
PgPlan pg_plan(int M, int N, int K, bool packed, size_t room) {
    PgPlan p{};
    const int rows = pg_rows(M);
    auto blocks = [&](int mg, int ng) { return ((rows + 16 * mg - 1) / (16 * mg)) * ((N + 64 * ng - 1) / (64 * ng)); };
    p.NG = 2;
    if (rows <= 32 && K % 256 == 0) {
        p.MG = rows <= 16 ? 1 : 2;
        // k_sgemm where K is short and the pairs do not outnumber the two workgroups per CU: 16 rows
        // onto 3072 x 2048 in 9.8 us against 11.2, 16384 x 2048 in 18.0 against 19.3, 768 x 768 in
        // 6.0; longer K streams from too few workgroups (2048 x 8192: 31 us against 15.6)
        p.skinny = !packed && rows <= 16 && K <= 2048 && N <= 16384;
        if (p.skinny) return p;
    } else if (rows <= 64 || blocks(8, 2) * (K / 512) < 512) {
        p.MG = 4;
        if (rows <= 64 && blocks(4, 4) >= 96) p.NG = 4;
    } else {
        p.MG = 8;
        if (blocks(8, 4) >= 384 || (K >= 8192 && blocks(8, 4) >= 128)) p.NG = 4;
    }
    p.nblk_m = (rows + 16 * p.MG - 1) / (16 * p.MG);
    p.nblk_n = (N + 64 * p.NG - 1) / (64 * p.NG);
    const int nb = p.nblk_m * p.nblk_n, tile = p.MG * p.NG * 1024;
    p.units = (int)std::min<size_t>(room / tile, kPgUnits);
    p.S = pg_ranges(nb, p.MG, K, p.units);
    p.grid = 8 * p.nblk_m * ((p.nblk_n + 7) / 8) * p.S;
    if (packed) {
        // the most any number of row blocks asks for
        int part = 0;
        p.S = 1;
        for (int m = 1; m <= p.nblk_m; ++m) {
            const int S = pg_ranges(m * p.nblk_n, p.MG, K, p.units);
            p.grid = std::max(p.grid, 8 * m * ((p.nblk_n + 7) / 8) * S);
            p.S = std::max(p.S, S);
            if (S > 1) part = std::max(part, m * p.nblk_n * S);
        }
        p.part = (size_t)part * tile;
        return p;
    }
    p.part = p.S > 1 ? (size_t)nb * p.S * tile : 0;
    return p;
}

static void sg_launch(hipStream_t s, ProfEntry* pe, int mode, const PgArgs& a) {
    const dim3 grid(a.pairs), blk(256);
    hipEvent_t ea = pe ? pe->a : nullptr, eb = pe ? pe->b : nullptr;
    if (mode == kEpiStore) hipExtLaunchKernelGGL((k_sgemm<kEpiStore>), grid, blk, 0, s, ea, eb, 0, a);
    else if (mode == kEpiAdd) hipExtLaunchKernelGGL((k_sgemm<kEpiAdd>), grid, blk, 0, s, ea, eb, 0, a);
    else if (mode == kEpiSwiglu) hipExtLaunchKernelGGL((k_sgemm<kEpiSwiglu>), grid, blk, 0, s, ea, eb, 0, a);
    else hipExtLaunchKernelGGL((k_sgemm<kEpiQkv>), grid, blk, 0, s, ea, eb, 0, a);
}

template <int MG, int NG, int KB, int WD>
static void pg_launch(hipStream_t s, ProfEntry* pe, int mode, dim3 grid, const PgArgs& a) {
    const dim3 blk(256);
    hipEvent_t ea = pe ? pe->a : nullptr, eb = pe ? pe->b : nullptr;
    if (mode == kEpiStore) hipExtLaunchKernelGGL((k_pgemm<MG, NG, KB, WD, kEpiStore>), grid, blk, 0, s, ea, eb, 0, a);
    else if (mode == kEpiAdd) hipExtLaunchKernelGGL((k_pgemm<MG, NG, KB, WD, kEpiAdd>), grid, blk, 0, s, ea, eb, 0, a);
    else if (mode == kEpiSwiglu) hipExtLaunchKernelGGL((k_pgemm<MG, NG, KB, WD, kEpiSwiglu>), grid, blk, 0, s, ea, eb, 0, a);
    else hipExtLaunchKernelGGL((k_pgemm<MG, NG, KB, WD, kEpiQkv>), grid, blk, 0, s, ea, eb, 0, a);
}

bool launch_pgemm(Engine* e, hipStream_t s, const WsCall& c) {
    Workspace& ws = e->ws;
    if (c.K % 128 || (c.nseg != 1 && c.mode != kEpiQkv && c.mode != kEpiSwiglu)) return false;
    PgArgs a{};
    a.M = c.M; a.Mp = pg_rows(c.M); a.K = c.K;
    a.planes = c.planes;
    if (!a.planes) {
        // the MLP's planes are free outside a layer
        if (c.M > e->maxm || pg_plane_bytes(c.M, c.K) > ws.ffh_n) return false;
        PlaneArgs x{};
        x.X = c.X; x.in_map = c.in_map; x.Mp = a.Mp; x.K = c.K; x.gamma = (const uint16_t*)c.gamma;
        x.planes = (uint16_t*)ws.ffh;
        prof_begin(e, kProfOther, 0.0);
        k_planes<<<dim3(c.M, (c.K + kPlaneCols - 1) / kPlaneCols), 256, 0, s>>>(x);
        prof_end(e);
        a.planes = x.planes;
    }
    if (c.gamma) {
        a.ss = c.ss; a.in_map = c.in_map; a.nss = c.nss; a.eps = c.eps;
    }
    int N = 0;
    for (int i = 0; i < 3; ++i) {
        a.W[i] = i < c.nseg ? (const uint16_t*)c.W[i] : nullptr;
        if (i < c.nseg) N += c.seg_rows[i];
    }
    const PgPlan p = pg_plan(c.M, N, c.K, c.m_live != nullptr, ws.ws_part_n);
    a.m_live = c.m_live; a.units = p.units;
    a.S = p.S; a.nblk_m = p.nblk_m; a.nblk_n = p.nblk_n;
    a.nbs = 8 * p.nblk_m * ((p.nblk_n + 7) / 8);
    if (c.mode == kEpiSwiglu) {
        a.pairs = a.tiles = c.seg_rows[0] / 16;
    } else {
        a.tiles = N / 16;
        a.pairs = (a.tiles + 1) / 2;
    }
    if (c.mode == kEpiQkv) {
        a.seg_pairs[0] = c.seg_rows[0] / 32;
        a.seg_pairs[1] = c.seg_rows[1] / 32;
    }
    a.Y = c.Y; a.ldy = c.ldy; a.out_map = c.out_map; a.ss_out = c.ss_out;
    a.yplanes = c.yplanes; a.ygamma = (const uint16_t*)c.ygamma; a.part = c.part; a.cnt = c.cnt;
    a.H = c.H; a.Hkv = c.Hkv; a.hd = c.hd; a.row_pos = c.row_pos; a.row_seq = c.row_seq;
    a.rcos = c.rcos; a.rsin = c.rsin; a.qout = c.qout; a.kc = c.kc; a.vc = c.vc;
    a.cap = c.cap; a.max_batch = c.max_batch; a.layer = c.layer; a.ubias = c.ubias; a.ub_ld = c.ub_ld;
    ProfEntry* pe = prof_slot(e, kProfGemv, (double)N * c.K * 2.0 + (double)c.M * c.K * 4.0 + (double)c.M * N * 4.0);
    if (p.skinny) sg_launch(s, pe, c.mode, a);
    else if (p.MG == 1) pg_launch<1, 2, 4, 1>(s, pe, c.mode, dim3(p.grid), a);
    else if (p.MG == 2) pg_launch<2, 2, 4, 1>(s, pe, c.mode, dim3(p.grid), a);
    else if (p.MG == 4 && p.NG == 4) pg_launch<4, 4, 1, 2>(s, pe, c.mode, dim3(p.grid), a);
    else if (p.MG == 4) pg_launch<4, 2, 2, 2>(s, pe, c.mode, dim3(p.grid), a);
    else if (p.NG == 2) pg_launch<8, 2, 1, 2>(s, pe, c.mode, dim3(p.grid), a);
    else pg_launch<8, 4, 1, 1>(s, pe, c.mode, dim3(p.grid), a);
    if (pe) prof_commit(e);
    return true;
}

}  // namespace sd2
