// Grouped-query causal attention over the fp32 KV cache for a block of query rows per sequence:
// k_vattn for few rows (decode steps, verify passes), k_pattn for many (prefill chunks, the
// training objective).  Both split the cache positions of a group over workgroups where that fills
// the chip (every span writes an un-normalised output, max and sum, and the last one to arrive
// merges them in span order, see arrive_last).  The causal mask is key position <= query position;
// rows with position -1 are inactive and produce zeros.
#include <math.h>

#include <algorithm>

#include <hip/hip_ext.h>

#include "attn_part.h"
#include "device_common.h"
#include "engine.h"
#include "pgemm.h"

namespace sd2 {

constexpr int kSplit = 128;   // cache positions of the smallest span: the partials have room for spans of these

struct AttnArgs {
    const float* q;
    int q_stride;
    const float *kc, *vc;
    float* out;
    uint16_t* planes;  // output as planes of Mp rows (see pgemm.hip), in place of out; or null
    int Mp;
    const int32_t* row_pos;
    const int32_t* row_off;  // packed rows: first row of every sequence (its rows: up to the next one's), or null
    int rps, H, Hkv, hd, cap, max_batch, layer;
    int nseq;   // sequences
    float scale;
    float* part;     // partials of the spans (see attn_part.h)
    int32_t* cnt;    // one arrival counter per workgroup of the split-free grid
};

// First row and number of rows of sequence b.
__device__ __forceinline__ int attn_rows(const AttnArgs& a, int b, int& n) {
    n = a.row_off ? a.row_off[b + 1] - a.row_off[b] : a.rps;
    return a.row_off ? a.row_off[b] : b * a.rps;
}

// One output value, or four neighbouring ones: column c of row `row`.
__device__ __forceinline__ void attn_put1(const AttnArgs& a, size_t row, int c, float v) {
    if (a.planes) pg_put1(a.planes, a.Mp, row, c, v);
    else a.out[row * a.H * a.hd + c] = v;
}
__device__ __forceinline__ void attn_put4(const AttnArgs& a, size_t row, int c, float4 v) {
    if (a.planes) pg_put4(a.planes, a.Mp, row, c, v);
    else *(float4*)(a.out + row * a.H * a.hd + c) = v;
}

// ---------------------------------------------------------------------------------------------
// Blocks of many rows per sequence (prefill chunks, the
// training-objective forward): causal flash attention on fp32 matrix cores.  A workgroup owns
// 16 consecutive query rows of one sequence, one KV head and one span of key tiles; each of its
// 4 waves takes the query heads wave, wave + 4, ... of that KV head.  Per 16-position key tile,
// K and V are staged in LDS once for all the group's heads (the next tile is requested into
// registers while the current one is used).  A wave computes the transposed products, with
// v_mfma_f32_16x16x4_f32 (fp32 operands keep the cache's precision):
//   S^T = K Q^T   (16 keys x 16 queries; the head dimension walked as dim = g * HD/4 + s for
//                  lane group g and step s, so a lane's K operands are HD/4 adjacent floats)
//   O^T += V^T P^T (HD/16 tiles; output dim = i * HD/16 + t for tile row i and tile t, so a
//                  lane's V operands are HD/16 adjacent floats per key)
// In the result layout of S^T a lane holds four keys of one query (its column), which is also
// the layout P^T needs as an operand and the layout of that query's O^T rows: the online softmax
// runs in registers, with its max and sum taken over the four lane groups of a column by two
// lane-swap steps, and P never goes through LDS.  With few (sequence, KV head, row block)
// groups the keys are split into at most 16 spans of span_t tiles (about eight workgroups per
// compute unit): every span writes an un-normalised partial and
// the last span of a group to arrive merges them in span order, all spans' loads at once.
// ---------------------------------------------------------------------------------------------
constexpr int kPaQ = 16;                  // query rows per workgroup
constexpr int kPaK = 16;                  // key positions per tile
constexpr int kPaMaxSpans = 16;           // spans per group (one merge batch)
typedef float pf4 __attribute__((ext_vector_type(4)));
typedef float pf2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4_t __attribute__((ext_vector_type(4)));

// Max and sum over the four 16-lane groups of a wave (lanes l, l^16, l^32, l^48 hold one column).
__device__ __forceinline__ float pa_colmax(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float pa_colsum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The last span of a (sequence, KV head, row block) group to finish merges the live spans in
// span order: a thread per (row, head, 4 dimensions), every span's (max, sum) and output
// requested at once.  qpos holds the block's row positions (-1: no row).
template <int HD>
__device__ void pa_span_merge(const AttnArgs& a, int grp_id, int nspan, int span_t, int ntile_all, int b, int kvh,
                              int i0, int rbase, int nrows, const int* qpos, int* last_flag) {
    if (!arrive_last(a.cnt + grp_id, nspan, last_flag)) return;
    const int tid = threadIdx.x, G = a.H / a.Hkv;
    const int nlive = min(nspan, ntile_all > 0 ? (ntile_all - 1) / span_t + 1 : 0);
    constexpr int D4 = HD / 4;
    for (int idx = tid; idx < kPaQ * G * D4; idx += 256) {
        const int i = idx / (G * D4), hh = (idx / D4) % G, d = (idx % D4) * 4;
        const int row = i0 + i;
        if (row >= nrows) continue;
        const size_t orow = (size_t)(rbase + row);
        const int h = kvh * G + hh;
        float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
        if (qpos[i] >= 0 && nlive > 0) {
            float m2[kPaMaxSpans], l2[kPaMaxSpans];
            float4 o2[kPaMaxSpans];
#pragma unroll
            for (int s2 = 0; s2 < kPaMaxSpans; ++s2) {
                const int sp = min(s2, nlive - 1);
                const pf2 ml = *(const pf2*)(a.part + part_ml((size_t)a.nseq * a.rps, a.H, HD, grp_id * G + hh, nspan, sp, i));
                m2[s2] = ml[0];
                l2[s2] = ml[1];
                o2[s2] = *(const float4*)(a.part + part_out(orow, a.H, h, nspan, sp, HD) + d);
            }
            float M = -INFINITY;
#pragma unroll
            for (int s2 = 0; s2 < kPaMaxSpans; ++s2) M = s2 < nlive ? fmaxf(M, m2[s2]) : M;
            float L = 0.f;
#pragma unroll
            for (int s2 = 0; s2 < kPaMaxSpans; ++s2) {
                const float w = (s2 < nlive && m2[s2] != -INFINITY) ? expf(m2[s2] - M) : 0.f;
                L += w * l2[s2];
                res.x += w * o2[s2].x;
                res.y += w * o2[s2].y;
                res.z += w * o2[s2].z;
                res.w += w * o2[s2].w;
            }
            const float inv = L > 0.f ? 1.f / L : 0.f;
            res = make_float4(res.x * inv, res.y * inv, res.z * inv, res.w * inv);
        }
        attn_put4(a, orow, h * HD + d, res);
    }
}

template <int HD>
__global__ __launch_bounds__(256) void k_pattn(AttnArgs a, int nspan, int span_t) {
    constexpr int KL = HD + 4;                            // padded LDS row of K and V
    constexpr int F4 = (kPaK * HD / 4 + 255) / 256;       // float4 of a K (or V) tile per thread
    constexpr int QD = HD / 4;                            // head dims per lane group in S^T
    constexpr int VD = HD / 16;                           // output dims per lane and key in O^T
    static_assert(QD % 4 == 0 && (VD % 4 == 0 || VD == 2), "head dim");
    __shared__ __attribute__((aligned(16))) float ks[kPaK * KL];
    __shared__ __attribute__((aligned(16))) float vs[kPaK * KL];
    __shared__ __attribute__((aligned(16))) float ot[4 * kPaQ * KL];  // per wave: O rows of one head
    __shared__ int qpos[kPaQ];
    __shared__ int maxpos_s;
    __shared__ int last_flag;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int G = a.H / a.Hkv;
    const int nqb = (a.rps + kPaQ - 1) / kPaQ;
    const int grp_id = blockIdx.x / nspan, sp = blockIdx.x % nspan;
    const int qb = grp_id % nqb;
    const int kvh = (grp_id / nqb) % a.Hkv;
    const int b = grp_id / (nqb * a.Hkv);
    const int i0 = qb * kPaQ;
    int nrows;
    const int rbase = attn_rows(a, b, nrows);
    if (i0 >= nrows) return;  // (uniform)
    if (tid == 0) maxpos_s = -1;
    __syncthreads();
    if (tid < kPaQ) {
        int p = -1;
        if (i0 + tid < nrows) p = a.row_pos[rbase + i0 + tid];
        qpos[tid] = p;
        if (p >= 0) atomicMax(&maxpos_s, p);
    }
    __syncthreads();
    const int maxpos = maxpos_s;
    const int ntile_all = maxpos >= 0 ? maxpos / kPaK + 1 : 0;
    // this workgroup's key tiles: all of them, or one span
    const int t0 = nspan == 1 ? 0 : sp * span_t;
    const int t1 = nspan == 1 ? ntile_all : min(ntile_all, t0 + span_t);
    const size_t kvoff = (((size_t)a.layer * a.max_batch + b) * a.Hkv + kvh) * (size_t)a.cap * HD;
    const float* kg = a.kc + kvoff;
    const float* vg = a.vc + kvoff;
    const int col = lane & 15, grp = lane >> 4;  // MFMA layouts: column / row-group of this lane
    const int myq = qpos[col];                    // position of this lane's query row (-1: none)
    auto fetch = [&](int kt, float4 (&pk)[F4], float4 (&pv)[F4]) {
#pragma unroll
        for (int i = 0; i < F4; ++i) {
            const int e4 = tid + 256 * i;
            const int j = (e4 * 4) / HD, d = (e4 * 4) % HD, pos = kt * kPaK + j;
            pk[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            pv[i] = pk[i];
            if (e4 < kPaK * HD / 4 && pos <= maxpos) {
                pk[i] = *(const float4*)(kg + (size_t)pos * HD + d);
                pv[i] = *(const float4*)(vg + (size_t)pos * HD + d);
            }
        }
    };
    for (int hp = 0; hp * 4 < G; ++hp) {
        const int hh = hp * 4 + wave;
        const bool active = hh < G && t0 < t1;
        const int h = kvh * G + (hh < G ? hh : 0);
        // Q as the B operand of S^T: lane holds Q[row col][grp * QD + s], pre-scaled (rows past
        // the block re-read row 0 and are zeroed by the scale: no load depends on a branch,
        // which would cost one memory round trip per load)
        float qf[QD];
        {
            const int qrow = i0 + col;
            const bool ok = qrow < nrows;
            const float* qp = a.q + (size_t)(rbase + (ok ? qrow : 0)) * a.q_stride + h * HD + grp * QD;
            const float qs = ok ? a.scale : 0.f;
#pragma unroll
            for (int s = 0; s < QD; s += 4) {
                const pf4 x = *(const pf4*)(qp + s) * qs;
                qf[s] = x[0]; qf[s + 1] = x[1]; qf[s + 2] = x[2]; qf[s + 3] = x[3];
            }
        }
        pf4 o[VD];  // o[t][r] = O[query col][(4 grp + r) * VD + t]
#pragma unroll
        for (int t = 0; t < VD; ++t) o[t] = pf4{0.f, 0.f, 0.f, 0.f};
        float m_run = -INFINITY, l_run = 0.f;
        float4 pk[F4], pv[F4];
        if (t0 < t1) fetch(t0, pk, pv);
        for (int kt = t0; kt < t1; ++kt) {
            // stage this tile's K and V rows (positions past maxpos are zeros), request the next
            __syncthreads();
#pragma unroll
            for (int i = 0; i < F4; ++i) {
                const int e4 = tid + 256 * i;
                if (e4 < kPaK * HD / 4) {
                    const int j = (e4 * 4) / HD, d = (e4 * 4) % HD;
                    *(float4*)(ks + j * KL + d) = pk[i];
                    *(float4*)(vs + j * KL + d) = pv[i];
                }
            }
            __syncthreads();
            if (kt + 1 < t1) fetch(kt + 1, pk, pv);
            if (!active) continue;
            // operands from LDS, all requested before the first product: K[key col][grp*QD + s]
            // and V[key 4 grp + r][col * VD + t]
            float kf[QD], vf[4][VD];
#pragma unroll
            for (int s = 0; s < QD; s += 4) {
                const pf4 x = *(const pf4*)(ks + col * KL + grp * QD + s);
                kf[s] = x[0]; kf[s + 1] = x[1]; kf[s + 2] = x[2]; kf[s + 3] = x[3];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float* vr = vs + (4 * grp + r) * KL + col * VD;
                if constexpr (VD == 2) {
                    const pf2 x = *(const pf2*)vr;
                    vf[r][0] = x[0]; vf[r][1] = x[1];
                } else {
#pragma unroll
                    for (int t = 0; t < VD; t += 4) {
                        const pf4 x = *(const pf4*)(vr + t);
                        vf[r][t] = x[0]; vf[r][t + 1] = x[1]; vf[r][t + 2] = x[2]; vf[r][t + 3] = x[3];
                    }
                }
            }
            // S^T = K Q^T in four independent accumulation chains; this lane then holds
            // S[query col][key 4 grp + r]
            pf4 sc4[4];
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) sc4[c4] = pf4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < QD; ++s)
                sc4[s & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s], qf[s], sc4[s & 3], 0, 0, 0);
            const pf4 sc = (sc4[0] + sc4[1]) + (sc4[2] + sc4[3]);
            // online softmax of query col over this tile's 16 keys
            const int kb = kt * kPaK + 4 * grp;
            float sv[4], mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sv[r] = (myq >= 0 && kb + r <= myq) ? sc[r] : -INFINITY;
                mx = fmaxf(mx, sv[r]);
            }
            mx = pa_colmax(mx);
            const float mnew = fmaxf(m_run, mx);
            float pr[4], sum = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                pr[r] = sv[r] == -INFINITY ? 0.f : expf(sv[r] - mnew);
                sum += pr[r];
            }
            sum = pa_colsum(sum);
            const float scl = m_run == -INFINITY ? 0.f : expf(m_run - mnew);
            l_run = l_run * scl + sum;
            m_run = mnew;
#pragma unroll
            for (int t = 0; t < VD; ++t) o[t] *= scl;
            // O^T += V^T P^T: step r pairs key 4 grp + r with this lane's k slot
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < VD; ++t)
                    o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][t], pr[r], o[t], 0, 0, 0);
        }
        // O through LDS into row-major order, then whole rows stored by the wave (a lane's own
        // values belong to one row: stored directly, each store would touch 16 rows)
        if (hh < G) {
            float* ow = ot + wave * (kPaQ * KL);
            const float inv = nspan == 1 ? ((myq >= 0 && l_run > 0.f) ? 1.f / l_run : 0.f) : 1.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* dst = ow + col * KL + (4 * grp + r) * VD;
                if constexpr (VD == 2) {
                    *(pf2*)dst = pf2{o[0][r] * inv, o[1][r] * inv};
                } else {
#pragma unroll
                    for (int t = 0; t < VD; t += 4)
                        *(pf4*)(dst + t) = pf4{o[t][r] * inv, o[t + 1][r] * inv, o[t + 2][r] * inv, o[t + 3][r] * inv};
                }
            }
            if (nspan > 1 && grp == 0 && i0 + col < nrows) {
                // this span's max and sum of the lane's row
                float* pp = a.part + part_ml((size_t)a.nseq * a.rps, a.H, HD, grp_id * G + hh, nspan, sp, col);
                store_through(pp, m_run);
                store_through(pp + 1, l_run);
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's rows are in LDS
            __builtin_amdgcn_wave_barrier();
            constexpr int RW = (HD + 63) / 64;  // values of one row per lane
            float rv[kPaQ][RW];                   // every row read before any is stored
#pragma unroll
            for (int i = 0; i < kPaQ; ++i)
#pragma unroll
                for (int j = 0; j < RW; ++j) rv[i][j] = ow[i * KL + min(lane + 64 * j, HD - 1)];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < kPaQ; ++i) {
                const size_t orow = (size_t)(rbase + i0 + i);
#pragma unroll
                for (int j = 0; j < RW; ++j) {
                    const int d = lane + 64 * j;
                    if (i0 + i < nrows && d < HD) {
                        if (nspan == 1) attn_put1(a, orow, h * HD + d, rv[i][j]);
                        else store_through(a.part + part_out(orow, a.H, h, nspan, sp, HD) + d, rv[i][j]);
                    }
                }
            }
        }
    }
    if (nspan == 1) return;
    pa_span_merge<HD>(a, grp_id, nspan, span_t, ntile_all, b, kvh, i0, rbase, nrows, qpos, &last_flag);
}

// ---------------------------------------------------------------------------------------------
// Blocks of fewer than 16 rows per sequence (decode steps, verify passes): flash attention on fp32
// matrix cores over packed query vectors.  The rps x G vectors (row, query head) of a sequence
// and KV head fill the 16 query columns of the products without gaps (rows alone would leave
// 16 - rps of them empty for every head); a workgroup owns up to 16 of them and one span of key
// tiles, and its 4 waves take the span's 16-key tiles in turn.  (Two column tiles per wave read K and V
// once for 32 vectors but measured slower at every shape: 77 against 72 us for 16 sequences of 8
// rows, 48 against 43 at the 70B shape; the second workgroup finds them in its XCD's L2.)
//
// A wave reads K and V from memory straight in the operand layout, with no LDS and no barrier in
// the key loop: S^T = K Q^T walks the head dimension as dim = 16 s4 + 4 g + e (lane group g, step
// 4 s4 + e), so that the four lanes of a key read 64 adjacent bytes per load, and O^T += V^T P^T
// numbers the output dims as 64 t4 + 4 i + e (tile row i, tile 4 t4 + e), so that the 16 lanes of
// a key read 256.  The online softmax stays in registers (see k_pattn); the waves' sums are merged
// through LDS, and the last live span of a group to arrive merges the spans.
//
// Bound: a tile's chain of loads, products and softmax.  The loop names a wave's next tile before it
// uses the current one, but nothing in it writes memory, and the compiler sinks the loads to their
// uses: at head dim 128 a tile's 16 loads are waited for one or two at a time among its 64 products
// (145 VGPRs; two tiles, the queries and the outputs would need 192).
// 4 sequences of 6 rows at 201 to 901 positions, 32/8 heads, head dim 128: 18 us (115 with the vector
// kernel before); 16 of 8 rows at 256 to 2048: 61 us (80 with two heads per tile staged through LDS).
// ---------------------------------------------------------------------------------------------
constexpr int kVaMinTiles = 8;  // key tiles per span: two per wave

template <int HD>
__global__ __launch_bounds__(256, 2) void k_vattn(AttnArgs a, int ncg, int nspan, int span_t) {
    constexpr int QD = HD / 4;                  // S^T steps: head dims per lane group
    constexpr int VD = HD / 16;                 // O^T tiles
    constexpr int VV = VD < 4 ? VD : 4;         // V values per load
    constexpr int NO = VD * 4 / VV;             // groups of VV adjacent output dims per lane
    typedef float vv_t __attribute__((ext_vector_type(VV)));
    __shared__ __attribute__((aligned(16))) float os[4][NO][64 * VV];
    __shared__ float ms[4][16], ls[4][16];
    __shared__ int last_flag;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int G = a.H / a.Hkv;
    // the column groups of one span, which read the same K/V, are 8 workgroups apart: on one XCD
    const int c8 = blockIdx.x / 8, cg = c8 % ncg;
    const int u = (c8 / ncg) * 8 + blockIdx.x % 8;
    // spans in the outer order: in the inner one a span count that is a multiple of 8 put the live
    // (first) spans of every group on the same few XCDs (4 sequences of 6 rows: 34 against 22 us)
    const int groups = a.nseq * a.Hkv, sp = u / groups, kvh = u % a.Hkv, b = (u % groups) / a.Hkv;
    if (sp >= nspan) return;  // grid padding
    int nrows;
    const int rbase = attn_rows(a, b, nrows), nv = nrows * G;
    // this lane's query vector and its position
    const int v = cg * 16 + col;
    const bool vok = v < nv;
    const int vrow = rbase + (vok ? v / G : 0), h = kvh * G + (vok ? v % G : 0);
    const int vpos = vok ? a.row_pos[vrow] : -1;
    int maxpos = vpos;
    const float* const qp = a.q + (size_t)vrow * a.q_stride + (size_t)h * HD + 4 * grp;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) maxpos = max(maxpos, __shfl_xor(maxpos, o, 16));
    maxpos = __builtin_amdgcn_readfirstlane(maxpos);
    const int ntile = maxpos >= 0 ? maxpos / 16 + 1 : 0;
    const int nlive = max(1, (ntile + span_t - 1) / span_t);  // spans that count in (one writes zeros)
    if (sp >= nlive) return;
    const int t0 = sp * span_t + wave, t1 = min(ntile, (sp + 1) * span_t);
    const size_t kvoff = (((size_t)a.layer * a.max_batch + b) * a.Hkv + kvh) * (size_t)a.cap * HD;
    const float* kg = a.kc + kvoff + 4 * grp;
    const float* vg = a.vc + kvoff + VV * col;
    struct Tile {
        pf4 k[QD / 4];
        vv_t v[4][VD / VV];
    };
    // positions past the last one re-read it (masked in the scores)
    auto load = [&](int kt, Tile& x) {
        const float* p = kg + (size_t)min(kt * 16 + col, maxpos) * HD;
#pragma unroll
        for (int s = 0; s < QD / 4; ++s) x.k[s] = *(const pf4*)(p + 16 * s);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float* pv = vg + (size_t)min(kt * 16 + 4 * grp + r, maxpos) * HD;
#pragma unroll
            for (int t = 0; t < VD / VV; ++t) x.v[r][t] = *(const vv_t*)(pv + 16 * VV * t);
        }
    };
    pf4 qf[QD / 4];
#pragma unroll
    for (int s = 0; s < QD / 4; ++s) qf[s] = *(const pf4*)(qp + 16 * s);
    Tile ta, tb;
    if (t0 < t1) load(t0, ta);
    const float qs = vok ? a.scale : 0.f;
#pragma unroll
    for (int s = 0; s < QD / 4; ++s) qf[s] *= qs;
    pf4 o[VD];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int d = 0; d < VD; ++d) o[d] = pf4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int kt, const Tile& x) {
        pf4 sc[2] = {pf4{0.f, 0.f, 0.f, 0.f}, pf4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < QD; ++s)
            sc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[s / 4][s % 4], qf[s / 4][s % 4], sc[s & 1], 0, 0, 0);
        // online softmax: this lane holds S[its query][key 4 grp + r]
        const int kb = kt * 16 + 4 * grp;
        float sv[4], pr[4], mx = -INFINITY, sum = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sv[r] = kb + r <= vpos ? sc[0][r] + sc[1][r] : -INFINITY;
            mx = fmaxf(mx, sv[r]);
        }
        mx = pa_colmax(mx);
        const float mnew = fmaxf(m_run, mx);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            pr[r] = sv[r] == -INFINITY ? 0.f : expf(sv[r] - mnew);
            sum += pr[r];
        }
        const float scl = m_run == -INFINITY ? 0.f : expf(m_run - mnew);
        l_run = l_run * scl + pa_colsum(sum);
        m_run = mnew;
#pragma unroll
        for (int d = 0; d < VD; ++d) o[d] *= scl;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int d = 0; d < VD; ++d)
                o[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[r][d / VV][d % VV], pr[r], o[d], 0, 0, 0);
    };
    // (past the last tile the current one is requested again: no branch around the loads)
    for (int kt = t0; kt < t1; kt += 8) {
        load(kt + 4 < t1 ? kt + 4 : kt, tb);
        step(kt, ta);
        if (kt + 4 >= t1) break;
        load(kt + 8 < t1 ? kt + 8 : kt, ta);
        step(kt + 4, tb);
    }
    // merge the waves: group i = (t4, r) of a lane is VV adjacent dims, 16 VV t4 + VV (4 grp + r), of
    // its query vector
#pragma unroll
    for (int t4 = 0; t4 < VD / VV; ++t4)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            vv_t x;
#pragma unroll
            for (int e = 0; e < VV; ++e) x[e] = o[VV * t4 + e][r];
            *(vv_t*)&os[wave][t4 * 4 + r][lane * VV] = x;
        }
    if (grp == 0) {
        ms[wave][col] = m_run;
        ls[wave][col] = l_run;
    }
    __syncthreads();
    // spans: outputs and (max, sum) pairs (see attn_part.h)
    const int rows = a.nseq * a.rps, block = (b * a.Hkv + kvh) * ncg + cg;
    const size_t ph0 = part_out(rbase, a.H, 0, nspan, 0, HD);  // the sequence's first
    const __amdgpu_buffer_rsrc_t prs =
        __builtin_amdgcn_make_buffer_rsrc(a.part + ph0, 0, nrows * a.H * nspan * HD * 4, 0x00027000);
    float w[4], M = -INFINITY, L = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) M = fmaxf(M, ms[k][col]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float m = ms[k][col];
        w[k] = m == -INFINITY ? 0.f : expf(m - M);
        L += w[k] * ls[k][col];
    }
    const float inv = nlive == 1 ? (L > 0.f ? 1.f / L : 0.f) : 1.f;
    const size_t ph = part_out(vrow, a.H, h, nspan, sp, HD);
#pragma unroll
    for (int i0 = 0; i0 < NO; i0 += 4) {
        const int i = i0 + wave;
        vv_t x = {};
#pragma unroll
        for (int k = 0; k < 4; ++k) x += *(const vv_t*)&os[k][i][lane * VV] * w[k];
        x *= inv;
        if (!vok) continue;
        const int d = 16 * VV * (i / 4) + VV * (4 * grp + i % 4);
        if (nlive == 1) {
            if constexpr (VV == 4) {
                attn_put4(a, vrow, h * HD + d, make_float4(x[0], x[1], x[2], x[3]));
            } else {
#pragma unroll
                for (int e = 0; e < VV; ++e) attn_put1(a, vrow, h * HD + d + e, x[e]);
            }
        } else if constexpr (VV == 4) {
            // (one 16-byte write-through store)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, x), prs, (int)((ph - ph0 + d) * 4), 0, 16);
        } else {
#pragma unroll
            for (int e = 0; e < VV; ++e) store_through(a.part + ph + d + e, x[e]);
        }
    }
    if (nlive > 1 && vok && grp == 0 && wave == 0) {
        float* const pml = a.part + part_ml(rows, a.H, HD, block, nspan, sp, col);
        store_through(pml, M);
        store_through(pml + 1, L);
    }
    if (nlive == 1) return;
    if (!arrive_last(a.cnt + block, nlive, &last_flag)) return;
    // the last live span merges: a thread per (vector, 4 dims), spans eight per round trip (loads
    // past the last live span re-read it and are not added)
    constexpr int D4 = HD / 4;
    for (int idx = tid; idx < 16 * D4; idx += 256) {
        const int v = cg * 16 + idx / D4, d = (idx % D4) * 4;
        if (v >= nv) break;
        const int h = kvh * G + v % G;
        const size_t row = (size_t)rbase + v / G;
        float M = -INFINITY, L = 0.f;
        pf4 O = {0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < nlive; s0 += 8) {
            pf4 ov[8];
            pf2 ml[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int s2 = min(s0 + k, nlive - 1);
                ov[k] = *(const pf4*)(a.part + part_out(row, a.H, h, nspan, s2, HD) + d);
                ml[k] = *(const pf2*)(a.part + part_ml(rows, a.H, HD, block, nspan, s2, idx / D4));
            }
            float Mn = M;
#pragma unroll
            for (int k = 0; k < 8; ++k) Mn = s0 + k < nlive ? fmaxf(Mn, ml[k][0]) : Mn;
            const float sc = M == -INFINITY ? 0.f : expf(M - Mn);
            L *= sc;
            O *= sc;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float w = s0 + k < nlive && ml[k][0] != -INFINITY ? expf(ml[k][0] - Mn) : 0.f;
                L += w * ml[k][1];
                O += ov[k] * w;
            }
            M = Mn;
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;
        O *= inv;
        attn_put4(a, row, h * HD + d, make_float4(O[0], O[1], O[2], O[3]));
    }
}

template <int HD>
static void launch_vattn(Engine& e, hipStream_t s, const AttnArgs& a) {
    const int ncg = (a.rps * (a.H / a.Hkv) + 15) / 16, groups = a.nseq * a.Hkv;
    // Key tiles per span: an eighth of the workgroups that share them, so that capacity-long
    // sequences come to about 8 x 193 workgroups at the 3081 positions swept; at least two per wave, one
    // with very few groups, and at most 48 spans to merge.  Measured best or within 5 % of it from 16
    // groups (2 sequences of 4 rows: 11.1 us with 4 tiles, 13.6 with 8) over 64 (4 of 6: 18.2 with 8,
    // 20.5 with 4, 22.8 with 16) to 256 (16 of 8: 60.7 with 32, 70.1 with 16, 88.6 with 64).  Large
    // ragged batches pull either way: a round of 128 sequences of 6 rows, d 2048 and 4 layers, takes 5.2 ms
    // with one of 5000 positions among 100s (4.5 with 8 tiles), 6.7 with lengths spread to 3000 (7.0).
    const int tiles = (a.cap + 15) / 16, ng = groups * ncg;
    int span_t = std::max(ng < 24 ? 4 : kVaMinTiles, ng / 8);
    span_t = (std::max(span_t, (tiles + 47) / 48) + 3) / 4 * 4;
    int nspan = (tiles + span_t - 1) / span_t;
    // the partials' and counters' room
    const size_t per = part_floats((size_t)a.nseq * a.rps, a.H, HD, ng);
    if ((size_t)ng > e.ws.cnt_n || per * nspan > e.ws.attn_part_n) {
        nspan = (size_t)ng > e.ws.cnt_n ? 1 : std::max<int>(1, e.ws.attn_part_n / per);
        span_t = ((tiles + nspan - 1) / nspan + 3) / 4 * 4;
        nspan = (tiles + span_t - 1) / span_t;
    }
    const dim3 grid((groups * nspan + 7) / 8 * 8 * ncg);
    ProfEntry* pe = prof_slot(&e, kProfAttn, 0.0);
    hipEvent_t ea = pe ? pe->a : nullptr, eb = pe ? pe->b : nullptr;
    hipExtLaunchKernelGGL((k_vattn<HD>), grid, dim3(256), 0, s, ea, eb, 0, a, ncg, nspan, span_t);
    if (pe) prof_commit(&e);
}

static void launch_pattn(Engine& e, hipStream_t s, AttnArgs a) {
    const int nqb = (a.rps + kPaQ - 1) / kPaQ;
    const int groups = a.nseq * a.Hkv * nqb;
    // few groups: split the keys into spans for about 2048 workgroups, eight per compute unit,
    // since spans past a sequence's length exit at once (at most 16 spans, within the decode
    // kernel's partial buffer and counters)
    int nspan = 1, span_t = 1;
    if (groups < kPattnGroups && (size_t)groups <= e.ws.cnt_n) {
        const int tiles = (a.cap + kPaK - 1) / kPaK;
        nspan = std::min(std::min(kPaMaxSpans, attn_nsplit(a.cap)), std::max(1, 2048 / groups));
        // (as many as the partials have room for)
        const size_t per = part_floats((size_t)a.nseq * a.rps, a.H, a.hd, (size_t)groups * (a.H / a.Hkv));
        nspan = std::max<int>(1, std::min<size_t>(nspan, e.ws.attn_part_n / per));
        span_t = (tiles + nspan - 1) / nspan;
        nspan = (tiles + span_t - 1) / span_t;
    }
    dim3 grid(groups * nspan);
    ProfEntry* pe = prof_slot(&e, kProfAttn, 0.0);
    hipEvent_t ea = pe ? pe->a : nullptr, eb = pe ? pe->b : nullptr;
    switch (a.hd) {
        case 32: hipExtLaunchKernelGGL(k_pattn<32>, grid, dim3(256), 0, s, ea, eb, 0, a, nspan, span_t); break;
        case 64: hipExtLaunchKernelGGL(k_pattn<64>, grid, dim3(256), 0, s, ea, eb, 0, a, nspan, span_t); break;
        case 128: hipExtLaunchKernelGGL(k_pattn<128>, grid, dim3(256), 0, s, ea, eb, 0, a, nspan, span_t); break;
        default: e.bad_launch = true; pe = nullptr; break;
    }
    if (pe) prof_commit(&e);
}

void launch_attn(Engine& e, hipStream_t s, ModelDev& m, int layer, int rows, int rps, const float* q, int q_stride) {
    const sd2_dims& dm = m.dm;
    AttnArgs a{};
    a.q = q; a.q_stride = q_stride; a.kc = m.kc; a.vc = m.vc; a.out = e.ws.attn;
    a.planes = e.ws.planes ? (uint16_t*)e.ws.attn : nullptr;
    a.Mp = pg_rows(rows);
    a.row_pos = e.ws.row_pos;
    a.row_off = e.live_off;
    a.rps = rps; a.H = dm.n_heads; a.Hkv = dm.n_kv_heads; a.hd = m.hd; a.cap = e.cap; a.max_batch = e.cfg.max_batch;
    a.layer = layer;
    a.nseq = rows / rps;
    a.scale = 1.0f / sqrtf((float)m.hd);
    a.part = e.ws.attn_part;
    a.cnt = e.ws.cnt;
    // the kernels read query rows and write output rows as 16-byte vectors
    if (a.q_stride % 4 || ((uintptr_t)a.q & 15) || ((uintptr_t)a.out & 15)) {
        e.bad_launch = true;
        return;
    }
    // from 16 rows a tile of one head's rows is full, and the keys staged once in LDS serve all heads
    if (rps > kVaMaxRows) {
        launch_pattn(e, s, a);
        return;
    }
    switch (m.hd) {
        case 32: launch_vattn<32>(e, s, a); break;
        case 64: launch_vattn<64>(e, s, a); break;
        case 128: launch_vattn<128>(e, s, a); break;
        default: e.bad_launch = true; break;
    }
}

// Arrival counters of attention launches of up to rps rows per sequence, one per group while the keys
// are split.  k_vattn: a group per sequence, KV head and 16 query vectors, unsplit from 8 of them per
// key tile, where a span holds all tiles (see launch_vattn).  k_pattn: per sequence, KV head and 16
// rows.
size_t attn_counters(int nseq, int rps, int H, int Hkv, int cap) {
    const int ng = nseq * Hkv * ((std::min(rps, kVaMaxRows) * (H / Hkv) + 15) / 16);
    const int groups = rps > kVaMaxRows ? nseq * Hkv * ((rps + kPaQ - 1) / kPaQ) : 0;
    return std::max(std::min(ng, 8 * ((cap + 15) / 16)), std::min(groups, kPattnGroups));
}

int attn_nsplit(int cap) { return (cap + kSplit - 1) / kSplit; }

}  // namespace sd2
