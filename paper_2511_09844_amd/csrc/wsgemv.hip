// Weight-streaming projection for bf16 weights and up to 16 fp32 activation rows per launch: the
// steering projections, and every projection of a static workspace without room for planes (see
// pgemm.hip for the others).
//
//   Y[m][n] (op)= sum_k W[n][k] * xn[m][k],   xn = x (optionally RMS-normalised and scaled by gamma)
//
// Workgroups are persistent: each stages the activation slice xn[:, k0:k0+KR) in LDS once,
// as a bf16 hi/lo pair (xn ~= hi + lo to ~16 significant bits), then walks a strided list of
// 16-row weight tiles.  Its NW waves split the K-range; every lane streams 16-byte fragments
// so that the four lanes sharing a weight row read one contiguous 128-byte segment, and the
// next tile's fragments are requested before the current tile is multiplied, so HBM traffic
// never waits on the MFMA/LDS work.  The contraction runs on v_mfma_f32_16x16x32_bf16 twice
// per fragment (hi and lo), i.e. fp32 activations against bf16 weights.  The NW partial tiles
// are summed in LDS.  Weights are read exactly once.
//
// When the activation slice of the whole K does not fit in LDS, K is cut into S ranges; each
// range writes a partial tile (write-through), and the last workgroup to finish a tile adds the
// S partials in range order and applies the epilogue (see arrive_last).
//
// Epilogues: plain store (optional output-row map), residual add (+ per-16-column sums of
// squares of the new residual, consumed by the next RMSNorm), SwiGLU on paired gate/up
// tiles, and Q|K|V with rotate-half RoPE and the append of K and V to the cache.
#include <hip/hip_ext.h>

#include "device_common.h"
#include "engine.h"

namespace sd2 {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

typedef float wf2_t __attribute__((ext_vector_type(2)));
typedef __bf16 wbf2_t __attribute__((ext_vector_type(2)));

// hi/lo bf16 split of two fp32 values, packed as two bf16 words each (element 0 in the low
// half): hi = x rounded to nearest even, lo = (x - hi) rounded likewise; one hardware packed
// conversion per word (integer rounding took about six VALU operations per value)
__device__ __forceinline__ void split_hilo(float x0, float x1, uint32_t& hi, uint32_t& lo) {
    const wf2_t v = {x0, x1};
    const wbf2_t h = __builtin_convertvector(v, wbf2_t);
    const wbf2_t l = __builtin_convertvector(v - __builtin_convertvector(h, wf2_t), wbf2_t);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

struct WsArgs {
    const float* X;
    int ldx;
    const int32_t* in_map;
    int M;     // rows in this launch (<= 16)
    int row0;  // first row (of X / Y / row plans) handled by this launch
    int K;
    const uint16_t* gamma;
    float eps;
    const float* ss;  // [rows][nss] partial sums of squares of X rows (norm input)
    int nss;
    const uint16_t* W[3];
    int seg_tiles[3];
    int nseg;
    int mode;
    int tiles;
    float* Y;
    int ldy;
    const int32_t* out_map;
    float* ss_out;
    int KR, S, Gt;  // K-range per workgroup, number of K ranges, workgroups per K range
    float* part;    // S > 1: [tiles][S][SUBS][256]
    int32_t* cnt;   // S > 1: arrival counter per tile
    // Q|K|V mode
    int H, Hkv, hd;
    const int32_t *row_pos, *row_seq;
    const float *rcos, *rsin;
    float *qout, *kc, *vc;
    int cap, max_batch, layer;
    // MLP steering: bias of the row's sequence (row_seq), added to up (SwiGLU) or to the output
    // (Add), or null
    const float* ubias;
    int ub_ld;
};

// Weight row streamed by lane column n of a tile (segment resolution and the Q|K|V pairing
// of rotate-half partners i and i + hd/2 inside one tile).
__device__ __forceinline__ const uint16_t* tile_row(const WsArgs& a, int tile, int sub, int n) {
    if (a.mode == kEpiSwiglu) return a.W[sub] + (size_t)(tile * 16 + n) * a.K;
    int seg = 0, lt = tile;
    while (seg + 1 < a.nseg && lt >= a.seg_tiles[seg]) { lt -= a.seg_tiles[seg]; ++seg; }
    int wrow;
    if (a.mode == kEpiQkv) {
        int per_head = a.hd / 16;
        int h = lt / per_head, j = lt % per_head;
        wrow = h * a.hd + (n < 8 ? 8 * j + n : a.hd / 2 + 8 * j + (n - 8));
    } else {
        wrow = lt * 16 + n;
    }
    return a.W[seg] + (size_t)wrow * a.K;
}

// Epilogue of one finished 16x16 tile; element (m, c) is held by thread t = 16m + c of the
// first 256 threads.  `v` holds the value per sub-tile.
template <int SUBS>
// Rows row0 .. row0 + nrows - 1 of the launch (at most 16).
__device__ __forceinline__ void tile_epilogue(const WsArgs& a, int tile, const float* v, int row0, int nrows) {
    const int tid = threadIdx.x;
    const int em = tid >> 4, ec = tid & 15;
    const bool valid = em < nrows;
    const int row = row0 + em;
    if (a.mode == kEpiStore) {
        if (valid) {
            int orow = a.out_map ? a.out_map[row] : row;
            if (orow >= 0) a.Y[(size_t)orow * a.ldy + tile * 16 + ec] = v[0];
        }
    } else if (a.mode == kEpiAdd) {
        float nv = 0.0f;
        if (valid) {
            float* yp = a.Y + (size_t)row * a.ldy + tile * 16 + ec;
            nv = *yp + v[0];
            if (a.ubias) nv += a.ubias[(size_t)a.row_seq[row] * a.ub_ld + tile * 16 + ec];
            *yp = nv;
        }
        float sq = nv * nv;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 16);
        if (valid && ec == 0) a.ss_out[(size_t)row * a.tiles + tile] = sq;
    } else if (a.mode == kEpiSwiglu) {
        if (valid) {
            float up = v[SUBS - 1];
            if (a.ubias) up += a.ubias[(size_t)a.row_seq[row] * a.ub_ld + tile * 16 + ec];
            a.Y[(size_t)row * a.ldy + tile * 16 + ec] = silu(v[0]) * up;
        }
    } else {
        float partner = __shfl_xor(v[0], 8, 16);
        if (!valid) return;
        int seg = 0, lt = tile;
        while (seg + 1 < a.nseg && lt >= a.seg_tiles[seg]) { lt -= a.seg_tiles[seg]; ++seg; }
        int per_head = a.hd / 16;
        int h = lt / per_head, j = lt % per_head;
        int half = a.hd / 2;
        int i = 8 * j + (ec & 7);
        int dim = ec < 8 ? i : half + i;
        int pos = a.row_pos[row];
        float out = v[0];
        if (seg < 2) {
            int pp = pos < 0 ? 0 : pos;
            float c = a.rcos[(size_t)pp * half + i], sn = a.rsin[(size_t)pp * half + i];
            out = ec < 8 ? v[0] * c - partner * sn : v[0] * c + partner * sn;
        }
        if (seg == 0) {
            a.qout[(size_t)row * a.H * a.hd + h * a.hd + dim] = out;
        } else if (pos >= 0) {
            int b = a.row_seq[row];
            size_t idx = ((((size_t)a.layer * a.max_batch + b) * a.Hkv + h) * a.cap + pos) * a.hd + dim;
            if (seg == 1) a.kc[idx] = out;
            else a.vc[idx] = out;
        }
    }
}

// Sum of one row's slice sums of squares over a wave (lane l takes slices l, l + 64, ...): loads in
// batches of eight per lane with clamped indexes, so that none waits for the one before it.
// row < 0: 0.
__device__ __forceinline__ float row_sumsq(const float* ss, int nss, int row, int lane) {
    const float* rp = ss + (size_t)max(row, 0) * nss;
    float sm = 0.0f;
    for (int t0 = 0; t0 < nss; t0 += 512) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = rp[min(t0 + lane + 64 * u, nss - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) sm += (row >= 0 && t0 + lane + 64 * u < nss) ? v[u] : 0.f;
    }
    return sm;
}

template <int NW, int STEPS, int SUBS>
__global__ __launch_bounds__(NW * 64) void k_wsgemv(WsArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ float inv_rms[16];
    __shared__ int src_row[16];
    __shared__ int last_flag;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int M = a.M;
    const int KR = a.KR;
    const int ldk = KR + 8;  // padded row stride (bf16 elements) of the LDS slices
    const int s = blockIdx.x % a.S;
    const int g = blockIdx.x / a.S;
    const int k0 = s * KR;
    uint16_t* xh = (uint16_t*)smem;
    uint16_t* xl = xh + (size_t)M * ldk;
    float* red = (float*)(xl + (size_t)M * ldk);  // [NW][256]

    const int n = lane & 15, q = lane >> 4;
    const int kw0 = wave * (KR / NW);

    // The workgroup's work is a sequence of sub-tiles u = 0, 1, ...: tile g + (u / SUBS) * Gt,
    // sub-tile u % SUBS (SwiGLU: gate then up).  Two sub-tiles of weight fragments are kept in
    // flight in two register buffers.
    const int ntile_mine = a.tiles > g ? (a.tiles - g + a.Gt - 1) / a.Gt : 0;
    const int nsub_mine = ntile_mine * SUBS;
    u32x4_t wa[STEPS][2], wb[STEPS][2];
    auto issue = [&](u32x4_t (&buf)[STEPS][2], int u) {
        const int tile = g + (u / SUBS) * a.Gt;
        const uint16_t* wp = tile_row(a, tile, u % SUBS, n) + k0 + kw0 + 16 * q;
#pragma unroll
        for (int st = 0; st < STEPS; ++st)
#pragma unroll
            for (int h = 0; h < 2; ++h) buf[st][h] = *(const u32x4_t*)(wp + st * 64 + 8 * h);
    };

    // ---- prologue.  Loads return in issue order, so the small activation loads go first, then
    //      the first weight sub-tile, then the RMSNorm statistics (needed only by the epilogue:
    //      the row scale 1/rms is applied to the outputs, the gain to the staged activations) ----
    if (tid < 16) {
        int src = -1;
        if (tid < M) src = a.in_map ? a.in_map[a.row0 + tid] : a.row0 + tid;
        src_row[tid] = src;
        inv_rms[tid] = 1.0f;
    }
    __syncthreads();
    constexpr int XB = 16;  // activation float4 loads per thread issued ahead of the weights
    const int n4 = KR / 4;
    const int nx = M * n4;  // float4 groups of the slice, row-major
    float4 xv[XB];
#pragma unroll
    for (int i = 0; i < XB; ++i) {
        const int idx = tid + i * NW * 64;
        if (idx < nx) {
            const int m = idx / n4, kk = (idx % n4) * 4;
            const int src = src_row[m];
            xv[i] = src >= 0 ? *(const float4*)(a.X + (size_t)src * a.ldx + k0 + kk) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    // the gain words of the same columns, all requested before any is used (a load under a
    // per-element test would wait for everything in flight, the weights included)
    uint2 gv[XB];
    if (a.gamma) {
#pragma unroll
        for (int i = 0; i < XB; ++i) {
            const int idx = min(tid + i * NW * 64, nx - 1);
            gv[i] = *(const uint2*)(a.gamma + k0 + (idx % n4) * 4);
        }
    } else {
#pragma unroll
        for (int i = 0; i < XB; ++i) gv[i] = make_uint2(0x3f803f80u, 0x3f803f80u);  // bf16 ones
    }
    if (nsub_mine > 0) issue(wa, 0);
    float ssum = 0.0f;
    const int ss_row = wave < M ? src_row[wave] : -1;
    if (a.gamma) ssum = row_sumsq(a.ss, a.nss, ss_row, lane);
    auto stage = [&](const float4& v, int idx, uint2 gw) {
        const int m = idx / n4, kk = (idx % n4) * 4;
        float gm[4] = {1.f, 1.f, 1.f, 1.f};
        if (a.gamma) {
            gm[0] = bf16_lo(gw.x); gm[1] = bf16_hi(gw.x); gm[2] = bf16_lo(gw.y); gm[3] = bf16_hi(gw.y);
        }
        uint32_t h0, h1, l0, l1;
        split_hilo(v.x * gm[0], v.y * gm[1], h0, l0);
        split_hilo(v.z * gm[2], v.w * gm[3], h1, l1);
        *(uint2*)(xh + (size_t)m * ldk + kk) = make_uint2(h0, h1);
        *(uint2*)(xl + (size_t)m * ldk + kk) = make_uint2(l0, l1);
    };
#pragma unroll
    for (int i = 0; i < XB; ++i) {
        const int idx = tid + i * NW * 64;
        if (idx < nx) stage(xv[i], idx, gv[i]);
    }
    // slices larger than XB float4 per thread (not used by the planned shapes) stage the rest here
    for (int idx = tid + XB * NW * 64; idx < nx; idx += NW * 64) {
        const int m = idx / n4, kk = (idx % n4) * 4;
        const int src = src_row[m];
        float4 v = src >= 0 ? *(const float4*)(a.X + (size_t)src * a.ldx + k0 + kk) : make_float4(0.f, 0.f, 0.f, 0.f);
        const uint2 gw = a.gamma ? *(const uint2*)(a.gamma + k0 + kk) : make_uint2(0x3f803f80u, 0x3f803f80u);
        stage(v, idx, gw);
    }
    if (nsub_mine > 1) issue(wb, 1);
    if (a.gamma) {
        ssum = wave_sum(ssum);
        if (lane == 0 && wave < M) inv_rms[wave] = rsqrtf(ssum / (float)a.K + a.eps);
        // rows beyond the number of waves (M > NW)
        for (int m = NW + wave; m < M; m += NW) {
            float sm = row_sumsq(a.ss, a.nss, src_row[m], lane);
            sm = wave_sum(sm);
            if (lane == 0) inv_rms[m] = rsqrtf(sm / (float)a.K + a.eps);
        }
    }
    __syncthreads();

    const bool arow = n < M;
    float stash = 0.0f;  // gate value of the current SwiGLU tile (threads < 256)
    auto compute = [&](u32x4_t (&buf)[STEPS][2], int u) {
        floatx4_t acc = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int kk = kw0 + st * 64 + 16 * q + 8 * h;
                bf16x8_t ah = bf16x8_t{0, 0, 0, 0, 0, 0, 0, 0}, al = ah;
                if (arow) {
                    ah = *(const bf16x8_t*)(xh + (size_t)n * ldk + kk);
                    al = *(const bf16x8_t*)(xl + (size_t)n * ldk + kk);
                }
                bf16x8_t b = __builtin_bit_cast(bf16x8_t, buf[st][h]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b, acc, 0, 0, 0);
            }
        }
        // sum the NW waves' tiles: element (m, c) = (t / 16, t % 16); scale by the row's 1/rms
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wave * 256 + (4 * q + i) * 16 + n] = acc[i];
        __syncthreads();
        const int tile = g + (u / SUBS) * a.Gt;
        const int sub = u % SUBS;
        float x = 0.0f;
        if (tid < 256) {
#pragma unroll
            for (int w = 0; w < NW; ++w) x += red[w * 256 + tid];
            x *= inv_rms[tid >> 4];
        }
        if (SUBS == 2 && sub == 0) {
            stash = x;
        } else if (a.S == 1) {
            float v[2] = {SUBS == 2 ? stash : x, x};
            if (tid < 256) tile_epilogue<SUBS>(a, tile, v, a.row0, a.M);
        } else {
            // K split over S workgroups: the last to finish this tile adds the partials in order
            float* pt = a.part + (size_t)tile * a.S * SUBS * 256;
            if (tid < 256) {
                store_through(pt + (size_t)s * SUBS * 256 + tid, SUBS == 2 ? stash : x);
                if (SUBS == 2) store_through(pt + (size_t)s * SUBS * 256 + 256 + tid, x);
            }
            if (arrive_last(a.cnt + tile, a.S, &last_flag) && tid < 256) {
                float p0[8], p1[8];
                float v[2] = {0.f, 0.f};
                for (int s0 = 0; s0 < a.S; s0 += 8) {
                    const int ns = min(8, a.S - s0);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if (i < ns) {
                            p0[i] = pt[(size_t)(s0 + i) * SUBS * 256 + tid];
                            if (SUBS == 2) p1[i] = pt[(size_t)(s0 + i) * SUBS * 256 + 256 + tid];
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if (i < ns) {
                            v[0] += p0[i];
                            if (SUBS == 2) v[1] += p1[i];
                        }
                    }
                }
                if (SUBS == 1) v[1] = v[0];
                tile_epilogue<SUBS>(a, tile, v, a.row0, a.M);
            }
        }
        __syncthreads();
    };

    // ---- sub-tile loop: after a buffer is consumed it is refilled two sub-tiles ahead ----
    for (int u = 0; u < nsub_mine; u += 2) {
        compute(wa, u);
        if (u + 2 < nsub_mine) issue(wa, u + 2);
        if (u + 1 >= nsub_mine) break;
        compute(wb, u + 1);
        if (u + 3 < nsub_mine) issue(wb, u + 3);
    }
}

constexpr int kLdsBudget = 160 * 1024 - 2048;
// Activation bytes a workgroup stages: K is split until each workgroup's slice of the rows fits
// this (16 rows of 2048 columns would be 128 KB read from L2 by every workgroup for one 64 KB
// weight tile, at one workgroup per CU); without such a split, the smallest that fits LDS.
constexpr size_t kWsStageMax = 64 * 1024;

static size_t lds_bytes(int rows, int KR, int NW) {
    return (size_t)rows * (KR + 8) * 2 * 2 + (size_t)NW * 256 * 4;
}

// Plan: number of K ranges S (1 when the whole activation row fits in LDS), K-range KR,
// waves NW and fragment steps per lane, and how many workgroups walk the tiles.
WsPlan ws_plan(int M, int N, int K, int mode) {
    WsPlan p{};
    int rows = M < 16 ? M : 16;
    (void)mode;
    p.tiles = N / 16;
    // first pass: the smallest split whose staged slice fits kWsStageMax; second: any that fits
    for (int pass = 0; pass < 2 && !p.S; ++pass)
    for (int S = 1; S <= K / 256; ++S) {
        if (K % S) continue;
        int KR = K / S;
        if (KR % 256) continue;
        if (pass == 0 && (size_t)rows * KR * 4 > kWsStageMax) continue;
        // waves: each a multiple of 64 columns; two fragment buffers of 8*steps VGPRs each must
        // leave room in the 512-entry register file (8 steps with <= 8 waves, 4 with 16 waves)
        int NW = 0, steps = 0;
        for (int nw = 4; nw <= 16; nw *= 2) {
            if (KR % (nw * 64)) continue;
            int st = KR / (nw * 64);
            if (st > (nw == 16 ? 4 : 8)) continue;
            NW = nw;
            steps = st;
            break;
        }
        if (!NW) continue;
        if (lds_bytes(rows, KR, NW) > (size_t)kLdsBudget) continue;
        p.S = S;
        p.KR = KR;
        p.NW = NW;
        p.steps = steps;
        break;
    }
    if (!p.S) return p;
    size_t lds = lds_bytes(rows, p.KR, p.NW);
    int per_cu = (int)((160 * 1024) / (lds + 1024));
    if (per_cu < 1) per_cu = 1;
    if (per_cu > 2) per_cu = 2;
    int want = 256 * per_cu;
    int gt = want / p.S;
    if (gt < 1) gt = 1;
    if (gt > p.tiles) gt = p.tiles;
    p.Gt = gt;
    p.lds = lds;
    return p;
}

void launch_wsgemv(Engine* e, hipStream_t s, const WsCall& c) {
    // rows that come as planes, and more than one 16-row group, run on the plane kernel
    // (pgemm.hip); up to 16 fp32 rows (the steering projections) save the launch that makes planes
    if ((c.planes || c.M > 16) && launch_pgemm(e, s, c)) return;
    if (c.planes) {  // there are no fp32 rows to fall back on
        if (e) e->bad_launch = true;
        return;
    }
    for (int r0 = 0; r0 < c.M; r0 += 16) {
        int M = c.M - r0 < 16 ? c.M - r0 : 16;
        WsArgs a{};
        a.X = c.X; a.ldx = c.K; a.in_map = c.in_map; a.M = M; a.row0 = r0; a.K = c.K;
        a.gamma = (const uint16_t*)c.gamma; a.eps = c.eps; a.ss = c.ss; a.nss = c.nss;
        int tiles = 0;
        for (int i = 0; i < 3; ++i) {
            a.W[i] = i < c.nseg ? (const uint16_t*)c.W[i] : nullptr;
            a.seg_tiles[i] = i < c.nseg ? c.seg_rows[i] / 16 : 0;
            if (c.mode != kEpiSwiglu) tiles += a.seg_tiles[i];
        }
        if (c.mode == kEpiSwiglu) tiles = c.seg_rows[0] / 16;
        a.nseg = c.nseg; a.mode = c.mode; a.tiles = tiles;
        a.Y = c.Y; a.ldy = c.ldy; a.out_map = c.out_map; a.ss_out = c.ss_out;
        WsPlan p = ws_plan(M, tiles * 16, c.K, c.mode);
        a.KR = p.KR; a.S = p.S; a.Gt = p.Gt;
        a.part = c.part;
        a.cnt = c.cnt;
        a.H = c.H; a.Hkv = c.Hkv; a.hd = c.hd; a.row_pos = c.row_pos; a.row_seq = c.row_seq;
        a.rcos = c.rcos; a.rsin = c.rsin; a.qout = c.qout; a.kc = c.kc; a.vc = c.vc;
        a.cap = c.cap; a.max_batch = c.max_batch; a.layer = c.layer;
        a.ubias = c.ubias; a.ub_ld = c.ub_ld;
        int subs = c.mode == kEpiSwiglu ? 2 : 1;
        bool launched = false;
        if (p.S) {
            dim3 grid(p.S * p.Gt);
            double wbytes = (double)tiles * 16 * subs * c.K * 2.0;
            ProfEntry* pe = prof_slot(e, kProfGemv, wbytes + (double)M * c.K * 4.0 + (double)M * tiles * 16 * 4.0);
#define SD2_WS_CASE(NWV, ST, SB)                                                                     \
    if (!launched && p.NW == NWV && p.steps == ST && subs == SB) {                                    \
        if (pe)                                                                                       \
            hipExtLaunchKernelGGL((k_wsgemv<NWV, ST, SB>), grid, dim3(NWV * 64), p.lds, s, pe->a, pe->b, 0, a); \
        else                                                                                          \
            k_wsgemv<NWV, ST, SB><<<grid, NWV * 64, p.lds, s>>>(a);                                   \
        launched = true;                                                                              \
    }
#define SD2_WS_STEPS8(NWV, SB)                                                    \
    SD2_WS_CASE(NWV, 1, SB) SD2_WS_CASE(NWV, 2, SB) SD2_WS_CASE(NWV, 3, SB) SD2_WS_CASE(NWV, 4, SB) \
    SD2_WS_CASE(NWV, 5, SB) SD2_WS_CASE(NWV, 6, SB) SD2_WS_CASE(NWV, 7, SB) SD2_WS_CASE(NWV, 8, SB)
            SD2_WS_STEPS8(4, 1) SD2_WS_STEPS8(8, 1) SD2_WS_STEPS8(4, 2) SD2_WS_STEPS8(8, 2)
            SD2_WS_CASE(16, 1, 1) SD2_WS_CASE(16, 2, 1) SD2_WS_CASE(16, 3, 1) SD2_WS_CASE(16, 4, 1)
            SD2_WS_CASE(16, 1, 2) SD2_WS_CASE(16, 2, 2) SD2_WS_CASE(16, 3, 2) SD2_WS_CASE(16, 4, 2)
#undef SD2_WS_STEPS8
#undef SD2_WS_CASE
            if (pe && launched) prof_commit(e);
        }
        if (!launched && e) e->bad_launch = true;
    }
}

}  // namespace sd2
