// Attention over the retrieved KV (paper Sec. V-A (2)): vector-ALU split-KV
// kernel (bf16 pages, values stored [T][D]) and the combine kernel that
// merges the per-split partials of every kernel family.
//
// Work decomposition:
//   rows     the unit's G*Tq query rows, row r = t*G + g, in tiles of 16
//   chunks   32 tokens inside one page; a unit has n_sel * ceil(T/32) chunks
//   splits   contiguous chunk ranges; one workgroup per (split, row tile, unit)
// Each workgroup keeps an online softmax in the log2 domain (logits are
// multiplied by log2(e)/sqrt(D) once) and writes (max, sum, unnormalised O).
#include <type_traits>

#include "mosaic_internal.h"
#include "attend_reps_device.h"

namespace mosaic {

namespace {

__device__ __forceinline__ void load8f(const unsigned short *p, float (&v)[8]) {
    const uint4 a = *reinterpret_cast<const uint4 *>(p);
    const unsigned int w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
template <typename E> __device__ __forceinline__ void store_out(E *p, float v);
template <> __device__ __forceinline__ void store_out<float>(float *p, float v) { *p = v; }
template <> __device__ __forceinline__ void store_out<unsigned short>(unsigned short *p, float v) {
    *p = f32_to_bf16_rne(v);
}

__device__ __forceinline__ float group16_max(float x) {
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 16));
    return x;
}
__device__ __forceinline__ float group16_sumf(float x) {
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) x += __shfl_xor(x, o, 16);
    return x;
}

// grid (n_units * n_splits [+ n_units with the global-representative augmentation], NT), 256 threads:
// thread (row = tid/16, tl = tid%16)
template <int D>
__global__ __launch_bounds__(kBlock) void k_attend_valu(const DeviceView *self, int u0, int n_units, const unsigned short *q,
                                                        int Tq, int B) {
    const DeviceView dv = device_view(self);
    typedef unsigned short E;
    constexpr int DPT = D / 16;   // output channels per thread
    constexpr int CG = D / 8;     // 8-element groups per token row
    if ((int)blockIdx.x >= B) {   // extra columns: the global representatives' part (augmentation)
        __shared__ float lds[kF32MergeFloats<D>];
        attend_reps_partial<E, D>(dv, u0, (int)blockIdx.x - B, blockIdx.y, q, Tq, lds);
        return;
    }
    const SplitSlot slot = split_slot<false>(dv.n_sel + u0, n_units, B, blockIdx.x);
    if (slot.uc < 0) return;      // block-uniform: no barrier reached yet
    const int split = slot.split, n_splits = slot.S, tile = blockIdx.y, uc = slot.uc, u = u0 + uc;
    const int NT = gridDim.y, tid = threadIdx.x, row = tid / 16, tl = tid % 16;
    const int G = dv.G, Hq = dv.Hq, T = dv.T;
    const int lc = uc / dv.Hkv, h = u % dv.Hkv, R = Tq * G;
    __shared__ float q_sh[kRowTile][D];
    __shared__ float k_sh[kChunk][D + 1];
    __shared__ float v_sh[kChunk][D];
    __shared__ float p_sh[kRowTile][kChunk];

    const float sl2 = 1.4426950408889634f / sqrtf((float)D);
    for (int idx = tid; idx < kRowTile * D; idx += kBlock) {
        const int rr = idx / D, d = idx % D, gr = tile * kRowTile + rr;
        float v = 0.f;
        if (gr < R) {
            const int t = gr / G, g = gr % G;
            v = bf16_to_f32(q[(((size_t)lc * Tq + t) * Hq + (size_t)h * G + g) * D + d]) * sl2;
        }
        q_sh[rr][d] = v;
    }
    const int cpp = dv.chunks_per_page;
    const int NC = dv.n_sel[u] * cpp;
    const int cps = (NC + n_splits - 1) / n_splits;
    const int c0 = split * cps, c1 = min(NC, c0 + cps);
    const int *sel = dv.sel_pages + (size_t)u * dv.F;

    float m = -INFINITY, l = 0.f, acc[DPT];
#pragma unroll
    for (int i = 0; i < DPT; ++i) acc[i] = 0.f;
    __syncthreads();

    for (int c = c0; c < c1; ++c) {
        const int page = sel[c / cpp], t0 = (c % cpp) * kChunk, nt = min(kChunk, T - t0);
        const E *kp = reinterpret_cast<const E *>(k_page(dv, u, page)) + (size_t)t0 * D;
        const E *vp = reinterpret_cast<const E *>(v_page(dv, u, page)) + (size_t)t0 * D;
        for (int item = tid; item < kChunk * CG; item += kBlock) {
            const int tok = item / CG, cg = item % CG;
            float kv[8], vv[8];
            if (tok < nt) {
                load8f(kp + (size_t)tok * D + cg * 8, kv);
                load8f(vp + (size_t)tok * D + cg * 8, vv);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) { kv[i] = 0.f; vv[i] = 0.f; }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) { k_sh[tok][cg * 8 + i] = kv[i]; v_sh[tok][cg * 8 + i] = vv[i]; }
        }
        __syncthreads();
        float s0 = 0.f, s1 = 0.f;
        for (int d = 0; d < D; ++d) {
            const float qv = q_sh[row][d];
            s0 += qv * k_sh[tl][d];
            s1 += qv * k_sh[tl + 16][d];
        }
        if (tl >= nt) s0 = -INFINITY;
        if (tl + 16 >= nt) s1 = -INFINITY;
        const float mnew = fmaxf(m, group16_max(fmaxf(s0, s1)));
        const float alpha = exp2f(m - mnew);
        const float p0 = exp2f(s0 - mnew), p1 = exp2f(s1 - mnew);
        l = l * alpha + group16_sumf(p0 + p1);
        m = mnew;
        p_sh[row][tl] = p0;
        p_sh[row][tl + 16] = p1;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < DPT; ++i) acc[i] *= alpha;
        for (int t = 0; t < kChunk; ++t) {
            const float p = p_sh[row][t];
#pragma unroll
            for (int i = 0; i < DPT; ++i) acc[i] += p * v_sh[t][tl + 16 * i];
        }
        __syncthreads();
    }
    const size_t entry = (size_t)slot.base * NT + (size_t)tile * n_splits + split;
#pragma unroll
    for (int i = 0; i < DPT; ++i) dv.part_o[(entry * kRowTile + row) * D + tl + 16 * i] = acc[i];
    if (tl == 0) {     // fp32 weights: the two normalisers coincide
        dv.part_ml[entry * kMlRows * kRowTile + row] = m;
        dv.part_ml[entry * kMlRows * kRowTile + kRowTile + row] = l;
        dv.part_ml[entry * kMlRows * kRowTile + 2 * kRowTile + row] = l;
    }
}

// Weighted sum of one unit's split partials for 32 output channels of one row tile
// (the per-thread share): log-sum-exp weights into w_sh, row maxima and normalisers
// into M_sh / L_sh, partial sums into acc.  The workgroup takes rows rbase .. rbase + nr - 1 of the
// tile; RMAX = 4, 8 or 16 bounds nr, MAXS the splits handled.  A thread keeps 128
// partial values in registers per pass, i.e. 64 splits of 16 rows or 128 splits of 8
// rows; MAXS beyond that (a unit that retrieved far more than the others of its launch)
// takes further passes, each one more memory round trip.
// The partial loads of the first pass are issued first, ahead of the (independent) loads
// and barriers of the weight computation: the partials were written by other compute
// units, so every load is a full memory round trip, and the two round trips overlap.
// Split and row indices are clamped instead of tested, so the loads are unconditional
// (straight-line code); what a clamped load brings is never used.
template <int D, int MAXS, int RMAX>
__device__ __forceinline__ void combine_accumulate(const DeviceView &dv, size_t e0, int n_splits, int rbase, int nr, int dg,
                                                   float (*w_sh)[kRowTile], float (*pm)[kRowTile],
                                                   float (*pl)[kRowTile], float (*px)[kRowTile], float *M_sh,
                                                   float *L_sh, float *X_sh, float (&acc)[kRowTile]) {
    constexpr int SPP = 64 * (kRowTile / RMAX);  // splits per pass (128 partial values per thread) ...
    constexpr int NB = (MAXS < SPP ? MAXS : SPP) / 8;   // ... in batches of 8 (fewer when the unit cannot have that many)
    const int tid = threadIdx.x, sg = tid / 32, col = tid % 32;
    float v[NB][RMAX];
    auto load_pass = [&](int s0) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int s = min(s0 + sg + 8 * i, max(n_splits - 1, 0));
            const float *po = dv.part_o + (e0 + s) * kRowTile * D + dg * 32 + col;
#pragma unroll
            for (int r = 0; r < RMAX; ++r) v[i][r] = po[(size_t)(rbase + min(r, nr - 1)) * D];
        }
    };
    load_pass(0);
    {   // per-row maximum and normaliser over the splits
        const int row = tid % 16, part = tid / 16;
        float mr[MAXS / 16], lr[MAXS / 16], xr[MAXS / 16];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < MAXS / 16; ++i) {
            const int s = part + 16 * i;
            mr[i] = -INFINITY; lr[i] = 0.f; xr[i] = 0.f;
            if (s < n_splits) {
                mr[i] = dv.part_ml[(e0 + s) * kMlRows * kRowTile + row];
                lr[i] = dv.part_ml[(e0 + s) * kMlRows * kRowTile + kRowTile + row];
                xr[i] = dv.part_ml[(e0 + s) * kMlRows * kRowTile + 2 * kRowTile + row];
            }
            mx = fmaxf(mx, mr[i]);
        }
        pm[part][row] = mx;
        __syncthreads();
        float M = -INFINITY;
#pragma unroll
        for (int p = 0; p < 16; ++p) M = fmaxf(M, pm[p][row]);
        float ls = 0.f, xs = 0.f;
#pragma unroll
        for (int i = 0; i < MAXS / 16; ++i) {
            const int s = part + 16 * i;
            if (s < n_splits) {
                const float w = M > -INFINITY ? exp2f(mr[i] - M) : 0.f;
                w_sh[s][row] = w;
                ls += w * lr[i];
                xs += w * xr[i];
            }
        }
        pl[part][row] = ls;
        px[part][row] = xs;
        __syncthreads();
        if (part == 0) {
            // (in pairs: sixteen sums one after the other made up most of the output's error where many splits are merged;
            // fp32 steps over 512 tokens in 32 splits 1.1e-7 -> 8.0e-8 of the output's norm, 36 streams of six other shapes
            // 0.73 to 1.04 -> 0.64 to 0.81 of what fewer and longer splits had; the launch no longer than before)
            float l16[16], x16[16];
#pragma unroll
            for (int p = 0; p < 16; ++p) { l16[p] = pl[p][row]; x16[p] = px[p][row]; }
            M_sh[row] = M;
            L_sh[row] = pair_sum<16>(l16);
            X_sh[row] = pair_sum<16>(x16);
        }
    }
#pragma unroll
    for (int r = 0; r < kRowTile; ++r) acc[r] = 0.f;
    for (int s0 = 0; s0 < (MAXS > SPP ? n_splits : 1); s0 += SPP) {
        if (MAXS > SPP && s0 > 0) load_pass(s0);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int s = s0 + sg + 8 * i;
            if (s < n_splits) {
#pragma unroll
                for (int r = 0; r < RMAX; ++r) acc[r] += w_sh[s][min(rbase + r, kRowTile - 1)] * v[i][r];
            }
        }
    }
}

// N neighbouring output values (channels ch ..) of row r of a tile, with the representatives' part merged in, and the row's
// log-sum-exp.  Lr: normaliser of the output (the weights the value contraction used, bf16-rounded in the MFMA kernels); Xr: the
// same sum over the unrounded fp32 weights, for the log-sum-exp; Mr: the row's reference (log2 domain).
template <typename E, int D, int N>
__device__ __forceinline__ void combine_store(const DeviceView &dv, int u, int lc, int h, int tile, int r, int ch, int Tq,
                                              float (&o)[N], float Lr, float Xr, float Mr, E *out, float *lse) {
    const int G = dv.G, Hq = dv.Hq;
    if (dv.aug_reps) {                            // one more partial: the representatives' part
        const size_t ae = (size_t)u * dv.nt_max + tile;
        const float ma = dv.aug_ml[ae * 2 * kRowTile + r], la = dv.aug_ml[ae * 2 * kRowTile + kRowTile + r];
        const float *oa = dv.aug_o + (ae * kRowTile + r) * D + ch;
        const float Mn = fmaxf(Mr, ma);
        const float wa = Mr > -INFINITY ? exp2f(Mr - Mn) : 0.f, wb = ma > -INFINITY ? exp2f(ma - Mn) : 0.f;
#pragma unroll
        for (int i = 0; i < N; ++i) o[i] = o[i] * wa + oa[i] * wb;
        Lr = Lr * wa + la * wb;
        Xr = Xr * wa + la * wb;                   // (the representatives' weights are fp32)
        Mr = Mn;
    }
    const int gr = tile * kRowTile + r, t = gr / G, g = gr - t * G;
    const size_t orow = ((size_t)lc * Tq + t) * Hq + (size_t)h * G + g;
#pragma unroll
    for (int i = 0; i < N; ++i) store_out<E>(out + orow * D + ch + i, Lr > 0.f ? o[i] / Lr : 0.f);
    if (ch == 0 && lse != nullptr)
        lse[orow] = Xr > 0.f ? (Mr + log2f(Xr)) * 0.6931471805599453f : -INFINITY;
}

// Merge of the per-split partials (log-sum-exp weights), normalisation, output, for one
// row tile (a decode step).  grid (D/32 * RS, n_units), 256 threads.  A workgroup owns 32
// output channels; its 8 groups of 32 threads share the splits, so the partial buffer is
// read with many independent 128-byte loads in flight.
template <typename E, int D>
__global__ __launch_bounds__(kBlock) void k_attend_combine(const DeviceView *self, int u0, int n_units, int Tq,
                                                           int B, int uniform_S, E *out, float *lse) {
    const DeviceView dv = device_view<0, 2, 8>(self);
    // grid.x = (D / 32) * RS: RS workgroups share a tile's rows (a decode step's heaviest unit has up to 256
    // partials to merge, and the launch lasts as long as that unit's workgroups: with its rows shared by two
    // workgroups each thread reads half as much, all of it in one pass)
    constexpr int DG = D / 32;
    const int dg = blockIdx.x % DG, rs = blockIdx.x / DG, RS = gridDim.x / DG;
    const int uc = blockIdx.y, u = u0 + uc;
    const int tid = threadIdx.x;
    const int lc = uc / dv.Hkv, h = u % dv.Hkv, rows = Tq * dv.G;
    const int rper = (rows + RS - 1) / RS, rbase = rs * rper, nr = min(rper, rows - rbase);
    if (nr <= 0) return;                         // block-uniform: no barrier reached yet
    // uniform_S > 0: every unit has exactly that many splits (the fused decode step); else the
    // splits were shared out by retrieved size and split_slot() says how
    SplitSlot slot{uc, 0, uniform_S, uc * uniform_S, 0};
    if (uniform_S <= 0) slot = split_slot<true>(dv.n_sel + u0, n_units, B, uc);
    const int n_splits = slot.S;                 // 0 if the unit retrieved nothing
    const size_t e0 = (size_t)slot.base;
    __shared__ float w_sh[kMaxUnitSplits][kRowTile];
    __shared__ float pm[16][kRowTile], pl[16][kRowTile], px[16][kRowTile];
    __shared__ float M_sh[kRowTile], L_sh[kRowTile], X_sh[kRowTile];
    __shared__ float red[8][kRowTile][33];
    const int sg = tid / 32, col = tid % 32;
    float acc[kRowTile];
#define MOSAIC_COMBINE(MAXS, RMAX) \
    combine_accumulate<D, MAXS, RMAX>(dv, e0, n_splits, rbase, nr, dg, w_sh, pm, pl, px, M_sh, L_sh, X_sh, acc)
    if (rper <= 1) {             // block-uniform choices
        if (n_splits <= 64) MOSAIC_COMBINE(64, 1);
        else if (n_splits <= 128) MOSAIC_COMBINE(128, 1);
        else MOSAIC_COMBINE(kMaxUnitSplits, 1);
    } else if (rper <= 2) {
        if (n_splits <= 64) MOSAIC_COMBINE(64, 2);
        else if (n_splits <= 128) MOSAIC_COMBINE(128, 2);
        else MOSAIC_COMBINE(kMaxUnitSplits, 2);
    } else if (rper <= 4) {
        if (n_splits <= 32) MOSAIC_COMBINE(32, 4);
        else if (n_splits <= 64) MOSAIC_COMBINE(64, 4);
        else if (n_splits <= 128) MOSAIC_COMBINE(128, 4);
        else MOSAIC_COMBINE(kMaxUnitSplits, 4);
    } else if (rper <= 8) {
        if (n_splits <= 16) MOSAIC_COMBINE(16, 8);
        else if (n_splits <= 32) MOSAIC_COMBINE(32, 8);
        else if (n_splits <= 64) MOSAIC_COMBINE(64, 8);
        else if (n_splits <= 128) MOSAIC_COMBINE(128, 8);
        else MOSAIC_COMBINE(kMaxUnitSplits, 8);
    } else {
        if (n_splits <= 16) MOSAIC_COMBINE(16, 16);
        else if (n_splits <= 64) MOSAIC_COMBINE(64, 16);
        else MOSAIC_COMBINE(kMaxUnitSplits, 16);
    }
#undef MOSAIC_COMBINE
#pragma unroll
    for (int r = 0; r < kRowTile; ++r) red[sg][r][col] = acc[r];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int rl = sg + 8 * j;                    // row inside this workgroup's share
        if (rl >= nr) continue;
        const int r = rbase + rl;
        float o8[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) o8[q] = red[q][rl][col];
        float o[1] = {pair_sum<8>(o8)};
        combine_store<E, D, 1>(dv, u, lc, h, 0, r, dg * 32 + col, Tq, o, L_sh[r], X_sh[r], M_sh[r], out, lse);
    }
}

// The merge for questions (NT > 1).  It reads every partial once; what bounds it is the latency of those reads, which are
// other compute units' stores.  A workgroup merges CW channels of one tile; its SG = BLK / (4 CW) (at most 1: BLK threads own
// the tile's 16 x CW values) split groups take every SG-th split each.  A thread owns four channels of a row (16-byte loads; the
// lanes of a row side by side) and keeps its rows' statistics itself, kMergeBatch splits of values and statistics in flight, so that
// up to the exchange between split groups nothing is shared and no barrier is met.
// Many tiles: CW = D, one split group, no LDS (32 tokens on 28 layers, 1568 tiles of 2.3 splits on average 49 -> 21.5 us against a
// workgroup per 32 channels with its weights through LDS; 256 tokens, 448 tiles of 9 splits 15.7 -> 10.6).  Fewer tiles: 1024
// threads, two or four split groups (160 tiles of 16 splits 10.8 -> 9.6; 240 of 11 with representatives 10.3 -> 9.5, in the narrow form
// 13.6 and 17.3).  Few tiles with many splits: 32 channels and eight split groups (28 rows in 4 units, 64 splits 13.4 -> 8.3 us;
// fp32, 48 tiles of 21 splits 22.5 -> 5.8).
// grid (D / CW, NT, n_units), BLK threads.
constexpr int kMergeBatch = 8;
template <typename E, int D, int CW, int BLK>
__global__ __launch_bounds__(BLK) void k_combine_question(const DeviceView *self, int u0, int n_units, int Tq, int B, int G, E *out,
                                                          float *lse) {
    const DeviceView dv = device_view(self);
    constexpr int TPS = 16 * CW / 4 < BLK ? 16 * CW / 4 : BLK, SG = BLK / TPS, RPT = 16 * CW / 4 / TPS;   // threads of a split group, groups, rows per thread
    constexpr int LPR = CW / 4, RSTEP = TPS / LPR;          // lanes of a row, rows between a thread's rows
    const int tile = blockIdx.y, uc = blockIdx.z, u = u0 + uc, NT = gridDim.y, tid = threadIdx.x;
    const int lc = uc / dv.Hkv, h = u % dv.Hkv, rows = min(kRowTile, Tq * dv.G - tile * kRowTile);
    const int sg = tid / TPS, row0 = tid % TPS / LPR, ch = blockIdx.x * CW + tid % LPR * 4;
    int n_splits, base;                          // n_splits is 0 if the unit retrieved nothing
    if (G > 0) {
        const EvenShare sh = even_share<kShareOfUnit, sizeof(E) == 4>(dv.n_sel + u0, n_units, ChunkSize<sizeof(E) == 4>(dv), G, uc);
        n_splits = sh.splits();
        base = sh.base();
    } else {                                     // (the bf16 vector-ALU kernel)
        const SplitSlot slot = split_slot<true>(dv.n_sel + u0, n_units, B, uc);
        n_splits = slot.S;
        base = slot.base;
    }
    const size_t e0 = (size_t)base * NT + (size_t)tile * n_splits;
    const float *po = dv.part_o + (e0 * kRowTile + row0) * D + ch, *ml = dv.part_ml + e0 * kMlRows * kRowTile + row0;
    float M[RPT], L[RPT], X[RPT], acc[RPT][4];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        M[j] = -INFINITY; L[j] = 0.f; X[j] = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[j][c] = 0.f;
    }
    const int last = n_splits - 1;
    for (int s0 = sg; s0 < n_splits; s0 += SG * kMergeBatch) {
        float4 v[RPT][kMergeBatch];
        float mm[RPT][kMergeBatch], ll[RPT][kMergeBatch], xx[RPT][kMergeBatch];
#pragma unroll
        for (int i = 0; i < kMergeBatch; ++i) {
            const int s = min(s0 + SG * i, last);           // (clamped: every load is unconditional)
#pragma unroll
            for (int j = 0; j < RPT; ++j) {
                v[j][i] = *reinterpret_cast<const float4 *>(po + ((size_t)s * kRowTile + RSTEP * j) * D);
                const float *p = ml + (size_t)s * kMlRows * kRowTile + RSTEP * j;
                mm[j][i] = p[0]; ll[j][i] = p[kRowTile]; xx[j][i] = p[2 * kRowTile];
            }
        }
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            float mx = M[j];
#pragma unroll
            for (int i = 0; i < kMergeBatch; ++i) mx = fmaxf(mx, mm[j][i]);
            const float a = M[j] > -INFINITY ? exp2f(M[j] - mx) : 0.f;
            M[j] = mx;
            L[j] *= a; X[j] *= a;
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[j][c] *= a;
            float p[6][kMergeBatch];            // the batch's terms of L, X and the four channels, added in pairs
#pragma unroll
            for (int i = 0; i < kMergeBatch; ++i) {
                const bool in = s0 + SG * i <= last;        // (the same for a whole split group)
                const float w = in && mx > -INFINITY ? exp2f(mm[j][i] - mx) : 0.f;
                const float t[6] = {ll[j][i], xx[j][i], v[j][i].x, v[j][i].y, v[j][i].z, v[j][i].w};
#pragma unroll
                for (int c = 0; c < 6; ++c) p[c][i] = in ? w * t[c] : 0.f;
            }
            L[j] += pair_sum<kMergeBatch>(p[0]); X[j] += pair_sum<kMergeBatch>(p[1]);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[j][c] += pair_sum<kMergeBatch>(p[2 + c]);
        }
    }
    if constexpr (SG > 1) {
        static_assert(RPT == 1, "split groups exchange one row per thread");
        __shared__ float4 o_sh[SG][TPS];
        __shared__ float m_sh[SG][16], l_sh[SG][16], x_sh[SG][16];
        o_sh[sg][tid % TPS] = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
        if (tid % LPR == 0) { m_sh[sg][row0] = M[0]; l_sh[sg][row0] = L[0]; x_sh[sg][row0] = X[0]; }
        __syncthreads();
        if (sg != 0) return;
        float mx = -INFINITY;
#pragma unroll
        for (int g = 0; g < SG; ++g) mx = fmaxf(mx, m_sh[g][row0]);
        M[0] = mx;
        // (in pairs as above: six fp32 questions 0.79 to 1.05 -> 0.72 to 0.89 of the error with a split count per unit, the call's
        // time the same)
        float p[6][SG];
#pragma unroll
        for (int g = 0; g < SG; ++g) {
            const float mg = m_sh[g][row0], w = mx > -INFINITY ? exp2f(mg - mx) : 0.f;
            const float4 o = o_sh[g][tid];
            const float t[6] = {l_sh[g][row0], x_sh[g][row0], o.x, o.y, o.z, o.w};
#pragma unroll
            for (int c = 0; c < 6; ++c) p[c][g] = w * t[c];
        }
        L[0] = pair_sum<SG>(p[0]); X[0] = pair_sum<SG>(p[1]);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[0][c] = pair_sum<SG>(p[2 + c]);
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = row0 + RSTEP * j;
        if (r < rows) combine_store<E, D, 4>(dv, u, lc, h, tile, r, ch, Tq, acc[j], L[j], X[j], M[j], out, lse);
    }
}

} // namespace

hipError_t launch_attend_valu(const DeviceView &dv, int u0, int n_units, const void *q, int Tq,
                              int n_splits, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const int NT = (Tq * dv.G + kRowTile - 1) / kRowTile;
    const int B = n_units * n_splits;
    const dim3 grid(B + (dv.aug_reps ? n_units : 0), NT), block(kBlock);
    const unsigned short *qq = (const unsigned short *)q;
    if (dv.D == 64) launch_timed((k_attend_valu<64>), grid, block, 0, s, ev0, ev1, dv.self, u0, n_units, qq, Tq, B);
    else launch_timed((k_attend_valu<128>), grid, block, 0, s, ev0, ev1, dv.self, u0, n_units, qq, Tq, B);
    return hipGetLastError();
}

hipError_t launch_attend_combine(const DeviceView &dv, int u0, int n_units, int Tq, int n_splits,
                                 void *out, float *lse, hipStream_t s, bool uniform, Shares shares) {
    const int us = uniform ? n_splits : 0;
    const int NT = (Tq * dv.G + kRowTile - 1) / kRowTile;
    const int B = n_units * n_splits;
    if (NT > 1) {
        // A workgroup of 256 per tile where that alone is one per CU or a unit has one batch of splits on average, one of 1024
        // for 64 tiles and more, else 1024 per 32 channels (see the kernel).
        const long long tiles = (long long)NT * n_units;
        const int form = tiles >= 256 || n_splits <= kMergeBatch ? 0 : tiles >= 64 ? 1 : 2;
        const dim3 gq(form == 2 ? dv.D / 32 : 1, NT, n_units);
        auto go = [&](auto kern, int blk, auto *o) { kern<<<gq, blk, 0, s>>>(dv.self, u0, n_units, Tq, B, shares.groups, o, lse); };
        auto pick = [&](auto *o, auto d) {
            using E = std::remove_pointer_t<decltype(o)>;
            constexpr int D = decltype(d)::value;
            if (form == 0) go(k_combine_question<E, D, D, 256>, 256, o);
            else if (form == 1) go(k_combine_question<E, D, D, 1024>, 1024, o);
            else go(k_combine_question<E, D, 32, 1024>, 1024, o);
        };
        auto by_d = [&](auto *o) {
            if (dv.D == 64) pick(o, std::integral_constant<int, 64>{});
            else pick(o, std::integral_constant<int, 128>{});
        };
        if (dv.esize == 4) by_d((float *)out); else by_d((unsigned short *)out);
        return hipGetLastError();
    }
    // One row tile (a decode step) of a few units: up to eight workgroups share a tile's rows, as long as the launch
    // stays within about two workgroups per CU (per-layer launch of config 2: 1075 -> 1048 / 1033 / 1027 us per step
    // with 2 / 4 / 8; the all-layers launch, 112 units, is left alone: 542 -> 562 us with 8).
    const int RS = std::max(1, std::min(8, 512 / (n_units * (dv.D / 32))));
    const dim3 grid(dv.D / 32 * RS, n_units);
    if (dv.esize == 4) {
        if (dv.D == 64) k_attend_combine<float, 64><<<grid, kBlock, 0, s>>>(dv.self, u0, n_units, Tq, B, us, (float *)out, lse);
        else k_attend_combine<float, 128><<<grid, kBlock, 0, s>>>(dv.self, u0, n_units, Tq, B, us, (float *)out, lse);
    } else {
        if (dv.D == 64) k_attend_combine<unsigned short, 64><<<grid, kBlock, 0, s>>>(dv.self, u0, n_units, Tq, B, us, (unsigned short *)out, lse);
        else k_attend_combine<unsigned short, 128><<<grid, kBlock, 0, s>>>(dv.self, u0, n_units, Tq, B, us, (unsigned short *)out, lse);
    }
    return hipGetLastError();
}

} // namespace mosaic
