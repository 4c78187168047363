// Attention on the fp32 matrix instruction, device side: one wavefront reduces 16 tokens at a
// time for R row tiles of 16 query rows, all operands straight from global memory (no LDS staging,
// no transposes).  Shared by the fp32 attention kernel and by the workgroups that attend to the
// global representatives (whose tables are fp32 whatever the page type).
//
// Operand layout of v_mfma_f32_16x16x4_f32 (lane = 16*g + n):
//   A (16 x 4): lane holds A[n][g]      B (4 x 16): lane holds B[g][n]
//   D (16 x 16): lane holds D[4g + i][n], i = 0..3
// The contraction index may be permuted freely as long as both operands agree, which is what makes
// 16-byte loads possible:
//   Logits:  A = keys, row slot n = token n, step (j, x): channel 16j + 4g + x, so a lane's operands
//            of four steps are one float4 of its token's row; B = Q^T likewise.  Lane (g, n) then
//            owns the logits of tokens 4g + v (v = 0..3) for query row n, which is the B operand
//            of step v of the
//   Output:  A = V^T with the contraction over tokens {4g + v}: row slot n of block (bb, x) = channel
//            64bb + 4n + x, so a lane's operands of four blocks are one float4 of token 4g + v.
//            D = O^T: lane holds, for query row n, channels 64bb + 16g + 4i + x.
// Logits, weights and outputs of a row sit in the same lanes, so the online softmax needs cross-lane
// traffic only for the rare rescale.
#pragma once
#include "mosaic_internal.h"

namespace mosaic {

typedef float f32v4 __attribute__((ext_vector_type(4)));

// See the bf16 kernels: the running reference of a row is raised only when a logit exceeds it by
// more than this (log2 domain); weights are then at most 2^8.
constexpr float kLazyF32 = 8.0f;

template <int D> struct F32Operands {
    f32v4 k[D / 16];                // [j]: key channels 16j + 4g .. + 3 of token n
    f32v4 v[4][D / 64];             // [v][bb]: value channels 64bb + 4n .. + 3 of token 4g + v
    int row[4];                     // rows of tokens 4g + v, negative: no such token
};

template <bool STREAM> __device__ __forceinline__ f32v4 ld_f32v4(const float *p) {
    return STREAM ? __builtin_nontemporal_load(reinterpret_cast<const f32v4 *>(p)) : *reinterpret_cast<const f32v4 *>(p);
}

// Issues the operand loads of one group.  row_k: row of token n in the [rows][D] arrays kb and vb,
// or ~(some valid row) if the token does not exist (it is loaded all the same and gets weight 0).
template <int D, bool STREAM>
__device__ __forceinline__ void f32_issue(const float *kb, const float *vb, int row_k, int g, int n, F32Operands<D> &o) {
    const float *kr = kb + (size_t)(row_k < 0 ? ~row_k : row_k) * D + 4 * g;
#pragma unroll
    for (int j = 0; j < D / 16; ++j) o.k[j] = ld_f32v4<STREAM>(kr + 16 * j);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        o.row[v] = __shfl(row_k, 4 * g + v, 64);
        const float *vr = vb + (size_t)(o.row[v] < 0 ? ~o.row[v] : o.row[v]) * D + 4 * n;
#pragma unroll
        for (int bb = 0; bb < D / 64; ++bb) o.v[v][bb] = ld_f32v4<STREAM>(vr + 64 * bb);
    }
}

// Query rows of one tile, scaled to log2 logits once.  Lane (g, n): row n, channels 16j + 4g + x.
template <typename E, int D>
__device__ __forceinline__ void f32_load_q(const DeviceView &dv, const E *q, int lc, int h, int Tq, int row, int g,
                                           float sl2, f32v4 (&qf)[D / 16]) {
    const int G = dv.G;
    const bool some = row < Tq * G;
    const int rr = some ? row : 0, t = rr / G, gg = rr - t * G;
    const E *qr = q + (((size_t)lc * Tq + t) * dv.Hq + (size_t)h * G + gg) * D + 4 * g;
#pragma unroll
    for (int j = 0; j < D / 16; ++j) {
        f32v4 x;
        if constexpr (sizeof(E) == 4) {
            x = *reinterpret_cast<const f32v4 *>(qr + 16 * j);
        } else {
            const uint2 w = *reinterpret_cast<const uint2 *>(qr + 16 * j);
            x = f32v4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                      __uint_as_float(w.y & 0xffff0000u)};
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) qf[j][i] = some ? x[i] * sl2 : 0.f;
    }
}

// One group of 16 tokens for R row tiles.
template <int D, int R>
__device__ __forceinline__ void f32_step(F32Operands<D> &o, const f32v4 (&qf)[R][D / 16], f32v4 (&acc)[R][D / 16],
                                         float (&m)[R], float (&l)[R]) {
    constexpr int NJ = D / 16, NB = D / 64;
    f32v4 s[R][2];                  // two accumulation chains per tile
#pragma unroll
    for (int r = 0; r < R; ++r) s[r][0] = s[r][1] = f32v4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int r = 0; r < R; ++r)
                s[r][j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.k[j][x], qf[r][j][x], s[r][j & 1], 0, 0, 0);
    const bool ragged = __builtin_amdgcn_ballot_w64((o.row[0] | o.row[1] | o.row[2] | o.row[3]) < 0) != 0;
    f32v4 p[R];
#pragma unroll
    for (int r = 0; r < R; ++r) p[r] = s[r][0] + s[r][1];
    if (ragged) {                   // wave-uniform: some token does not exist -- no weight, and nothing of its value row
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool none = o.row[v] < 0;
#pragma unroll
            for (int r = 0; r < R; ++r) p[r][v] = none ? -INFINITY : p[r][v];
#pragma unroll
            for (int bb = 0; bb < NB; ++bb)
#pragma unroll
                for (int x = 0; x < 4; ++x) o.v[v][bb][x] = none ? 0.f : o.v[v][bb][x];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float cm = fmaxf(fmaxf(p[r][0], p[r][1]), fmaxf(p[r][2], p[r][3]));
        if (__builtin_amdgcn_ballot_w64(cm > m[r] + kLazyF32)) {            // rare, wave-uniform
            cm = fmaxf(cm, __shfl_xor(cm, 16, 64));
            cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
            // (a whole number: the weights of partials against each other are then powers of two, and exact)
            const float mnew = fmaxf(m[r], ceilf(cm));
            const float alpha = m[r] > -INFINITY ? __builtin_amdgcn_exp2f(m[r] - mnew) : 0.f;
            m[r] = mnew;
            l[r] *= alpha;
#pragma unroll
            for (int b = 0; b < NJ; ++b) acc[r][b] = acc[r][b] * alpha;
        }
        // (a row that has seen no token yet keeps m = -inf; its logits here are -inf too)
        const float ref = m[r] > -INFINITY ? m[r] : 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) p[r][v] = __builtin_amdgcn_exp2f(p[r][v] - ref);
        l[r] += (p[r][0] + p[r][1]) + (p[r][2] + p[r][3]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r][4 * bb + x] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.v[v][bb][x], p[r][v], acc[r][4 * bb + x], 0, 0, 0);
}

// Floats of LDS that f32_merge_waves needs.
template <int D, int NW = 4> constexpr int kF32MergeFloats = NW * D * (kRowTile + 1) + 2 * NW * kRowTile;

// Merge of the NW wavefronts' running (m, l, O) of one row tile.  All threads call it; thread
// (row, dl) = (tid / 16, tid % 16), row < 16, gets channels dl, dl + 16, ... of its row in o, and the row's M and L.
// Ends with the LDS free to be written again.
template <int D, int NW = 4>
__device__ __forceinline__ void f32_merge_waves(const f32v4 (&acc)[D / 16], float m, float l, float *lds, float (&o)[D / 16], float &M, float &L) {
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, g = lane / 16, n = lane % 16;
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    float (*o_sh)[D][kRowTile + 1] = reinterpret_cast<float (*)[D][kRowTile + 1]>(lds);
    float (*m_sh)[kRowTile] = reinterpret_cast<float (*)[kRowTile]>(lds + NW * D * (kRowTile + 1)), (*l_sh)[kRowTile] = m_sh + NW;
#pragma unroll
    for (int b = 0; b < D / 16; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) o_sh[wave][64 * (b / 4) + 16 * g + 4 * i + b % 4][n] = acc[b][i];
    if (g == 0) { m_sh[wave][n] = m; l_sh[wave][n] = l; }
    __syncthreads();
    const int row = NW == 4 ? tid / 16 : tid / 16 % kRowTile, dl = tid % 16;
    M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, m_sh[w][row]);
    float wgt[NW], x[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wgt[w] = m_sh[w][row] > -INFINITY ? __builtin_amdgcn_exp2f(m_sh[w][row] - M) : 0.f;
        x[w] = wgt[w] * l_sh[w][row];
    }
    L = pair_sum<NW>(x);
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
#pragma unroll
        for (int w = 0; w < NW; ++w) x[w] = wgt[w] * o_sh[w][dl + 16 * i][row];
        o[i] = pair_sum<NW>(x);
    }
    __syncthreads();
}

} // namespace mosaic
