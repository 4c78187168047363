// Page store + summaries (paper Sec. V-A (1), Sec. VI-A), device part.  store_key_page / store_value_page are run by one
// workgroup of NT threads per (unit, frame): the page goes to the arena's store (HBM
// tier) or the staging ring (host tier); the key summary (mean of the frame's T key
// vectors, fp64) goes to dv.summ and, if s_out is given, to that LDS array too.
#pragma once
#include "mosaic_internal.h"

namespace mosaic {

// NT threads share a row of D channels in pieces of 2048 / NT elements, so that whatever NT is, kStoreRows rows are summed side by side:
// the additions of a summary are the same.  512 threads in page stores (256 / 512: one frame of 28 layers 4.42 / 4.16 us, sixteen of four layers 6.29 /
// 5.70, sixteen of 28 layers 28.2 / 26.7), 256 where the assignment of the frame follows in the same workgroup (5.90 / 6.39).
constexpr int kStoreBlock = 512;
template <int D> constexpr int kStoreRows = 2048 / D;

constexpr int kStoreTile = 64;          // tokens of a value page transposed at a time (two chunks)
template <int D> union StoreShared {    // LDS of a page store
    double red[kStoreRows<D>][D];
    unsigned short tile[kStoreTile][D + 2];
};

// BEYOND: the store is far beyond the caches (see issue_chunk() for the loads of such pages), and so its pages are written with the hint, too.
// Re-clustered ingest of 28 layers, page stores beside the K-means rounds of the batch before: a round's assignment 34.7 -> 32.4 us, its
// update 27.1 -> 22.8 us on average, a page store 26.8 -> 25.8.  Not in one-frame calls (5.83 -> 6.06 us), nor where the next question finds the pages in a cache.
template <bool BEYOND, typename W> __device__ __forceinline__ void keep_words(W *p, W w) {
    if constexpr (BEYOND) __builtin_nontemporal_store(w, p);
    else *p = w;
}

// N elements of a row of D.  The caller's rows are read once: their loads carry the non-temporal hint, so that they displace less of what the kernels
// beside and after a page store work with.  What a lane takes of more than 16 bytes are pieces of 16, as far apart as the row has pieces: a wavefront's load is
// then whole lines.  (With 32 bytes side by side each of the two loads takes half of every line, and a hinted line is fetched for both.)
// One frame of 112 units in one call, assignment included, us; without the hint / hinted, 32 bytes side by side / hinted, 16-byte pieces.
// Frames that lie in no cache: bf16, 196 tokens of 128 channels 9.4 / - / 8.8, fp32 14.2 / 14.0 / 12.4, fp32, 64 channels 9.2 / 8.6 / 7.6; frames that a kernel
// has just written: 6.6 / - / 5.7, 11.6 / 12.4 / 10.7, 5.8 / 5.8 / 5.0.  (A frame that an earlier call took, and nothing has
// written since, is faster without it: 7.9 / 8.8 in bf16, 11.5 / 14.0 / 12.4 in fp32.)
template <typename E, int D, int N> struct RowPiece {
    static constexpr int W = N * (int)sizeof(E) / 4, PIECES = W > 4 ? W / 4 : 1, PW = W / PIECES, PN = N / PIECES;
    typedef unsigned int Words __attribute__((ext_vector_type(PW)));
    Words w[PIECES];
    static __device__ __forceinline__ int first(int lane) { return lane * PN; }                       // a lane's first channel,
    static __device__ __forceinline__ constexpr int next(int i) { return i / PN * (D / PIECES) + i % PN; }    // and its i-th from there
    __device__ __forceinline__ unsigned int word(int i) const { return w[i / PW][i % PW]; }
    __device__ __forceinline__ void load(const E *p) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) w[i] = __builtin_nontemporal_load(reinterpret_cast<const Words *>(p + i * (D / PIECES)));
    }
    template <bool BEYOND> __device__ __forceinline__ void store(E *p) const {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) keep_words<BEYOND>(reinterpret_cast<Words *>(p + i * (D / PIECES)), w[i]);
    }
    __device__ __forceinline__ void unpack(float (&v)[N]) const {
#pragma unroll
        for (int i = 0; i < W; ++i) {
            if constexpr (sizeof(E) == 4) v[i] = __uint_as_float(word(i));
            else {
                v[2 * i] = __uint_as_float(word(i) << 16);
                v[2 * i + 1] = __uint_as_float(word(i) & 0xffff0000u);
            }
        }
    }
};

template <typename E, int D, int NT, bool BEYOND>
__device__ __forceinline__ void store_key_page(const DeviceView &dv, const E *k_in, char *kdst_base, int u, int fl,
                                               int f, StoreShared<D> &sh, double *s_out) {
    constexpr int RP = kStoreRows<D>, LPR = NT / RP, N = D / LPR;      // rows per pass, lanes per row, elements each
    const int tid = threadIdx.x, c0 = RowPiece<E, D, N>::first(tid % LPR), r0 = tid / LPR;
    const int T = dv.T;
    const size_t in_page = ((size_t)fl * dv.U + u) * (size_t)T * D;
    const size_t page = (size_t)u * dv.F + f;          // summary slot
    const bool host = dv.tier == MOSAIC_TIER_HOST;
    const size_t spage = host ? (size_t)(f % dv.SN) * dv.U + u : (size_t)u * dv.PU + f;
    const E *src = k_in + in_page + c0;
    // (a thread's channels lie in one of the pieces that bf16 keys are stored in; fp32 pages are row by row)
    E *dst = reinterpret_cast<E *>(kdst_base) + spage * (size_t)T * D + c0 / 32 * dv.k_ps() + c0 % 32;
    double acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.0;
    // four rows' loads in flight (row clamped, loads unconditional): one row at a time, a load waits for the store before
    // it, which may alias it for all the compiler knows, and a 64-token page is four trips to memory instead of one (28
    // layers, one frame a call: 12.2 -> 9.0 us a frame; 64 a call, C = 20: 6.5 -> 4.9)
    for (int t0 = r0; t0 < T; t0 += 4 * RP) {
        RowPiece<E, D, N> x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k].load(src + (size_t)min(t0 + k * RP, T - 1) * D);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (t0 + k * RP < T) {
                float v[N];
                x[k].unpack(v);
                x[k].template store<BEYOND>(dst + (size_t)(t0 + k * RP) * dv.k_rs());
#pragma unroll
                for (int i = 0; i < N; ++i) acc[i] += (double)v[i];
            }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) sh.red[r0][c0 + RowPiece<E, D, N>::next(i)] = acc[i];
    __syncthreads();
    if (tid < D) {
        double sm = 0.0;
        for (int rr = 0; rr < RP; ++rr) sm += sh.red[rr][tid];
        sm /= (double)T;
        dv.summ[page * D + tid] = sm;
        if (s_out) s_out[tid] = sm;
    }
}

template <typename E, int D, int NT, bool BEYOND>
__device__ __forceinline__ void store_value_page(const DeviceView &dv, const E *v_in, char *vdst_base, int u, int fl,
                                                 int f, StoreShared<D> &sh) {
    constexpr int RP = kStoreRows<D>, LPR = NT / RP, N = D / LPR;
    const int tid = threadIdx.x, c0 = RowPiece<E, D, N>::first(tid % LPR), r0 = tid / LPR;
    const int T = dv.T;
    const size_t in_page = ((size_t)fl * dv.U + u) * (size_t)T * D;
    const size_t page = (size_t)u * dv.F + f;
    const bool host = dv.tier == MOSAIC_TIER_HOST;
    const size_t spage = host ? (size_t)(f % dv.SN) * dv.U + u : (size_t)u * dv.PU + f;
    // With the global-representative augmentation on, the frame's value summary (mean of
    // its T value vectors, fp64) is formed next to the copy, like the key summary.
    const E *src = v_in + in_page + c0;
    if (!dv.v_transposed) {
        E *dst = reinterpret_cast<E *>(vdst_base) + spage * (size_t)T * D + c0;
        double acc[N];
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = 0.0;
        for (int t0 = r0; t0 < T; t0 += 4 * RP) {      // (as in store_key_page)
            RowPiece<E, D, N> x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k].load(src + (size_t)min(t0 + k * RP, T - 1) * D);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (t0 + k * RP < T) {
                    x[k].template store<BEYOND>(dst + (size_t)(t0 + k * RP) * D);
                    if (dv.vsumm) {
                        float v[N];
                        x[k].unpack(v);
#pragma unroll
                        for (int i = 0; i < N; ++i) acc[i] += (double)v[i];
                    }
                }
        }
        if (dv.vsumm) {
#pragma unroll
            for (int i = 0; i < N; ++i) sh.red[r0][c0 + RowPiece<E, D, N>::next(i)] = acc[i];
            __syncthreads();
            if (tid < D) {
                double sv = 0.0;
                for (int rr = 0; rr < RP; ++rr) sv += sh.red[rr][tid];
                dv.vsumm[page * D + tid] = sv / (double)T;
            }
        }
        return;
    }
    // Transposed, chunk-blocked value page [Tp/32][D][32] (2-byte elements only):
    // 8 consecutive tokens of one channel form one 16-byte operand of the PV
    // contraction, and the 16 channels x 32 tokens a wavefront loads at once
    // are one contiguous KiB.  Tokens T..Tp-1 are written as zeros.
    if constexpr (sizeof(E) == 2) {
        constexpr int TC = kStoreTile;
        const int Tp = dv.Tp;
        double vacc = 0.0;
        unsigned short *dst = reinterpret_cast<unsigned short *>(vdst_base) + spage * (size_t)D * Tp;
        // a tile's rows are loaded together (row clamped, loads unconditional), the next tile's while this one is written out
        constexpr int RPT = TC / RP;                 // rows per thread and tile
        RowPiece<E, D, N> w[RPT];
        auto load_tile = [&](int tc0) {
#pragma unroll
            for (int k = 0; k < RPT; ++k) w[k].load(src + (size_t)min(tc0 + r0 + k * RP, T - 1) * D);
        };
        load_tile(0);
        for (int tc0 = 0; tc0 < Tp; tc0 += TC) {
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                const bool in = tc0 + r0 + k * RP < T;
                unsigned int *row = reinterpret_cast<unsigned int *>(&sh.tile[r0 + k * RP][c0]);
#pragma unroll
                for (int i = 0; i < RowPiece<E, D, N>::W; ++i) row[i] = in ? w[k].word(i) : 0u;
            }
            if (tc0 + TC < Tp) load_tile(tc0 + TC);
            __syncthreads();
            if (dv.vsumm && tid < D) {
                const int nt = min(TC, T - tc0);     // real tokens in this tile
                for (int t = 0; t < nt; ++t) vacc += (double)bf16_to_f32(sh.tile[t][tid]);
            }
            const int ntg = (min(TC, Tp - tc0)) / 8;  // token groups of 8 in this tile
            for (int id = tid; id < D * ntg; id += NT) {
                const int d = id / ntg, tg = id % ntg;
                unsigned int o[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o[j] = (unsigned int)sh.tile[tg * 8 + 2 * j][d] |
                           ((unsigned int)sh.tile[tg * 8 + 2 * j + 1][d] << 16);
                const int tok = tc0 + tg * 8;         // first of the 8 tokens
                typedef unsigned int Words __attribute__((ext_vector_type(4)));
                keep_words<BEYOND>(reinterpret_cast<Words *>(dst + ((size_t)(tok / kChunk) * D + d) * kChunk + tok % kChunk), Words{o[0], o[1], o[2], o[3]});
            }
            __syncthreads();
        }
        if (dv.vsumm && tid < D) dv.vsumm[page * D + tid] = vacc / (double)T;
    }
}

} // namespace mosaic
