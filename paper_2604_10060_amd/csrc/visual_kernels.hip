// Visual level of the nested visual-semantic hierarchy (paper Sec. V-B (1)):
// the per-frame visual embeddings are clustered once per stream, with the same
// modified K-means as the key summaries (cosine criterion, representative =
// mean of the members, Eq. 1 / Eq. 3), into P partitions that every unit's
// semantic clustering is then confined to.
//   k_visual_store   warm-up embeddings (fp32) -> the visual level's fp64 state array
//   k_visual_seed / k_visual_lloyd_assign / _update   initial P-means over the warm-up embeddings
//   k_visual_assign  greedy assignment + running-mean update
// One stream has one visual level and P <= 64: the online kernel is a single wide
// workgroup (frames depend on the frames before them), the K-means rounds spread frames
// and centroids over workgroups.  Dot products of frames and centroids are fp64 matrix
// products, the Dv channels shared out over a workgroup's wavefronts.
#include "mosaic_internal.h"
#include "assign_device.h"

namespace mosaic {

namespace {

constexpr int kVisBlock = 1024, kVisWaves = kVisBlock / 64;

// (every call site has the whole wavefront active)
__device__ __forceinline__ double wave_sum(double x) { return wave64_sum(x); }
// grid (n_frames), 256 threads
__global__ __launch_bounds__(256) void k_visual_store(DeviceView dv, const float *e_in, int f0) {
    const int i = blockIdx.x;
    const float *src = e_in + (size_t)i * dv.Dv;
    double *dst = dv.vemb + (size_t)(f0 + i) * dv.Dv;
    for (int d = threadIdx.x; d < dv.Dv; d += 256) dst[d] = (double)src[d];
}

// Sum of one value per thread over the workgroup, in a fixed order.  Every thread
// gets the result.  red: NW doubles of LDS, one per wavefront.
template <int NW>
__device__ __forceinline__ double block_sum(double x, double *red) {
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    x = wave_sum(x);
    __syncthreads();                 // the previous use of red is over
    if (lane == 0) red[wave] = x;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += red[w];
    return t;
}

// This wavefront's share of the matrix products of 16 embeddings (rows base + i * Dv, i < n_rows, the rest repeat the
// last one) with the P centroids, 16 columns per accumulator, and with each other (GRAM: the last accumulator): channels
// [ks, ke).  Layout of v_mfma_f64_16x16x4_f64: A lane (row lane%16, k lane/16), B lane (column lane%16, k lane/16),
// result register v = (row 4v + lane/16, column lane%16); step x of 16 channels from c takes channels c + 4 (lane/16) + x.
// VEC: Dv is a multiple of 4 (16-byte loads).
constexpr int kVisTiles = 4;                // P <= 64
template <typename E, bool VEC, bool GRAM>
__device__ __forceinline__ void visual_products(const DeviceView &dv, const E *base, int n_rows, int ks, int ke,
                                                f64x4 (&acc)[kVisTiles + 1]) {
    const int lane = threadIdx.x % 64, g = lane / 16, n = lane % 16, Dv = dv.Dv, P = dv.P;
    const E *row = base + (size_t)min(n, n_rows - 1) * Dv;
#pragma unroll
    for (int t = 0; t <= kVisTiles; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    auto load4 = [&](const auto *p, int c, double (&o)[4]) {
        if constexpr (VEC) {                // (c is a multiple of 4: wholly inside or outside)
            const bool in = c < ke;
            const auto *q = p + (in ? c : 0);
#pragma unroll
            for (int x = 0; x < 4; ++x) o[x] = (double)q[x];
            if (!in)
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = 0.0;
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x) o[x] = c + x < ke ? (double)p[c + x] : 0.0;
        }
    };
#pragma unroll 2
    for (int c0 = ks; c0 < ke; c0 += 16) {
        double a[4], b[kVisTiles][4];
        load4(row, c0 + 4 * g, a);
#pragma unroll
        for (int t = 0; t < kVisTiles; ++t)
            if (16 * t < P) load4(dv.vr + (size_t)min(16 * t + n, P - 1) * Dv, c0 + 4 * g, b[t]);     // (uniform)
#pragma unroll
        for (int t = 0; t < kVisTiles; ++t)
            if (16 * t < P)
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[t][x], acc[t], 0, 0, 0);
        if constexpr (GRAM)
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[kVisTiles] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], a[x], acc[kVisTiles], 0, 0, 0);
    }
}

// Initial clustering of the visual level over the first W embeddings: seeds =
// embeddings of frames floor(p*W/P), every centroid live in the first
// assignment round, `iters` rounds; a centroid left without members keeps its
// vector and is skipped afterwards.  Three small kernels per round trip of the
// algorithm, launched back to back on the stream:
//   k_visual_seed          grid (P): copy the seed embedding, its norm
//   k_visual_lloyd_assign  grid (ceil(W/16)), 256 threads: 16 frames, the channels shared by four wavefronts
//                          (W = 1024, P = 16, Dv = 1024: 73 -> 13.6 us against a wavefront per frame)
//   k_visual_lloyd_update  grid (P): members listed, then summed in ascending frame order with 32 loads in flight
//                          (159 -> 38 us against a test per frame and channel)
__global__ __launch_bounds__(kVisBlock) void k_visual_seed(DeviceView dv, int W) {
    const int tid = threadIdx.x, p = blockIdx.x, Dv = dv.Dv;
    __shared__ double red[kVisWaves];
    const double *src = dv.vemb + (size_t)(((long long)p * W) / dv.P) * Dv;
    double sq = 0.0;
    for (int d = tid; d < Dv; d += kVisBlock) { const double v = src[d]; dv.vr[(size_t)p * Dv + d] = v; sq += v * v; }
    sq = block_sum<kVisWaves>(sq, red);
    if (tid == 0) { dv.vrn[p] = sqrt(sq); dv.vn[p] = 0; }
}

template <bool VEC>
__global__ __launch_bounds__(256) void k_visual_lloyd_assign(DeviceView dv, int W, int live_all) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, P = dv.P, Dv = dv.Dv;
    const int f0 = blockIdx.x * 16, nf = min(16, W - f0);
    __shared__ double sim_sh[4][16][64];
    f64x4 acc[kVisTiles + 1];
    const int share = ((Dv + 63) / 64) * 16, ks = wave * share;
    visual_products<double, VEC, false>(dv, dv.vemb + (size_t)f0 * Dv, nf, ks, min(Dv, ks + share), acc);
#pragma unroll
    for (int t = 0; t < kVisTiles; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) sim_sh[wave][4 * v + lane / 16][16 * t + lane % 16] = acc[t][v];
    // the non-empty centroid with the largest e.r / |r| (|e| is the same factor for all of them), ties to the lowest id;
    // where that is infinite the cosine is not a number, and no candidate
    const bool live = lane < P && (live_all != 0 || dv.vn[min(lane, P - 1)] > 0);
    const double rn = dv.vrn[min(lane, P - 1)];
    __syncthreads();
    for (int i = wave; i < nf; i += 4) {
        const double x = (sim_sh[0][i][lane] + sim_sh[1][i][lane]) + (sim_sh[2][i][lane] + sim_sh[3][i][lane]);
        double c = rn == 0.0 ? 0.0 : x / rn;
        if (!live || !(fabs(c) < INFINITY)) c = -INFINITY;
        int bi = c == -INFINITY ? 0x7fffffff : lane;
        wave_best_ascending(c, bi);
        if (lane == 0) dv.part[f0 + i] = bi == 0x7fffffff ? 0 : bi;
    }
}

__global__ __launch_bounds__(kVisBlock) void k_visual_lloyd_update(DeviceView dv, int W) {
    constexpr int CH = kVisBlock * kListPer;
    const int tid = threadIdx.x, p = blockIdx.x, Dv = dv.Dv;
    __shared__ double red[kVisWaves];
    __shared__ int mem[CH];
    __shared__ int wtot[kVisWaves];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};   // channels tid, tid + 1024, ... (Dv <= 4096)
    int count = 0;
    for (int c0 = 0; c0 < W; c0 += CH) {
        const int m = list_members<kVisBlock>(dv.part, p, c0, W, mem, wtot);
        count += m;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int d = tid + kVisBlock * i;
            if (d < Dv) acc[i] = add_members<32>(acc[i], mem, m, [&](int f) { return dv.vemb[(size_t)f * Dv + d]; });
        }
    }
    if (count == 0) {                                    // workgroup-uniform
        if (tid == 0) dv.vn[p] = 0;
        return;
    }
    double sq = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int d = tid + kVisBlock * i;
        if (d < Dv) {
            const double rv = acc[i] / (double)count;
            dv.vr[(size_t)p * Dv + d] = rv;
            sq += rv * rv;
        }
    }
    sq = block_sum<kVisWaves>(sq, red);
    if (tid == 0) { dv.vrn[p] = sqrt(sq); dv.vn[p] = count; }
}

// One frame by itself, all threads of a workgroup: the embedding is staged in LDS, a wavefront scores two
// centroids at a time (their rows' loads in flight together), all threads update the winner's row.  changed(a, n, norm) is
// called by thread 0 with the new size and norm of the row.  The caller orders calls by a barrier.
constexpr int kVisAssign = 512;             // threads of the online kernels
constexpr int kVisChannels = 4096;          // visual_dim at most
static_assert(chain_error(kVisChannels / (kVisAssign / 64) + kVisAssign / 64) < kChainMargin / 5,
              "a wavefront's share of the channels, then the wavefronts' sums");
struct VisualTurnShared {
    double e[kVisChannels], red[kVisAssign / 64], bv[kVisAssign / 64];
    int bi[kVisAssign / 64];
};
template <typename Changed>
__device__ __forceinline__ void visual_in_turn(const DeviceView &dv, const float *src, int f, VisualTurnShared &sh, Changed changed) {
    constexpr int NW = kVisAssign / 64;
    const int tid = threadIdx.x, lane = tid % 64, Dv = dv.Dv, P = dv.P;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    for (int d = tid; d < Dv; d += kVisAssign) {
        const double v = (double)src[d];
        sh.e[d] = v;
        dv.vemb[(size_t)f * Dv + d] = v;
    }
    __syncthreads();
    double en = 0.0;
    for (int d = lane; d < Dv; d += 64) en = __builtin_fma(sh.e[d], sh.e[d], en);
    en = sqrt(wave_sum(en));
    double bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int p = wave; p < P; p += 2 * NW) {
        const int p2 = p + NW < P ? p + NW : p;
        const double *ra = dv.vr + (size_t)p * Dv, *rb = dv.vr + (size_t)p2 * Dv;
        const int na = dv.vn[p], nb = p2 != p ? dv.vn[p2] : 0;
        const double rna = dv.vrn[p], rnb = dv.vrn[p2];
        double xa = 0.0, xb = 0.0;
#pragma unroll 8
        for (int d = lane; d < Dv; d += 64) { xa = __builtin_fma(sh.e[d], ra[d], xa); xb = __builtin_fma(sh.e[d], rb[d], xb); }
        xa = wave_sum(xa);
        xb = wave_sum(xb);
        const double ca = (en == 0.0 || rna == 0.0) ? 0.0 : xa / (en * rna), cb = (en == 0.0 || rnb == 0.0) ? 0.0 : xb / (en * rnb);
        if (na > 0 && ca > bv) { bv = ca; bi = p; }              // (ids ascend: a strict comparison keeps the lowest)
        if (nb > 0 && cb > bv) { bv = cb; bi = p2; }
    }
    if (lane == 0) { sh.bv[wave] = bv; sh.bi[wave] = bi; }
    __syncthreads();
    bv = -INFINITY;
    bi = 0x7fffffff;
#pragma unroll
    for (int w = 0; w < NW; ++w)
        if (sh.bv[w] > bv || (sh.bv[w] == bv && sh.bi[w] < bi)) { bv = sh.bv[w]; bi = sh.bi[w]; }
    const int a = bi == 0x7fffffff ? 0 : bi, na = dv.vn[a];
    const double y = __ddiv_rn(1.0, (double)na + 1.0);
    double sq = 0.0;
    for (int d = tid; d < Dv; d += kVisAssign) {
        const double x = eq3_channel((double)na, y, dv.vr[(size_t)a * Dv + d], sh.e[d]);
        dv.vr[(size_t)a * Dv + d] = x;
        sq = __builtin_fma(x, x, sq);
    }
    sq = block_sum<NW>(sq, sh.red);     // (its barriers also order the reads of vn[a] before the update)
    if (tid == 0) {
        const double norm = sqrt(sq);
        dv.vrn[a] = norm;
        dv.vn[a] = na + 1;
        dv.part[f] = a;
        changed(a, na + 1, norm);
    }
}

// Frames f0..f1-1: partition = most similar non-empty visual centroid, which then moves by Eq. 3.  grid (1), kVisAssign
// threads.  e_in: the fp32 embeddings of these frames as the caller passed them; the kernel also files them in the visual
// level's state array.  The frames are taken up to sixteen at a time, as k_assign_chain does for the semantic level (which
// says why the decisions are exact): products of the chunk with all centroids and with itself, the channels shared out
// over the wavefronts; the decisions from those; Eq. 3 on the rows of the centroids that the chunk moved, a thread per
// channel.  Where a chunk begins with a frame that is too close to call, its frames are taken in turn.  (16 frames, P = 16,
// Dv = 1024: 90.5 -> 26 us against one frame at a time.)
template <bool VEC>
__global__ __launch_bounds__(kVisAssign) void k_visual_assign(DeviceView dv, const float *e_in, int f0, int f1) {
    constexpr int NW = kVisAssign / 64, FR = kChainFrames, kNone = 0x7fffffff;
    const int tid = threadIdx.x, lane = tid % 64, Dv = dv.Dv, P = dv.P, g = lane / 16, n = lane % 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    __shared__ double part_sh[NW][256];
    __shared__ double sim_sh[FR * 64], gram_sh[FR][FR + 1], red[NW], irn_sh[64];
    __shared__ double ss_sh[FR], sn_sh[FR], isn_sh[FR], out_sh[FR], y_sh[FR];
    __shared__ VisualTurnShared turn_sh;
    __shared__ int vn_sh[64], slot_sh[64], lo_sh[FR], near_sh[FR], sure_sh[FR], w_sh[FR], p_sh[FR], slot_id[FR], n_slot_sh, nc_sh, tied_sh;
    if (tid < 64) {
        const double rn = tid < P ? dv.vrn[tid] : 0.0;
        vn_sh[tid] = tid < P ? dv.vn[tid] : 0;
        irn_sh[tid] = rn > 0.0 ? 1.0 / rn : 0.0;
        slot_sh[tid] = -1;
        if (tid < FR) lo_sh[tid] = 0;
    }
    const int share = (Dv + 16 * NW - 1) / (16 * NW) * 16, ks = min(Dv, wave * share);
    InTurn turn;
    for (int c0 = f0; c0 < f1;) {
        int nc = min(FR, f1 - c0);
        const float *e = e_in + (size_t)(c0 - f0) * Dv;
        bool in_turn = turn.left > 0;       // workgroup-uniform
        if (in_turn) {
            --turn.left;
        } else {
            // ---- products ----
            f64x4 acc[kVisTiles + 1];
            visual_products<float, VEC, true>(dv, e, nc, ks, min(Dv, ks + share), acc);
#pragma unroll
            for (int t = 0; t <= kVisTiles; ++t) {
                if (t < kVisTiles && 16 * t >= P) continue;              // workgroup-uniform
                __syncthreads();                // (the first one also orders the tables above and the chunk before)
#pragma unroll
                for (int v = 0; v < 4; ++v) part_sh[wave][(4 * v + g) * 16 + n] = acc[t][v];
                __syncthreads();
                if (tid < 256) {
                    double x = 0.0;
#pragma unroll
                    for (int w = 0; w < NW; ++w) x += part_sh[w][tid];
                    const int f = tid / 16, c = tid % 16, p = 16 * t + c;
                    if (t == kVisTiles) gram_sh[f][c] = x;
                    else if (p < P) sim_sh[f * P + p] = vn_sh[p] > 0 ? x : -INFINITY;
                }
            }
            __syncthreads();
            if (wave == 0) {
                const double ss = n < nc ? gram_sh[n][n] : 0.0, is = fast_rsqrt(ss);
                double x[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = gram_sh[4 * v + g][n] * is;
                wave_sync();
#pragma unroll
                for (int v = 0; v < 4; ++v) gram_sh[4 * v + g][n] = x[v];
                if (g == 0) { ss_sh[n] = ss; sn_sh[n] = ss * is; isn_sh[n] = is; }
            }
            __syncthreads();
            for (int f = wave; f < nc; f += NW) {                    // the nearest centroid under the table as it stands
                const double d = lane < P ? sim_sh[f * P + lane] : -INFINITY;
                double c = d == -INFINITY ? d : d * isn_sh[f] * irn_sh[lane];
                const bool odd = __ballot(!(c == c)) != 0;
                if (!(c == c)) c = -INFINITY;
                double bv = c;
                int bi = c == -INFINITY ? kNone : lane;
                wave_best_ascending(bv, bi);
                const double second = wave_max(lane == bi ? -INFINITY : c);
                bool sure = bi != kNone && !odd && bv - second > kChainMargin;
                if (ss_sh[f] == 0.0) {          // (wave-uniform) a zero embedding: similarity 0 with every live centroid, the lowest id
                    const unsigned long long live = __ballot(lane < P && vn_sh[lane] > 0);
                    bi = live ? __ffsll((long long)live) - 1 : kNone;
                    sure = live != 0;
                }
                if (lane == 0) { near_sh[f] = bi; out_sh[f] = second; sure_sh[f] = sure; }
            }
            __syncthreads();
            in_turn = !sure_sh[0];
            if (in_turn) turn.failed();
        }
        if (in_turn) {
            for (int fc = 0; fc < nc; ++fc) {
                visual_in_turn(dv, e + (size_t)fc * Dv, c0 + fc, turn_sh, [&](int a, int size, double norm) {
                    vn_sh[a] = size;
                    irn_sh[a] = norm > 0.0 ? 1.0 / norm : 0.0;
                });
                __syncthreads();
            }
            c0 += nc;
            continue;
        }
        // ---- decisions ----
        if (wave == 0) {
            int mine = lane < nc ? near_sh[lane] : -1;
            if (mine == kNone) mine = -1;   // (no live candidate: the chunk ends before the frame)
            unsigned long long left = __ballot(mine >= 0);
            int k = 0;
            while (left) {
                const int id = __builtin_amdgcn_readlane(mine, __ffsll((long long)left) - 1);
                if (lane == 0) { slot_id[k] = id; slot_sh[id] = k; }
                left &= ~__ballot(mine == id);
                ++k;
            }
            wave_sync();
            int w = n < nc && near_sh[n] != kNone ? slot_sh[near_sh[n]] : -1;
            bool tied;
            const int done =
                chain_decide({sim_sh, P, lo_sh, sn_sh, isn_sh, ss_sh, out_sh, gram_sh, slot_id, vn_sh, irn_sh}, nc, k, w, tied);
            if (lane < done) {
                const int id = slot_id[w];
                int p = vn_sh[id];
#pragma unroll
                for (int h = 0; h < FR - 1; ++h) p += h < lane && __builtin_amdgcn_readlane(w, h) == w ? 1 : 0;
                w_sh[lane] = w;
                p_sh[lane] = p;
                y_sh[lane] = __ddiv_rn(1.0, (double)p + 1.0);
                dv.part[c0 + lane] = id;
            }
            if (lane == 0) { nc_sh = done; n_slot_sh = k; tied_sh = tied; }
        }
        __syncthreads();
        nc = nc_sh;
        if (tied_sh) turn.failed();
        else turn.held();
        const int n_slot = n_slot_sh;
        // ---- Eq. 3 on the rows; the frames' states ----
        for (int k = 0; k < n_slot; ++k) {
            const int id = slot_id[k];
            int cnt = 0;
            for (int fc = 0; fc < nc; ++fc) cnt += w_sh[fc] == k;
            if (cnt > 0) {                  // workgroup-uniform
                double sq = 0.0;
                for (int d = tid; d < Dv; d += kVisAssign) {
                    const double xs = dv.vr[(size_t)id * Dv + d];
                    double x = xs;
                    float ev[FR];
#pragma unroll
                    for (int fc = 0; fc < FR; ++fc) ev[fc] = e[(size_t)min(fc, nc - 1) * Dv + d];
#pragma unroll
                    for (int fc = 0; fc < FR; ++fc)
                        if (fc < nc && w_sh[fc] == k) x = eq3_finite((double)p_sh[fc], y_sh[fc], x, (double)ev[fc]);
                    if (!(x == x)) {        // infinite states: over again
                        x = xs;
                        for (int fc = 0; fc < nc; ++fc)
                            if (w_sh[fc] == k) x = eq3_channel((double)p_sh[fc], y_sh[fc], x, (double)e[(size_t)fc * Dv + d]);
                    }
                    dv.vr[(size_t)id * Dv + d] = x;
                    sq = __builtin_fma(x, x, sq);
                }
                sq = block_sum<NW>(sq, red);
                if (tid == 0) {
                    const double rn = sqrt(sq);
                    vn_sh[id] += cnt;
                    irn_sh[id] = rn > 0.0 ? 1.0 / rn : 0.0;
                    dv.vn[id] = vn_sh[id];
                    dv.vrn[id] = rn;
                }
            }
            if (tid == 0) slot_sh[id] = -1;
        }
        for (int i = tid; i < nc * Dv; i += kVisAssign) dv.vemb[(size_t)c0 * Dv + i] = (double)e[i];
        c0 += nc;
        __syncthreads();
    }
}

// The same for calls of at most kVisFew frames, all of them in turn.  The chunk form's products, reductions and check cost 4
// us more for one frame (P = 10, Dv = 512, C = 120, whole call 16.6 against 12.2 us).
constexpr int kVisFew = 2;
__global__ __launch_bounds__(kVisAssign) void k_visual_assign_few(DeviceView dv, const float *e_in, int f0, int f1) {
    __shared__ VisualTurnShared sh;
    for (int f = f0; f < f1; ++f) {
        if (f > f0) __syncthreads();
        visual_in_turn(dv, e_in + (size_t)(f - f0) * dv.Dv, f, sh, [](int, int, double) {});
    }
}

hipError_t after_launch() {
    return hipGetLastError();
}

} // namespace

hipError_t launch_visual_store(const DeviceView &dv, const float *e_in, int f0, int n_frames, hipStream_t s) {
    k_visual_store<<<n_frames, 256, 0, s>>>(dv, e_in, f0);
    return after_launch();
}

hipError_t launch_visual_lloyd(const DeviceView &dv, int W, int iters, hipStream_t s) {
    k_visual_seed<<<dv.P, kVisBlock, 0, s>>>(dv, W);
    hipError_t e = after_launch();
    for (int it = 0; it < iters && e == hipSuccess; ++it) {
        if (dv.Dv % 4 == 0) k_visual_lloyd_assign<true><<<(W + 15) / 16, 256, 0, s>>>(dv, W, it == 0);
        else k_visual_lloyd_assign<false><<<(W + 15) / 16, 256, 0, s>>>(dv, W, it == 0);
        if ((e = after_launch()) != hipSuccess) break;
        k_visual_lloyd_update<<<dv.P, kVisBlock, 0, s>>>(dv, W);
        e = after_launch();
    }
    return e;
}

hipError_t launch_visual_assign(const DeviceView &dv, const float *e_in, int f0, int f1, hipStream_t s) {
    if (f1 - f0 <= kVisFew) k_visual_assign_few<<<1, kVisAssign, 0, s>>>(dv, e_in, f0, f1);
    else if (dv.Dv % 4 == 0) k_visual_assign<true><<<1, kVisAssign, 0, s>>>(dv, e_in, f0, f1);
    else k_visual_assign<false><<<1, kVisAssign, 0, s>>>(dv, e_in, f0, f1);
    return after_launch();
}

} // namespace mosaic
