// Visual level of the nested visual-semantic hierarchy (paper Sec. V-B (1)):
// the per-frame visual embeddings are clustered once per stream, with the same
// modified K-means as the key summaries (cosine criterion, representative =
// mean of the members, Eq. 1 / Eq. 3), into P partitions that every unit's
// semantic clustering is then confined to.
//   (warm-up embeddings (fp32) are filed in the visual level's fp64 state array by the page stores' launch)
//   k_visual_seed / k_visual_lloyd_assign / _update   initial P-means over the warm-up embeddings
//   k_visual_assign  greedy assignment + running-mean update
// One stream has one visual level and P <= 64: the online kernel is a single wide
// workgroup (frames depend on the frames before them), the K-means rounds spread frames
// and centroids over workgroups.  Dot products of frames and centroids are fp64 matrix
// products, the Dv channels shared out over a workgroup's wavefronts.
#include <type_traits>

#include "mosaic_internal.h"
#include "assign_device.h"
#include "page_store_device.h"

namespace mosaic {

namespace {

constexpr int kVisBlock = 1024, kVisWaves = kVisBlock / 64;

// (every call site has the whole wavefront active)
__device__ __forceinline__ double wave_sum(double x) { return wave64_sum(x); }
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
// TILES: columns (16 TILES >= P).  What bounds it is the trip to memory of its operands: up to eight steps' loads are in flight.
constexpr int kVisTiles = 4;                // at most
static_assert(16 * kVisTiles >= kMaxPartitions, "a column for every centroid");
template <typename E, bool VEC, bool GRAM, int TILES>
__device__ __forceinline__ void visual_products(const DeviceView &dv, const E *base, int n_rows, int ks, int ke,
                                                f64x4 (&acc)[TILES + 1]) {
    constexpr int UN = TILES == 1 ? 8 : TILES == 2 ? 4 : 2;
    const int lane = threadIdx.x % 64, g = lane / 16, n = lane % 16, Dv = dv.Dv, P = dv.P;
    const E *row = base + (size_t)min(n, n_rows - 1) * Dv;
#pragma unroll
    for (int t = 0; t <= TILES; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    auto load4 = [&](const auto *p, int c, auto (&o)[4]) {
        if constexpr (VEC) {                // (c is a multiple of 4: wholly inside or outside)
            const bool in = c < ke;
            const auto *q = p + (in ? c : 0);
#pragma unroll
            for (int x = 0; x < 4; ++x) o[x] = q[x];
            if (!in)
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = 0;
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const auto v = p[min(c + x, Dv - 1)];
                o[x] = c + x < ke ? v : 0;
            }
        }
    };
    for (int c0 = ks; c0 < ke; c0 += 16 * UN) {
        E a[UN][4];
        double b[UN][TILES][4];
#pragma unroll
        for (int s = 0; s < UN; ++s) {
            load4(row, c0 + 16 * s + 4 * g, a[s]);
#pragma unroll
            for (int t = 0; t < TILES; ++t) load4(dv.vr + (size_t)min(16 * t + n, P - 1) * Dv, c0 + 16 * s + 4 * g, b[s][t]);
        }
#pragma unroll
        for (int s = 0; s < UN; ++s) {
            if (s > 0 && c0 + 16 * s >= ke) break;                       // (uniform)
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[s][x], b[s][t][x], acc[t], 0, 0, 0);
            if constexpr (GRAM)
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[TILES] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[s][x], (double)a[s][x], acc[TILES], 0, 0, 0);
        }
    }
}

// While the initial clustering runs, a centroid's squared norm is sixteen sums, one per wavefront that a workgroup of kVisBlock threads
// with a thread per channel would have (in the partitions' key-space representatives, which are formed after it).
__device__ __forceinline__ double *visual_norm_parts(const DeviceView &dv, int p) {
    static_assert(kVisWaves <= 64, "a partition's row of representatives holds the parts");
    return dv.pr + (size_t)p * kVisWaves;
}
__device__ __forceinline__ double visual_norm(const DeviceView &dv, int p) {
    const double *part = visual_norm_parts(dv, p);
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kVisWaves; ++w) t += part[w];
    return sqrt(t);
}

// Initial clustering of the visual level over the first W embeddings: seeds =
// embeddings of frames floor(p*W/P), every centroid live in the first
// assignment round, `iters` rounds; a centroid left without members keeps its
// vector and is skipped afterwards.  Three small kernels per round trip of the
// algorithm, launched back to back on the stream:
//   k_visual_seed          grid (P): copy the seed embedding, its norm
//   k_visual_lloyd_assign  grid (ceil(W/16)), 256 threads: 16 frames, the channels shared by four wavefronts
//                          (W = 1024, P = 16, Dv = 1024: a wavefront per frame 73 us, operands in eight trips to memory 13.4, in two 10.7)
//   k_visual_lloyd_update  grid (P, 4), 256 threads: members listed, then summed in ascending frame order with 32 loads in flight
//                          (159 us with a test per frame and channel, 38 with a workgroup of 1024 per centroid, whose CU takes in
//                          what it can, now 17)
__global__ __launch_bounds__(kVisBlock) void k_visual_seed(const DeviceView *self, int W) {
    const DeviceView dv = device_view(self);
    const int tid = threadIdx.x, p = blockIdx.x, Dv = dv.Dv;
    const double *src = dv.vemb + (size_t)(((long long)p * W) / dv.P) * Dv;
    double sq = 0.0;
    for (int d = tid; d < Dv; d += kVisBlock) { const double v = src[d]; dv.vr[(size_t)p * Dv + d] = v; sq += v * v; }
    sq = wave_sum(sq);
    if (tid % 64 == 0) visual_norm_parts(dv, p)[tid / 64] = sq;
    if (tid == 0) dv.vn[p] = 0;
}

// the norms of all centroids from their parts.  grid (1), 64 threads
__global__ __launch_bounds__(64) void k_visual_norms(const DeviceView *self) {
    const DeviceView dv = device_view(self);
    if ((int)threadIdx.x < dv.P) dv.vrn[threadIdx.x] = visual_norm(dv, threadIdx.x);
}

template <bool VEC, int TILES>
__global__ __launch_bounds__(256) void k_visual_lloyd_assign(const DeviceView *self, int W, int live_all) {
    const DeviceView dv = device_view(self);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, P = dv.P, Dv = dv.Dv;
    const int f0 = blockIdx.x * 16, nf = min(16, W - f0);
    __shared__ double sim_sh[4][16][64];
    f64x4 acc[TILES + 1];
    const int share = ((Dv + 63) / 64) * 16, ks = min(Dv, wave * share);
    visual_products<double, VEC, false, TILES>(dv, dv.vemb + (size_t)f0 * Dv, nf, ks, min(Dv, ks + share), acc);
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) sim_sh[wave][4 * v + lane / 16][16 * t + lane % 16] = acc[t][v];
    // the non-empty centroid with the largest e.r / |r| (|e| is the same factor for all of them), ties to the lowest id;
    // where that is infinite the cosine is not a number, and no candidate
    const bool live = lane < P && (live_all != 0 || dv.vn[min(lane, P - 1)] > 0);
    const double rn = visual_norm(dv, min(lane, P - 1));
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

constexpr int kVisUpdate = 256;             // threads; workgroup y has channels 256 y .. 256 y + 255, and those 1024, 2048, 3072 further on
__global__ __launch_bounds__(kVisUpdate) void k_visual_lloyd_update(const DeviceView *self, int W) {
    const DeviceView dv = device_view(self);
    constexpr int CH = kVisUpdate * kListPer;
    const int tid = threadIdx.x, p = blockIdx.x, Dv = dv.Dv, c = blockIdx.y * kVisUpdate + tid;
    __shared__ int mem[CH];
    __shared__ int wtot[kVisUpdate / 64];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};   // channels c, c + 1024, ... (Dv <= 4096)
    int count = 0;
    for (int c0 = 0; c0 < W; c0 += CH) {
        const int m = list_members<kVisUpdate>(dv.part, p, c0, W, mem, wtot);
        count += m;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int d = c + kVisBlock * i;
            if (d < Dv) acc[i] = add_members<32>(acc[i], mem, m, [&](int f) { return dv.vemb[(size_t)f * Dv + d]; });
        }
    }
    if (blockIdx.y == 0 && tid == 0) dv.vn[p] = count;
    if (count == 0) return;                 // workgroup-uniform: it keeps its vector
    double sq = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int d = c + kVisBlock * i;
        if (d < Dv) {
            const double rv = acc[i] / (double)count;
            dv.vr[(size_t)p * Dv + d] = rv;
            sq += rv * rv;
        }
    }
    sq = wave_sum(sq);
    if (tid % 64 == 0) visual_norm_parts(dv, p)[c / 64] = sq;
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

// Frames f0..f1-1: partition = most similar non-empty visual centroid, which then moves by Eq. 3.  One workgroup, kVisAssign
// threads.  e_in: the fp32 embeddings of these frames as the caller passed them; they are also filed in the visual
// level's state array.  The frames are taken up to sixteen at a time, as k_assign_chain does for the semantic level (which
// says why the decisions are exact): products of the chunk with all centroids and with itself, the channels shared out
// over the wavefronts; the decisions from those; Eq. 3 on the rows of the centroids that the chunk moved, a thread per
// channel.  Where a chunk begins with a frame that is too close to call, its frames are taken in turn.  What bounds it is its chain of trips to
// memory: operands of the products, embeddings by channel (on their way while the frames are decided), a row per moved centroid.
// 16 frames, P = 16, Dv = 1024: 90.5 us one frame at a time, 25.2 with a product's operands in four trips and the embeddings read anew for every moved
// centroid, now 19.
struct VisualShared {
    static constexpr int NW = kVisAssign / 64, FR = kChainFrames;
    union {
        struct { double part[NW][256], sim[FR * 64]; };
        VisualTurnShared turn;
    };
    double gram[FR][FR + 1], irn[64], ss[FR], sn[FR], isn[FR], out[FR], y[FR], norm[FR][NW];
    int vn[64], slot[64], lo[FR], near_id[FR], sure[FR], w[FR], p[FR], slot_id[FR], n_slot, nc, tied;
};

__device__ __forceinline__ void visual_assign(const DeviceView &dv, const float *e_in, int f0, int f1, VisualShared &sh) {
    constexpr int NW = VisualShared::NW, FR = kChainFrames, kNone = 0x7fffffff, CPT = 2;
    const int tid = threadIdx.x, lane = tid % 64, Dv = dv.Dv, P = dv.P, g = lane / 16, n = lane % 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    if (tid < 64) {
        const double rn = tid < P ? dv.vrn[tid] : 0.0;
        sh.vn[tid] = tid < P ? dv.vn[tid] : 0;
        sh.irn[tid] = rn > 0.0 ? 1.0 / rn : 0.0;
        sh.slot[tid] = -1;
        if (tid < FR) sh.lo[tid] = 0;
    }
    const int share = (Dv + 16 * NW - 1) / (16 * NW) * 16, ks = min(Dv, wave * share);
    InTurn turn;
    for (int c0 = f0; c0 < f1;) {
        int nc = min(FR, f1 - c0);
        const float *e = e_in + (size_t)(c0 - f0) * Dv;
        bool in_turn = turn.left > 0;       // workgroup-uniform
        // the chunk's embeddings, CPT channels per thread from kVisAssign * CPT * cb on
        float ev[CPT][FR];
        auto load_channels = [&](int cb) {
#pragma unroll
            for (int i = 0; i < CPT; ++i)
#pragma unroll
                for (int fc = 0; fc < FR; ++fc) ev[i][fc] = e[(size_t)min(fc, nc - 1) * Dv + min(tid + kVisAssign * (CPT * cb + i), Dv - 1)];
        };
        if (in_turn) {
            --turn.left;
        } else {
            // ---- products ----
            auto products = [&](auto vec, auto tiles) {
                constexpr int TILES = decltype(tiles)::value;
                f64x4 acc[TILES + 1];
                visual_products<float, decltype(vec)::value, true, TILES>(dv, e, nc, ks, min(Dv, ks + share), acc);
#pragma unroll
                for (int t = 0; t <= TILES; ++t) {
                    __syncthreads();            // (the first one also orders the tables above and the chunk before)
#pragma unroll
                    for (int v = 0; v < 4; ++v) sh.part[wave][(4 * v + g) * 16 + n] = acc[t][v];
                    __syncthreads();
                    if (tid < 256) {
                        double x = 0.0;
#pragma unroll
                        for (int w = 0; w < NW; ++w) x += sh.part[w][tid];
                        const int f = tid / 16, c = tid % 16, p = 16 * t + c;
                        if (t == TILES) sh.gram[f][c] = x;
                        else if (p < P) sh.sim[f * P + p] = sh.vn[p] > 0 ? x : -INFINITY;
                    }
                }
            };
            auto by_tiles = [&](auto vec) {
                if (P <= 16) products(vec, std::integral_constant<int, 1>{});
                else if (P <= 32) products(vec, std::integral_constant<int, 2>{});
                else products(vec, std::integral_constant<int, kVisTiles>{});
            };
            if (Dv % 4 == 0) by_tiles(std::true_type{});                 // (16-byte loads)
            else by_tiles(std::false_type{});
            load_channels(0);
            __syncthreads();
            if (wave == 0) {
                const double ss = n < nc ? sh.gram[n][n] : 0.0, is = fast_rsqrt(ss);
                double x[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = sh.gram[4 * v + g][n] * is;
                wave_sync();
#pragma unroll
                for (int v = 0; v < 4; ++v) sh.gram[4 * v + g][n] = x[v];
                if (g == 0) { sh.ss[n] = ss; sh.sn[n] = ss * is; sh.isn[n] = is; }
            }
            lds_barrier();
            for (int f = wave; f < nc; f += NW) {                    // the nearest centroid under the table as it stands
                const double d = lane < P ? sh.sim[f * P + lane] : -INFINITY;
                double c = d == -INFINITY ? d : d * sh.isn[f] * sh.irn[lane];
                const bool odd = __ballot(!(c == c)) != 0;
                if (!(c == c)) c = -INFINITY;
                double bv = c;
                int bi = c == -INFINITY ? kNone : lane;
                wave_best_ascending(bv, bi);
                const double second = wave_max(lane == bi ? -INFINITY : c);
                bool sure = bi != kNone && !odd && bv - second > kChainMargin;
                if (sh.ss[f] == 0.0) {          // (wave-uniform) a zero embedding: similarity 0 with every live centroid, the lowest id
                    const unsigned long long live = __ballot(lane < P && sh.vn[lane] > 0);
                    bi = live ? __ffsll((long long)live) - 1 : kNone;
                    sure = live != 0;
                }
                if (lane == 0) { sh.near_id[f] = bi; sh.out[f] = second; sh.sure[f] = sure; }
            }
            lds_barrier();
            in_turn = !sh.sure[0];
            if (in_turn) turn.failed();
        }
        if (in_turn) {
            __syncthreads();                // (the frames in turn use the products' LDS)
            for (int fc = 0; fc < nc; ++fc) {
                visual_in_turn(dv, e + (size_t)fc * Dv, c0 + fc, sh.turn, [&](int a, int size, double norm) {
                    sh.vn[a] = size;
                    sh.irn[a] = norm > 0.0 ? 1.0 / norm : 0.0;
                });
                __syncthreads();
            }
            c0 += nc;
            continue;
        }
        // ---- decisions ----
        if (wave == 0) {
            int mine = lane < nc ? sh.near_id[lane] : -1;
            if (mine == kNone) mine = -1;   // (no live candidate: the chunk ends before the frame)
            unsigned long long left = __ballot(mine >= 0);
            int k = 0;
            while (left) {
                const int id = __builtin_amdgcn_readlane(mine, __ffsll((long long)left) - 1);
                if (lane == 0) { sh.slot_id[k] = id; sh.slot[id] = k; }
                left &= ~__ballot(mine == id);
                ++k;
            }
            wave_sync();
            int w = n < nc && sh.near_id[n] != kNone ? sh.slot[sh.near_id[n]] : -1;
            bool tied;
            const int done =
                chain_decide({sh.sim, P, sh.lo, sh.sn, sh.isn, sh.ss, sh.out, sh.gram, sh.slot_id, sh.vn, sh.irn}, nc, k, w, tied);
            if (lane < done) {
                const int id = sh.slot_id[w];
                int p = sh.vn[id];
#pragma unroll
                for (int h = 0; h < FR - 1; ++h) p += h < lane && __builtin_amdgcn_readlane(w, h) == w ? 1 : 0;
                sh.w[lane] = w;
                sh.p[lane] = p;
                sh.y[lane] = __ddiv_rn(1.0, (double)p + 1.0);
                dv.part[c0 + lane] = id;
            }
            if (lane == 0) { sh.nc = done; sh.n_slot = k; sh.tied = tied; }
        }
        lds_barrier();
        nc = sh.nc;
        if (sh.tied) turn.failed();
        else turn.held();
        const int n_slot = sh.n_slot, n_cb = (Dv + kVisAssign * CPT - 1) / (kVisAssign * CPT);
        // ---- Eq. 3 on the rows; the frames' states ----
        // (a frame's slot, size and reciprocal from lane `frame`: the loops below branch on them, and would wait for LDS at every frame)
        const int w_lane = sh.w[n], p_lane = sh.p[n];
        const double y_lane = sh.y[n];
        double next[CPT];                   // the next slot's row (one block of channels: on its way while the slot before it is worked on)
        auto load_row = [&](int k, int cb) {
#pragma unroll
            for (int i = 0; i < CPT; ++i)
                next[i] = dv.vr[(size_t)sh.slot_id[min(k, n_slot - 1)] * Dv + min(tid + kVisAssign * (CPT * cb + i), Dv - 1)];
        };
        load_row(0, 0);
        for (int k = 0; k < n_slot; ++k) {
            const int id = sh.slot_id[k];
            int cnt = 0;
#pragma unroll
            for (int fc = 0; fc < FR; ++fc) cnt += fc < nc && __builtin_amdgcn_readlane(w_lane, fc) == k;
            double sq = 0.0;
            for (int cb = 0; cb < n_cb; ++cb) {
                if (n_cb > 1) {
                    nc = min(FR, f1 - c0);  // (rows that may be read)
                    load_channels(cb);
                    nc = sh.nc;
                    if (cb > 0) load_row(k, cb);
                }
                double xs[CPT];
#pragma unroll
                for (int i = 0; i < CPT; ++i) xs[i] = next[i];
                if (cb == n_cb - 1) load_row(k + 1, 0);
                if (cnt == 0) continue;     // workgroup-uniform
#pragma unroll
                for (int i = 0; i < CPT; ++i) {
                    const int d = tid + kVisAssign * (CPT * cb + i);
                    if (d >= Dv) continue;
                    double x = xs[i];
#pragma unroll
                    for (int fc = 0; fc < FR; ++fc)
                        if (fc < nc && __builtin_amdgcn_readlane(w_lane, fc) == k)
                            x = eq3_finite((double)__builtin_amdgcn_readlane(p_lane, fc), readlane_f64(y_lane, fc), x, (double)ev[i][fc]);
                    if (!(x == x)) {        // infinite states: over again
                        x = xs[i];
                        for (int fc = 0; fc < nc; ++fc)
                            if (sh.w[fc] == k) x = eq3_channel((double)sh.p[fc], sh.y[fc], x, (double)e[(size_t)fc * Dv + d]);
                    }
                    dv.vr[(size_t)id * Dv + d] = x;
                    sq = __builtin_fma(x, x, sq);
                }
            }
            sq = wave_sum(sq);
            if (lane == 0) sh.norm[k][wave] = sq;
        }
        if (n_cb == 1) {
#pragma unroll
            for (int i = 0; i < CPT; ++i)
#pragma unroll
                for (int fc = 0; fc < FR; ++fc)
                    if (fc < nc && tid + kVisAssign * i < Dv) dv.vemb[(size_t)(c0 + fc) * Dv + tid + kVisAssign * i] = (double)ev[i][fc];
        } else {
            for (int i = tid; i < nc * Dv; i += kVisAssign) dv.vemb[(size_t)c0 * Dv + i] = (double)e[i];
        }
        lds_barrier();
        if (tid < n_slot) {
            const int id = sh.slot_id[tid];
            int cnt = 0;
            for (int fc = 0; fc < nc; ++fc) cnt += sh.w[fc] == tid;
            if (cnt > 0) {
                double sq = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) sq += sh.norm[tid][w];
                const double rn = sqrt(sq);
                sh.vn[id] += cnt;
                sh.irn[id] = rn > 0.0 ? 1.0 / rn : 0.0;
                dv.vn[id] = sh.vn[id];
                dv.vrn[id] = rn;
            }
            sh.slot[id] = -1;
        }
        c0 += nc;
        __syncthreads();                    // (the next chunk reads the rows)
    }
}

__global__ __launch_bounds__(kVisAssign, 2) void k_visual_assign(const DeviceView *self, const float *e_in, int f0, int f1) {
    const DeviceView dv = device_view(self);
    __shared__ VisualShared sh;
    visual_assign(dv, e_in, f0, f1, sh);
}

// The page stores of the same frames beside it (the visual level reads nothing that they write): grid (1 + 2 U n), workgroup 0 the visual
// level, the others a page each.  (16 frames, 4 layers of 4 heads, T = 64: 5.4 + 25.2 us in two launches, now 21.6; of 28 layers of 4 heads a call of 16 frames, assignment included, 65.3 -> 51.7.)
template <typename E, int D>
__global__ __launch_bounds__(kVisAssign, 2) void k_store_visual_assign(const DeviceView *self, const E *k_in, const E *v_in, const float *e_in, int f0, int f1,
                                                                       int beyond) {
    const DeviceView dv = device_view(self);
    static_assert(kStoreBlock == kVisAssign, "one workgroup size");
    __shared__ union { VisualShared visual; StoreShared<D> store; } sh;
    if (blockIdx.x == 0) {
        visual_assign(dv, e_in, f0, f1, sh.visual);
        return;
    }
    const int i = (int)blockIdx.x - 1, u = i / 2 % dv.U, fl = i / 2 / dv.U;
    if (i % 2 == 0) {
        if (beyond) store_key_page<E, D, kStoreBlock, true>(dv, k_in, dv.k_store, u, fl, f0 + fl, sh.store, nullptr);
        else store_key_page<E, D, kStoreBlock, false>(dv, k_in, dv.k_store, u, fl, f0 + fl, sh.store, nullptr);
    } else {
        if (beyond) store_value_page<E, D, kStoreBlock, true>(dv, v_in, dv.v_store, u, fl, f0 + fl, sh.store);
        else store_value_page<E, D, kStoreBlock, false>(dv, v_in, dv.v_store, u, fl, f0 + fl, sh.store);
    }
}

// The same for calls of at most kVisFew frames, all of them in turn.  The chunk form's products, reductions and check cost 4
// us more for one frame (P = 10, Dv = 512, C = 120, whole call 16.6 against 12.2 us).
constexpr int kVisFew = 2;
__global__ __launch_bounds__(kVisAssign) void k_visual_assign_few(const DeviceView *self, const float *e_in, int f0, int f1) {
    const DeviceView dv = device_view(self);
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

hipError_t launch_visual_lloyd(const DeviceView &dv, int W, int iters, hipStream_t s) {
    k_visual_seed<<<dv.P, kVisBlock, 0, s>>>(dv.self, W);
    hipError_t e = after_launch();
    for (int it = 0; it < iters && e == hipSuccess; ++it) {
        auto go = [&](auto kern) { kern<<<(W + 15) / 16, 256, 0, s>>>(dv.self, W, it == 0); };
        auto by_tiles = [&](auto vec) {
            constexpr bool VEC = decltype(vec)::value;
            if (dv.P <= 16) go(k_visual_lloyd_assign<VEC, 1>);
            else if (dv.P <= 32) go(k_visual_lloyd_assign<VEC, 2>);
            else go(k_visual_lloyd_assign<VEC, kVisTiles>);
        };
        if (dv.Dv % 4 == 0) by_tiles(std::true_type{});
        else by_tiles(std::false_type{});
        if ((e = after_launch()) != hipSuccess) break;
        k_visual_lloyd_update<<<dim3(dv.P, kVisBlock / kVisUpdate), kVisUpdate, 0, s>>>(dv.self, W);
        e = after_launch();
    }
    if (e == hipSuccess) {
        k_visual_norms<<<1, 64, 0, s>>>(dv.self);
        e = after_launch();
    }
    return e;
}

hipError_t launch_visual_assign(const DeviceView &dv, const float *e_in, int f0, int f1, hipStream_t s) {
    if (f1 - f0 <= kVisFew) k_visual_assign_few<<<1, kVisAssign, 0, s>>>(dv.self, e_in, f0, f1);
    else k_visual_assign<<<1, kVisAssign, 0, s>>>(dv.self, e_in, f0, f1);
    return after_launch();
}

// (a launch holds fewer than 2^32 threads in a dimension: 37449 frames of 112 units; what is larger goes to launches of its own)
bool store_visual_assign_takes(const DeviceView &dv, int n_frames) {
    return n_frames > kVisFew && (1 + 2 * (long long)n_frames * dv.U) * kVisAssign < (1ll << 32);
}

hipError_t launch_store_visual_assign(const DeviceView &dv, const void *k_in, const void *v_in, const float *e_in, int f0, int f1, bool beyond,
                                      hipStream_t s) {
    const int grid = 1 + 2 * dv.U * (f1 - f0);
    auto go = [&](auto kern, auto *k) { kern<<<grid, kVisAssign, 0, s>>>(dv.self, k, (decltype(k))v_in, e_in, f0, f1, beyond); };
    if (dv.esize == 4) {
        if (dv.D == 64) go(k_store_visual_assign<float, 64>, (const float *)k_in);
        else go(k_store_visual_assign<float, 128>, (const float *)k_in);
    } else {
        if (dv.D == 64) go(k_store_visual_assign<unsigned short, 64>, (const unsigned short *)k_in);
        else go(k_store_visual_assign<unsigned short, 128>, (const unsigned short *)k_in);
    }
    return after_launch();
}

} // namespace mosaic
