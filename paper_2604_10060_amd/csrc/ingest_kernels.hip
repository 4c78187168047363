// Frame Encoding kernels (paper Sec. V-A (1), Sec. VI-A, Sec. V-B):
//   k_store_summary  copy a frame's K/V pages into the arena and form the
//                    frame's key summary (mean of its T keys) in fp64
//   k_assign_update  greedy cosine assignment + running-mean update (Eq. 3),
//                    sequential over the frames of a batch, one workgroup per unit
//   k_lloyd_*        cosine K-means rounds for the initial clustering and the
//                    periodic warm-started re-clustering
// All decision arithmetic is fp64: on CDNA4 the fp64 vector rate equals the
// non-packed fp32 rate, so exact-to-rounding decisions cost only table bytes.
#include <type_traits>

#include <algorithm>
#include "mosaic_internal.h"
#include "maintain_device.h"
#include "page_store_device.h"
#include "assign_device.h"

namespace mosaic {

namespace {

// (every call site has all 16 lanes of the group active)
__device__ __forceinline__ double group16_sum(double x) { return row16_sum(x); }
// (every call site has the whole wavefront active)
__device__ __forceinline__ double wave_sum(double x) { return wave64_sum(x); }
// (value, id) ordered by value descending then id ascending
__device__ __forceinline__ bool better(double v, int i, double bv, int bi) {
    return v > bv || (v == bv && i < bi);
}
// Best (value, id) of a wavefront, left in every lane: a butterfly inside each row of 16
// lanes with data-parallel primitives (the order is total, so every lane of a row ends
// with the same pair), then the four rows' pairs are read from their first lanes.
template <int CTRL> __device__ __forceinline__ void best_step(double &bv, int &bi) {
    const double ov = dpp_f64<CTRL>(bv);
    const int oi = dpp_i32<CTRL>(bi);
    if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
}
__device__ __forceinline__ void wave_best(double &bv, int &bi) {
    best_step<kDppXor8>(bv, bi);
    best_step<kDppXor7>(bv, bi);
    best_step<kDppXor3>(bv, bi);
    best_step<kDppXor1>(bv, bi);
    const long long b = __double_as_longlong(bv);
    const int lo = (int)b, hi = (int)(b >> 32);
    double rv[4];
    int ri[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int l = __builtin_amdgcn_readlane(lo, 16 * r), h = __builtin_amdgcn_readlane(hi, 16 * r);
        rv[r] = __longlong_as_double(((long long)h << 32) | (long long)(unsigned int)l);
        ri[r] = __builtin_amdgcn_readlane(bi, 16 * r);
    }
    bv = rv[0]; bi = ri[0];
#pragma unroll
    for (int r = 1; r < 4; ++r)
        if (better(rv[r], ri[r], bv, bi)) { bv = rv[r]; bi = ri[r]; }
}

// ---------------------------------------------------------------------------
// Page store + summaries: page_store_device.h.
// grid (U, n_frames, 2 or 3): z = 0 keys, z = 1 values, z = 2 the embeddings e_in of the n_emb first frames (nested hierarchy, warm-up), into the
// visual level's fp64 state array.  (A launch of their own cost 3.6 us.)
template <typename E, int D, bool BEYOND>
__global__ __launch_bounds__(kStoreBlock) void k_store_summary(const DeviceView *self, const E *k_in,
                                                          const E *v_in, int f0, const float *e_in, int n_emb) {
    const DeviceView dv = device_view(self);
    __shared__ StoreShared<D> store_sh;
    const int u = blockIdx.x, fl = blockIdx.y;
    const bool host = dv.tier == MOSAIC_TIER_HOST;
    if (blockIdx.z == 0) store_key_page<E, D, kStoreBlock, BEYOND>(dv, k_in, host ? dv.stage_k : dv.k_store, u, fl, f0 + fl, store_sh, nullptr);
    else if (blockIdx.z == 1) store_value_page<E, D, kStoreBlock, BEYOND>(dv, v_in, host ? dv.stage_v : dv.v_store, u, fl, f0 + fl, store_sh);
    else if (fl < n_emb)
        for (int d = u * kStoreBlock + threadIdx.x; d < dv.Dv; d += dv.U * kStoreBlock) dv.vemb[(size_t)(f0 + fl) * dv.Dv + d] = (double)e_in[(size_t)fl * dv.Dv + d];
}

// ---------------------------------------------------------------------------
// Retrieval augmentation, global representatives (paper Sec. V-C): the value of a
// cluster's pseudo token is the mean of its member frames' value summaries, its key the
// cluster's representative.  grid (U, C), 128 threads: one workgroup per cluster lists
// the cluster's frames in ascending order and adds their value summaries in that order, so
// the sum is one fixed sequence of additions: the same bits on every run, whatever the
// order in which workgroups are scheduled.  It then writes the fp32 key / value rows of
// the pseudo-token tables (zero rows for empty clusters).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(128) void k_value_reps(const DeviceView *self, int n_frames) {
    const DeviceView dv = device_view(self);
    constexpr int NT = 128, CH = NT * kListPer;
    const int u = blockIdx.x, j = blockIdx.y, tid = threadIdx.x, C = dv.C;
    __shared__ int mem[CH];
    __shared__ int wtot[NT / 64];
    const size_t row = (size_t)u * C + j;
    const int nj = dv.n[row];                       // workgroup-uniform
    const double *vb = dv.vsumm + (size_t)u * dv.F * D + tid;
    double acc = 0.0;
    for (int c0 = 0; nj > 0 && c0 < n_frames; c0 += CH) {
        const int m = list_members<NT>(dv.assign + (size_t)u * dv.F, j, c0, n_frames, mem, wtot);
        if (tid < D) acc = add_members<16>(acc, mem, m, [&](int f) { return vb[(size_t)f * D]; });
    }
    if (tid < D) {
        dv.rvsum[row * D + tid] = acc;
        dv.rep_k[row * D + tid] = nj > 0 ? (float)dv.r[row * D + tid] : 0.f;
        dv.rep_v[row * D + tid] = nj > 0 ? (float)(acc / (double)nj) : 0.f;
    }
}

// ---------------------------------------------------------------------------
// Online assignment + Eq. 3, frames f0..f1-1 in order, the table read from global memory for every frame.  grid (U),
// 256 threads.  With the maintainer, and without it for calls of one or two frames on tables of more than 256 clusters
// (2 layers, whole calls with the page store, this / k_assign_chain: C = 1000, one frame a call 8.4 / 11.7 us, two
// 11.2 / 12; three 14.8 / 12.9; C = 300, three 16.1 / 15.1).
// ---------------------------------------------------------------------------
// With MAINT the insertion procedure of the self-adaptive maintainer (Sec. VI,
// Alg. 1 lines 1-10) follows the update: running variance (Eq. 4), threshold
// (Eq. 5) at the size before the insertion, then absorb / split / defer.
enum { kActAbsorb = 1, kActSplit = 2, kActDefer = 3, kActForced = 4 };

template <int D, bool MAINT>
__global__ __launch_bounds__(kBlock) void k_assign_update(const DeviceView *self, int f0, int f1) {
    const DeviceView dv = device_view(self);
    constexpr int EPL = D / 16;  // elements per lane in a 16-lane row group
    const int u = blockIdx.x, tid = threadIdx.x, C = dv.C;
    const int lr = tid % 16, row0 = tid / 16, wave = tid / 64, lane = tid % 64;
    __shared__ double s_sh[D];
    __shared__ double dot_sh[1024];
    __shared__ double red_v[4];
    __shared__ int red_i[4];
    __shared__ double snorm_sh, nsum_sh[2], dsum_sh[2], psum_sh[2];
    __shared__ int act_sh;
    __shared__ SplitShared<MAINT ? D : 16> split_sh;   // (small placeholder when the maintainer is off)
    double *r = dv.r + (size_t)u * C * D;
    double *rn = dv.rnorm + (size_t)u * C;
    int *n = dv.n + (size_t)u * C;

    const bool nested = dv.P > 0;
    // the summary of the next frame travels while the current frame is processed
    double s_ahead = tid < D ? dv.summ[((size_t)u * dv.F + f0) * D + tid] : 0.0;
    for (int f = f0; f < f1; ++f) {
        // candidates: every cluster id, or (nested hierarchy, Sec. V-B) the ids of the frame's
        // visual partition only
        const int part_f = nested ? dv.part[f] : 0;
        // (maintainer: only the ids in use, [0, n_slots), can have members; the table behind them is not read)
        const int lo = nested ? part_f * dv.Cs : 0, hi = nested ? lo + dv.Cs : (MAINT ? min(C, max(dv.n_slots[u], 1)) : C);
        if (tid < D) {
            s_sh[tid] = s_ahead;
            if (f + 1 < f1) s_ahead = dv.summ[((size_t)u * dv.F + f + 1) * D + tid];
        }
        __syncthreads();
        if (wave == 0) {
            double x = 0.0;
            if constexpr (MAINT) {
                for (int d = lane; d < D; d += 64) x += s_sh[d] * s_sh[d];
                x = wave_sum(x);
            } else {            // (in the order of the kernels that share this state)
                double sl[EPL];
#pragma unroll
                for (int e = 0; e < EPL; ++e) sl[e] = s_sh[lr * EPL + e];
                x = row16_sum(square_channels(sl, true));
            }
            if (lane == 0) snorm_sh = sqrt(x);
        }
        // sizes and norms of this thread's candidates (at most four: C <= 1024), fetched ahead of the rows
        int nj[4];
        double rnj[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int j = min(lo + tid + kBlock * x, hi - 1);
            nj[x] = n[j]; rnj[x] = rn[j];
        }
        // Dot products with the candidates' rows, eight rows of a 16-lane group in flight at a time
        // (row index clamped, loads unconditional, no test of the size: a row nobody reads costs
        // nothing extra, a dependent load per row costs a trip to L2)
        for (int jb = lo; jb < hi; jb += 16 * 8) {
            const int passes = min(8, (hi - jb + 15) / 16);   // workgroup-uniform
            const int j0 = jb + row0;
            auto rows = [&](auto full) {      // full: all eight passes (straight-line code); else only `passes`
                double rv[8][EPL];
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    if (decltype(full)::value || x < passes) {
                        const double *rj = r + (size_t)min(j0 + 16 * x, hi - 1) * D + lr * EPL;
#pragma unroll
                        for (int i = 0; i < EPL; ++i) rv[x][i] = rj[i];
                    }
                }
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    if (decltype(full)::value || x < passes) {
                        double p = 0.0;
#pragma unroll
                        for (int i = 0; i < EPL; ++i) p = __builtin_fma(s_sh[lr * EPL + i], rv[x][i], p);
                        p = group16_sum(p);
                        if (lr == 0 && j0 + 16 * x < hi) dot_sh[j0 + 16 * x] = p;
                    }
                }
            };
            if (passes == 8) rows(std::true_type{});
            else rows(std::false_type{});
        }
        __syncthreads();
        // argmax of the cosine over non-empty clusters, ties to the lowest id
        double bv = -INFINITY;
        int bi = 0x7fffffff;
        const double sn = snorm_sh;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int j = lo + tid + kBlock * x;
            if (j < hi && nj[x] > 0) {
                const double c = (sn == 0.0 || rnj[x] == 0.0) ? 0.0 : dot_sh[j] / (sn * rnj[x]);
                if (better(c, j, bv, bi)) { bv = c; bi = j; }
            }
        }
        wave_best(bv, bi);
        if (lane == 0) { red_v[wave] = bv; red_i[wave] = bi; }
        __syncthreads();
        // every thread merges the four wavefronts' winners itself
        bv = red_v[0]; bi = red_i[0];
#pragma unroll
        for (int w = 1; w < 4; ++w)
            if (better(red_v[w], red_i[w], bv, bi)) { bv = red_v[w]; bi = red_i[w]; }
        const int a = bi == 0x7fffffff ? lo : bi;
        const int na_i = n[a];
        const double na = (double)na_i;
        double sq = 0.0, dq = 0.0;
        if (tid < D) {
            const double rv = __builtin_fma(na, r[(size_t)a * D + tid], s_sh[tid]) / (na + 1.0);      // Eq. 3 (as eq3_channel)
            r[(size_t)a * D + tid] = rv;
            if constexpr (!MAINT) dot_sh[tid] = rv;  // (the dot products have been read)
            sq = rv * rv;
            const double t = s_sh[tid] - rv;
            dq = t * t;
        }
        if (MAINT && wave < 2) {
            sq = wave_sum(sq);
            dq = wave_sum(dq);
            if (lane == 0) { nsum_sh[wave] = sq; dsum_sh[wave] = dq; }
        }
        // nested hierarchy: the partition's representative in this unit's key space follows the
        // same running mean (Eq. 3 one level up)
        int pn_i = 0;
        if (nested) {
            double *prow = dv.pr + ((size_t)u * dv.P + part_f) * D;
            pn_i = dv.pn[(size_t)u * dv.P + part_f];
            double pv = 0.0;
            if (tid < D) {
                pv = eq3_channel((double)pn_i, __ddiv_rn(1.0, (double)pn_i + 1.0), prow[tid], s_sh[tid]);
                prow[tid] = pv;
            }
            if (wave < 2) {
                const double psq = wave_square_sum(pv);
                if (lane == 0) psum_sh[wave] = psq;
            }
        }
        __syncthreads();   // all threads have read n[a] and written r before the scalars change
        if (!MAINT && wave == 0) {      // (the norm's additions in the order of the kernels that share this state)
            double x[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) x[e] = dot_sh[lr * EPL + e];
            const double sum = row16_sum(square_channels(x, row_second_first(C, a)));
            if (lane == 0) nsum_sh[0] = sum;
        }
        if (tid == 0) {
            if (nested) {
                dv.prn[(size_t)u * dv.P + part_f] = sqrt(D > 64 ? psum_sh[0] + psum_sh[1] : psum_sh[0]);
                dv.pn[(size_t)u * dv.P + part_f] = pn_i + 1;
            }
            rn[a] = sqrt(MAINT && D > 64 ? nsum_sh[0] + nsum_sh[1] : nsum_sh[0]);
            int act = kActAbsorb;
            if (MAINT) {
                const double dist2 = D > 64 ? dsum_sh[0] + dsum_sh[1] : dsum_sh[0];
                double *var = dv.var + (size_t)u * C;
                const double var_new = (na * var[a] + dist2) / (na + 1.0);                          // Eq. 4
                const double tau = dv.tau_min + (dv.tau_max - dv.tau_min) * exp(-na / dv.tau_n0);   // Eq. 5
                var[a] = var_new;
                const bool on_gpu = dv.maint_mode == MOSAIC_MAINT_EAGER || dv.resident[(size_t)u * C + a] != 0;
                if (var_new <= tau) act = kActAbsorb;
                else if (on_gpu) act = kActSplit;
                else if (dv.n_buf[u] < dv.buf_max) act = kActDefer;
                else act = kActForced;
                if (act == kActDefer || act == kActForced) dv.lazy[(size_t)u * C + a] = 1;
                if (act == kActDefer) {
                    const int b = dv.n_buf[u];
                    dv.buf_frame[(size_t)u * dv.buf_max + b] = f;
                    dv.buf_owner[(size_t)u * dv.buf_max + b] = a;
                    dv.n_buf[u] = b + 1;
                    dv.mt_cnt[(size_t)u * 4 + 2] += 1;
                }
                if (act == kActForced) dv.mt_cnt[(size_t)u * 4 + 3] += 1;
                act_sh = act;
            }
            if (act == kActDefer) {                     // held in the buffer on behalf of cluster a
                dv.assign[(size_t)u * dv.F + f] = -2 - a;
                dv.pos[(size_t)u * dv.F + f] = 0;
            } else {
                n[a] = na_i + 1;
                dv.assign[(size_t)u * dv.F + f] = a;
                dv.pos[(size_t)u * dv.F + f] = na_i;
            }
        }
        __syncthreads();
        if constexpr (MAINT) {
            if (act_sh == kActSplit) {                  // workgroup-uniform
                const int fresh = mt_split_cluster<D>(dv, u, a, f + 1, false, split_sh);
                if (tid == 0) dv.mt_cnt[(size_t)u * 4 + (fresh >= 0 ? 0 : 3)] += 1;
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// Online assignment + Eq. 3 without the maintainer, frames f0..f1-1 in order.  grid (U), kChainBlock threads.
//
// Eq. 3 makes frame t depend on frame t - 1, but only through the one representative that t - 1 moved, and moving it
// changes dot products by a known amount: r' = (n r + s) / (n + 1) gives r'.x = (n r.x + s.x) / (n + 1).  So the frames
// are taken a chunk of up to 16 at a time:
//   1. the chunk's summaries times the whole table, and times each other, on the fp64 matrix instruction (all
//      wavefronts); every frame's nearest cluster under the table as it stands;
//   2. those clusters -- almost always the only ones the chunk will move -- become "slots"; a frame's second best
//      similarity of step 1 bounds what it can have with any cluster that is not a slot;
//   3. wavefront 0 assumes that every frame joins its nearest cluster of step 1.  Then all sums are known: by the
//      identity a slot's dot product with a frame is n r.x plus the products with the frames that joined it before
//      (and |n r + ...|^2 likewise), so all frames are checked at once, a lane per (frame, slot).  Where a frame's best
//      slot is another one than assumed, the first such frame is corrected and the rest checked again;
//   4. with the winners known, Eq. 3 is applied to the rows themselves: a thread per (slot, channel) runs through the
//      slot's frames in order.
// Decisions are exact: the similarities of steps 1 and 3 differ from those of the rows by rounding (chain_error: differences
// by less than 5e-13 at D = 128), and they only decide where the best is ahead by more than kChainMargin.  At a frame that is closer than that, or whose best slot does not exceed the
// bound of step 2, the chunk ends, and the frames after it are taken in turn: in the order of operations of the one-frame
// kernel, ties to the lowest id, the products of a chunk's frames with the rows formed in one pass over them and those with
// a row that moves formed anew.  So ids and representatives are the same bits for any split of the stream into calls.  (A
// zero summary needs no product: it has similarity 0 with every cluster.)  Frames in turn cost 2 us each, more for large
// tables: 16 a call, page store included, on streams whose clusters lie along six directions, taken in turn by a pass over
// the products each / now / by the kernels before this one: C = 64 67 / 46 / 33 us, C = 200 200 / 63 / 46, C = 300 186 / 74
// / 103, C = 1000 456 / 169 / 260; on zero summaries C = 64 146 / 16 / 32 us, C = 1000 913 / 86 / 262.
// What bounds it (16 frames, D = 128, one chunk; cycles of one workgroup): the trip to memory for table and summaries
// 4 k (11 k while page stores saturate the memory system), the fp64 products 6-8 k, nearest clusters 3 k, decisions
// 3.5 k, Eq. 3 on the rows 7 k (seven dependent fp64 operations per frame).  A kernel that takes the frames one after
// the other -- table in registers, dot products, search, update, two barriers per frame -- needs 77 k.  Launch: 4 layers,
// C = 512 in 16 partitions 48.7 -> 15.6 us, 28 layers, C = 128, beside page stores 37.1 -> 22.3 us.
// ---------------------------------------------------------------------------
constexpr int kChainBlock = 512, kChainSims = 8192;

template <int D>
__global__ __launch_bounds__(kChainBlock) void k_assign_chain(const DeviceView *self, int f0, int f1) {
    const DeviceView dv = device_view(self);
    constexpr int EPL = D / 16, NG = kChainBlock / 16, NW = kChainBlock / 64, KS = D / 8, SPB = kChainBlock / D;
    constexpr int FR = kChainFrames, kNone = 0x7fffffff, TW = FR / 4;
    const int u = blockIdx.x, tid = threadIdx.x, lane = tid % 64, lr = tid % 16, grp = tid / 16, C = dv.C;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), g = lane / 16, n = lane % 16;
    __shared__ __attribute__((aligned(16))) double s_sh[FR][D + 2];     // (row padding: 16 rows' operand reads spread over the banks)
    __shared__ double sim_sh[kChainSims];           // [frame][candidate] dot products, -inf for an empty cluster
    __shared__ double gram_sh[FR][FR + 1];          // s_f . s_g / |s_g|
    __shared__ double rn_sh[1024], irn_sh[1024];    // |r_j|; 1 / |r_j|, 0 for a zero row
    __shared__ int n_sh[1024];                      // sizes
    __shared__ signed char slot_sh[1024];           // slot of a cluster, -1
    __shared__ double ss_sh[FR], sn_sh[FR], isn_sh[FR], out_v[FR], y_sh[FR], row_sh[SPB][D];
    __shared__ double red_v[TW];
    __shared__ int red_i[TW];
    __shared__ int near_sh[FR], sure_sh[FR], lo_sh[FR], w_sh[FR], p_sh[FR], slot_id[FR], n_slot_sh, nc_sh, tied_sh;
    double *r = dv.r + (size_t)u * C * D;
    const bool nested = dv.P > 0;
    const int width = nested ? dv.Cs : C;           // candidates per frame: ids lo .. lo + width - 1
    const int NI = (width + 63) / 64;               // ... lane l takes NI consecutive ones, so that ids ascend with the lane
    const int NF = min(FR, kChainSims / width), tiles = (C + 15) / 16;
    for (int j = tid; j < C; j += kChainBlock) {
        const double rn = dv.rnorm[(size_t)u * C + j];
        n_sh[j] = dv.n[(size_t)u * C + j];
        rn_sh[j] = rn;
        irn_sh[j] = rn > 0.0 ? 1.0 / rn : 0.0;
        slot_sh[j] = -1;
    }
    auto resize = [&](int j, int size, double norm) {               // a cluster's new size and norm
        n_sh[j] = size;
        rn_sh[j] = norm;
        irn_sh[j] = norm > 0.0 ? 1.0 / norm : 0.0;
        dv.n[(size_t)u * C + j] = size;
        dv.rnorm[(size_t)u * C + j] = norm;
    };
    // nested hierarchy: the partitions' representatives in this unit's key space follow the same running mean (Eq. 3 one
    // level up), one wavefront, two channels per lane, a partition's row in registers until another's turn comes
    auto partition_reps = [&](int nc) {
        constexpr int CPL = D / 64;
        const int own = lane < nc ? lo_sh[lane] / dv.Cs : -1;
        int size = lane < nc ? dv.pn[(size_t)u * dv.P + own] : 0;
#pragma unroll
        for (int h = 0; h < FR - 1; ++h) size += h < lane && __builtin_amdgcn_readlane(own, h) == own ? 1 : 0;
        const double yl = __ddiv_rn(1.0, (double)size + 1.0);
        double pv[CPL];
        int at = -1, pn = 0;
        auto leave = [&]() {
            double psq = 0.0;
#pragma unroll
            for (int x = 0; x < CPL; ++x) {
                dv.pr[((size_t)u * dv.P + at) * D + lane + 64 * x] = pv[x];
                const double w = wave_square_sum(pv[x]);
                psq = x == 0 ? w : psq + w;
            }
            if (lane == 0) {
                dv.prn[(size_t)u * dv.P + at] = sqrt(psq);
                dv.pn[(size_t)u * dv.P + at] = pn;
            }
        };
        for (int fc = 0; fc < nc; ++fc) {
            const int p = __builtin_amdgcn_readlane(own, fc);
            if (p != at) {
                if (at >= 0) leave();
                at = p;
#pragma unroll
                for (int x = 0; x < CPL; ++x) pv[x] = dv.pr[((size_t)u * dv.P + at) * D + lane + 64 * x];
            }
            pn = __builtin_amdgcn_readlane(size, fc) + 1;
            const double ny = readlane_f64(yl, fc);
#pragma unroll
            for (int x = 0; x < CPL; ++x) pv[x] = eq3_channel((double)(pn - 1), ny, pv[x], s_sh[fc][lane + 64 * x]);
        }
        leave();
    };
    InTurn turn;
    for (int c0 = f0; c0 < f1;) {
        int nc = min(NF, f1 - c0);
        const bool in_turn = turn.left > 0;         // workgroup-uniform
        // ---- 1. the chunk against the whole table and against itself ----
        // operand layout of v_mfma_f64_16x16x4_f64: A lane (row lane%16, k lane/16), B lane (column lane%16, k lane/16),
        // result register v = (row 4v + lane/16, column lane%16); lane group k holds channels 8s + 2k, + 1 of step s
        f64x2 b[KS];
        auto load_rows = [&](int t) {
            const double *rj = r + (size_t)min(16 * t + n, C - 1) * D + 2 * g;
#pragma unroll
            for (int s = 0; s < KS; ++s) b[s] = *reinterpret_cast<const f64x2 *>(rj + 8 * s);
        };
        if (!nested && !in_turn && wave < tiles) load_rows(wave);   // travels with the summaries
        {
            const double *src = dv.summ + ((size_t)u * dv.F + c0) * D;
            for (int i = tid; i < nc * D / 2; i += kChainBlock)
                *reinterpret_cast<f64x2 *>(&s_sh[2 * i / D][2 * i % D]) = *reinterpret_cast<const f64x2 *>(src + 2 * i);
            if (tid < nc) lo_sh[tid] = nested ? dv.part[c0 + tid] * dv.Cs : 0;
        }
        __syncthreads();
        auto times_s = [&]() {                      // the chunk's summaries (rows) times the operand in b (columns)
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const f64x2 a = *reinterpret_cast<const f64x2 *>(&s_sh[n][8 * s + 2 * g]);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b[s].x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b[s].y, acc, 0, 0, 0);
            }
            return acc;
        };
        for (int t = wave; t < tiles && !in_turn; t += NW) {
            if (nested) {                           // tiles that no frame of the chunk asks for are not read
                const int lo = lo_sh[min(lane, nc - 1)];
                if (__ballot(lo < 16 * t + 16 && lo + width > 16 * t) == 0) continue;
            }
            if (nested || t != wave) load_rows(t);
            const f64x4 acc = times_s();
            const int j = 16 * t + n;
            const bool live = j < C && n_sh[min(j, C - 1)] > 0;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int fc = 4 * v + g;
                if (fc < nc && j < C) {
                    const int cj = j - lo_sh[fc];
                    if (cj >= 0 && cj < width) sim_sh[fc * width + cj] = live ? acc[v] : -INFINITY;
                }
            }
        }
        if (wave == NW - 1 && !in_turn) {           // (the wavefront with the fewest tiles)
#pragma unroll
            for (int s = 0; s < KS; ++s) b[s] = *reinterpret_cast<const f64x2 *>(&s_sh[n][8 * s + 2 * g]);
            const f64x4 acc = times_s();            // (rows and columns beyond the chunk: whatever the LDS held, never read)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * v + g == n) ss_sh[n] = n < nc ? acc[v] : 0.0;
            wave_sync();
            const double is = fast_rsqrt(ss_sh[n]);
#pragma unroll
            for (int v = 0; v < 4; ++v) gram_sh[4 * v + g][n] = acc[v] * is;
            if (g == 0) { isn_sh[n] = is; sn_sh[n] = ss_sh[n] * is; }
        }
        __syncthreads();
        for (int fc = wave; fc < nc && !in_turn; fc += NW) {        // the nearest cluster under the table as it stands
            const double is = isn_sh[fc];
            const int lo = lo_sh[fc];
            double bv = -INFINITY, sv = -INFINITY;
            int bi = kNone;
            bool odd = false;
            for (int i = 0; i < NI; ++i) {
                const int cj = lane * NI + i;
                if (cj < width) {
                    const double d = sim_sh[fc * width + cj], c = d == -INFINITY ? d : d * is * irn_sh[lo + cj];
                    odd |= !(c == c);
                    if (c > bv) { sv = bv; bv = c; bi = lo + cj; }
                    else if (c > sv) sv = c;
                }
            }
            const double own = bv;
            const int own_i = bi;
            wave_best_ascending(bv, bi);
            const double second = wave_max(own_i == bi ? sv : own);
            bool sure = bi != kNone && __ballot(odd) == 0 && bv - second > kChainMargin;
            if (ss_sh[fc] == 0.0) {                 // (wave-uniform) a zero summary: similarity 0 with every live cluster, the lowest id
                int first = kNone;
                for (int i = NI - 1; i >= 0; --i) {
                    const int cj = lane * NI + i;
                    if (cj < width && n_sh[lo + cj] > 0) first = lo + cj;
                }
                bi = __builtin_amdgcn_readlane(first, max(__ffsll((long long)__ballot(first != kNone)) - 1, 0));
                sure = bi != kNone;
            }
            if (lane == 0) { near_sh[fc] = bi; sure_sh[fc] = sure; out_v[fc] = second; }
        }
        __syncthreads();
        if (in_turn || !sure_sh[0]) {               // workgroup-uniform: the frames in turn
            // In the one-frame kernel's order of operations, but a row is read once for all frames of the chunk: the frames'
            // products with every row (a 16-lane group per row, four at a time), then frame by frame the search, Eq. 3 on the
            // winner -- by a group per frame, so that each has the new row -- and the later frames' products with it.
            if (in_turn) --turn.left;
            else turn.failed();
            unsigned long long parts = 0;           // partitions that the chunk asks for
            if (nested)
                for (int fc = 0; fc < nc; ++fc) parts |= 1ull << (lo_sh[fc] / dv.Cs);
            auto next = [&](int j) {
                do j += NG;
                while (j < C && nested && !((parts >> (j / dv.Cs)) & 1));
                return j;
            };
            auto fetch = [&](int j, double (&o)[EPL]) {
                const double *rj = r + (size_t)min(j, C - 1) * D + lr * EPL;
#pragma unroll
                for (int e = 0; e < EPL; ++e) o[e] = rj[e];
            };
            auto summary = [&](int fc, double (&o)[EPL]) {
#pragma unroll
                for (int e = 0; e < EPL; ++e) o[e] = s_sh[fc][lr * EPL + e];
            };
            auto product = [&](int fc, int j, const double (&sl)[EPL], const double (&row)[EPL]) {  // (uniform within a group)
                const double p = row16_sum(dot_channels(sl, row));
                const int cj = j - lo_sh[fc];
                if (lr == 0 && cj >= 0 && cj < width) sim_sh[fc * width + cj] = p;
            };
            double row[EPL], sl[EPL];
            for (int j = next(grp - NG); j < C;) {
                constexpr int RB = 4;
                double rows[RB][EPL];
                int id[RB];
#pragma unroll
                for (int x = 0; x < RB; ++x) {
                    id[x] = j;
                    fetch(j, rows[x]);
                    if (j < C) j = next(j);
                }
                for (int fc = 0; fc < nc; ++fc) {
                    summary(fc, sl);
#pragma unroll
                    for (int x = 0; x < RB; ++x) product(fc, id[x] < C ? id[x] : -1, sl, rows[x]);
                }
            }
            if (grp < nc) {
                summary(grp, sl);
                const double norm = sqrt(row16_sum(square_channels(sl, true)));
                if (lr == 0) sn_sh[grp] = norm;
            }
            if (nested && wave == NW - 1) partition_reps(nc);       // (the summaries alone decide these)
            __syncthreads();
            // (The loop waits for no store: moved rows stay in LDS until the chunk is done, the k-th one in place of the summary
            // of frame k, which has had its turn by then.  Four wavefronts, one per SIMD: a group per frame, and up to four
            // consecutive candidates per thread, so that ids ascend with the thread.)
            const int per = (width + 64 * TW - 1) / (64 * TW);
            int a1 = -1, n1 = 0, used = 0;          // the cluster of the frame before, with its new size and norm; `row` is its row
            double rn1 = 0.0;
            for (int fc = 0; fc < nc; ++fc) {
                const int lo = lo_sh[fc];
                double bv = -INFINITY;
                int bi = kNone;
                if (wave < TW) {
                    const double sn = sn_sh[fc];
                    for (int cj = tid * per; cj < min(width, tid * per + per); ++cj) {
                        const int id = lo + cj, size = id == a1 ? n1 : n_sh[id];
                        const double rn = id == a1 ? rn1 : rn_sh[id];
                        const double c = (sn == 0.0 || rn == 0.0) ? 0.0 : sim_sh[fc * width + cj] / (sn * rn);
                        if (size > 0 && c > bv) { bv = c; bi = id; }
                    }
                    wave_best_ascending(bv, bi);
                    if (lane == 0) { red_v[wave] = bv; red_i[wave] = bi; }
                }
                lds_barrier();
                int a = lo, size = 0, slot = -1;
                double norm = 0.0;
                if (wave < TW) {
                    bv = red_v[0]; bi = red_i[0];
#pragma unroll
                    for (int w = 1; w < TW; ++w)
                        if (red_v[w] > bv) { bv = red_v[w]; bi = red_i[w]; }
                    if (bi != kNone) a = bi;
                    size = a == a1 ? n1 : n_sh[a];
                    slot = slot_sh[a];
                    const double y = __ddiv_rn(1.0, (double)size + 1.0);
                    if (a != a1) {
                        if (slot < 0) fetch(a, row);
                        else
#pragma unroll
                            for (int e = 0; e < EPL; ++e) row[e] = s_sh[slot][lr * EPL + e];
                    }
#pragma unroll
                    for (int e = 0; e < EPL; ++e) row[e] = eq3_channel((double)size, y, row[e], s_sh[fc][lr * EPL + e]);
                    if (grp > fc && grp < nc) product(grp, a, sl, row);
                    norm = sqrt(row16_sum(square_channels(row, row_second_first(C, a))));
                    if (slot < 0) slot = used++;
                    a1 = a; n1 = size + 1; rn1 = norm;
                }
                lds_barrier();                      // the old row, size and norm have been read
                if (grp == 0) {
#pragma unroll
                    for (int e = 0; e < EPL; ++e) s_sh[slot][lr * EPL + e] = row[e];
                    if (lr == 0) {
                        slot_sh[a] = slot;
                        slot_id[slot] = a;
                        n_slot_sh = used;
                        resize(a, size + 1, norm);
                        dv.assign[(size_t)u * dv.F + c0 + fc] = a;
                        dv.pos[(size_t)u * dv.F + c0 + fc] = size;
                    }
                }
            }
            __syncthreads();
            for (int i = tid; i < n_slot_sh * D; i += kChainBlock) r[(size_t)slot_id[i / D] * D + i % D] = s_sh[i / D][i % D];
            if (tid < n_slot_sh) slot_sh[slot_id[tid]] = -1;
            __syncthreads();
            c0 += nc;
            continue;
        }
        // ---- 2. slots ----
        if (wave == 0) {
            int mine = lane < nc ? near_sh[lane] : -1;
            if (mine == kNone) mine = -1;           // (no live candidate: the chunk ends before the frame)
            unsigned long long left = __ballot(mine >= 0);
            int k = 0;
            while (left) {
                const int id = __builtin_amdgcn_readlane(mine, __ffsll((long long)left) - 1);
                if (lane == 0) { slot_id[k] = id; slot_sh[id] = k; }
                left &= ~__ballot(mine == id);
                ++k;
            }
            if (lane == 0) n_slot_sh = k;
        }
        __syncthreads();
        const int n_slot = n_slot_sh;
        double x0 = 0.0;                            // step 4's first rows travel meanwhile
        if (tid / D < n_slot) x0 = r[(size_t)slot_id[tid / D] * D + tid % D];
        // ---- 3. the decisions: lane (g, n) looks at frame n and slots g, g + 4, ... ----
        if (wave == 0) {
            int w = n < nc && near_sh[n] != kNone ? slot_sh[near_sh[n]] : -1;       // the frame's winner, as assumed
            bool tied;
            const int done =
                chain_decide({sim_sh, width, lo_sh, sn_sh, isn_sh, ss_sh, out_v, gram_sh, slot_id, n_sh, irn_sh}, nc, n_slot, w, tied);
            if (lane < done) {
                int p = n_sh[slot_id[w]];
#pragma unroll
                for (int h = 0; h < FR - 1; ++h) p += h < lane && __builtin_amdgcn_readlane(w, h) == w ? 1 : 0;
                w_sh[lane] = w;
                p_sh[lane] = p;
                y_sh[lane] = __ddiv_rn(1.0, (double)p + 1.0);
                dv.assign[(size_t)u * dv.F + c0 + lane] = slot_id[w];
                dv.pos[(size_t)u * dv.F + c0 + lane] = p;
            }
            if (lane == 0) { nc_sh = done; tied_sh = tied; }
        }
        __syncthreads();
        nc = nc_sh;
        if (tied_sh) turn.failed();
        else turn.held();
        if (nested && wave == NW - 1) partition_reps(nc);
        // ---- 4. Eq. 3 on the rows ----
        for (int kb = 0; kb < n_slot; kb += SPB) {  // workgroup-uniform
            const int k = kb + tid / D, d = tid % D;                    // wave-uniform k
            int mine = 0;
            if (k < n_slot) {
                const double xs = kb == 0 ? x0 : r[(size_t)slot_id[k] * D + d];
                double x = xs;
                int w1 = w_sh[0], p1 = p_sh[0];     // (the next frame's operands are read ahead of this one's arithmetic)
                double y1 = y_sh[0], s1 = s_sh[0][d];
                for (int fc = 0; fc < nc; ++fc) {
                    const int w = __builtin_amdgcn_readfirstlane(w1), p = p1, fn = min(fc + 1, FR - 1);
                    const double y = y1, sv = s1;
                    w1 = w_sh[fn]; p1 = p_sh[fn]; y1 = y_sh[fn]; s1 = s_sh[fn][d];
                    if (w != k) continue;
                    x = eq3_finite((double)p, y, x, sv);
                    ++mine;
                }
                if (!(x == x)) {                    // infinite states: over again
                    x = xs;
                    for (int fc = 0; fc < nc; ++fc)
                        if (w_sh[fc] == k) x = eq3_channel((double)p_sh[fc], y_sh[fc], x, s_sh[fc][d]);
                }
                if (mine > 0) r[(size_t)slot_id[k] * D + d] = x;
                row_sh[tid / D][d] = x;
            }
            __syncthreads();
            const int kn = kb + grp;                // norm of slot kn, and its new size
            if (grp < SPB && kn < n_slot) {
                double x[EPL];
#pragma unroll
                for (int e = 0; e < EPL; ++e) x[e] = row_sh[grp][lr * EPL + e];
                const double sq = row16_sum(square_channels(x, row_second_first(C, slot_id[kn])));
                int cnt = 0;
                for (int fc = 0; fc < nc; ++fc) cnt += w_sh[fc] == kn;
                if (lr == 0) {
                    const int j = slot_id[kn];
                    if (cnt > 0) resize(j, n_sh[j] + cnt, sqrt(sq));
                    slot_sh[j] = -1;
                }
            }
            __syncthreads();
        }
        c0 += nc;
        __syncthreads();                            // before the next chunk overwrites the staged summaries
    }
}

// ---------------------------------------------------------------------------
// Online assignment + Eq. 3 without the maintainer for calls of a few frames, tables of up to THREADS / 2 clusters, one
// frame after the other.  grid (U), THREADS threads.  Each 16-lane group keeps its RPG rows of the unit's table
// (row j = group + (THREADS/16) i) in registers for the whole call, sizes and norms sit in LDS, and the winner's row is
// updated in place, so nothing in the per-frame chain waits on memory.  The operations of a similarity, of Eq. 3 and of a
// norm are those of the one-frame kernel and of k_assign_chain's frames in turn, in their order.
// What k_assign_chain pays per call whatever the number of frames -- sixteen frames' worth of matrix products, the nearest
// clusters, slots, the check -- is more than up to four frames in turn (4 layers, 700 frames, C = 180, whole calls with the
// page store, in turn / chain: 2 a call 11.0 / 13.4 us, 4 a call 14.9 / 16.2; 5 a call 17.2 / 17.0, 8 a call 23.3 / 20.7).
// ---------------------------------------------------------------------------
constexpr int kRegFrames = 4;

// Of this kernel and the one-frame kernel, whose 16-lane groups hold the table's rows in registers (rr[i]: row group + NG i).
// Dot products of the summary (sl: this lane's channels) with the rows, into dot, four rows at a time written out side by
// side: four independent multiply-add chains, then their 16-lane reductions step by step in lockstep, so that one chain's
// latency is filled by the other three (a loop over the rows with the block-uniform test per row kept every row's chain in
// a basic block of its own: 2100 cycles per frame for 210 instructions).  Rows beyond the table or of empty clusters give
// values nobody reads.  The group also forms |s| from its own share of the channels, the same bits in every group.
template <int EPL, int NG, int RPG>
__device__ __forceinline__ double held_products(const double (&sl)[EPL], const double (&rr)[RPG][EPL], int C, double *dot) {
    const int lr = threadIdx.x % 16, grp = threadIdx.x / 16;
    double ssq = 0.0;
#pragma unroll
    for (int h = 0; h < RPG / 4; ++h) {
        if (h > 0 && NG * 4 * h >= C) break;                  // block-uniform: passes beyond the table
        double p[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = __builtin_fma(sl[e], rr[4 * h + k][e], p[k]);
            if (h == 0) ssq = square_step<EPL>(ssq, sl, e, true);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] += dpp_f64<kDppXor8>(p[k]);
        if (h == 0) ssq += dpp_f64<kDppXor8>(ssq);
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] += dpp_f64<kDppXor7>(p[k]);
        if (h == 0) ssq += dpp_f64<kDppXor7>(ssq);
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] += dpp_f64<kDppXor3>(p[k]);
        if (h == 0) ssq += dpp_f64<kDppXor3>(ssq);
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] += dpp_f64<kDppXor1>(p[k]);
        if (h == 0) ssq += dpp_f64<kDppXor1>(ssq);
        if (lr == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) dot[grp + NG * (4 * h + k)] = p[k];
        }
    }
    return sqrt(ssq);
}
// The most similar candidate of each wavefront, ties to the lowest id (at most one candidate per thread: ids lo + thread)
__device__ __forceinline__ void held_nearest(int lo, int hi, const int *size, const double *norm, const double *dot, double sn,
                                             double *best_v, int *best_i) {
    const int j = lo + threadIdx.x;
    double bv = -INFINITY;
    int bi = 0x7fffffff;
    if (j < hi && size[j] > 0) {
        bv = (sn == 0.0 || norm[j] == 0.0) ? 0.0 : dot[j] / (sn * norm[j]);
        bi = j;
    }
    wave_best_ascending(bv, bi);
    if (threadIdx.x % 64 == 0) { best_v[threadIdx.x / 64] = bv; best_i[threadIdx.x / 64] = bi; }
}

template <int D, int THREADS>
__global__ __launch_bounds__(THREADS) void k_assign_update_reg(const DeviceView *self, int f0, int f1) {
    const DeviceView dv = device_view(self);
    constexpr int EPL = D / 16, NG = THREADS / 16, RPG = 8, NW = THREADS / 64, ROWS = NG * RPG;
    const int u = blockIdx.x, tid = threadIdx.x, C = dv.C;
    const int lr = tid % 16, grp = tid / 16, wave = tid / 64, lane = tid % 64;
    __shared__ __attribute__((aligned(16))) double s_sh[kRegFrames][D];
    __shared__ double dot_sh[ROWS], rn_sh[ROWS];
    __shared__ int n_sh[ROWS];
    __shared__ int a_out[kRegFrames], p_out[kRegFrames];
    __shared__ int chg_sh[ROWS];                // 1 = the cluster's size and norm changed in this call
    __shared__ double red_v[NW];
    __shared__ int red_i[NW];
    __shared__ double psum_sh[2];
    double *r = dv.r + (size_t)u * C * D;
    double rr[RPG][EPL];
#pragma unroll
    for (int i = 0; i < RPG; ++i) {
        const double *rj = r + (size_t)min(grp + NG * i, C - 1) * D + lr * EPL;
        if (NG * i < C) {                 // block-uniform: passes beyond the table are not loaded
#pragma unroll
            for (int e = 0; e < EPL; ++e) rr[i][e] = rj[e];
        } else {
#pragma unroll
            for (int e = 0; e < EPL; ++e) rr[i][e] = 0.0;
        }
    }
    for (int j = tid; j < ROWS; j += THREADS) {
        n_sh[j] = j < C ? dv.n[(size_t)u * C + j] : 0;
        rn_sh[j] = j < C ? dv.rnorm[(size_t)u * C + j] : 0.0;
        chg_sh[j] = 0;
    }
    const bool nested = dv.P > 0;
    // The barriers inside the frame loop order LDS traffic only, and the loop touches no global memory: the
    // call's summaries are staged in LDS, the winner's row stays in registers and is written back once after the last
    // frame, sizes and norms live in LDS, the frames' ids and ranks collect in LDS until the end.  A full __syncthreads() waits for every outstanding global access of the wavefront, and so
    // does any wait the compiler places for a register a load is still to fill: with the next frame's summary
    // fetched inside the loop and the winner's row written through in every frame, each frame waited once for
    // that load, issued a moment before, and once for the store's acknowledgement.  The nested hierarchy's
    // partition representatives and sizes do go through global memory from one frame to the next, so there the
    // barriers stay full ones.
    auto frame_barrier = [&]() {
        if (nested) __syncthreads();          // workgroup-uniform
        else lds_barrier();
    };
    unsigned int dirty = 0;                   // bit i: this group's row i changed in this call
    // a one-frame call is all latency: its results go straight to memory, with no collection and no write-back pass
    const bool single = f1 - f0 == 1;
    {
        const double *src = dv.summ + ((size_t)u * dv.F + f0) * D;
        for (int i = tid; i < (f1 - f0) * D / 2; i += THREADS)
            *reinterpret_cast<double2 *>(&s_sh[0][0] + 2 * i) = *reinterpret_cast<const double2 *>(src + 2 * i);
    }
    __syncthreads();
    for (int fc = 0; fc < f1 - f0; ++fc) {
        const int f = f0 + fc;
        const double *sv = s_sh[fc];
        const int part_f = nested ? dv.part[f] : 0;
        const int lo = nested ? part_f * dv.Cs : 0, hi = nested ? lo + dv.Cs : C;
        double sl[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) sl[e] = sv[lr * EPL + e];
        const double sn = held_products<EPL, NG>(sl, rr, C, dot_sh);
        frame_barrier();
        // argmax of the cosine over the candidates, ties to the lowest id (THREADS >= C: at
        // most one candidate per thread)
        held_nearest(lo, hi, n_sh, rn_sh, dot_sh, sn, red_v, red_i);
        // nested hierarchy: the partition's representative follows the same running mean
        int pn_i = 0;
        if (nested) {
            double *prow = dv.pr + ((size_t)u * dv.P + part_f) * D;
            pn_i = dv.pn[(size_t)u * dv.P + part_f];
            double pv = 0.0;
            if (tid < D) {
                pv = eq3_channel((double)pn_i, __ddiv_rn(1.0, (double)pn_i + 1.0), prow[tid], sv[tid]);
                prow[tid] = pv;
            }
            if (wave < 2) {
                const double psq = wave_square_sum(pv);
                if (lane == 0) psum_sh[wave] = psq;
            }
        }
        frame_barrier();
        // every thread merges the wavefronts' winners itself (no second barrier for one thread's merge)
        double bv = red_v[0];
        int bi = red_i[0];
#pragma unroll
        for (int w = 1; w < NW; ++w)
            if (better(red_v[w], red_i[w], bv, bi)) { bv = red_v[w]; bi = red_i[w]; }
        const int a = bi == 0x7fffffff ? lo : bi;
        const int ai = __builtin_amdgcn_readfirstlane(a / NG);      // workgroup-uniform: a scalar
        if (grp == a % NG) {                                  // the group that holds row a
            const int na_i = n_sh[a];
            const double na = (double)na_i;
            const double ny = __ddiv_rn(1.0, na + 1.0);
            double sq = 0.0;
#pragma unroll
            for (int i = 0; i < RPG; ++i) {
                if (i == ai) {                                // scalar branch: one pass runs
#pragma unroll
                    for (int e = 0; e < EPL; ++e) {
                        const double rv = eq3_channel(na, ny, rr[i][e], sl[e]);
                        rr[i][e] = rv;
                        if (single) r[(size_t)a * D + lr * EPL + e] = rv;
                    }
                    sq = square_channels(rr[i], i == 0);                      // (row_second_first: a < NG)
                }
            }
            if (!single) dirty |= 1u << ai;
            sq = row16_sum(sq);
            if (lr == 0) {
                const double nr = sqrt(sq);
                if (single) {
                    dv.rnorm[(size_t)u * C + a] = nr;
                    dv.n[(size_t)u * C + a] = na_i + 1;
                    dv.assign[(size_t)u * dv.F + f] = a;
                    dv.pos[(size_t)u * dv.F + f] = na_i;
                } else {
                    rn_sh[a] = nr;
                    n_sh[a] = na_i + 1;
                    chg_sh[a] = 1;
                    a_out[fc] = a;
                    p_out[fc] = na_i;
                }
            }
        }
        if (nested && tid == 0) {
            dv.prn[(size_t)u * dv.P + part_f] = sqrt(D > 64 ? psum_sh[0] + psum_sh[1] : psum_sh[0]);
            dv.pn[(size_t)u * dv.P + part_f] = pn_i + 1;
        }
        if (single) return;                   // workgroup-uniform: nothing follows the only frame
        frame_barrier();
    }
    // the frames' ids and ranks (the barrier that ended the last one made them visible)
    if (tid < f1 - f0) {
        dv.assign[(size_t)u * dv.F + f0 + tid] = a_out[tid];
        dv.pos[(size_t)u * dv.F + f0 + tid] = p_out[tid];
    }
    // write back what changed: rows, sizes and norms
#pragma unroll
    for (int i = 0; i < RPG; ++i) {
        if ((dirty >> i) & 1u) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) r[(size_t)(grp + NG * i) * D + lr * EPL + e] = rr[i][e];
        }
    }
    for (int j = tid; j < C; j += THREADS) {
        if (chg_sh[j]) {
            dv.n[(size_t)u * C + j] = n_sh[j];
            dv.rnorm[(size_t)u * C + j] = rn_sh[j];
        }
    }
}

// ---------------------------------------------------------------------------
// One frame in one launch (maintainer off, C <= 128, HBM tier, online phase).
// grid (U, 2), kOneBlock threads: y = 0 key page + summary + assignment + Eq. 3, y = 1 value page.
// The table is in flight -- eight rows per 16-lane group -- before the page store begins; what follows it runs out of
// registers and LDS.  (The page's loads first, so that it could be summed while the table is on its way: 5.90 -> 7.28 us.)  The same operations on the same operands as k_assign_chain, element by element.
// ---------------------------------------------------------------------------
constexpr int kOneBlock = 256;
template <typename E, int D>
__global__ __launch_bounds__(kOneBlock) void k_ingest_one(const DeviceView *self, const E *k_in, const E *v_in, int f) {
    const DeviceView dv = device_view<0, 1, 3>(self);
    constexpr int EPL = D / 16, NG = kOneBlock / 16, RPG = 128 / NG, NW = kOneBlock / 64, ROWS = NG * RPG;
    __shared__ StoreShared<D> store_sh;
    const int u = blockIdx.x;
    if (blockIdx.y == 1) {
        store_value_page<E, D, kOneBlock, false>(dv, v_in, dv.v_store, u, 0, f, store_sh);         // HBM tier only
        return;
    }
    const int tid = threadIdx.x, C = dv.C;
    const int lr = tid % 16, grp = tid / 16, wave = tid / 64, lane = tid % 64;
    __shared__ double s_sh[D], dot_sh[ROWS], rn_sh[ROWS];
    __shared__ int n_sh[ROWS];
    __shared__ double red_v[NW];
    __shared__ int red_i[NW];
    __shared__ double psum_sh[2];
    double *r = dv.r + (size_t)u * C * D;
    double rr[RPG][EPL];
#pragma unroll
    for (int i = 0; i < RPG; ++i) {
        const double *rj = r + (size_t)min(grp + NG * i, C - 1) * D + lr * EPL;
        if (NG * i < C) {                 // block-uniform: passes beyond the table are not loaded
#pragma unroll
            for (int e = 0; e < EPL; ++e) rr[i][e] = rj[e];
        } else {
#pragma unroll
            for (int e = 0; e < EPL; ++e) rr[i][e] = 0.0;
        }
    }
    if (tid < ROWS) {
        n_sh[tid] = tid < C ? dv.n[(size_t)u * C + tid] : 0;
        rn_sh[tid] = tid < C ? dv.rnorm[(size_t)u * C + tid] : 0.0;
    }
    const bool nested = dv.P > 0;
    const int part_f = nested ? dv.part[f] : 0;
    const int lo = nested ? part_f * dv.Cs : 0, hi = nested ? lo + dv.Cs : C;
    store_key_page<E, D, kOneBlock, false>(dv, k_in, dv.k_store, u, 0, f, store_sh, s_sh);
    __syncthreads();
    double sl[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) sl[e] = s_sh[lr * EPL + e];
    const double sn = held_products<EPL, NG>(sl, rr, C, dot_sh);
    __syncthreads();
    // argmax of the cosine over the candidates, ties to the lowest id (at most one candidate per thread)
    held_nearest(lo, hi, n_sh, rn_sh, dot_sh, sn, red_v, red_i);
    // nested hierarchy: the partition's representative in this unit's key space follows the same running mean
    int pn_i = 0;
    if (nested) {
        double *prow = dv.pr + ((size_t)u * dv.P + part_f) * D;
        pn_i = dv.pn[(size_t)u * dv.P + part_f];
        double pv = 0.0;
        if (tid < D) {
            pv = eq3_channel((double)pn_i, __ddiv_rn(1.0, (double)pn_i + 1.0), prow[tid], s_sh[tid]);
            prow[tid] = pv;
        }
        if (wave < 2) {
            const double psq = wave_square_sum(pv);
            if (lane == 0) psum_sh[wave] = psq;
        }
    }
    __syncthreads();
    // every thread merges the wavefronts' winners itself (no second barrier for one thread's merge)
    double bv = red_v[0];
    int bi = red_i[0];
#pragma unroll
    for (int w = 1; w < NW; ++w)
        if (better(red_v[w], red_i[w], bv, bi)) { bv = red_v[w]; bi = red_i[w]; }
    const int a = bi == 0x7fffffff ? lo : bi;
    const int ai = __builtin_amdgcn_readfirstlane(a / NG);      // workgroup-uniform: a scalar
    if (grp == a % NG) {                                  // the group that holds row a: Eq. 3 as in k_assign_chain
        const int na_i = n_sh[a];
        const double na = (double)na_i, ny = __ddiv_rn(1.0, na + 1.0);
        double sq = 0.0;
#pragma unroll
        for (int i = 0; i < RPG; ++i) {
            if (i == ai) {                                // scalar branch: one pass runs
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    rr[i][e] = eq3_channel(na, ny, rr[i][e], sl[e]);
                    r[(size_t)a * D + lr * EPL + e] = rr[i][e];
                }
                sq = square_channels(rr[i], row_second_first(C, a));
            }
        }
        sq = row16_sum(sq);
        if (lr == 0) {
            dv.rnorm[(size_t)u * C + a] = sqrt(sq);
            dv.n[(size_t)u * C + a] = na_i + 1;
            dv.assign[(size_t)u * dv.F + f] = a;
            dv.pos[(size_t)u * dv.F + f] = na_i;
        }
    }
    if (nested && tid == 0) {
        dv.prn[(size_t)u * dv.P + part_f] = sqrt(D > 64 ? psum_sh[0] + psum_sh[1] : psum_sh[0]);
        dv.pn[(size_t)u * dv.P + part_f] = pn_i + 1;
    }
}

// ---------------------------------------------------------------------------
// Lloyd: seeds from the warm-up buffer.  grid (U), 256 threads.
// r_j = summary of frame floor(j*W/C); every cluster counts as non-empty for
// the first assignment round (n_j = 1 as a placeholder).
// ---------------------------------------------------------------------------
// With the maintainer on only the first c_init ids are seeded (the rest of the
// table is empty until splits fill it) and the maintainer's state is cleared.
template <int D>
__global__ __launch_bounds__(kBlock) void k_lloyd_seed(const DeviceView *self, int W) {
    const DeviceView dv = device_view(self);
    constexpr int EPL = D / 16;
    const int u = blockIdx.x, tid = threadIdx.x, C = dv.C;
    const int Cl = dv.maint_mode ? dv.c_init : C;
    const int lr = tid % 16, row0 = tid / 16;
    for (int j = row0; j < C; j += 16) {
        double *rj = dv.r + ((size_t)u * C + j) * D + lr * EPL;
        if (j >= Cl) {
#pragma unroll
            for (int i = 0; i < EPL; ++i) rj[i] = 0.0;
            if (lr == 0) { dv.rnorm[(size_t)u * C + j] = 0.0; dv.n[(size_t)u * C + j] = 0; }
            continue;
        }
        const int src = (int)(((long long)j * W) / Cl);
        const double *s = dv.summ + ((size_t)u * dv.F + src) * D + lr * EPL;
        double sq = 0.0;
#pragma unroll
        for (int i = 0; i < EPL; ++i) { rj[i] = s[i]; sq += s[i] * s[i]; }
        sq = group16_sum(sq);
        if (lr == 0) { dv.rnorm[(size_t)u * C + j] = sqrt(sq); dv.n[(size_t)u * C + j] = 1; }
    }
    if (dv.maint_mode) {
        for (int j = tid; j < C; j += kBlock) {
            dv.var[(size_t)u * C + j] = 0.0;
            dv.lazy[(size_t)u * C + j] = 0;
            dv.resident[(size_t)u * C + j] = 0;
        }
        if (tid == 0) { dv.n_slots[u] = Cl; dv.n_buf[u] = 0; }
        if (tid < 4) dv.mt_cnt[(size_t)u * 4 + tid] = 0;
    }
}

// ---------------------------------------------------------------------------
// Seeds under the nested hierarchy (Sec. V-B).  grid (U, ceil(C/64)), 256 threads: 64 cluster ids each.
// Cluster id j = p*Cs + jj belongs to visual partition p.  With np warm-up
// frames in p and L = min(Cs, np), id j is started (n_j = 1 as a placeholder)
// from the summary of the partition's member floor(jj*np/L) if jj < L and is
// left empty otherwise.  A wavefront per partition walks the frame -> partition map 64 frames at a time -- once
// to count, once to meet the members its lanes' clusters start from -- instead of a thread per partition one frame
// at a time for all ids of a unit (W = 1024, P = 16, C = 512: 250 -> 24 us).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kBlock) void k_lloyd_seed_nested(const DeviceView *self, int W) {
    const DeviceView dv = device_view(self);
    constexpr int EPL = D / 16;
    const int u = blockIdx.x, tid = threadIdx.x, lane = tid % 64, C = dv.C, Cs = dv.Cs;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lr = tid % 16, grp = tid / 16;
    const int j0 = blockIdx.y * 64, j1 = min(C, j0 + 64);
    __shared__ int src_sh[64];                // frame that starts cluster j0 + i, -1: stays empty
    for (int p = j0 / Cs + wave; p <= (j1 - 1) / Cs; p += kBlock / 64) {
        int np = 0;
        for (int f0 = 0; f0 < W; f0 += 64)
            np += __popcll(__ballot(f0 + lane < W && dv.part[min(f0 + lane, W - 1)] == p));
        const int jj = j0 + lane - p * Cs, L = min(Cs, np);
        const bool mine = j0 + lane < j1 && jj >= 0 && jj < Cs;
        const int want = mine && jj < L ? (int)(((long long)jj * np) / L) : -1;
        int src = -1, seen = 0;
        for (int f0 = 0; f0 < W; f0 += 64) {
            unsigned long long m = __ballot(f0 + lane < W && dv.part[min(f0 + lane, W - 1)] == p);
            const int here = __popcll(m), t = want - seen;
            for (int i = 0; m; ++i, m &= m - 1)                      // the i-th member of these 64 frames
                if (t == i) src = f0 + __ffsll((long long)m) - 1;
            seen += here;
        }
        if (mine) src_sh[lane] = src;
    }
    __syncthreads();
    for (int i = grp; j0 + i < j1; i += kBlock / 16) {
        const size_t j = (size_t)u * C + j0 + i;
        const int src = src_sh[i];
        const double *s = dv.summ + ((size_t)u * dv.F + max(src, 0)) * D + lr * EPL;
        double sq = 0.0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
            const double x = src >= 0 ? s[e] : 0.0;
            dv.r[j * D + lr * EPL + e] = x;
            sq += x * x;
        }
        sq = group16_sum(sq);
        if (lr == 0) { dv.rnorm[j] = sqrt(sq); dv.n[j] = src >= 0 ? 1 : 0; }
    }
}

// ---------------------------------------------------------------------------
// Partition representatives from the member lists: per unit and visual
// partition the mean of the key summaries of the partition's frames, in
// ascending frame order.  grid (U, P), 128 threads (thread d owns channel d; the
// members are listed first, then sixteen loads are in flight: 73 -> 13 us for 1024 frames).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(128) void k_partition_reps(const DeviceView *self, int n_frames) {
    const DeviceView dv = device_view(self);
    constexpr int NT = 128, CH = NT * kListPer;
    const int u = blockIdx.x, p = blockIdx.y, tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    __shared__ double nsum_sh[2];
    __shared__ int mem[CH];
    __shared__ int wtot[NT / 64];
    const double *sb = dv.summ + (size_t)u * dv.F * D + tid;
    double acc = 0.0;
    int count = 0;
    for (int c0 = 0; c0 < n_frames; c0 += CH) {
        const int m = list_members<NT>(dv.part, p, c0, n_frames, mem, wtot);
        if (tid < D) acc = add_members<16>(acc, mem, m, [&](int f) { return sb[(size_t)f * D]; });
        count += m;
    }
    double sq = 0.0;
    if (tid < D) {
        const double rv = count > 0 ? acc / (double)count : 0.0;
        dv.pr[((size_t)u * dv.P + p) * D + tid] = rv;
        sq = rv * rv;
    }
    sq = wave_sum(sq);
    if (lane == 0) nsum_sh[wave] = sq;
    __syncthreads();
    if (tid == 0) {
        dv.prn[(size_t)u * dv.P + p] = sqrt(nsum_sh[0] + nsum_sh[1]);
        dv.pn[(size_t)u * dv.P + p] = count;
    }
}

// ---------------------------------------------------------------------------
// Intra-cluster variance from the member lists (Eq. 2), after a K-means run.
// grid (U, clusters), 256 threads: 16-lane groups take members in turn, the
// group partials are added in a fixed order.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kBlock) void k_exact_var(const DeviceView *self, int n_frames) {
    const DeviceView dv = device_view(self);
    constexpr int EPL = D / 16, NG = kBlock / 16;
    const int u = blockIdx.x, j = blockIdx.y, tid = threadIdx.x, C = dv.C;
    const int lr = tid % 16, grp = tid / 16;
    __shared__ double part[NG];
    const int *assign = dv.assign + (size_t)u * dv.F;
    const double *rj = dv.r + ((size_t)u * C + j) * D + lr * EPL;
    double rv[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) rv[i] = rj[i];
    double acc = 0.0;
    for (int f = grp; f < n_frames; f += NG) {
        if (assign[f] != j) continue;                    // uniform within the 16-lane group
        const double *s = dv.summ + ((size_t)u * dv.F + f) * D + lr * EPL;
        double p = 0.0;
#pragma unroll
        for (int i = 0; i < EPL; ++i) { const double t = s[i] - rv[i]; p += t * t; }
        acc += group16_sum(p);
    }
    if (lr == 0) part[grp] = acc;
    __syncthreads();
    if (tid == 0) {
        double tot = 0.0;
        for (int g = 0; g < NG; ++g) tot += part[g];
        const int cnt = dv.n[(size_t)u * C + j];
        dv.var[(size_t)u * C + j] = cnt > 0 ? tot / (double)cnt : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Lloyd assignment round: similarity table = summaries x representatives^T, a
// dense fp64 contraction, on the matrix cores (v_mfma_f64_16x16x4_f64: A lane
// (row = lane%16, k = lane/16), B lane (col = lane%16, k = lane/16), result
// register v of a lane = element (row 4v + lane/16, col lane%16)).
// grid (U, ceil(F/64)), 256 threads: a wavefront owns 16 frames, keeps their
// summaries in registers as the A operand for the whole call, and sweeps the
// representatives 16 at a time (each tile staged once per workgroup in LDS,
// double buffered, the next tile in flight behind the current tile's MFMAs).  Lane group k
// holds channels 8s + 2k and 8s + 2k + 1 of k-step s (one 16-byte load feeds two
// MFMAs); the order of the additions inside a dot product is therefore not the
// channel order, which moves a similarity by rounding only.
// ---------------------------------------------------------------------------

// Rounds that change nothing are skipped: a round `it` that moved no frame of a unit leaves the same
// members, hence (the sums being one fixed sequence of additions) the same representatives bit for
// bit, hence the same assignments in every later round.  moved[u][it % 3] counts the frames round
// `it` moved; a round whose predecessor moved none returns at once (and so does its update kernel).
// The slot of the round after is cleared by this launch, which neither reads nor counts in it.
//
// Frames whose assignment cannot change are skipped as well, by the distance bounds of accelerated
// K-means (Hamerly, SDM 2010; bounds by groups of representatives: Ding et al., ICML 2015) taken on the unit sphere, where the largest
// cosine is the smallest chord d(s, r) = |s/|s| - r/|r|| = sqrt(2 - 2 cos): a round that computes a frame's similarities leaves
// ub = d(own representative) and, for each group of representatives, lb = the least d to one of the group other than its own; an update that
// moves representative j by delta_j = d(old r_j, new r_j) can change any frame's distance to it by at most delta_j, so after it
// ub + delta_own still bounds the own distance from above and lb - max delta_j over the group the others from below (triangle
// inequality).  While ub < lb for every group, by more than the rounding of the similarities (> 5e-13 in the cosine), the own representative
// wins and the full computation would return the same id: such a frame only gets the moved bounds stored.  Any other is computed again
// against the groups that fail and its own, whose bounds are then exact again.  Round 0 computes everything.
// The assignments are the same as without the test, by construction: a similarity is the same sum whichever others are formed beside it.
// Bounds are whole multiples of 2^-14, rounded outwards: ub < lb then means a distance of at least that.  A frame's eight, 16 bytes: ub, then
// seven groups' lb.  (One lb for all other representatives, sixteen consecutive frames at a time: a representative that jumps far made every row of its unit live
// again, 45 % of the frame-candidate pairs of the second round of 112 units x 1536 frames and 10 to 60 % of those after it; by groups and single
// frames 3 and 0.1 to 3 %.)
constexpr int kChordOne = 1 << 14, kChordNever = 65534, kChordNone = 65535;    // 1.0; an ub no lb exceeds; the lb of a group without candidates
constexpr int kChordLost = 65535;                                              // the movement of a representative whose chords are, or were, no number
__device__ __forceinline__ int chord_up(double d) { return d < 2.0 ? (int)(d * kChordOne) + 1 : 2 * kChordOne; }          // (also where d is no number)
__device__ __forceinline__ int chord_down(double d) { return d > 0.0 ? (int)fmin(d * kChordOne, 2.0 * kChordOne) : 0; }

// (written out: the compiler's own fmaxf first makes a quiet number of every operand that comes from another lane)
__device__ __forceinline__ float max_f32(float a, float b) { float r; asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
__device__ __forceinline__ float min_f32(float a, float b) { float r; asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
__device__ __forceinline__ float max3_f32(float a, float b, float c) { float r; asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c)); return r; }
template <int CTRL> __device__ __forceinline__ float dpp_f32(float x) { return __int_as_float(dpp_i32<CTRL>(__float_as_int(x))); }
// largest and second largest of x over the 16 lanes of a row, in every lane
__device__ __forceinline__ void row16_top2(float x, float &m1, float &m2) {
    float o = dpp_f32<kDppXor8>(x);
    m2 = min_f32(x, o);
    m1 = max_f32(x, o);
    o = dpp_f32<kDppXor7>(m1);
    m2 = max3_f32(m2, dpp_f32<kDppXor7>(m2), min_f32(m1, o));
    m1 = max_f32(m1, o);
    o = dpp_f32<kDppXor3>(m1);
    m2 = max3_f32(m2, dpp_f32<kDppXor3>(m2), min_f32(m1, o));
    m1 = max_f32(m1, o);
    o = dpp_f32<kDppXor1>(m1);
    m2 = max3_f32(m2, dpp_f32<kDppXor1>(m2), min_f32(m1, o));
    m1 = max_f32(m1, o);
}
template <int CTRL> __device__ __forceinline__ unsigned int or_step(unsigned int x) { return x | (unsigned int)dpp_i32<CTRL>((int)x); }
__device__ __forceinline__ unsigned int row16_or(unsigned int x) {
    return or_step<kDppXor1>(or_step<kDppXor3>(or_step<kDppXor7>(or_step<kDppXor8>(x))));
}

// Round 0: grid (U, ceil(F/64)), a workgroup's four wavefronts take 16 consecutive frames each.  LATER, the instantiation for the rounds after
// it: grid (U, ceil(F/128)); a workgroup tests 128 frames, a thread each, and its wavefronts then take the live ones 16 at a time, in order,
// so that those taken together mostly ask for the same tiles.  A tile of 16 representatives that no frame of a wavefront asks for is not multiplied, one that
// none of the workgroup's asks for is not staged.  (256 frames a workgroup: where most are live its tasks follow one another, 10 us longer.)
// 112 units, C = 128, 512 to 1536 frames, a later round on average, nothing beside it: rows of sixteen consecutive frames, live or not by one bound, in a
// list that a launch of its own made, all tiles for each: 7.6 + 57 us; now 35 us (18 us where little is live).  4 units of C = 512 in 16
// partitions: 6.1 + 39.5 us; now 16 us; round 0, where tiles of other partitions are no longer multiplied, 59 -> 40 us.
constexpr int kLloydTest = 128;
template <int D, bool LATER, bool NESTED>
__global__ __launch_bounds__(kBlock, LATER ? 2 : 3) void k_lloyd_assign(const DeviceView *self, int n_frames, int it) {
    const DeviceView dv = device_view(self);
    constexpr int KS = D / 8;
    static_assert(kLloydTiles <= kBlock, "a thread per tile writes its group");
    static_assert(kLloydTest <= kBlock && kLloydTest % 64 == 0, "a thread per frame, whole wavefronts");
    const int u = blockIdx.x, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, C = dv.C;
    const int row = lane % 16, kq = lane / 16;
    int *moved = dv.lloyd_moved + (size_t)u * 3;
    if (blockIdx.y == 0 && tid == 0) moved[(it + 1) % 3] = 0;
    const double *r = dv.r + (size_t)u * C * D;
    const int n_tiles = (C + 15) / 16;
    const LloydGroups groups(dv.P, dv.Cs, C);
    ChordBounds *bounds = dv.lloyd_bounds + (size_t)u * dv.F;
    // A tile of 16 representatives is shared by the four wavefronts through LDS (each row is read
    // from L2 once per workgroup); rows are padded by 16 bytes so that the 16 lanes of a k group hit
    // 16 different 16-byte bank groups.  The next tile travels global -> registers while one is used.
    constexpr int LROW = D + 2, PPT = 16 * D / 2 / kBlock;        // doubles per LDS row; 16-byte pieces per thread
    __shared__ __attribute__((aligned(16))) double b_lds[2][16][LROW];
    f64x2 stg[PPT];
    auto fetch_tile = [&](int ct) {
#pragma unroll
        for (int i = 0; i < PPT; ++i) {
            const int p = tid + kBlock * i, trow = p / (D / 2), seg = p % (D / 2);
            stg[i] = *reinterpret_cast<const f64x2 *>(r + (size_t)min(16 * ct + trow, C - 1) * D + 2 * seg);
        }
    };
    auto stage_tile = [&](int buf) {
#pragma unroll
        for (int i = 0; i < PPT; ++i) {
            const int p = tid + kBlock * i, trow = p / (D / 2), seg = p % (D / 2);
            *reinterpret_cast<f64x2 *>(&b_lds[buf][trow][2 * seg]) = stg[i];
        }
    };
    // The ranking of a frame's similarities does not need the division by |s| |r_j| per candidate: |s| is the
    // same positive factor for every j, so the winner is argmax_j dot_j * (1 / |r_j|).  The fp64 matrix
    // instruction runs on the vector unit's fp64 lanes (counters: no cycle in which both execute), so every
    // vector instruction of the tile epilogue is time taken from the contraction: per candidate one fused
    // multiply-add, dot * scale_j + offset_j, with the pair formed once per workgroup in LDS: (1 / |r_j|, 0) for
    // a candidate, (0, 0) for a zero representative (its cosine is 0), (0, -inf) for an empty cluster and past
    // the table's end.  An all-zero summary gives 0 for every candidate and so the lowest id, as its cosines
    // (all 0) do.
    __shared__ __attribute__((aligned(16))) f64x2 scale_sh[1024 + 16];    // the cluster-count limit of a context, rounded up to tiles
    __shared__ double sn_sh[4][16];
    __shared__ unsigned long long tiles_sh[4];
    __shared__ unsigned char group_sh[kLloydTiles];                       // group of a tile, counted from the frame's first
    // LATER: a tile's largest movement of a representative * 16 + 15 - whose, and its second largest; the live frames, and the tiles they ask for
    __shared__ unsigned short delta_sh[LATER ? 1024 + 16 : 1];            // what the last update moved a representative by, at most, or kChordLost
    __shared__ unsigned char odd_sh[kLloydTiles];                         // a tile with a live representative that is not finite
    __shared__ int top_sh[LATER ? kLloydTiles : 1], second_sh[LATER ? kLloydTiles : 1], live_sh[LATER ? 4 : 1];
    __shared__ unsigned char list_sh[LATER ? kLloydTest : 1];
    __shared__ unsigned long long need_sh[LATER ? kLloydTest : 1];
    const int f0 = blockIdx.y * (LATER ? kLloydTest : 64);
    int n_live = min(64, n_frames - f0);
    ChordBounds cb{};
    int own = 0, plo_t = 0, moved_before = 1;
    // (loads without a condition, before anything waits for one)
    int nj = dv.n[(size_t)u * C + min(tid, C - 1)];
    double rnj = dv.rnorm[(size_t)u * C + min(tid, C - 1)], dj = 0.0;
    if constexpr (LATER) {
        const int f = min(f0 + tid, n_frames - 1);
        dj = dv.lloyd_delta[(size_t)u * C + min(tid, C - 1)];
        cb = bounds[f];
        own = dv.assign[(size_t)u * dv.F + f];
        if constexpr (NESTED) plo_t = dv.part[f] * dv.Cs;
        moved_before = moved[(it - 1) % 3];
        if (moved_before == 0) return;                         // workgroup-uniform: converged in an earlier round
    }
    for (int j = tid; j < 16 * n_tiles; j += kBlock) {
        if (j >= kBlock) {
            nj = dv.n[(size_t)u * C + min(j, C - 1)];
            rnj = dv.rnorm[(size_t)u * C + min(j, C - 1)];
            if constexpr (LATER) dj = dv.lloyd_delta[(size_t)u * C + min(j, C - 1)];
        }
        f64x2 e = {0.0, -INFINITY};
        if (j < C && nj > 0) {
            e.x = rnj == 0.0 ? 0.0 : 1.0 / rnj;
            e.y = 0.0;
        }
        scale_sh[j] = e;
        const bool odd = j < C && nj > 0 && !(rnj < INFINITY);
        const unsigned long long odd_lanes = __ballot(odd);
        if (row == 0) odd_sh[j / 16] = (odd_lanes >> lane & 0xffff) != 0;
        if constexpr (LATER) {
            if (j >= C) dj = 0.0;
            const int d = dj == 0.0 ? 0 : chord_up(dj);
            delta_sh[j] = (unsigned short)(odd || dj != dj ? kChordLost : d);
            int top = 16 * d + 15 - row;
            top = max(top, dpp_i32<kDppXor8>(top));
            top = max(top, dpp_i32<kDppXor7>(top));
            top = max(top, dpp_i32<kDppXor3>(top));
            top = max(top, dpp_i32<kDppXor1>(top));
            int second = row == 15 - top % 16 ? 0 : d;
            second = max(second, dpp_i32<kDppXor8>(second));
            second = max(second, dpp_i32<kDppXor7>(second));
            second = max(second, dpp_i32<kDppXor3>(second));
            second = max(second, dpp_i32<kDppXor1>(second));
            if (row == 0) { top_sh[j / 16] = top; second_sh[j / 16] = second; }
        }
    }
    if (tid < groups.span) group_sh[tid] = (unsigned char)groups.of(tid);
    if constexpr (LATER) {
        // the test
        __syncthreads();
        const int t0 = plo_t / 16, t1 = (NESTED ? plo_t + dv.Cs - 1 : C - 1) / 16 + 1;
        const bool in = tid < kLloydTest && f0 + tid < n_frames;
        const int ub = min((int)cb.ub + (int)delta_sh[own], kChordNever);
        const bool lost = delta_sh[own] == kChordLost;                      // every other candidate may win, a later one than any bound knows of too
        unsigned long long need = 0;
#pragma unroll
        for (int g = 0; g < kLloydGroups; ++g) {
            int d = 0;
            for (int t = groups.lo(g); t < groups.lo(g + 1); ++t) {         // (uniform)
                const int tt = min(t0 + t, n_tiles - 1), top = top_sh[tt];
                const int dt = tt == own / 16 && top % 16 == 15 - own % 16 ? second_sh[tt] : top / 16;
                d = t0 + t < t1 ? max(d, dt) : d;
            }
            const int lb = cb.lb[g] == kChordNone ? kChordNone : max(0, (int)cb.lb[g] - d);
            cb.lb[g] = (unsigned short)lb;
            if (ub >= lb || lost) need |= groups.tiles(g, t0, t1);
        }
        cb.ub = (unsigned short)ub;
        if (in) bounds[f0 + tid] = cb;
        const bool live = in && need != 0;
        if (live) need |= groups.tiles(group_sh[own / 16 - t0], t0, t1);    // the own group: the exact own distance, and its bound if the frame leaves
        if (tid < kLloydTest) need_sh[tid] = need;
        const unsigned long long lv = __ballot(live);
        if (lane == 0) live_sh[wave] = __popcll(lv);
        __syncthreads();
        int at = __popcll(lv & ((1ull << lane) - 1));
        n_live = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) { at += w < wave ? live_sh[w] : 0; n_live += live_sh[w]; }
        if (n_live == 0) return;                                // workgroup-uniform
        if (live) list_sh[at] = (unsigned char)tid;
        __syncthreads();
    }
    for (int task = 0; task < n_live; task += 64) {
        const int k0 = task + 16 * wave;                        // this wavefront's frames: k0 .. of the live ones
        const bool busy = k0 < n_live;
        auto frame = [&](int i) {                               // the i-th of them (the last live one past the end)
            const int k = min(k0 + i, n_live - 1);
            return f0 + (LATER ? (int)list_sh[k] : k);
        };
        f64x2 a[KS];
        unsigned long long mine = 0;                            // tiles that the frames of this lane's row ask for
        if (busy) {
            const int f = frame(row);
            const double *sp = dv.summ + ((size_t)u * dv.F + f) * D + 2 * kq;
#pragma unroll
            for (int s = 0; s < KS; ++s) a[s] = *reinterpret_cast<const f64x2 *>(sp + 8 * s);
            if constexpr (LATER) mine = need_sh[f - f0];
            else {
                const int lo = NESTED ? dv.part[f] * dv.Cs : 0, hi = NESTED ? lo + dv.Cs : C;
                mine = (~0ull >> (63 - (hi - 1) / 16 + lo / 16)) << (lo / 16);
            }
            mine = ((unsigned long long)row16_or((unsigned int)(mine >> 32)) << 32) | row16_or((unsigned int)mine);
        }
        mine = ((unsigned long long)(unsigned int)__builtin_amdgcn_readfirstlane((int)(mine >> 32)) << 32) |
               (unsigned int)__builtin_amdgcn_readfirstlane((int)mine);
        if (lane == 0) tiles_sh[wave] = mine;
        int fv[4], plo[4], phi[4], bi[4];
        double bv[4];
        float g1[4], g2[4];              // of group `row`: largest and second largest similarity (times |s|)
#pragma unroll
        for (int v = 0; v < 4; ++v) {    // the four result rows of this lane
            bv[v] = -INFINITY; bi[v] = 0x7fffffff; g1[v] = -INFINITY; g2[v] = -INFINITY;
            fv[v] = frame(4 * v + kq); plo[v] = 0; phi[v] = C;
            if constexpr (NESTED) {        // nested hierarchy: only the ids of the frame's visual partition are candidates
                plo[v] = dv.part[fv[v]] * dv.Cs;
                phi[v] = plo[v] + dv.Cs;
            }
        }
        __syncthreads();
        unsigned long long left = tiles_sh[0] | tiles_sh[1] | tiles_sh[2] | tiles_sh[3];
        left = ((unsigned long long)(unsigned int)__builtin_amdgcn_readfirstlane((int)(left >> 32)) << 32) |
               (unsigned int)__builtin_amdgcn_readfirstlane((int)left);
        int ct = __ffsll((long long)left) - 1, buf = 0;
        fetch_tile(ct);
        int a_was[4] = {0, 0, 0, 0};     // the frames' ids before this round, for the lane that finishes them
        if (busy) {
#pragma unroll
            for (int v = 0; v < 4; ++v) a_was[v] = dv.assign[(size_t)u * dv.F + fv[v]];
            double sq = 0.0;
#pragma unroll
            for (int s = 0; s < KS; ++s) sq += a[s].x * a[s].x + a[s].y * a[s].y;
            sq += __shfl_xor(sq, 16, 64);
            sq += __shfl_xor(sq, 32, 64);
            if (kq == 0) sn_sh[wave][row] = sqrt(sq);
        }
        stage_tile(0);
        __syncthreads();
        for (;;) {
            left &= left - 1;
            const int next = left ? __ffsll((long long)left) - 1 : ct;
            fetch_tile(next);
            if ((mine >> ct) & 1) {                             // wave-uniform
                f64x2 b[KS];
#pragma unroll
                for (int s = 0; s < KS; ++s) b[s] = *reinterpret_cast<const f64x2 *>(&b_lds[buf][row][8 * s + 2 * kq]);
                const f64x2 sc = scale_sh[16 * ct + row];
                // one accumulator chain: back-to-back matrix instructions on the same accumulator sustain 70 TFLOP/s
                // in a probe of nothing else, two alternating accumulators 66, four 58
                f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s].x, b[s].x, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s].y, b[s].y, acc, 0, 0, 0);
                }
                const int j = 16 * ct + row;
                // A lane meets its candidates in ascending id order, so a strict comparison keeps the lowest id of equals.
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    double c = __builtin_fma(acc[v], sc.x, sc.y);
                    if (NESTED && (j < plo[v] || j >= phi[v])) c = -INFINITY;
                    bi[v] = c > bv[v] ? j : bi[v];
                    bv[v] = max_f64(bv[v], c);
                    // the tile's two largest join those of its group (lane `row` keeps group `row`)
                    const int t = ct - plo[v] / 16;
                    const bool here = row == (int)group_sh[NESTED ? min(max(t, 0), groups.span - 1) : ct];
                    float m1, m2;
                    row16_top2((float)c, m1, m2);
                    m1 = here ? m1 : -INFINITY;                 // (no branch: the four rows' chains interleave)
                    m2 = here ? m2 : -INFINITY;
                    g2[v] = max3_f32(g2[v], m2, min_f32(g1[v], m1));
                    g1[v] = max_f32(g1[v], m1);
                }
            }
            if (left == 0) break;                               // workgroup-uniform
            stage_tile(buf ^ 1);            // the other buffer: last read before the previous barrier
            __syncthreads();
            ct = next;
            buf ^= 1;
        }
        const unsigned long long odd_tiles = __ballot(lane < n_tiles && odd_sh[lane]);
        if (busy) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                // best over the 16 columns a lane group covers (lanes 16k .. 16k + 15)
                best_step<kDppXor8>(bv[v], bi[v]);
                best_step<kDppXor7>(bv[v], bi[v]);
                best_step<kDppXor3>(bv[v], bi[v]);
                best_step<kDppXor1>(bv[v], bi[v]);
                if (k0 + 4 * v + kq >= n_live) continue;
                const int f = fv[v];
                const bool none = bv[v] == -INFINITY;            // no candidate at all: the first id of the range
                const int a_new = none ? plo[v] : bi[v];
                if (row == 0 && a_was[v] != a_new) {
                    dv.assign[(size_t)u * dv.F + f] = a_new;
                    atomicAdd(&moved[it % 3], 1);
                    // both clusters' sums change; every other cluster's update is skipped (round 0 updates all)
                    dv.lloyd_changed[(size_t)u * C + a_new] = 1;
                    if (a_was[v] >= 0 && a_was[v] < C) dv.lloyd_changed[(size_t)u * C + a_was[v]] = 1;
                }
                // Chords to the winner (lane 7) and to the best other candidate of group `row` (a frame without a winner, or whose
                // summary is all zeros or nearly, is never skipped).  A representative that is not finite is no candidate as long as it is not, and may
                // be finite after the next update: its group has no bound.  Roots in fp32, pushed outwards (relative error below 2e-7 with the
                // conversion); a similarity that has been rounded to fp32 is pushed upwards first.
                const double sn = sn_sh[wave][4 * v + kq], inv = 1.0 / sn;
                const bool sound = !none && sn > 1e-30 && sn < 1e30;         // (what fp32 similarities hold)
                const int t0 = plo[v] / 16, t1 = (phi[v] - 1) / 16 + 1;
                const unsigned long long gt = row < kLloydGroups ? groups.tiles(row, t0, t1) : 0ull;
                const float sim = row == (int)group_sh[sound ? a_new / 16 - t0 : 0] ? g2[v] : g1[v];
                const double cos = row == 7 ? bv[v] * inv : ((double)sim + fabs((double)sim) * 1.2e-7) * inv;
                const double chord = (double)sqrtf((float)fmax(0.0, 2.0 - 2.0 * cos));
                unsigned short *o = reinterpret_cast<unsigned short *>(bounds + f);
                if (row == 7) o[0] = (unsigned short)(sound ? chord_up(chord * (1.0 + 1e-6) + 1e-9) : kChordNever);
                else if (row < kLloydGroups && (mine & gt) == gt)
                    o[1 + row] = (unsigned short)(!sound || (gt & odd_tiles) ? 0 : sim == -INFINITY ? kChordNone : chord_down(chord * (1.0 - 1e-6) - 1e-9));
            }
        }
        if constexpr (!LATER) break;
        __syncthreads();                                        // (the buffers and masks are written again)
    }
}

// ---------------------------------------------------------------------------
// Lloyd update round.  grid (U, C), 128 threads (thread d owns channel d).
// Members are found by an order-preserving compaction of the assignment array,
// 2048 frames at a time: the assignments are staged in LDS with coalesced loads,
// every thread then looks at 16 consecutive frames, a scan over the threads' match
// counts gives each match its slot, and the member summaries are added in ascending
// frame order, so the mean is the same sequence of additions a sequential loop would
// perform.  The launch reads every fp64 summary of every unit once (1 KB per frame and
// unit: 470 MB at 112 units x 4096 frames), which is what bounds it.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(128) void k_lloyd_update(const DeviceView *self, int n_frames, int it) {
    const DeviceView dv = device_view(self);
    constexpr int NT = 128, FPT = 16, CH = NT * FPT;
    const int u = blockIdx.x, j = blockIdx.y, tid = threadIdx.x, C = dv.C;
    // (a round that moved no frame would rebuild the same sums: see k_lloyd_assign)
    if (it > 0 && dv.lloyd_moved[(size_t)u * 3 + it % 3] == 0) return;
    // A cluster that no frame entered or left in this round (flags set by k_lloyd_assign) has the same
    // members, so the same sums bit for bit: it is not recomputed, and its representative has not moved.
    // Round 0 recomputes every cluster (the online running means are not the ordered sums).
    int *changed = dv.lloyd_changed + (size_t)u * C + j;
    double *delta = dv.lloyd_delta + (size_t)u * C + j;
    if (it > 0 && *changed == 0) {                   // workgroup-uniform: the flag is cleared only after the last barrier
        if (tid == 0) *delta = 0.0;
        return;
    }
    const double norm_old = dv.rnorm[(size_t)u * C + j];
    const int wave = tid / 64, lane = tid % 64;
    __shared__ int a_sh[CH];
    __shared__ int mem[CH];
    __shared__ int wtot[2];
    __shared__ double nsum_sh[2], dsum_sh[2];
    const int *assign = dv.assign + (size_t)u * dv.F;
    int *pos = dv.pos + (size_t)u * dv.F;
    double acc = 0.0;
    int count = 0;
    for (int c0 = 0; c0 < n_frames; c0 += CH) {
        const int cend = min(n_frames, c0 + CH);
#pragma unroll
        for (int i = 0; i < FPT; ++i) {
            const int f = c0 + tid + NT * i;
            a_sh[tid + NT * i] = f < cend ? assign[f] : -1;
        }
        __syncthreads();
        unsigned int mask = 0;               // bit i: frame c0 + 16 tid + i belongs to cluster j
#pragma unroll
        for (int i = 0; i < FPT; ++i) mask |= (a_sh[tid * FPT + i] == j ? 1u : 0u) << i;
        const int mine = __popc(mask);
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        int slot = incl - mine + (wave == 1 ? wtot[0] : 0);
        const int filled = wtot[0] + wtot[1];   // members found in this chunk (same in every thread)
        while (mask) {
            const int i = __ffs((int)mask) - 1;
            mask &= mask - 1;
            const int f = c0 + tid * FPT + i;
            mem[slot] = f;
            pos[f] = count + slot;
            ++slot;
        }
        __syncthreads();
        if (tid < D) {
            // sixteen members' loads in flight at a time (index clamped, loads unconditional), added in order
            // (thirty-two: slower, 75 against 68 us on average over a pass of config 2)
            constexpr int NL = 16;
            const double *sb = dv.summ + (size_t)u * dv.F * D + tid;
            for (int m0 = 0; m0 < filled; m0 += NL) {
                double v[NL];
#pragma unroll
                for (int x = 0; x < NL; ++x) v[x] = sb[(size_t)mem[min(m0 + x, filled - 1)] * D];
#pragma unroll
                for (int x = 0; x < NL; ++x)
                    if (m0 + x < filled) acc += v[x];
            }
        }
        count += filled;
    }
    if (count == 0) {                      // keeps its representative, skipped from now on
        if (tid == 0) { dv.n[(size_t)u * C + j] = 0; *delta = 0.0; *changed = 0; }
        return;
    }
    double sq = 0.0, rv = 0.0, r_old = 0.0;
    if (tid < D) {
        r_old = dv.r[((size_t)u * C + j) * D + tid];
        rv = acc / (double)count;
        dv.r[((size_t)u * C + j) * D + tid] = rv;
        sq = rv * rv;
    }
    sq = wave_sum(sq);
    if (lane == 0) nsum_sh[wave] = sq;
    __syncthreads();
    // how far the representative moved on the unit sphere (chord between the old and the new direction): what
    // k_lloyd_assign's bounds are moved by; 2, the largest chord there is, if either is the zero vector
    const double norm_new = sqrt(nsum_sh[0] + nsum_sh[1]);
    const bool both = norm_old > 0.0 && norm_new > 0.0;
    double dd = 0.0;
    if (tid < D && both) {
        const double t = r_old / norm_old - rv / norm_new;
        dd = t * t;
    }
    dd = wave_sum(dd);
    if (lane == 0) dsum_sh[wave] = dd;
    __syncthreads();
    if (tid == 0) {
        dv.rnorm[(size_t)u * C + j] = norm_new;
        dv.n[(size_t)u * C + j] = count;
        *delta = both ? sqrt(dsum_sh[0] + dsum_sh[1]) : 2.0;
        *changed = 0;
    }
}

// ---------------------------------------------------------------------------
// Assignments of frames f0 .. f0+n-1, compacted: a host-tier batch's straight into pinned memory, an observer's into
// scratch.  grid (U, blocks of frames).
__global__ __launch_bounds__(kBlock) void k_gather_assign(const DeviceView *self, int *rows, int f0, int n) {
    const DeviceView dv = device_view(self);
    const int u = blockIdx.x;
    for (int i = blockIdx.y * kBlock + threadIdx.x; i < n; i += gridDim.y * kBlock)
        rows[(size_t)u * n + i] = dv.assign[(size_t)u * dv.F + f0 + i];
}

// ---------------------------------------------------------------------------
// Host tier: store staged pages into their cluster's slab in pinned host memory
// (device stores over PCIe, 16 bytes per lane, whole pages contiguous).
// Sixteen workgroups share the (unit, frame, keys | values) items: the launch
// runs on the copy stream beside the next batch's staging and assignment, and
// one workgroup per page would hold the chip while it waits for the link.
// ---------------------------------------------------------------------------
constexpr int kOffloadXcds = 8;
__global__ __launch_bounds__(kBlock) void k_offload(const DeviceView *self, const int *dest, int f0, int n) {
    const DeviceView dv = device_view(self);
    // The page table is in pinned host memory: a workgroup fetches the entries of its next 256 items in one trip.
    // Only workgroups 0, 8, 16, ... work: workgroups go to the eight XCDs in turn, so these share one XCD, and its path to
    // the fabric is the only one that fills up with posted stores to the link.  Spread over all XCDs the same stores hold
    // up every other kernel's memory traffic (a page store beside it 217 us instead of 12).
    __shared__ int hp_sh[kBlock];
    if (blockIdx.x % kOffloadXcds) return;
    const int n_items = dv.U * n * 2, stride = gridDim.x / kOffloadXcds;
    for (int i0 = blockIdx.x / kOffloadXcds; i0 < n_items; i0 += kBlock * stride) {
        const long long mine = i0 + (long long)threadIdx.x * stride;
        if (mine < n_items) hp_sh[threadIdx.x] = dest[(size_t)(((int)mine >> 1) % dv.U) * dv.SN + ((int)mine >> 1) / dv.U];
        __syncthreads();
        for (int k = 0; k < kBlock && i0 + k * stride < n_items; ++k) {
            const int it = i0 + k * stride, val = it & 1, u = (it >> 1) % dv.U, f = f0 + (it >> 1) / dv.U;
            const size_t bytes = val ? dv.vpage : dv.kpage, hbytes = val ? dv.hvpage : dv.kpage;
            const size_t spage = (size_t)(f % dv.SN) * dv.U + u;
            const int hp = hp_sh[k];                           // page within the unit's host pool
            const size_t hoff = (size_t)u * dv.h_ustride + (size_t)(hp / dv.SFh) * dv.h_bstride + (size_t)(hp % dv.SFh) * hbytes;
            const uint4 *src = reinterpret_cast<const uint4 *>((val ? dv.stage_v : dv.stage_k) + spage * bytes);
            uint4 *dst = reinterpret_cast<uint4 *>((val ? dv.host_v : dv.host_k) + hoff);
            const int tail = val ? dv.htail : 0;
            const size_t n16 = (hbytes - (size_t)dv.D * tail * 8) / 16;
            for (size_t i = threadIdx.x; i < n16; i += kBlock) dst[i] = src[i];
            // (the last block: the first units of 8 bytes of each channel's 64, two units a store)
            const uint2 *s2 = reinterpret_cast<const uint2 *>(src + n16);
            for (int i = threadIdx.x; i < dv.D * tail / 2; i += kBlock) {
                const uint2 a = s2[2 * i / tail * 8 + 2 * i % tail], b = s2[(2 * i + 1) / tail * 8 + (2 * i + 1) % tail];
                dst[n16 + i] = make_uint4(a.x, a.y, b.x, b.y);
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Host tier: cluster fetch.  One launch moves every missing page of a layer's
// selection from the pinned slabs into the GPU cluster cache: the kernel loads
// straight from host memory over PCIe (16 bytes per lane), which streams at the
// rate of a large DMA copy and costs one launch instead of one runtime call per
// slab.  grid: a few dozen workgroups that share the (unit, page, keys | values) items.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_fetch(const DeviceView *self, int u0, int n_units, int max_moves) {
    const DeviceView dv = device_view(self);
    // items = (unit, move, keys | values), dealt round-robin to a SMALL fixed number of workgroups: the link
    // needs ~150 KB in flight, and workgroups parked on PCIe loads would otherwise hold the wave slots and
    // registers that the attention and selection kernels of the neighbouring layers are waiting for
    const int n_items = n_units * max_moves * 2;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int val = it & 1, i = (it >> 1) % max_moves, u = u0 + (it >> 1) / max_moves;
        if (i >= dv.n_moves[u]) continue;                                   // block-uniform
        const int hp = dv.moves[((size_t)u * dv.F + i) * 2], cp = dv.moves[((size_t)u * dv.F + i) * 2 + 1];
        const size_t bytes = val ? dv.vpage : dv.kpage, hbytes = val ? dv.hvpage : dv.kpage;
        const char *src = (val ? dv.host_v : dv.host_k) + (size_t)u * dv.h_ustride +
                          (size_t)(hp / dv.SFh) * dv.h_bstride + (size_t)(hp % dv.SFh) * hbytes;
        char *dst = (val ? dv.v_store + (size_t)u * dv.v_ustride : dv.k_store + (size_t)u * dv.k_ustride) + (size_t)cp * bytes;
        const uint4 *s4 = reinterpret_cast<const uint4 *>(src);
        uint4 *d4 = reinterpret_cast<uint4 *>(dst);
        const int tail = val ? dv.htail : 0;
        const size_t n16 = (hbytes - (size_t)dv.D * tail * 8) / 16;
        // the last block of a V page, 16 bytes of its rows of 64 per thread; in flight beside the rest
        constexpr int kTail = 128 * 4 / kBlock;
        uint2 t[kTail][2];
        if (tail) {
            const uint2 *s2 = reinterpret_cast<const uint2 *>(s4 + n16);
#pragma unroll
            for (int q = 0; q < 2 * kTail; ++q) {
                const int i = threadIdx.x + q / 2 * kBlock, ch = i / 4, unit = i % 4 * 2 + q % 2;
                t[q / 2][q % 2] = ch < dv.D && unit < tail ? s2[ch * tail + unit] : make_uint2(0, 0);
            }
        }
        for (size_t j = threadIdx.x; j < n16; j += 4 * kBlock) {           // four 16-byte loads in flight per thread
            uint4 x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = s4[min(j + (size_t)q * kBlock, n16 - 1)];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (j + (size_t)q * kBlock < n16) d4[j + (size_t)q * kBlock] = x[q];
        }
        if (tail) {
#pragma unroll
            for (int q = 0; q < kTail; ++q)
                if ((int)threadIdx.x + q * kBlock < dv.D * 4)
                    d4[n16 + threadIdx.x + q * kBlock] = make_uint4(t[q][0].x, t[q][0].y, t[q][1].x, t[q][1].y);
        }
    }
}

template <typename F> hipError_t checked(F &&launch) {
    launch();
    return hipGetLastError();
}

} // namespace

hipError_t launch_store_summary(const DeviceView &dv, const void *k_in, const void *v_in, int f0,
                                int n_frames, bool beyond, const float *e_in, int n_emb, hipStream_t s) {
    const dim3 grid(dv.U, n_frames, n_emb > 0 ? 3 : 2);
    auto go = [&](auto kern, auto *k) { kern<<<grid, kStoreBlock, 0, s>>>(dv.self, k, (decltype(k))v_in, f0, e_in, n_emb); };
    auto pick = [&](auto *k, auto d) {
        using E = std::remove_const_t<std::remove_pointer_t<decltype(k)>>;
        constexpr int D = decltype(d)::value;
        if (beyond) go(k_store_summary<E, D, true>, k);
        else go(k_store_summary<E, D, false>, k);
    };
    return checked([&] {
        auto by_d = [&](auto *k) {
            if (dv.D == 64) pick(k, std::integral_constant<int, 64>{});
            else pick(k, std::integral_constant<int, 128>{});
        };
        if (dv.esize == 4) by_d((const float *)k_in);
        else by_d((const unsigned short *)k_in);
    });
}

hipError_t launch_ingest_one(const DeviceView &dv, const void *k_in, const void *v_in, int f, hipStream_t s) {
    dim3 grid(dv.U, 2);
    return checked([&] {
        if (dv.esize == 4) {
            if (dv.D == 64) k_ingest_one<float, 64><<<grid, kOneBlock, 0, s>>>(dv.self, (const float *)k_in, (const float *)v_in, f);
            else k_ingest_one<float, 128><<<grid, kOneBlock, 0, s>>>(dv.self, (const float *)k_in, (const float *)v_in, f);
        } else {
            if (dv.D == 64) k_ingest_one<unsigned short, 64><<<grid, kOneBlock, 0, s>>>(dv.self, (const unsigned short *)k_in, (const unsigned short *)v_in, f);
            else k_ingest_one<unsigned short, 128><<<grid, kOneBlock, 0, s>>>(dv.self, (const unsigned short *)k_in, (const unsigned short *)v_in, f);
        }
    });
}

hipError_t launch_value_reps(const DeviceView &dv, int n_frames, hipStream_t s) {
    const dim3 grid(dv.U, dv.C);
    return checked([&] {
        if (dv.D == 64) k_value_reps<64><<<grid, 128, 0, s>>>(dv.self, n_frames);
        else k_value_reps<128><<<grid, 128, 0, s>>>(dv.self, n_frames);
    });
}

hipError_t launch_gather_assign(const DeviceView &dv, int *rows, int f0, int n, hipStream_t s) {
    const dim3 grid(dv.U, std::min((n + kBlock - 1) / kBlock, 1024));
    return checked([&] { k_gather_assign<<<grid, kBlock, 0, s>>>(dv.self, rows, f0, n); });
}

hipError_t launch_offload(const DeviceView &dv, const int *dest, int f0, int n, hipStream_t s) {
    // 16 working workgroups, all on one XCD (2 layers of 4 heads, 196-token pages, 16 frames a call, 512 frames, offloaded and
    // assigned: 10.9 ms with 16 workgroups spread over the XCDs, 9.3 with 16 on one, 10.4 with 16 on two; more
    // workgroups, or more loads in flight per thread, slow the staging and assignment kernels beside them).
    const long long items = (long long)dv.U * n * 2;
    const int blocks = (int)std::min<long long>(items, 16) * kOffloadXcds;
    return checked([&] { k_offload<<<blocks, kBlock, 0, s>>>(dv.self, dest, f0, n); });
}

hipError_t launch_fetch(const DeviceView &dv, int u0, int n_units, int max_moves, hipStream_t s) {
    if (max_moves <= 0) return hipSuccess;
    // 64 workgroups (measured on config 3: 16 / 32 / 64 / 96 / 128 / 256 / one per page and operand give a warm
    // decode step of 6.15 / 6.19 / 6.01 / 6.28 / 6.25 / 6.53 / 6.71 ms and 53.4 .. 55.2 GB/s over the link)
    const long long items = (long long)n_units * max_moves * 2;
    const int blocks = (int)std::min<long long>(items, 64);
    return checked([&] { k_fetch<<<blocks, kBlock, 0, s>>>(dv.self, u0, n_units, max_moves); });
}

hipError_t launch_assign_update(const DeviceView &dv, int f0, int f1, hipStream_t s) {
    return checked([&] {
        if (dv.maint_mode) {
            if (dv.D == 64) k_assign_update<64, true><<<dv.U, kBlock, 0, s>>>(dv.self, f0, f1);
            else k_assign_update<128, true><<<dv.U, kBlock, 0, s>>>(dv.self, f0, f1);
        } else if (f1 - f0 <= kRegFrames && dv.C <= 128) {
            if (dv.D == 64) k_assign_update_reg<64, 256><<<dv.U, 256, 0, s>>>(dv.self, f0, f1);
            else k_assign_update_reg<128, 256><<<dv.U, 256, 0, s>>>(dv.self, f0, f1);
        } else if (f1 - f0 <= kRegFrames && dv.C <= 256) {
            if (dv.D == 64) k_assign_update_reg<64, 512><<<dv.U, 512, 0, s>>>(dv.self, f0, f1);
            else k_assign_update_reg<128, 512><<<dv.U, 512, 0, s>>>(dv.self, f0, f1);
        } else if (f1 - f0 <= 2 && dv.C > 256) {
            if (dv.D == 64) k_assign_update<64, false><<<dv.U, kBlock, 0, s>>>(dv.self, f0, f1);
            else k_assign_update<128, false><<<dv.U, kBlock, 0, s>>>(dv.self, f0, f1);
        } else {
            if (dv.D == 64) k_assign_chain<64><<<dv.U, kChainBlock, 0, s>>>(dv.self, f0, f1);
            else k_assign_chain<128><<<dv.U, kChainBlock, 0, s>>>(dv.self, f0, f1);
        }
    });
}

hipError_t launch_lloyd(const DeviceView &dv, int n_frames, int iters, bool seed_from_warmup,
                        hipStream_t s) {
    hipError_t e = hipSuccess;
    if (seed_from_warmup) {
        e = checked([&] {
            if (dv.P > 0) {
                const dim3 gs(dv.U, (dv.C + 63) / 64);
                if (dv.D == 64) k_lloyd_seed_nested<64><<<gs, kBlock, 0, s>>>(dv.self, n_frames);
                else k_lloyd_seed_nested<128><<<gs, kBlock, 0, s>>>(dv.self, n_frames);
            } else {
                if (dv.D == 64) k_lloyd_seed<64><<<dv.U, kBlock, 0, s>>>(dv.self, n_frames);
                else k_lloyd_seed<128><<<dv.U, kBlock, 0, s>>>(dv.self, n_frames);
            }
        });
        if (e != hipSuccess) return e;
    }
    const dim3 gu(dv.U, dv.C);
    // the rounds' moved-frame counters and, behind them, the clusters' changed flags
    if ((e = hipMemsetAsync(dv.lloyd_moved, 0, ((size_t)dv.U * 3 + (size_t)dv.U * dv.C) * 4, s)) != hipSuccess) return e;
    for (int it = 0; it < iters; ++it) {
        e = checked([&] {
            const int per = it == 0 ? 64 : kLloydTest;
            const dim3 g(dv.U, (n_frames + per - 1) / per);
            auto go = [&](auto kern) { kern<<<g, kBlock, 0, s>>>(dv.self, n_frames, it); };
            auto pick = [&](auto d, auto later) {
                constexpr int D = decltype(d)::value;
                constexpr bool LATER = decltype(later)::value;
                if (dv.P > 0) go(k_lloyd_assign<D, LATER, true>);
                else go(k_lloyd_assign<D, LATER, false>);
            };
            auto by_d = [&](auto later) {
                if (dv.D == 64) pick(std::integral_constant<int, 64>{}, later);
                else pick(std::integral_constant<int, 128>{}, later);
            };
            if (it == 0) by_d(std::false_type{});
            else by_d(std::true_type{});
        });
        if (e != hipSuccess) return e;
        e = checked([&] {
            if (dv.D == 64) k_lloyd_update<64><<<gu, 128, 0, s>>>(dv.self, n_frames, it);
            else k_lloyd_update<128><<<gu, 128, 0, s>>>(dv.self, n_frames, it);
        });
        if (e != hipSuccess) return e;
    }
    if (dv.maint_mode) {
        const dim3 gv(dv.U, dv.c_init);
        e = checked([&] {
            if (dv.D == 64) k_exact_var<64><<<gv, kBlock, 0, s>>>(dv.self, n_frames);
            else k_exact_var<128><<<gv, kBlock, 0, s>>>(dv.self, n_frames);
        });
    }
    return e;
}

hipError_t launch_partition_reps(const DeviceView &dv, int n_frames, hipStream_t s) {
    const dim3 g(dv.U, dv.P);
    return checked([&] {
        if (dv.D == 64) k_partition_reps<64><<<g, 128, 0, s>>>(dv.self, n_frames);
        else k_partition_reps<128><<<g, 128, 0, s>>>(dv.self, n_frames);
    });
}

} // namespace mosaic
