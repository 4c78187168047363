// A latency-bound decode step in one launch: selection (paper Sec. V-C) and attention over the retrieved pages (Sec. V-A (2)).
#include <type_traits>

#include "attend_mfma_device.h"
#include "attend_reps_device.h"

namespace mosaic {

namespace {

__device__ __forceinline__ double to_f64(float v) { return (double)v; }
__device__ __forceinline__ double to_f64(unsigned short v) { return (double)bf16_to_f32(v); }

// ---------------------------------------------------------------------------
// Fused decode step (one row tile, per-layer call): selection and attention in one
// launch.  grid (n_units * S [+ n_units with the global-representative augmentation]),
// kFusedBlock threads; workgroup = (unit, split), S uniform.
// Every workgroup of a unit first repeats the unit's selection for itself -- mean
// query, scores of the C <= 256 representatives, ranks of the k best, page offsets --
// which costs it the table's C x D x 8 bytes through L2 (the longest part of its life: the query is
// back after ~2 k cycles, the table after 6-7 k) and ~4 k cycles of arithmetic, but
// removes the separate selection launch and the two dependent round trips (sizes,
// page ids) at the start of the attention kernel; it then lists the pages of its own
// contiguous chunk range in LDS and reduces them like k_attend_decode_mfma (bf16) or
// k_attend_fp32 (fp32 pages: chunks of 16 tokens across pages).  Split 0
// of each unit also writes the selection (scores, ids, page list, counts) to memory,
// so the observers and a later mosaic_attend see what mosaic_retrieve would have left.
// Same arithmetic, lane for lane, as k_retrieve (scores, ranking) and as the decode
// kernels (chunk steps), hence the same ids, token lists and -- up to the order in
// which partials are merged -- outputs.
// Against the two calls, us a layer (eight layers in turn; 64 tokens a frame, C = 64, k = 8, D = 128, 4 KV heads), at 4 / 10 / 16 /
// 24 / 36 MiB of K/V: bf16 14.6, 15.6, 18.4, 21.2, 28.1 against 17.0, 18.0, 20.3, 22.9, 28.0; fp32 16.6, 23.0, 23.5, 23.6, 29.7 against
// 20.5, 24.3, 25.1, 24.6, 31.7; with window and representatives 15.2, 16.6, 19.3, 22.4, 29.6 against 18.9, 19.6, 22.1, 24.5, 29.6.
// ---------------------------------------------------------------------------
constexpr int kFusedMaxC = 256, kFusedList = 2048;
// Threads of a workgroup, one workgroup per CU.  Eight wavefronts halve the selection's and the pages' trips (bf16, 1 to 36 MiB a
// layer: 0.4 to 0.9 us less than four; fp32 at D = 64 1 us less).  Four where a wavefront's accumulators are large and there
// are more of them to merge (fp32 at D = 128: 16 to 38 us a layer with four, 1 to 2 us more with eight), and with the
// representatives, whose workgroups have to find a place beside the others (a window alone takes the same instantiation).
template <typename E, int D, bool AUG> constexpr int kFusedBlock = AUG || (sizeof(E) == 4 && D == 128) ? 256 : 512;

__device__ __forceinline__ double group16_sum_f64(double x) { return row16_sum(x); }   // as in k_retrieve

template <typename E, int D, bool AUG, bool STREAM>
__global__ __launch_bounds__((kFusedBlock<E, D, AUG>), AUG ? 2 : 1) void k_decode_fused(const DeviceView *self, int u0, int n_units, const E *q, int Tq,
                                                         int S, int n_frames, int score_mode) {
    const DeviceView dv = device_view<0, 1, 2, 3>(self);
    constexpr bool FP32 = sizeof(E) == 4;
    constexpr int BLK = kFusedBlock<E, D, AUG>, NW = BLK / 64;
    constexpr int KK = D / 32, DB = D / 16, EPL = D / 16, NG = BLK / 16, RPF = 128 / NG, FPT = 2048 / BLK;
    static_assert(BLK >= kFusedMaxC && BLK >= D, "a thread per table entry and per channel");
    static_assert(128 % NG == 0 && 1024 % BLK == 0, "whole passes of prefetched rows, frames and window frames");
    __shared__ float lds[FP32 || (AUG && kF32MergeFloats<D> > kMergeFloats<D, kFusedBlock<E, D, AUG> / 64>)
                             ? kF32MergeFloats<D, kFusedBlock<E, D, AUG> / 64> : kMergeFloats<D, kFusedBlock<E, D, AUG> / 64>];
    if constexpr (AUG) {
        if ((int)blockIdx.x >= n_units * S) {      // extra workgroups: the global representatives' part (augmentation)
            attend_reps_partial<E, D>(dv, u0, (int)blockIdx.x - n_units * S, 0, q, Tq, lds);
            return;
        }
    }
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, g = lane / 16, n = lane % 16;
    const int lr = tid % 16, grp = tid / 16;
    const int uc = (int)blockIdx.x / S, split = (int)blockIdx.x % S, u = u0 + uc;
    const int C = dv.C, k = dv.k, G = dv.G, Hq = dv.Hq, T = dv.T, F = dv.F, cpp = dv.chunks_per_page;
    const int lc = uc / dv.Hkv, h = u % dv.Hkv, R = Tq * G;
    __shared__ double qbar[D];
    __shared__ double sc_sh[kFusedMaxC], rn_sh[kFusedMaxC];
    __shared__ int n_sh[kFusedMaxC], rank_sh[kFusedMaxC], cnt_sh[kFusedMaxC], ids_sh[kFusedMaxC], off_sh[kFusedMaxC + 1], wcnt_sh[AUG ? kFusedMaxC : 1];
    __shared__ int list_sh[kFusedList];
    __shared__ int n_live_sh;
    const double *r = dv.r + (size_t)u * C * D;
    const int *assign = dv.assign + (size_t)u * F;
    const int *pos = dv.pos + (size_t)u * F;

    // ---- independent loads, all issued up front ----
    const float sl2 = 1.4426950408889634f / sqrtf((float)D);
    bf16x8 qf[KK];
    f32v4 qf32[1][D / 16];
    if constexpr (FP32) f32_load_q<float, D>(dv, q, lc, h, Tq, n, g, sl2, qf32[0]);
    else load_q<D>(dv, q, lc, h, Tq, n, g, qf);
    int fa[FPT], fp[FPT];
#pragma unroll
    for (int i = 0; i < FPT; ++i) {
        const int f = tid + BLK * i;
        fa[i] = f < n_frames ? assign[f] : -1;
        fp[i] = f < n_frames ? pos[f] : 0;
    }
    for (int j = tid; j < C; j += BLK) {
        n_sh[j] = dv.n[(size_t)u * C + j];
        rn_sh[j] = dv.rnorm[(size_t)u * C + j];
        cnt_sh[j] = 0;
        if constexpr (AUG) wcnt_sh[j] = 0;
    }
    // the local window (augmentation): its frames are listed once, after the clusters; they are the last members of
    // their clusters (ranks ascend with the frame id), so a cluster's list is cut short by its number of window members
    const int w0 = AUG && dv.aug_window > 0 ? max(0, n_frames - dv.aug_window) : n_frames;
    constexpr int WPT = 1024 / BLK;               // aug_window <= 1024 (checked at create)
    int wa[WPT];
    if constexpr (AUG) {
#pragma unroll
        for (int i = 0; i < WPT; ++i) wa[i] = w0 + tid + BLK * i < n_frames ? assign[w0 + tid + BLK * i] : -1;
    }
    if (tid == 0) n_live_sh = 0;
    double rpre[RPF][EPL];
#pragma unroll
    for (int i = 0; i < RPF; ++i) {
        if (NG * i < C) {               // workgroup-uniform: passes beyond the table are not loaded
            const double *rj = r + (size_t)min(grp + NG * i, C - 1) * D + lr * EPL;
#pragma unroll
            for (int e = 0; e < EPL; ++e) rpre[i][e] = rj[e];
        }
    }
    if (tid < D) {      // mean query over the Tq tokens and the G query heads of this KV head
        // (R <= 16: two batches of eight loads, row index clamped, loads unconditional)
        const E *qb = q + (size_t)lc * Tq * Hq * D + (size_t)h * G * D + tid;
        double a = 0.0;
        for (int r0 = 0; r0 < R; r0 += 8) {
            E v[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const int rr = min(r0 + x, R - 1), t = rr / G, gg = rr - t * G;
                v[x] = qb[((size_t)t * Hq + gg) * D];
            }
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (r0 + x < R) a += to_f64(v[x]);
        }
        qbar[tid] = a / (double)R;
    }
    __syncthreads();
    if constexpr (AUG) {         // (read after the scores' barriers)
#pragma unroll
        for (int i = 0; i < WPT; ++i)
            if (wa[i] >= 0) atomicAdd(&wcnt_sh[wa[i]], 1);
    }
    // ---- scores: score_j = (qbar . r_j) / |r_j|   (plain dot product in score_mode 1) ----
    // the 16-lane groups leave the raw dot products in LDS; thread j then finishes entry j
    // (one fp64 division per thread instead of one per row on a single lane)
    // (no lane-dependent branch around a row: the rows' reduction chains interleave; a row
    // beyond the table repeats the last one and is not stored)
#pragma unroll
    for (int i = 0; i < RPF; ++i) {
        const int j = grp + NG * i;
        if (NG * i < C) {                                     // workgroup-uniform
            double p = 0.0;
#pragma unroll
            for (int e = 0; e < EPL; ++e) p += qbar[lr * EPL + e] * rpre[i][e];
            p = group16_sum_f64(p);
            if (lr == 0 && j < C) sc_sh[j] = p;
        }
    }
    for (int j = grp + NG * RPF; j < C; j += NG) {
        const double *rj = r + (size_t)j * D + lr * EPL;
        double p = 0.0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) p += qbar[lr * EPL + e] * rj[e];
        p = group16_sum_f64(p);
        if (lr == 0) sc_sh[j] = p;
    }
    __syncthreads();
    float *key_sh = reinterpret_cast<float *>(off_sh);     // (the page offsets are formed after the ranking)
    if (tid < C) {
        double sc = -INFINITY;
        if (n_sh[tid] > 0) {
            const double p = sc_sh[tid], nr = rn_sh[tid];
            sc = score_mode == 1 ? p : (nr == 0.0 ? 0.0 : p / nr);
        }
        if (split == 0) dv.scores[(size_t)u * dv.SC + tid] = sc;
        if (n_sh[tid] > 0) sc = rank_score(sc);
        sc_sh[tid] = sc;
        key_sh[tid] = (float)sc;          // fp32 rounding for the pair count below
    }
    __syncthreads();
    // ---- ranks by (score descending, id ascending) among the non-empty clusters ----
    {   // 2^pl threads per entry (the largest power of two that fits the workgroup: shifts, no divisions);
        // pairs compared on the fp32 roundings (monotone, so a strict fp32 order is the fp64 order; fp64
        // compares run at a quarter of the rate), collisions settled exactly below
        const int pl = 31 - __clz(BLK / C);
        const int j = tid >> pl, part = tid & ((1 << pl) - 1);
        if (j < C && n_sh[j] > 0) {
            const float fj = key_sh[j];
            const int i0 = (C * part) >> pl, i1 = (C * (part + 1)) >> pl;
            int c = 0, ceq = 0;  // (an empty cluster carries -inf and neither outranks nor equals a live one)
#pragma unroll 8
            for (int i = i0; i < i1; ++i) {
                const float fi = key_sh[i];
                c += fi > fj;
                ceq += fi == fj;
            }
            atomicAdd(&cnt_sh[j], c + (ceq << 16));     // c <= 256, ceq <= 256
        }
    }
    __syncthreads();
    {   // C <= kFusedMaxC <= BLK: thread j owns entry j; live entries counted with one atomic per wavefront
        const bool live = tid < C && n_sh[tid] > 0;
        int rk = -1;
        if (live) {
            const int v = cnt_sh[tid];
            rk = v & 0xffff;
            if ((v >> 16) > 1) {                        // collisions (the entry itself counts once): exact order among them
                const float fj = key_sh[tid];
                const double sj = sc_sh[tid];
                for (int i = 0; i < C; ++i) {
                    if (i == tid || key_sh[i] != fj) continue;
                    const double si = sc_sh[i];
                    rk += (si > sj) || (si == sj && i < tid);
                }
            }
            if (rk < k) ids_sh[rk] = tid; else rk = -1;
        }
        if (tid < C) rank_sh[tid] = rk;
        const unsigned long long lb = __ballot(live);
        if (lane == 0 && lb) atomicAdd(&n_live_sh, __popcll(lb));
    }
    __syncthreads();
    const int n_ids = min(k, n_live_sh);
    if (wave == 0) {     // page offsets of the selected clusters: running sums of their sizes, 64 at a time
        int run = 0;
        for (int i0 = 0; i0 < n_ids; i0 += 64) {
            const int i = i0 + lane;
            int sz = i < n_ids ? n_sh[ids_sh[i]] : 0;
            if constexpr (AUG) { if (i < n_ids) sz -= wcnt_sh[ids_sh[i]]; }
            int incl = sz;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(incl, o, 64);
                if (lane >= o) incl += t;
            }
            if (i < n_ids) off_sh[i + 1] = run + incl;
            run += __shfl(incl, 63, 64);
        }
        if (lane == 0) {
            off_sh[0] = 0;
            if (split == 0) { dv.n_ids[u] = n_ids; dv.n_sel[u] = run + (n_frames - w0); }
        }
    }
    if (split == 0)
        for (int i = tid; i < k; i += BLK) dv.ids[(size_t)u * k + i] = i < n_ids ? ids_sh[i] : -1;
    __syncthreads();
    // ---- this workgroup's chunk range and its pages ----
    const int n_sel = off_sh[n_ids] + (n_frames - w0);
    const int NC = FP32 ? (n_sel * T + kGroup - 1) / kGroup : n_sel * cpp;
    const int cps = (NC + S - 1) / S;
    const int c0 = split * cps, c1 = min(NC, c0 + cps);
    const int p_lo = FP32 ? c0 * kGroup / T : c0 / cpp;
    const int p_hi = c1 > c0 ? (FP32 ? (min(n_sel * T, c1 * kGroup) - 1) / T : (c1 - 1) / cpp) : p_lo - 1;
    int *sel = dv.sel_pages + (size_t)u * F;
    auto place = [&](int f, int a, int ps) {   // (no early exits: the LDS look-ups of a batch overlap)
        const int rk = rank_sh[max(a, 0)];
        const bool sel_f = a >= 0 && (rk >= 0 || f >= w0);
        const int p = f >= w0 ? off_sh[n_ids] + (f - w0) : off_sh[max(rk, 0)] + ps;
        if (sel_f && p >= p_lo && p <= p_hi) list_sh[p - p_lo] = f;
        if (sel_f && split == 0) sel[p] = f;
    };
#pragma unroll
    for (int i = 0; i < FPT; ++i) place(tid + BLK * i, fa[i], fp[i]);
    for (int f0 = tid + BLK * FPT; f0 < n_frames; f0 += BLK * FPT) {      // further batches of FPT loads
#pragma unroll
        for (int i = 0; i < FPT; ++i) {
            const int f = f0 + BLK * i;
            fa[i] = f < n_frames ? assign[f] : -1;
            fp[i] = f < n_frames ? pos[f] : 0;
        }
#pragma unroll
        for (int i = 0; i < FPT; ++i) place(f0 + BLK * i, fa[i], fp[i]);
    }
    __syncthreads();

    // ---- attention over chunks c0 + wave, + NW, ... of the range ----
    const int first = c0 + wave;
    const int n_my = first < c1 ? (c1 - first + NW - 1) / NW : 0;
    if constexpr (FP32) {
        const float *kb = reinterpret_cast<const float *>(k_page(dv, u, 0)), *vb = reinterpret_cast<const float *>(v_page(dv, u, 0));
        // cursor over the wave's chunks: page (index into the selection) and token offset of a chunk's first token
        const int dq = NW * kGroup / T, dr = NW * kGroup - dq * T;
        int cp = first * kGroup / T, cr = first * kGroup - cp * T;
        const int inv = 65536 / T + 1;      // floor(x / T) = (x * inv) >> 16 for x < T + 16 <= 32
        auto issue = [&](F32Operands<D> &o) {      // the cursor's chunk (token n is this lane's; past the last one: another, of no weight)
            int off = cr + n;
            const int d = T >= kGroup ? (off >= T ? 1 : 0) : (off * inv) >> 16;
            off -= d * T;
            const int id = list_sh[min(cp + d, p_hi) - p_lo];
            f32_issue<D, STREAM>(kb, vb, cp + d < n_sel ? id * T + off : ~(id * T), g, n, o);
            cp += dq;
            cr += dr;
            if (cr >= T) { cr -= T; ++cp; }
            cp = min(cp, n_sel);
        };
        f32v4 acc[1][D / 16];
        float m[1] = {-INFINITY}, l[1] = {0.f};
#pragma unroll
        for (int b = 0; b < D / 16; ++b) acc[0][b] = f32v4{0.f, 0.f, 0.f, 0.f};
        F32Operands<D> oa, ob;
        if (n_my > 0) {
            issue(oa);
            int i = 0;
            for (; i + 2 < n_my; i += 2) {
                issue(ob);
                __builtin_amdgcn_sched_barrier(0);
                f32_step<D, 1>(oa, qf32, acc, m, l);
                issue(oa);
                __builtin_amdgcn_sched_barrier(0);
                f32_step<D, 1>(ob, qf32, acc, m, l);
            }
            if (i + 2 == n_my) {
                issue(ob);
                __builtin_amdgcn_sched_barrier(0);
                f32_step<D, 1>(oa, qf32, acc, m, l);
                f32_step<D, 1>(ob, qf32, acc, m, l);
            } else {
                f32_step<D, 1>(oa, qf32, acc, m, l);
            }
        }
        float o[D / 16], M, L;
        f32_merge_waves<D, NW>(acc[0], m[0], l[0], lds, o, M, L);
        const size_t entry = (size_t)uc * S + split;
        const int rw = tid / 16, dl = tid % 16;
        if (rw >= kRowTile) return;
        float *po = dv.part_o + (entry * kRowTile + rw) * D;
#pragma unroll
        for (int i = 0; i < D / 16; ++i) po[dl + 16 * i] = o[i];
        if (dl == 0) {                      // fp32 weights throughout: the two normalisers coincide
            float *ml = dv.part_ml + entry * kMlRows * kRowTile;
            ml[rw] = M;
            ml[kRowTile + rw] = L;
            ml[2 * kRowTile + rw] = L;
        }
    } else {
        f32x4 acc[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m = -INFINITY, l = 0.f, lx = 0.f;
        bf16x8 kA[2 * KK], vA[DB], kB[2 * KK], vB[DB];
        int ccA = 0, ccB = 0;
        auto issue = [&](int c, bf16x8 (&kf)[2 * KK], bf16x8 (&vf)[DB], int &cc) {
            const int pi = c / cpp;
            cc = c - pi * cpp;
            const int page = list_sh[pi - p_lo];
            const char *kp = k_page(dv, u, page);
            const char *vp = v_page(dv, u, page);
            issue_chunk<D, STREAM>(dv, reinterpret_cast<const unsigned short *>(kp),
                                   reinterpret_cast<const unsigned short *>(vp) + (size_t)cc * D * 32,
                                   cc * kChunk, g, n, kf, vf);
        };
        auto step = [&](const bf16x8 (&kf)[2 * KK], const bf16x8 (&vf)[DB], int cc) {
            chunk_step<D>(kf, vf, qf, min(kChunk, T - cc * kChunk), g, sl2, acc, m, l, lx);
        };
        if (n_my > 0) {
            issue(first, kA, vA, ccA);
            int i = 0;
            for (; i + 2 < n_my; i += 2) {
                issue(first + NW * (i + 1), kB, vB, ccB);
                __builtin_amdgcn_sched_barrier(0);
                step(kA, vA, ccA);
                issue(first + NW * (i + 2), kA, vA, ccA);
                __builtin_amdgcn_sched_barrier(0);
                step(kB, vB, ccB);
            }
            if (i + 2 == n_my) {
                issue(first + NW * (i + 1), kB, vB, ccB);
                __builtin_amdgcn_sched_barrier(0);
                step(kA, vA, ccA);
                step(kB, vB, ccB);
            } else {
                step(kA, vA, ccA);
            }
        }
        merge_waves_store<D, NW>(dv, acc, m, l, lx, R, (size_t)uc * S + split, lds);
    }
}

} // namespace

hipError_t launch_decode_fused(const DeviceView &dv, int u0, int n_units, const void *q, int Tq, int n_splits,
                               int n_frames, int score_mode, bool stream_kv, hipStream_t s, hipEvent_t ev0,
                               hipEvent_t ev1) {
    const bool aug = dv.aug_reps || dv.aug_window > 0;
    const dim3 grid(n_units * n_splits + (dv.aug_reps ? n_units : 0));
    auto go = [&](auto kern, int blk, auto *qq) { launch_timed(kern, grid, dim3(blk), 0, s, ev0, ev1, dv.self, u0, n_units, qq, Tq, n_splits, n_frames, score_mode); };
    auto pick = [&](auto *qq, auto d) {
        using E = std::remove_const_t<std::remove_pointer_t<decltype(qq)>>;
        constexpr int D = decltype(d)::value, A = kFusedBlock<E, D, true>, P = kFusedBlock<E, D, false>;
        if (aug) stream_kv ? go(k_decode_fused<E, D, true, true>, A, qq) : go(k_decode_fused<E, D, true, false>, A, qq);
        else stream_kv ? go(k_decode_fused<E, D, false, true>, P, qq) : go(k_decode_fused<E, D, false, false>, P, qq);
    };
    auto by_d = [&](auto *qq) {
        if (dv.D == 64) pick(qq, std::integral_constant<int, 64>{});
        else pick(qq, std::integral_constant<int, 128>{});
    };
    if (dv.esize == 4) by_d((const float *)q); else by_d((const unsigned short *)q);
    return hipGetLastError();
}

} // namespace mosaic
