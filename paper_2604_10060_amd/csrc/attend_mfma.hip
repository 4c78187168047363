// Attention over the retrieved KV on the matrix cores (bf16 pages); paper
// Sec. V-A (2).  The G*Tq query rows of a unit form the small dense operand, so
// both the logits (K Q^T) and the output (V^T P^T) are 16x16x32 bf16 MFMA
// contractions fed straight from global memory with 16-byte loads: no LDS
// staging and no register transposes.
//
// Value pages are stored chunk-blocked and transposed, [chunk][D][32 tokens], so
// that every operand load of a wavefront covers one contiguous KiB.
//
// Operand layout of v_mfma_f32_16x16x32_bf16 (lane = 16*g + n):
//   A (16 x 32): lane holds A[n][8g .. 8g+7]
//   B (32 x 16): lane holds B[8g .. 8g+7][n]
//   D (16 x 16): lane holds D[4g + i][n], i = 0..3
// Logits:  A = keys (row slot n of tile tau holds token t0 + 8*(n/4) + 4*tau + n%4),
//          B = Q^T; lane (g, n) then owns, for query row n, the logits of tokens
//          t0 + 8g + j, j = 0..7 -- exactly the B operand P^T[8g+j][n] of
// Output:  A = V^T (row slot n = channel 16*db + n, k-slots = tokens t0 + 8g + j),
//          D = O^T[16*db + 4g + i][n].

#include "mosaic_internal.h"
#include "attend_mfma_device.h"
#include "attend_reps_device.h"

namespace mosaic {

namespace {

// ---------------------------------------------------------------------------
// Decode shape: at most 16 query rows per unit (one row tile).
// grid (n_units * n_splits), 4 waves; split_slot() shares the workgroups out
// over the units by retrieved size.  Inside a unit chunks are dealt round-robin:
// wave w of split s takes chunks s + S*(w + 4*i); the next chunk's operands are
// in flight while the current one is reduced.
// ---------------------------------------------------------------------------
template <int D, bool AUG, bool STREAM>
__global__ __launch_bounds__(kBlock, 2) void k_attend_decode_mfma(const DeviceView *self, int u0, int n_units,
                                                                  const unsigned short *q, int Tq, int B) {
    const DeviceView dv = device_view(self);
    constexpr int KK = D / 32, DB = D / 16;
    if constexpr (AUG) {
        if ((int)blockIdx.x >= B) {   // extra workgroups: the global representatives' part (augmentation)
            __shared__ float lds[kF32MergeFloats<D>];
            attend_reps_partial<unsigned short, D>(dv, u0, (int)blockIdx.x - B, 0, q, Tq, lds);
            return;
        }
    }
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, g = lane / 16, n = lane % 16;
    const SplitSlot slot = split_slot<false>(dv.n_sel + u0, n_units, B, blockIdx.x);
    if (slot.uc < 0) return;                       // block-uniform: no barrier reached yet
    const int uc = slot.uc, u = u0 + uc, split = slot.split, S = slot.S;
    const int T = dv.T, F = dv.F, cpp = dv.chunks_per_page;
    const int lc = uc / dv.Hkv, h = u % dv.Hkv, R = Tq * dv.G;
    const int *sel = dv.sel_pages + (size_t)u * F;
    // wave-uniform chunk walk: wave w of split s takes chunks first + stride * i
    const int stride = __builtin_amdgcn_readfirstlane(4 * S);
    const int first = __builtin_amdgcn_readfirstlane(split + S * wave);

    bf16x8 qf[KK];
    load_q<D>(dv, q, lc, h, Tq, n, g, qf);

    const float sl2 = 1.4426950408889634f / sqrtf((float)D);

    f32x4 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f, lx = 0.f;

    const int NC = __builtin_amdgcn_readfirstlane(slot.n) * cpp;
    const int n_my = __builtin_amdgcn_readfirstlane(first < NC ? (NC - first + stride - 1) / stride : 0);

    // The page id of a chunk is read (a wave-uniform scalar load) one step before the
    // chunk's operand loads are issued, the cursor that walks the selection advances by
    // increments (no division in the loop), and inside the steady-state loop every load
    // is issued unconditionally, so the operand loads of chunk i+1 stay in flight across
    // the whole reduction of chunk i.
    bf16x8 kA[2 * KK], vA[DB], kB[2 * KK], vB[DB];
    int ccA = 0, ccB = 0;                             // chunk index inside its page
    const int sq = __builtin_amdgcn_readfirstlane(stride / cpp), sr = __builtin_amdgcn_readfirstlane(stride % cpp);
    int lq = __builtin_amdgcn_readfirstlane(first / cpp), lr = __builtin_amdgcn_readfirstlane(first % cpp), lj = 0;
    auto lookup = [&](int &page, int &cc) {           // page and in-page chunk of the cursor's chunk
        page = sel[lq]; cc = lr;
        if (lj + 1 < n_my) {                          // advance, stopping at the wave's last chunk
            ++lj; lq += sq; lr += sr;
            if (lr >= cpp) { lr -= cpp; ++lq; }
        }
    };
    auto issue = [&](int page, int cc_in, bf16x8 (&kf)[2 * KK], bf16x8 (&vf)[DB], int &cc) {
        cc = cc_in;
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
        int pg, cc, pg_n, cc_n;
        lookup(pg, cc);
        lookup(pg_n, cc_n);
        issue(pg, cc, kA, vA, ccA);
        int i = 0;
        for (; i + 2 < n_my; i += 2) {                // A holds chunk i; (pg_n, cc_n) is chunk i+1
            issue(pg_n, cc_n, kB, vB, ccB);
            lookup(pg_n, cc_n);
            __builtin_amdgcn_sched_barrier(0);        // keep the loads ahead of the arithmetic
            step(kA, vA, ccA);
            issue(pg_n, cc_n, kA, vA, ccA);
            lookup(pg_n, cc_n);
            __builtin_amdgcn_sched_barrier(0);
            step(kB, vB, ccB);
        }
        if (i + 2 == n_my) {
            issue(pg_n, cc_n, kB, vB, ccB);
            __builtin_amdgcn_sched_barrier(0);
            step(kA, vA, ccA);
            step(kB, vB, ccB);
        } else {
            step(kA, vA, ccA);
        }
    }
    // merge the four waves, write one partial per workgroup
    __shared__ float lds[kMergeFloats<D>];
    merge_waves_store<D>(dv, acc, m, l, lx, R, (size_t)slot.base + split, lds);   // one row tile
}

} // namespace

hipError_t launch_attend_mfma(const DeviceView &dv, int u0, int n_units, const void *q, int Tq,
                              int n_splits, Shares shares, bool stream_kv, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const int NT = (Tq * dv.G + kRowTile - 1) / kRowTile;
    const unsigned short *qq = (const unsigned short *)q;
    const dim3 block(kBlock);
    if (NT == 1) {
        const int B = n_units * n_splits;
        const dim3 grid(B + (dv.aug_reps ? n_units : 0));
        auto go = [&](auto kern) { launch_timed(kern, grid, block, 0, s, ev0, ev1, dv.self, u0, n_units, qq, Tq, B); };
        if (dv.aug_reps) {
            if (dv.D == 64) stream_kv ? go(k_attend_decode_mfma<64, true, true>) : go(k_attend_decode_mfma<64, true, false>);
            else stream_kv ? go(k_attend_decode_mfma<128, true, true>) : go(k_attend_decode_mfma<128, true, false>);
        } else {
            if (dv.D == 64) stream_kv ? go(k_attend_decode_mfma<64, false, true>) : go(k_attend_decode_mfma<64, false, false>);
            else stream_kv ? go(k_attend_decode_mfma<128, false, true>) : go(k_attend_decode_mfma<128, false, false>);
        }
    } else {
        return launch_attend_prefill(dv, u0, n_units, qq, Tq, shares, s, ev0, ev1);
    }
    return hipGetLastError();
}

} // namespace mosaic
