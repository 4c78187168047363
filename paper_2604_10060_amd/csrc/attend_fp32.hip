// Attention over the retrieved KV with fp32 pages (paper Sec. V-A (2)) on the fp32 matrix
// instruction: exact fp32 products, fp32 accumulation (operand layout in attend_fp32_device.h).
// Against the vector-ALU kernel it replaces (a row of K and V at a time through LDS, scalar LDS reads in the inner
// loops, nothing prefetched): a decode step's launch at D = 128, 33 k tokens in four units 61 -> 14 us, at D = 64,
// 512 tokens 25.7 -> 8.8 us, an 84-row question at D = 64 61 -> 14 us; 1792-row question 100 TFLOP/s.  Its error
// against 64 bits, averaged over a few streams, is 0.09 to 0.74 of that kernel's (decode steps and questions of 17 shapes;
// D = 128, 33 k tokens 2.0e-7 -> 1.2e-7 of the output's norm); on a single stream either can be the larger.
//
// What bounds it.  A decode step (one row tile) reads 2 * D * 4 bytes per token and spends 4 * D / 16 matrix
// instructions of 32 cycles on 16 tokens, about 40 % of the time the bytes take at the HBM rate: memory, and on the
// small launches of one layer the latency of two or three dependent loads.  A question of many tokens is bound by
// the fp32 matrix rate (153 TFLOP/s measured for a large product), so R row tiles share a wavefront's operands.
#include "attend_fp32_device.h"
#include "attend_reps_device.h"

namespace mosaic {

namespace {

// grid B [+ n_units with the global-representative augmentation] for one row tile (R = 1), else the (group, row block) pairs in
// xcd_run() order [+ n_units * row blocks], 4 wavefronts.  A unit's tokens are one flat sequence in gather order (token
// i = token i % T of page i / T of the selection), taken 16 at a time whatever T is, so that only the very last group of
// 16 is padded.  One row tile: split_slot() shares the workgroups out over the units by retrieved size, wavefront w of
// split s takes 16s number s + S * w + 4 * S * i.  Questions: a workgroup takes a contiguous run of 16s, an equal share of all
// units' or the part of one that lies in one unit (even_share), its wavefronts every fourth.
// The page ids of group i + 2 and the operands of group i + 1 are in flight while group i is reduced.
template <int D, int R, bool STREAM>
__global__ __launch_bounds__(kBlock, R == 1 || D == 64 ? 2 : 1) void k_attend_fp32(const DeviceView *self, int u0, int n_units, const float *q,
                                                                        int Tq, int NT, int G, int B, int n_row_blocks) {
    const DeviceView dv = device_view<0, 1, 2, 8>(self);
    __shared__ float lds[kF32MergeFloats<D>];
    const int first_extra = R == 1 ? B : (B * n_row_blocks + 7) / 8 * 8;
    if ((int)blockIdx.x >= first_extra) {      // extra workgroups: the global representatives' part (augmentation)
        const int idx = (int)blockIdx.x - first_extra, rb = idx % n_row_blocks;
        for (int r = 0; r < R; ++r) {
            const int tile = rb * R + r;
            if (tile < NT) attend_reps_partial<float, D>(dv, u0, idx / n_row_blocks, tile, q, Tq, lds);
        }
        return;
    }
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, g = lane / 16, n = lane % 16, T = dv.T;
    int grp = (int)blockIdx.x, yb = 0;
    if constexpr (R > 1) {
        const int pair = xcd_run((int)blockIdx.x, B * n_row_blocks);
        if (pair < 0) return;       // block-uniform: no barrier reached yet
        grp = pair / n_row_blocks; yb = pair % n_row_blocks;
    }
    const ChunkSize<true> cs(dv);
    ShareWalk<true> w;
    if constexpr (R == 1) {
        const SplitSlot slot = split_slot<false>(dv.n_sel + u0, n_units, B, grp);
        if (slot.uc < 0) return;                                                       // block-uniform as well
        w.uc = __builtin_amdgcn_readfirstlane(slot.uc); w.n = __builtin_amdgcn_readfirstlane(slot.n);
        w.base = __builtin_amdgcn_readfirstlane(slot.base); w.S = __builtin_amdgcn_readfirstlane(slot.S);
        w.split = __builtin_amdgcn_readfirstlane(slot.split);
    } else {
        if (!w.start(dv.n_sel + u0, n_units, cs, G, grp, B == G)) return;              // (B > G: slots)
    }
  do {
    int n_ = n, g_ = g, t_ = tid;   // (opaque copies: what only a unit's first loads and last stores need of the lane is worked out there)
    asm volatile("" : "+v"(n_), "+v"(g_), "+v"(t_));
    const int uc = w.uc, u = u0 + uc, S = w.S;
    const int lc = uc / dv.Hkv, h = u % dv.Hkv;
    const int *sel = dv.sel_pages + (size_t)u * dv.F;
    const float *kb = reinterpret_cast<const float *>(k_page(dv, u, 0)), *vb = reinterpret_cast<const float *>(v_page(dv, u, 0));
    const int n_sel = w.n;
    const int first = __builtin_amdgcn_readfirstlane(R == 1 ? w.split + S * wave : w.c0 + wave);
    const int stride = R == 1 ? 4 * S : 4;
    const int groups = R == 1 ? cs.of(n_sel) : w.c1;       // (where this workgroup's end)
    const int n_my = __builtin_amdgcn_readfirstlane(first < groups ? (groups - first + stride - 1) / stride : 0);

    // wave-uniform cursor over the groups: page (index into the selection) and token offset of a group's first token
    const int dq = __builtin_amdgcn_readfirstlane(stride * kGroup / T), dr = __builtin_amdgcn_readfirstlane(stride * kGroup % T);
    int cp = __builtin_amdgcn_readfirstlane(first * kGroup / T), cr = __builtin_amdgcn_readfirstlane(first * kGroup % T);
    const int inv = 65536 / T + 1;  // floor(x / T) = (x * inv) >> 16 for x < T + 16 <= 32
    int id = 0, at = 0;             // this lane's token (token n of the cursor's group): page id, ~offset if there is none
    auto lookup = [&]() {           // (past the last group: the last page again)
        int off = cr + n;
        const int d = T >= kGroup ? (off >= T ? 1 : 0) : (off * inv) >> 16;
        off -= d * T;
        const bool some = cp + d < n_sel;
        id = sel[min(cp + d, n_sel - 1)];
        at = some ? off : ~0;
        cp += dq;
        cr += dr;
        if (cr >= T) { cr -= T; ++cp; }
        cp = min(cp, n_sel);
    };
    // the cursor's group; then the cursor moves on -- its page id is loaded ahead of the operands, so that waiting for it is not
    // waiting for them (behind them: decode step of four layers over 69 MB each 133 -> 140 us)
    auto issue = [&](F32Operands<D> &o, bool more = true) {
        const int row = at < 0 ? ~(id * T) : id * T + at;
        if (more) lookup();
        f32_issue<D, STREAM>(kb, vb, row, g, n, o);
    };

    const float sl2 = 1.4426950408889634f / sqrtf((float)D);
    f32v4 qf[R][D / 16], acc[R][D / 16];
    float m[R], l[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        f32_load_q<float, D>(dv, q, lc, h, Tq, (yb * R + r) * kRowTile + n_, g_, sl2, qf[r]);
        m[r] = -INFINITY;
        l[r] = 0.f;
#pragma unroll
        for (int b = 0; b < D / 16; ++b) acc[r][b] = f32v4{0.f, 0.f, 0.f, 0.f};
    }
    // Questions: a share of a long one is hundreds of groups, and one fp32 sum over all of them errs with the root of their
    // number (in equal shares, 182 tokens over 1200 frames 2.3e-5 of the output's norm, 30 over 752 8.9e-7).  So the sums of
    // kSumGroups groups are added to a second level in LDS: 1.7e-6 and 1.3e-7 (with a split count per unit, two to six times as
    // many, 8.4e-6 and 1.4e-7).  Four groups, not eight: 176 tokens over 378 frames 9.4e-8 against 2.4e-7 (8.9e-8 with a split
    // count per unit), for 4 % of a long question's time (60 tokens, 246 k retrieved: 580 -> 605 us, as long as with a split count).
    constexpr int kSumGroups = 4;
    __shared__ f32v4 sum_sh[R == 1 ? 1 : 4 * R * (D / 16) * 64];
    float msum[R], lsum[R];
    bool summed = false;            // wave-uniform
#pragma unroll
    for (int r = 0; r < R; ++r) { msum[r] = -INFINITY; lsum[r] = 0.f; }
    auto sum_up = [&](bool last) {  // what acc and l hold joins the second level; last: and comes back
        if constexpr (R > 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float a = msum[r] > -INFINITY ? __builtin_amdgcn_exp2f(msum[r] - m[r]) : 0.f;      // (m is no lower)
                lsum[r] = lsum[r] * a + l[r];
                msum[r] = m[r];
                l[r] = last ? lsum[r] : 0.f;
#pragma unroll
                for (int b = 0; b < D / 16; ++b) {
                    f32v4 *const at_sum = &sum_sh[((wave * R + r) * (D / 16) + b) * 64 + lane];
                    f32v4 x = acc[r][b];
                    if (summed) x = *at_sum * a + x;
                    if (!last) *at_sum = x;
                    acc[r][b] = last ? x : f32v4{0.f, 0.f, 0.f, 0.f};
                }
            }
            summed = true;
        }
    };
    F32Operands<D> oa, ob;
    if (n_my > 0) {                 // then n_sel > 0
        lookup();
        issue(oa);
        int i = 0;
        for (; i + 2 < n_my; i += 2) {
            if (R > 1 && i % kSumGroups == 0 && i > 0) sum_up(false);
            issue(ob);
            __builtin_amdgcn_sched_barrier(0);
            f32_step<D, R>(oa, qf, acc, m, l);
            issue(oa);
            __builtin_amdgcn_sched_barrier(0);
            f32_step<D, R>(ob, qf, acc, m, l);
        }
        if (i + 2 == n_my) {
            issue(ob, false);
            __builtin_amdgcn_sched_barrier(0);
            f32_step<D, R>(oa, qf, acc, m, l);
            f32_step<D, R>(ob, qf, acc, m, l);
        } else {
            f32_step<D, R>(oa, qf, acc, m, l);
        }
    }
    if (summed) sum_up(true);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int tile = yb * R + r;
        if (tile >= NT) break;      // block-uniform
        float o[D / 16], M, L;
        f32_merge_waves<D>(acc[r], m[r], l[r], lds, o, M, L);
        const int rw = t_ / 16, dl = t_ % 16;
        const size_t entry = (size_t)w.base * NT + (size_t)tile * S + w.split;
        float *po = dv.part_o + (entry * kRowTile + rw) * D;
#pragma unroll
        for (int i = 0; i < D / 16; ++i) po[dl + 16 * i] = o[i];
        if (dl == 0) {              // fp32 weights throughout: the two normalisers coincide
            float *ml = dv.part_ml + entry * kMlRows * kRowTile;
            ml[rw] = M;
            ml[kRowTile + rw] = L;
            ml[2 * kRowTile + rw] = L;
        }
    }
  } while (R > 1 && w.next(dv.n_sel + u0, cs));
}

} // namespace

hipError_t launch_attend_fp32(const DeviceView &dv, int u0, int n_units, const float *q, int Tq, int n_splits,
                              Shares shares, bool stream_kv, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const int NT = (Tq * dv.G + kRowTile - 1) / kRowTile, R = NT == 1 ? 1 : kFp32Tiles, rb = (NT + R - 1) / R;
    const int B = NT == 1 ? n_units * n_splits : shares.walk ? shares.groups : shares.groups + n_units - 1;
    const dim3 grid((NT == 1 ? B : (B * rb + 7) / 8 * 8) + (dv.aug_reps ? n_units * rb : 0)), block(kBlock);
    auto go = [&](auto kern) { launch_timed(kern, grid, block, 0, s, ev0, ev1, dv.self, u0, n_units, q, Tq, NT, shares.groups, B, rb); };
    if (NT == 1) {
        if (dv.D == 64) stream_kv ? go(k_attend_fp32<64, 1, true>) : go(k_attend_fp32<64, 1, false>);
        else stream_kv ? go(k_attend_fp32<128, 1, true>) : go(k_attend_fp32<128, 1, false>);
    } else {                        // several row blocks read a unit's pages: they find them in the caches
        if (dv.D == 64) go(k_attend_fp32<64, kFp32Tiles, false>);
        else go(k_attend_fp32<128, kFp32Tiles, false>);
    }
    return hipGetLastError();
}

} // namespace mosaic
