// Retrieval augmentation, global representatives (paper Sec. V-C), device side: the
// attention partial of one row tile over a unit's clusters as pseudo tokens.  The
// attention kernels run it in extra workgroups of their own launch (the part depends on
// the query and the clustering only), so it costs no kernel boundary of its own.
#pragma once
#include "mosaic_internal.h"
#include "attend_fp32_device.h"

namespace mosaic {

// Attention of one row tile over the unit's non-empty clusters as pseudo tokens (key = representative,
// value = mean of the members' values; fp32 tables rep_k / rep_v [C][D], built whenever the clustering
// changed), written as one more partial (running maximum in the log2 domain, sum, unnormalised output)
// that the combine kernel merges with the split partials.  One workgroup of 256 threads per (row tile,
// unit); lds: kF32MergeFloats<D> floats.
// The tables are a short run of fp32 tokens (C <= 1024), so this is the fp32 attention step: wavefront w takes
// clusters 16 (w + 4 i) .. + 15, the next group's rows and sizes in flight.  The launch lasts as long as its slowest
// workgroup, and a decode step's attention workgroups are done in about 10 us: as a chain of query, logits, statistics
// and value passes through LDS on the vector ALU this part took 23 us, in this form it is over before they are
// (C = 64, D = 128, four units: decode step of four layers 144 -> 86 us; other cards and streams 153 -> 93, 168 -> 112).
template <typename E, int D>
__device__ void attend_reps_partial(const DeviceView &dv, int u0, int uc, int tile, const E *q, int Tq, float *lds) {
    const int u = u0 + uc, tid = threadIdx.x, wave = tid / 64, lane = tid % 64, g = lane / 16, n = lane % 16;
    const int C = dv.C, lc = uc / dv.Hkv, h = u % dv.Hkv;
    const float *rk = dv.rep_k + (size_t)u * C * D, *rv = dv.rep_v + (size_t)u * C * D;
    const int *size = dv.n + (size_t)u * C;
    const int groups = (C + kGroup - 1) / kGroup;
    const float sl2 = 1.4426950408889634f / sqrtf((float)D);
    f32v4 acc[1][D / 16], qf[1][D / 16];
    float m[1] = {-INFINITY}, l[1] = {0.f};
#pragma unroll
    for (int b = 0; b < D / 16; ++b) acc[0][b] = f32v4{0.f, 0.f, 0.f, 0.f};
    F32Operands<D> oa, ob;
    int na = 0, nb = 0;             // size of the cluster whose key row this lane loads, 0 beyond the table
    auto issue = [&](int grp, F32Operands<D> &o, int &nn) {
        const int c = grp * kGroup + n;
        nn = size[min(c, C - 1)];
        if (c >= C) nn = 0;
        f32_issue<D, false>(rk, rv, min(c, C - 1), g, n, o);
    };
    auto step = [&](F32Operands<D> &o, int nn) {
#pragma unroll
        for (int v = 0; v < 4; ++v) o.row[v] = __shfl(nn, 4 * g + v, 64) > 0 ? 0 : -1;      // empty clusters are no tokens
        f32_step<D, 1>(o, qf, acc, m, l);
    };
    if (wave < groups) issue(wave, oa, na);
    f32_load_q<E, D>(dv, q, lc, h, Tq, tile * kRowTile + n, g, sl2, qf[0]);
    for (int grp = wave; grp < groups; grp += 8) {
        if (grp + 4 < groups) issue(grp + 4, ob, nb);
        step(oa, na);
        if (grp + 8 < groups) issue(grp + 8, oa, na);
        if (grp + 4 < groups) step(ob, nb);
    }
    float o[D / 16], M, L;
    f32_merge_waves<D>(acc[0], m[0], l[0], lds, o, M, L);
    const size_t entry = (size_t)u * dv.nt_max + tile;
    const int row = tid / 16, dl = tid % 16;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) dv.aug_o[(entry * kRowTile + row) * D + dl + 16 * i] = o[i];
    if (dl == 0) {
        dv.aug_ml[entry * 2 * kRowTile + row] = M;
        dv.aug_ml[entry * 2 * kRowTile + kRowTile + row] = L;
    }
}

} // namespace mosaic
