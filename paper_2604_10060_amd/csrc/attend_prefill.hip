// Multi-token questions (paper Sec. V-A (2): attention of a question chunk over the retrieved
// KV), MFMA-bound.  A workgroup of four wavefronts owns 4 * 16 * kPrefillTiles query rows: wave w
// holds kPrefillTiles row tiles of 16 in registers and all waves walk the same chunk range, so
// each 32-token K/V chunk is fetched from memory once per workgroup, placed in LDS and read as
// MFMA operands by every wave.  Two workgroups per CU.
//
// Global -> LDS without registers: every lane's 16-byte load is written by the memory pipeline
// straight into LDS (lane l of a wavefront's load lands at base + 16 l), so the copy holds no
// staging registers, issues no LDS stores and computes no store addresses; which 16 bytes a lane
// fetches is free, so the layout below is produced by choosing the SOURCE address per lane.
// LDS holds four key slots and four value slots of one chunk each (chunk c lives in slot c % 4).  Wavefronts
// 0 and 1 fetch the even and the odd chunks' keys, 2 and 3 their values, so that each keeps one cursor instead of two and
// moves it once per two chunks (scalar instructions per chunk and wavefront 67 -> 40).
//
// LDS layout (per 32-token chunk: 32 x D keys / D x 32 values, both unpadded):
//   keys    row slot s = 16 tau + 4 j + i holds token 8 j + 4 tau + i  (MFMA slot order: lane
//           (g, n) of key tile tau then owns the logits of tokens 8 g .. 8 g + 7, the k-slots of
//           the value contraction), 16-byte pieces of a row XOR-swizzled with the row number;
//   values  [channel][32 tokens] as in memory, pieces XOR-swizzled with channel / 4.
//   A 16-lane group's operand read (16 rows, one piece each) then covers all 64 banks once.
//
// What bounds it (D = 128, 256-token questions).  A wavefront issues 34 MFMAs per chunk (544 cycles of the matrix pipe),
// 63 vector instructions (16 of them exp2, twice as long) and 16 LDS reads; two vector instructions per MFMA hide behind it, more do
// not, so what counts is that they alternate and that nothing else is issued.  A wavefront's step therefore works on three chunks at once
// -- logits of chunk j + 1, softmax of chunk j, outputs of chunk j - 1 -- whose instructions do not depend on each other, cut into
// phases of two MFMAs, one LDS read and three or four vector instructions that the compiler may not reorder across.
// (With only the order of the statements to go by it moved one tile's softmax behind the next branch: 8 MFMAs with no vector
// instruction between them, then 26 with both tiles' softmax.)  A value operand is read into the registers of the key
// operand that the phase has used up, and the other way round, which is what lets the three chunks fit 256 registers.
// The reference of a row's weights is checked after the fact: the sum of a lane's weights, needed for the log-sum-exp
// anyway, tells whether any of them has grown too large; rarely it has, and the chunk's weights are formed over again
// with a new reference before anything has used them.  That is one compare per chunk instead of eight maxima.
// Launch of a 256-token question, 246 k retrieved tokens: 271 -> 217 us; 32 tokens on 28 layers: 501 -> 420 us.  The matrix pipe is
// busy 57 % of the cycles (43 before) and the chip lowers its clock with it (1.95 -> 1.86 GHz): 1.11 PFLOP/s
// of matrix instructions, the rate at which a large matrix product of the library runs on this card.  Repeated without a pause
// the clock falls further and the calls gain less (197 -> 177, 658 -> 600 us).
// Slower: the weights' row sums by a two-element dot product on the vector ALU instead of a 17th MFMA per tile (217 -> 247 us);
// four row tiles per wavefront, one wavefront per SIMD (556 us: accumulators in the other half of the
// register file, and nothing to fill a wavefront's waits).
//
// A group is an equal share of all units' retrieved chunks, or the part of one that lies in one unit (even_share); its
// n_row_blocks workgroups read the same K/V range, and xcd_run() says which id is which.
#include <mutex>
#include <type_traits>

#include "mosaic_internal.h"
#include "attend_mfma_device.h"
#include "attend_reps_device.h"

namespace mosaic {

namespace {

typedef __attribute__((address_space(1))) const void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

// maximum of three floats in one instruction (no NaNs reach it: logits are finite or -inf)
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

constexpr int kPrefillSlots = 4;   // LDS slots of one chunk per operand

template <int D, bool AUG>
__global__ __launch_bounds__(64 * kPrefillWaves, 2) void k_attend_prefill_mfma(const DeviceView *self, int u0, int n_units,
                                                                                    const unsigned short *q, int Tq,
                                                                                    int NT, int G, int n_groups, int n_row_blocks,
                                                                                    int group_blocks) {
    const DeviceView dv = device_view(self);
    constexpr int NW = kPrefillWaves;
    static_assert(!AUG || 64 * NW == kBlock, "the representatives' workgroups are written for kBlock threads");
    constexpr int KK = D / 32, DB = D / 16, RTW = kPrefillTiles;
    constexpr int KSEG = D / 8;                  // 16-byte pieces per key row
    constexpr int KRP = 16 / KSEG;               // key rows per 256 bytes (1 at D = 128, 2 at D = 64)
    constexpr int KBYTES = kChunk * D * 2, VBYTES = D * kChunk * 2;
    static_assert(NW == 4, "a wavefront for the even and one for the odd chunks of each operand");
    constexpr int NS = kPrefillSlots;
    constexpr int NL = KBYTES / 1024;            // wavefront-sized loads per chunk and operand
    static_assert(KBYTES == VBYTES, "the same loads for either operand");
    // LDS (dynamic): NS key slots, then NS value slots, one chunk each
    extern __shared__ __attribute__((aligned(1024))) unsigned char prefill_lds[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, n = lane % 16;
    if constexpr (AUG) {
        static_assert(kF32MergeFloats<D> * 4 <= NS * (KBYTES + VBYTES), "the representatives' merge fits the chunk slots");
        if ((int)blockIdx.x >= group_blocks) {   // extra workgroups: the global representatives' part (augmentation)
            const int idx = (int)blockIdx.x - group_blocks;
            attend_reps_partial<unsigned short, D>(dv, u0, idx / NT, idx % NT, q, Tq, reinterpret_cast<float *>(prefill_lds));
            return;
        }
    }
    const int pair = xcd_run((int)blockIdx.x, n_groups * n_row_blocks);
    if (pair < 0) return;                          // block-uniform: no barrier reached yet
    const int grp = pair / n_row_blocks, yb = pair % n_row_blocks;
    const int T = dv.T, F = dv.F, cpp = dv.chunks_per_page;
    const int tile0 = (yb * NW + wave) * RTW;
    const bool idle = tile0 >= NT;                 // wave-uniform: no rows for this wave; it only fetches
    const float sl2 = 1.4426950408889634f / sqrtf((float)D);

    // What this lane fetches of a chunk of its wavefront's operand, in bytes from the chunk's first: LDS pieces
    // 64 i + lane for load i.  Wavefronts 0 and 1 fetch keys, 2 and 3 values.
    const bool is_k = wave < 2;
    const int k_rs2 = dv.k_rs() * 2;
    unsigned ld_off[NL];
    auto k_tok = [](int P) {                       // token of the chunk whose piece goes to LDS piece P
        const int row = P / KSEG, rem = row % 16;
        return 8 * (rem / 4) + 4 * (row / 16) + rem % 4;
    };
    const int lane_tok = k_tok(lane);              // (k_tok(64 i + lane) = k_tok(64 i) + k_tok(lane))
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        if (is_k) {
            const int P = i * 64 + lane, row = P / KSEG, seg = P % KSEG ^ ((row / KRP) % KSEG);
            ld_off[i] = (unsigned)((k_tok(64 * i) + lane_tok) * k_rs2 + seg / 4 * (int)(dv.k_ps() * 2) + seg % 4 * 16);
        } else {
            const int P = i * 64 + lane, row = P / 4;
            ld_off[i] = row * (kChunk * 2) + (P % 4 ^ ((row / 4) % 4)) * 16;
        }
    }
    // ... and where it reads its operands: key rows 16 tau + n, pieces 4 kk + g; value rows 16 db + n, piece g
    int kr_off[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kr_off[kk] = n * (D * 2) + (((4 * kk + g) ^ ((n / KRP) % KSEG)) * 16);
    const int vr_off = n * (kChunk * 2) + ((g ^ ((n / 4) % 4)) * 16);

    // The group's chunks, unit by unit.
    const ChunkSize<false> cs(dv);
    ShareWalk<false> w;
    if (!w.start(dv.n_sel + u0, n_units, cs, G, grp, n_groups == G)) return;      // (n_groups > G: they are slots)
  do {
    // (opaque copies: what a unit's first loads and last stores derive from the lane is worked out there, and not kept in
    // registers across the loop over the chunks)
    int n_ = n, g_ = g;
    asm volatile("" : "+v"(n_), "+v"(g_));
    const int uc = w.uc, c0 = w.c0, c1 = w.c1;
    const int u = u0 + uc, lc = uc / dv.Hkv, h = u % dv.Hkv;
    bf16x8 qf[RTW][KK];
#pragma unroll
    for (int r = 0; r < RTW; ++r) load_q<D>(dv, q, lc, h, Tq, (tile0 + r) * kRowTile + n_, g_, qf[r]);
    // (a page id is read by a vector load: while a scalar load is on its way, no count of LDS reads still under way can be waited for,
    // only all of them)
    const int *const sel = dv.sel_pages + (size_t)u * F;
    int zero = 0;
    asm volatile("" : "+v"(zero));

    f32x4 acc[RTW][DB], l[RTW];                    // l: row sums, kept by an all-ones MFMA
    float nm[RTW], lx[RTW];                        // nm: minus the row's reference
#pragma unroll
    for (int r = 0; r < RTW; ++r) {
        nm[r] = INFINITY; l[r] = f32x4{0.f, 0.f, 0.f, 0.f}; lx[r] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[r][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // This wavefront's next chunk to fetch (f_idx of the unit's range): chunk f_cc of its f_pi-th page, f_page.  Page ids are read one fetch
    // ahead.  Past the end a cursor stays on the last chunk: such loads re-read valid memory and land in slots nobody reads.
    const int n_chunks = c1 - c0;
    const char *const base = is_k ? dv.k_store + (size_t)u * dv.k_ustride : dv.v_store + (size_t)u * dv.v_ustride;
    const size_t psize = is_k ? dv.kpage : dv.vpage;
    const int cbytes = is_k ? kChunk * k_rs2 : VBYTES;          // from a page's chunk to its next
    unsigned char *const slots = prefill_lds + (is_k ? 0 : NS * KBYTES);
    int f_idx = wave & 1, f_pi, f_cc, f_page;
    {
        const int c = c0 + min(f_idx, n_chunks - 1);
        f_pi = c / cpp; f_cc = c - f_pi * cpp; f_page = sel[f_pi + zero];
    }
    auto fetch = [&]() __attribute__((always_inline)) {
        const char *const p = base + (size_t)__builtin_amdgcn_readfirstlane(f_page) * psize + (size_t)f_cc * (unsigned)cbytes;
        unsigned char *const dst = slots + (f_idx & (NS - 1)) * KBYTES;
        const int last = T - 1 - f_cc * kChunk;      // the page's last token
        if (is_k && last < kChunk - 1) {             // a page's ragged last chunk: the last token again for those that are not there
            int over = lane_tok - last;
            asm volatile("" : "+v"(over));
#pragma unroll
            for (int i = 0; i < NL; ++i)
                __builtin_amdgcn_global_load_lds((gptr_t)(p + (ld_off[i] - (unsigned)(max(over + k_tok(64 * i), 0) * k_rs2))), (lptr_t)(dst + i * 1024), 16, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                unsigned off = ld_off[i];
                asm volatile("" : "+v"(off));       // (the offset stays 32 bits wide, beside a scalar base)
                __builtin_amdgcn_global_load_lds((gptr_t)(p + off), (lptr_t)(dst + i * 1024), 16, 0, 0);
            }
        }
        f_cc += min(f_idx + 2, n_chunks - 1) - min(f_idx, n_chunks - 1);
        f_idx += 2;
        if (f_cc >= cpp) { f_cc -= cpp; ++f_pi; }
        if (f_cc >= cpp) { f_cc -= cpp; ++f_pi; }
        f_page = sel[f_pi + zero];
    };
    auto publish = [&]() {
        __builtin_amdgcn_s_waitcnt(0x3f70);     // every load of this wavefront, and nothing else
        lds_barrier();
    };

    // ---- the pipeline -------------------------------------------------------------------------
    f32x4 S[RTW][2], S2[RTW][2];                     // logits of the chunk whose softmax is next, and of the one after it (in turn)
    bf16x8 kf[2 * KK], pf[RTW];                      // keys of the chunk whose logits are next; weights of the chunk before
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
    int c_cc = c0 - (c0 / cpp) * cpp;                // chunk inside its page, of the chunk whose softmax is next
    auto ldk = [&](int s, int i) {                   // (i = tau * KK + kk)
        const unsigned char *const kb = prefill_lds + s * KBYTES + i / KK * 16 * D * 2;
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(kb + kr_off[i % KK]));
    };
    auto ldv = [&](int s, int db) {
        const unsigned char *const vb = prefill_lds + NS * KBYTES + s * VBYTES + db * 16 * kChunk * 2;
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(vb + vr_off));
    };
    auto logits = [&](int i, f32x4 (&s)[RTW][2]) {
#pragma unroll
        for (int r = 0; r < RTW; ++r)
            s[r][i / KK] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i], qf[r][i % KK], i % KK == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[r][i / KK], 0, 0, 0);
    };
    auto output = [&](bf16x8 vf, int db) {
#pragma unroll
        for (int r = 0; r < RTW; ++r) acc[r][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[r], acc[r][db], 0, 0, 0);
    };
    auto output_sum = [&]() {
#pragma unroll
        for (int r = 0; r < RTW; ++r) l[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[r], l[r], 0, 0, 0);
    };
    struct Weights { float e[8]; unsigned int w[4]; float x; };
    // half-step i of a row tile's softmax: two weights, then their sum and their bf16 pair
    auto softmax_half = [&](int i, int r, const f32x4 (&s)[RTW][2], Weights &o) __attribute__((always_inline)) {
        const int j = i / 2 * 2;
        if (i % 2 == 0) {
#pragma unroll
            for (int x = j; x < j + 2; ++x) o.e[x] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r][x / 4][x % 4], sl2, nm[r]));
        } else {
            o.w[j / 2] = pack_bf16(o.e[j], o.e[j + 1]);
            o.x = j == 0 ? o.e[j] + o.e[j + 1] : o.x + (o.e[j] + o.e[j + 1]);
        }
    };
    auto raise = [&](int r, const f32x4 (&s)[RTW][2]) __attribute__((always_inline)) {
        float cm = max3(s[r][0][0], s[r][0][1], s[r][0][2]);
        cm = max3(cm, s[r][0][3], s[r][1][0]);
        cm = max3(cm, s[r][1][1], s[r][1][2]);
        cm = max3(cm, s[r][1][3], s[r][1][3]) * sl2;
        cm = fmaxf(cm, __shfl_xor(cm, 16, 64));
        cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
        const float mnew = fmaxf(-nm[r], cm);
        const float alpha = __builtin_amdgcn_exp2f(-nm[r] - mnew);
        l[r] = l[r] * alpha;
        lx[r] = lx[r] * alpha;
        nm[r] = -mnew;
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[r][db] = acc[r][db] * alpha;
    };
    auto mask = [&](int n_valid, f32x4 (&s)[RTW][2]) __attribute__((always_inline)) {
        if (n_valid < kChunk) {             // ragged last chunk of a page (wave-uniform)
            int valid = n_valid - 8 * g;    // of this lane's eight tokens
            asm volatile("" : "+v"(valid));
#pragma unroll
            for (int r = 0; r < RTW; ++r)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j >= valid) s[r][j / 4][j % 4] = -INFINITY;
        }
    };
    auto fresh = [&](int r, const f32x4 (&s)[RTW][2], Weights &o) __attribute__((always_inline)) {
        raise(r, s);
#pragma unroll
        for (int i = 0; i < 8; ++i) softmax_half(i, r, s, o);
    };
    auto take = [&](int r, const Weights &o) {
        pf[r] = __builtin_bit_cast(bf16x8, make_uint4(o.w[0], o.w[1], o.w[2], o.w[3]));
        lx[r] += o.x;
    };
    // A step: outputs of chunk j - 1 (values in slot sv), softmax of chunk j (logits S, n_valid of its tokens exist), logits Sn of
    // chunk j + 1 (keys in kf), keys of chunk j + 2 from slot sk.  The compiler may move vector and scalar instructions across a phase's MFMAs,
    // its LDS read only after them (the wait before an MFMA is for every LDS read issued so far).
    // A chunk whose weights add up to more than kRaise in some lane is done over with the row's reference raised; weights stay below it, far from
    // what fp32 sums and bf16 hold.
    constexpr float kRaise = 4096.f;
    auto step = [&](int sv, int sk, int n_valid, f32x4 (&S)[RTW][2], f32x4 (&Sn)[RTW][2]) __attribute__((always_inline)) {
        bf16x8 vf[DB];
        Weights o[RTW];
        mask(n_valid, S);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int HALVES = 8 * RTW, PER = (HALVES + 2 * KK + DB - 1) / (2 * KK + DB);
        auto vector_part = [&](int ph) {
#pragma unroll
            for (int x = 0; x < PER; ++x) {
                const int i = ph * PER + x;
                if (i < HALVES) softmax_half(i % 8, i / 8, S, o[i / 8]);
            }
        };
#pragma unroll
        for (int i = 0; i < 2 * KK; ++i) {
            logits(i, Sn);
            __builtin_amdgcn_sched_barrier(0x406);
            if (i < DB - 1) vf[i] = ldv(sv, i);
            if (i == DB - 2) vf[i + 1] = ldv(sv, i + 1);
            vector_part(i);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < DB; ++i) {
            output(vf[i], i);
            __builtin_amdgcn_sched_barrier(0x406);
            if (i < DB - 1) kf[i] = ldk(sk, i);
            if (i == DB - 2) kf[i + 1] = ldk(sk, i + 1);
            vector_part(2 * KK + i);
            __builtin_amdgcn_sched_barrier(0);
        }
        output_sum();
        float tot = o[0].x;
#pragma unroll
        for (int r = 1; r < RTW; ++r) tot += o[r].x;
        if (__builtin_amdgcn_ballot_w64(!(tot <= kRaise))) {       // rare, wave-uniform
#pragma unroll
            for (int r = 0; r < RTW; ++r)
                if (__builtin_amdgcn_ballot_w64(!(o[r].x <= kRaise / RTW))) fresh(r, S, o[r]);
        }
#pragma unroll
        for (int r = 0; r < RTW; ++r) take(r, o[r]);
    };
    auto next_valid = [&]() {                         // tokens of the chunk; advances the in-page cursor
        const int nv = min(kChunk, T - c_cc * kChunk);
        c_cc = c_cc + 1 == cpp ? 0 : c_cc + 1;
        return nv;
    };

    {
        fetch();
        if (is_k) fetch();
        publish();                                    // K0 .. K3, V0, V1 are in LDS
        if (!idle) {
#pragma unroll
            for (int i = 0; i < 2 * KK; ++i) kf[i] = ldk(0, i);
        }
        lds_barrier();
        if (wave == 0) fetch();                       // K4 takes K0's place
        if (!idle) {
#pragma unroll
            for (int i = 0; i < 2 * KK; ++i) logits(i, S2);
#pragma unroll
            for (int i = 0; i < 2 * KK; ++i) kf[i] = ldk(1, i);
            mask(next_valid(), S2);
            Weights o[RTW];
#pragma unroll
            for (int r = 0; r < RTW; ++r) { fresh(r, S2, o[r]); take(r, o[r]); }
#pragma unroll
            for (int i = 0; i < 2 * KK; ++i) logits(i, S);
#pragma unroll
            for (int i = 0; i < 2 * KK; ++i) kf[i] = ldk(2, i);
        }
        publish();
        int j = 1;
        // Two steps per barrier interval: read are V(j - 1), V(j), K(j + 2), K(j + 3), fetched are K(j + 4), K(j + 5), V(j + 1), V(j + 2), in
        // slots last read one interval ago.
        auto interval = [&](auto odd) __attribute__((always_inline)) {               // steps j and j + 1
            constexpr int s = decltype(odd)::value ? 2 : 0;
            fetch();
            if (!idle) {
                step(s, (s + 3) % NS, next_valid(), S, S2);
                if (j + 1 < n_chunks) step(s + 1, s, next_valid(), S2, S);
            }
            publish();
            j += 2;
        };
        while (j < n_chunks) {
            interval(std::false_type{});
            if (j >= n_chunks) break;
            interval(std::true_type{});
        }
        if (!idle) {
#pragma unroll
            for (int i = 0; i < DB; ++i) output(ldv((n_chunks - 1) & 3, i), i);
            output_sum();
        }
        lds_barrier();                                // (the next unit's first chunks go to slots read here)
    }
#pragma unroll
    for (int r = 0; r < RTW; ++r) {
        const int tile = tile0 + r;
        if (tile >= NT) break;
        const float lr = l[r][0];
        float xr = lx[r];                              // this lane's 8 tokens per chunk: add the four lane groups
        xr += __shfl_xor(xr, 16, 64);
        xr += __shfl_xor(xr, 32, 64);
        const size_t entry = (size_t)w.base * NT + (size_t)tile * w.S + w.split;
        float *po = dv.part_o + (entry * kRowTile + n_) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
            *reinterpret_cast<float4 *>(po + 16 * db + 4 * g_) =
                make_float4(acc[r][db][0], acc[r][db][1], acc[r][db][2], acc[r][db][3]);
        if (g_ == 0) {
            dv.part_ml[entry * kMlRows * kRowTile + n_] = -nm[r];
            dv.part_ml[entry * kMlRows * kRowTile + kRowTile + n_] = lr;
            dv.part_ml[entry * kMlRows * kRowTile + 2 * kRowTile + n_] = xr;
        }
    }
  } while (w.next(dv.n_sel + u0, cs));
}

} // namespace

hipError_t launch_attend_prefill(const DeviceView &dv, int u0, int n_units, const unsigned short *q, int Tq,
                                 Shares shares, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int NW = kPrefillWaves;
    const int NT = (Tq * dv.G + kRowTile - 1) / kRowTile;
    // dynamic LDS: key slots and value slots of one chunk (32 x D bf16) each
    const size_t lds = (size_t)2 * kPrefillSlots * (kChunk * dv.D * 2);
    static std::once_flag attr_once;          // process-wide, but set exactly once whichever handle comes first
    std::call_once(attr_once, [] {
        const int big = 2 * kPrefillSlots * kChunk * 128 * 2;
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attend_prefill_mfma<64, true>), hipFuncAttributeMaxDynamicSharedMemorySize, big);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attend_prefill_mfma<64, false>), hipFuncAttributeMaxDynamicSharedMemorySize, big);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attend_prefill_mfma<128, true>), hipFuncAttributeMaxDynamicSharedMemorySize, big);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attend_prefill_mfma<128, false>), hipFuncAttributeMaxDynamicSharedMemorySize, big);
    });
    const int n_groups = shares.walk ? shares.groups : shares.groups + n_units - 1, rb = (NT + NW * kPrefillTiles - 1) / (NW * kPrefillTiles);
    const int gb = (n_groups * rb + 7) / 8 * 8;
    const dim3 grid(gb + (dv.aug_reps ? n_units * NT : 0)), block(64 * NW);
    auto go = [&](auto kern) { launch_timed(kern, grid, block, lds, s, ev0, ev1, dv.self, u0, n_units, q, Tq, NT, shares.groups, n_groups, rb, gb); };
    if (dv.aug_reps) { if (dv.D == 64) go(k_attend_prefill_mfma<64, true>); else go(k_attend_prefill_mfma<128, true>); }
    else { if (dv.D == 64) go(k_attend_prefill_mfma<64, false>); else go(k_attend_prefill_mfma<128, false>); }
    return hipGetLastError();
}

} // namespace mosaic
