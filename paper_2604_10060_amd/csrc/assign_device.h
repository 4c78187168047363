// Device helpers of the online assignment (semantic and visual level): ordered member lists, Eq. 3 with a shared
// correctly rounded reciprocal, and the decision of a chunk of up to 16 frames from carried-over dot products.
#pragma once
#include "mosaic_internal.h"

namespace mosaic {

// fp64 max / min as single instructions (the builtins add an instruction per operand that quiets signalling NaNs);
// only used on values that are never NaN
__device__ __forceinline__ double max_f64(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double min_f64(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Best (value, id) of a wavefront when the ids ascend with the lane (at most one candidate per lane, -inf and
// 0x7fffffff in lanes without one; no NaN): the largest value by a max butterfly (three instructions per step
// against a dozen for the (value, id) pair), then the first lane that holds it, which is the lowest id.  Left in
// every lane.
__device__ __forceinline__ void wave_best_ascending(double &bv, int &bi) {
    double m = bv;
    m = max_f64(m, dpp_f64<kDppXor8>(m));
    m = max_f64(m, dpp_f64<kDppXor7>(m));
    m = max_f64(m, dpp_f64<kDppXor3>(m));
    m = max_f64(m, dpp_f64<kDppXor1>(m));
    const long long b = __double_as_longlong(m);
    const int lo = (int)b, hi = (int)(b >> 32);
    double wm = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int l = __builtin_amdgcn_readlane(lo, 16 * r), h = __builtin_amdgcn_readlane(hi, 16 * r);
        wm = fmax(wm, __longlong_as_double(((long long)h << 32) | (long long)(unsigned int)l));
    }
    const unsigned long long at = __ballot(bv == wm);
    const int first = __ffsll((long long)at) - 1;                       // some lane holds the maximum
    const int id = __builtin_amdgcn_readlane(bi, first);
    bv = wm;
    bi = wm == -INFINITY ? 0x7fffffff : id;
}

// LDS written by one lane and read by others of the same wavefront: the wavefront runs in lockstep and LDS is in order,
// so only the compiler has to be kept from moving the accesses across.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sums whose last bit decides between clusters that tie to the last bit.  Several kernels share the state they go into
// (which one runs depends on the frames per call), so every multiply-add is written out: left to the compiler, the order
// of the first two squares and which of them is rounded by itself differed from kernel to kernel.
//
// Products of a lane's channels, in their order
template <int N>
__device__ __forceinline__ double dot_channels(const double (&a)[N], const double (&b)[N]) {
    double p = 0.0;
#pragma unroll
    for (int e = 0; e < N; ++e) p = __builtin_fma(a[e], b[e], p);
    return p;
}
// Squares of a lane's channels: step e of the sum, channels in their order but for the first two, whose order is a choice
template <int N>
__device__ __forceinline__ double square_step(double sq, const double (&x)[N], int e, bool second_first) {
    const double v = e < 2 && second_first ? x[1 - e] : x[e];
    return e == 0 ? v * v : __builtin_fma(v, v, sq);
}
template <int N>
__device__ __forceinline__ double square_channels(const double (&x)[N], bool second_first) {
    double sq = 0.0;
#pragma unroll
    for (int e = 0; e < N; ++e) sq = square_step<N>(sq, x, e, second_first);
    return sq;
}
// ... which is: second first for a frame's summary, for the rows that a register kernel holds in its first pass (16
// rows of tables of up to 128 clusters, 32 of up to 256) and for all rows of larger tables
__device__ __forceinline__ bool row_second_first(int C, int id) { return C > 256 || id < (C > 128 ? 32 : 16); }

// One channel of Eq. 3, (n r + s) / (n + 1): n r + s in one rounding, the division in another.  y = RN(1 / (n + 1)).
// The division by n + 1, the same divisor for all channels: q = RN(x y) and two residual corrections
// q <- RN(q + RN(x - (n + 1) q) y), each residual exact in a fused multiply-add: the first leaves q within half an ulp
// and a little of x / (n + 1), and from such a q and a correctly rounded y the second returns the correctly rounded
// quotient (Markstein's theorem; n + 1 is a small integer, so its significand is not all ones, and nothing here is near
// the ends of the exponent range).  The compiler's own division hands a flag from its scaling step to its last step in
// VCC, so the divisions of several channels run one after the other.
// Where x is infinite the residuals are not a number and the last instruction, that of the compiler's own division, puts
// the infinity back.
__device__ __forceinline__ double eq3_channel(double n, double y, double r, double s) {
    const double nb = n + 1.0, x = __builtin_fma(n, r, s);
    double q = x * y;
    q = __builtin_fma(__builtin_fma(-nb, q, x), y, q);
    q = __builtin_fma(__builtin_fma(-nb, q, x), y, q);
    return __builtin_amdgcn_div_fixup(q, nb, x);
}
// The same in a chain of dependent updates, where that instruction would lengthen every link: not a number for an infinite
// x, which is left to the caller to see at the end and do over with eq3_channel.
__device__ __forceinline__ double eq3_finite(double n, double y, double r, double s) {
    const double nb = n + 1.0, x = __builtin_fma(n, r, s);
    double q = x * y;
    q = __builtin_fma(__builtin_fma(-nb, q, x), y, q);
    return __builtin_fma(__builtin_fma(-nb, q, x), y, q);
}

// The nested hierarchy's partition representatives follow the same running mean: eq3_channel per channel, and this per
// wavefront for the norm, whose squares are rounded before they are added (fused into the first addition, as the compiler
// does where it may, the two lanes of a pair get different sums)
__device__ __forceinline__ double wave_square_sum(double x) {
#pragma clang fp contract(off)
    const double sq = x * x;
    return wave64_sum(sq);
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Ordered member lists: the frames f in [c0, min(n, c0 + NT * kListPer)) with ids[f] == want, ascending, into mem; returns
// how many.  All NT threads call it (wtot: NT / 64 ints of LDS); it begins with a barrier, so mem may still be read by
// the threads when they call, and ends with one.
constexpr int kListPer = 16;
template <int NT>
__device__ __forceinline__ int list_members(const int *ids, int want, int c0, int n, int *mem, int *wtot) {
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int f0 = c0 + wave * (64 * kListPer) + lane;       // a wavefront owns 64 * kListPer consecutive frames
    int id[kListPer];
#pragma unroll
    for (int i = 0; i < kListPer; ++i) id[i] = ids[min(f0 + 64 * i, n - 1)];
    int mine = 0;
#pragma unroll
    for (int i = 0; i < kListPer; ++i) mine += __popcll(__ballot(id[i] == want && f0 + 64 * i < n));
    __syncthreads();
    if (lane == 0) wtot[wave] = mine;
    __syncthreads();
    int at = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) { at += w < wave ? wtot[w] : 0; all += wtot[w]; }
#pragma unroll
    for (int i = 0; i < kListPer; ++i) {
        const bool hit = id[i] == want && f0 + 64 * i < n;
        const unsigned long long m = __ballot(hit);
        if (hit) mem[at + __popcll(m & ((1ull << lane) - 1))] = f0 + 64 * i;
        at += __popcll(m);
    }
    __syncthreads();
    return all;
}
// acc + value(mem[0]) + value(mem[1]) + ..., in that order, UN loads in flight
template <int UN, typename F>
__device__ __forceinline__ double add_members(double acc, const int *mem, int m, F value) {
    for (int m0 = 0; m0 < m; m0 += UN) {
        double v[UN];
#pragma unroll
        for (int x = 0; x < UN; ++x) v[x] = value(mem[min(m0 + x, m - 1)]);
#pragma unroll
        for (int x = 0; x < UN; ++x)
            if (m0 + x < m) acc += v[x];
    }
    return acc;
}

constexpr int kChainFrames = 16;
constexpr double kChainMargin = 1e-11;          // in the cosine
// How far the difference of two carried-over cosines can be from that of the full computation; N: the longest chain of
// additions in a product of a chunk's products with the rows.  With u = 2^-53, v_0 = n r and v_i the frames that joined it:
// a product is off by at most (N + 1) u |v_i| |x|, and with what scales and adds up to 17 of them the numerator by
// (N + 22) u |x| sum |v_i|.  Every v_i joined at no more than a right angle (chain_decide stops after a winner that did
// not), so |sum v_i|^2 >= sum |v_i|^2 and sum |v_i| <= sqrt(17) |sum v_i|: numerators are off by sqrt(17) (N + 22) u, squared
// lengths by 17 (N + 22) u, cosines by less than 13 (N + 24) u, a difference of two by twice that.  The rounding of the rows
// themselves (three roundings an update) and of the full computation add less than 300 u.
constexpr double chain_error(int n) { return (26.0 * (n + 24) + 300.0) * 0x1p-53; }
static_assert(chain_error(128) < kChainMargin / 20, "semantic level: head sizes up to 128");

// Sum / maximum over a row of 16 lanes or a wavefront of values that may be -inf but not NaN.
__device__ __forceinline__ double row16_max(double m) {
    m = max_f64(m, dpp_f64<kDppXor8>(m));
    m = max_f64(m, dpp_f64<kDppXor7>(m));
    m = max_f64(m, dpp_f64<kDppXor3>(m));
    return max_f64(m, dpp_f64<kDppXor1>(m));
}
__device__ __forceinline__ double wave_max(double m) {
    m = row16_max(m);
    const long long b = __double_as_longlong(m);
    double wm = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int l = __builtin_amdgcn_readlane((int)b, 16 * r), h = __builtin_amdgcn_readlane((int)(b >> 32), 16 * r);
        wm = fmax(wm, __longlong_as_double(((long long)h << 32) | (long long)(unsigned int)l));
    }
    return wm;
}
// 1 / sqrt(x) and 1 / x to a few ulps (for similarities that only decide with a margin); 0 for x = 0
__device__ __forceinline__ double fast_rsqrt(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = y * (1.5 - 0.5 * x * y * y);
    y = y * (1.5 - 0.5 * x * y * y);
    return x > 0.0 ? y : 0.0;
}
__device__ __forceinline__ double fast_rcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
    return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double readlane_f64(double x, int l) {
    const long long b = __double_as_longlong(x);
    return __longlong_as_double(((long long)__builtin_amdgcn_readlane((int)(b >> 32), l) << 32) |
                                (long long)(unsigned int)__builtin_amdgcn_readlane((int)b, l));
}

// What the decision of a chunk works on (all in LDS); n frames, candidates lo .. lo + width - 1 of each.
struct ChainView {
    const double *sim;                          // [frame][width] s . r_j, -inf for an empty cluster
    int width;
    const int *lo;
    const double *sn, *isn, *ss;                // |s|, 1 / |s|, |s|^2
    const double *out;                          // no cluster outside the slots is more similar to the frame than this
    const double (*gram)[kChainFrames + 1];     // s_f . s_g / |s_g|
    const int *slot_id;
    const int *size;                            // [cluster]
    const double *irn;                          // [cluster] 1 / |r|, 0 for a zero row
};

// Decides the frames of a chunk, whose first one joins slot w of lane 0.  One wavefront; lane (g, n) = (lane / 16, lane % 16)
// looks at frame n and slots g, g + 4, ...  w: the slot every frame (lane n of each row of 16) is assumed to join (-1: it
// has no live candidate), replaced by the one it does join.  Returns the number of leading frames that are decided, at
// least one; tied: the frame after them is too close to call.
__device__ __forceinline__ int chain_decide(const ChainView &v, int nc, int n_slot, int &w, bool &tied) {
    constexpr int FR = kChainFrames;
    const int lane = threadIdx.x % 64, g = lane / 16, n = lane % 16;
    const int fn = min(n, nc - 1), lo = v.lo[fn];
    const double is = v.isn[fn], sn = v.sn[fn], ss = v.ss[fn], out = v.out[fn];
    const bool zero = ss == 0.0 && w >= 0;      // similarity 0 with every live cluster: it joins the lowest id, as assumed
    double gr[FR];                      // s_h . s_n / |s_n| of the earlier frames h
#pragma unroll
    for (int h = 0; h < FR; ++h) gr[h] = v.gram[h][fn];
    for (;;) {                          // (at most FR turns: the first frame that disagrees comes later in every one)
        double best = -INFINITY, next = -INFINITY;
        int bk = -1;
        bool odd = false, back = false;
        for (int kb = 0; kb < n_slot; kb += 4) {
            const int k = kb + g, id = v.slot_id[min(k, n_slot - 1)], cj = id - lo;
            const bool cand = k < n_slot && cj >= 0 && cj < v.width;
            const double n0 = (double)v.size[id], ir0 = v.irn[id];
            // (n r + the slot's earlier frames) . s_n / |s_n|, and the squared length of that vector
            double num = cand ? n0 * (v.sim[fn * v.width + (cand ? cj : 0)] * is) : 0.0;
#pragma unroll
            for (int h = 0; h < FR - 1; ++h)
                num += __builtin_amdgcn_readlane(w, h) == k && h < n ? gr[h] : 0.0;
            double t = w == k ? __builtin_fma(2.0 * num, sn, ss) : 0.0;
            back |= w == k && !(num >= 0.0);
            t += dpp_f64<0x111>(t);     // row_shr 1, 2, 4, 8: running sum over the frames
            t += dpp_f64<0x112>(t);
            t += dpp_f64<0x114>(t);
            t += dpp_f64<0x118>(t);
            const double len = (ir0 > 0.0 ? n0 * n0 * fast_rcp(ir0 * ir0) : 0.0) + dpp_f64<0x111>(t);
            const double c = cand && n0 > 0.0 ? num * fast_rsqrt(len) : -INFINITY;
            odd |= !(c == c);
            next = c > best ? best : fmax(next, c);
            bk = c > best ? k : bk;
            best = c > best ? c : best;
        }
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {            // over the four lanes that look at the frame
            const double ob = __shfl_xor(best, o, 64), on = __shfl_xor(next, o, 64);
            const int ok = __shfl_xor(bk, o, 64);
            next = fmax(fmax(next, on), fmin(best, ob));
            bk = ob > best ? ok : bk;
            best = fmax(best, ob);
        }
        const unsigned long long odds = __ballot(odd), backs = __ballot(back);
        const unsigned int odd16 = (unsigned int)(odds | odds >> 16 | odds >> 32 | odds >> 48) & 0xffffu;
        const unsigned int back16 = (unsigned int)(backs | backs >> 16 | backs >> 32 | backs >> 48) & 0xffffu;
        // (frame 0 joins slot 0 by construction)
        const bool clear = n == 0 || n >= nc || zero || (best - fmax(next, out) > kChainMargin && !((odd16 >> n) & 1));
        const unsigned int vague = (unsigned int)__ballot(!clear) & 0xffffu;
        const unsigned int other = (unsigned int)__ballot(clear && !zero && n > 0 && n < nc && bk != w) & 0xffffu;
        // a winner at more than a right angle shortens the representative: the rounding errors of its dot
        // products grow relative to it, so the frames after it are better taken from the rows
        const int stop = min(vague ? __ffs((int)vague) - 1 : nc, back16 ? __ffs((int)back16) : nc);
        const int at = other ? __ffs((int)other) - 1 : nc;
        if (at >= stop) {
            // (not a tie: a cluster outside the slots may be ahead, which the next chunk's products decide)
            const unsigned int behind = (unsigned int)__ballot(out - best > kChainMargin) & 0xffffu;
            tied = stop < nc && (((vague & ~behind) >> stop) & 1);
            return min(stop, nc);
        }
        if (n == at) w = bk;            // ... that frame's winner, and once more
    }
}

// How many chunks' worth of frames are taken in turn after a chunk that met a frame too close to call: one, and twice as
// many each time the next chunk fares no better.  A stream that ties at every frame (representatives along one direction)
// so pays for few products whose result it cannot use.
struct InTurn {
    int left = 0, next = 1;
    __device__ __forceinline__ void failed() { left = next; next = min(2 * next, 64); }
    __device__ __forceinline__ void held() { next = 1; }
};

} // namespace mosaic
