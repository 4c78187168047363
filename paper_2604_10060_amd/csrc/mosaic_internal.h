// Internal declarations shared by the HIP sources of libmosaic (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "../../include/mosaic.h"
#include "lloyd_groups.h"

namespace mosaic {

constexpr int kBlock = 256;       // threads per workgroup (4 wavefronts of 64)
constexpr int kRowTile = 16;      // query rows per attention tile
constexpr int kChunk = 32;        // tokens per attention step, always inside one page
constexpr int kGroup = 16;        // tokens a wavefront of the fp32 attention reduces per step, across pages
constexpr int kMaxSplits = 64;    // KV splits per (unit, row tile), average over the units of a launch
constexpr int kMaxUnitSplits = 256; // ... and the most one unit can be given when the units retrieve unequal amounts
constexpr int kPrefillTiles = 2;  // row tiles per wavefront in the multi-tile MFMA kernel
constexpr int kFp32Tiles = 2;     // row tiles per wavefront in the fp32 attention kernel when there is more than one
constexpr int kPrefillWaves = 4;  // wavefronts per workgroup of that kernel (64 * kPrefillTiles * 4 = 128 query rows)
constexpr int kMaxPartitions = 64;   // of the visual level
constexpr int kMlRows = 3;        // rows of 16 floats per attention partial besides O: max, normaliser, exact-weight sum

// A frame's K-means bounds, in units of 2^-14: its chord to its own representative from above, to the others of each group from below
struct __attribute__((aligned(16))) ChordBounds { unsigned short ub, lb[kLloydGroups]; };

// A pointer that the GPU loads from memory and uses as one to global memory (the compiler knows that of a kernel's arguments only)
#ifdef __HIP_DEVICE_COMPILE__
#define MOSAIC_GLOBAL __attribute__((address_space(1)))
#else
#define MOSAIC_GLOBAL
#endif
template <typename T> struct DevPtr {
    MOSAIC_GLOBAL T *p;
    DevPtr() = default;
    __host__ __device__ __forceinline__ DevPtr(T *q) : p((MOSAIC_GLOBAL T *)q) {}
    __host__ __device__ __forceinline__ operator T *() const { return (T *)p; }
};

// Device-side view of one context: plain pointers into the caller's arena.
struct alignas(64) DeviceView {
    const DeviceView *self;     // the copy of this struct that kernels read (in the arena)
    // geometry
    int L, Hq, Hkv, G, D, T, Tp, F, C, k, U;
    int esize;        // bytes per KV element
    int v_transposed; // not 0: V pages stored [Tp/32][D][32] (MFMA path, Tp = T rounded up to 32); 0: [T][D]
                      // 2: and K pages in pieces of 32 channels, [D/32][T][32]; else [T][D]
    // K pages: elements from one token to the next and from 32 channels to the next 32
    __device__ __forceinline__ int k_rs() const { return v_transposed == 2 ? 32 : D; }
    __device__ __forceinline__ size_t k_ps() const { return v_transposed == 2 ? (size_t)32 * T : 32; }
    int chunks_per_page;
    int tier;         // MOSAIC_TIER_*
    int PU;           // pages per unit in k_store / v_store: F (HBM tier) or the cluster-cache capacity (host tier)
    int SN;           // host tier: frames in the staging ring
    int SC;           // score columns per unit: C + buf_max
    // KV pages the attention kernels read, addressed through k_page()/v_page() below: two arrays,
    //   k_store [U][PU] K pages, v_store [U][PU] V pages.
    // HBM tier: page p = frame id (arrival order).  Host tier: page p = a slot of the unit's GPU
    //   cluster cache (slots are handed out frame by frame; a cluster's frames need not be adjacent).
    // A K page is [T][D] or, for the bf16 MFMA path on stores of at most 768 MiB, in pieces of 32 channels, [D/32][T][32].
    //   A V page is [T][D] or, for the bf16 MFMA path, [Tp/32][D][32].
    DevPtr<char> k_store;
    DevPtr<char> v_store;
    size_t kpage, vpage;           // bytes of one K / V page
    size_t k_ustride, v_ustride;   // bytes between units, K array / V array
    // latest selection per unit
    DevPtr<double> scores;   // [U][SC]
    DevPtr<int> ids;         // [U][k]
    DevPtr<int> n_ids;       // [U]
    DevPtr<int> sel_pages;   // [U][F]      frames of the selected clusters, gather order
    DevPtr<int> n_sel;       // [U]         number of selected frames
    // attention partials: entry e = base_slot(unit)*NT + tile*S(unit) + split, see split_slot()
    DevPtr<float> part_o;    // [entries][16][D]
    DevPtr<float> part_ml;   // [entries][3][16]  running max (log2 domain), sum of the weights the value contraction
                      //                   used (bf16-rounded in the MFMA kernels), sum of the unrounded weights
    int aug_reps, aug_window;       // retrieval augmentation (paper Sec. V-C); both 0 = off
    // clustering state (decision arithmetic in fp64)
    DevPtr<double> summ;     // [U][F][D]   per-frame key summaries
    DevPtr<double> r;        // [U][C][D]   representatives
    DevPtr<double> rnorm;    // [U][C]      |r_j|
    DevPtr<int> n;           // [U][C]      sizes in frames
    DevPtr<int> assign;      // [U][F]      frame -> cluster
    DevPtr<int> pos;         // [U][F]      rank of the frame among its cluster's members (ascending frame order)
    int maint_mode;          // self-adaptive maintainer (paper Sec. VI), 0 = off
    int P, Cs, top_p;        // nested visual-semantic hierarchy (paper Sec. V-B, V-C); P = 0: flat index
    // (what decode and questions read ends here: four lines of 64 bytes)
    // host tier: staging ring the ingest kernel writes (frame f at slot f % SN), and the
    // device-visible address of the pinned host pools the offload kernel writes
    DevPtr<char> stage_k, stage_v;   // [SN][U][page]
    // A V page in [Tp/32][D][32] leaves out what pads it there: whole blocks of 32 tokens as they are, then [D][4 * htail] of the last T % 32 tokens
    // (htail = 0: none, or so many that nothing is saved; the page is then as on the GPU).
    // The link bounds both directions: 512 frames of 196 tokens offloaded and four questions' clusters fetched back 15.35 -> 14.55 ms.
    DevPtr<char> host_k, host_v;     // pinned pools: [U][HP/SFh] slabs of [SFh K pages][SFh V pages]
    size_t h_ustride, h_bstride, hvpage;   // hvpage: bytes of a V page there
    int htail;
    int SFh;                   // frames per host slab
    int HP;                    // host pages per unit
    DevPtr<const int> dest;           // [2][U][SN] host page of each staged frame of a batch, two tables in turn (pinned memory)
    DevPtr<int> batch_assign;         // [U][n] a host-tier batch's gathered assignments (pinned memory)
    // fetch work lists, written by the host into pinned memory and read by k_fetch over PCIe
    DevPtr<const int> moves;          // [U][F][2] (host page, cache page)
    DevPtr<const int> n_moves;        // [U]
    DevPtr<long long> sel_flag;   // [U]    (launch number << 32 | retrieved pages) of the unit's last selection published inside a launch (k_decode_layer)
    DevPtr<int> sync_err;    // [1]         set if a bounded in-kernel wait ever ran out
    DevPtr<int> lloyd_moved; // [U][3]      frames moved by the K-means rounds it-1, it, it+1 (mod 3): converged units skip the rest
    DevPtr<int> lloyd_changed; // [U][C]    1 = a frame entered or left the cluster in the current round (its sums must be rebuilt)
    DevPtr<double> lloyd_delta; // [U][C]   chord by which the last update moved the representative's direction
    DevPtr<ChordBounds> lloyd_bounds; // [U][F]
    // self-adaptive maintainer (paper Sec. VI; empty arrays when it is off)
    int c_init, split_iters, buf_max;
    double tau_min, tau_max, tau_n0;
    DevPtr<double> var;      // [U][C]      running intra-cluster variance (Eq. 2 / Eq. 4)
    DevPtr<int> lazy;        // [U][C]      lazy-split flag
    DevPtr<int> resident;    // [U][C]      1 = selected by the unit's latest retrieval
    DevPtr<int> n_slots;     // [U]         cluster ids in use: [0, n_slots)
    DevPtr<int> buf_frame;   // [U][buf_max] buffered singletons: frame
    DevPtr<int> buf_owner;   // [U][buf_max]                       cluster they were assigned to
    DevPtr<int> n_buf;       // [U]
    DevPtr<long long> mt_cnt;// [U][4]      splits on insertion, deferred splits, buffered inserts, forced absorbs
    DevPtr<int> mt_mem, mt_side;   // [U][F] scratch of Split
    DevPtr<double> mt_nrm;          // [U][F]
    // retrieval augmentation (paper Sec. V-C)
    int nt_max;
    DevPtr<float> rep_k, rep_v;   // [U][C][D] fp32 pseudo-token tables: representative, value representative
    DevPtr<float> aug_o;     // [U][nt_max][16][D]  partial of the representatives' part, same form as part_o
    DevPtr<float> aug_ml;    // [U][nt_max][2][16]
    DevPtr<double> vsumm;    // [U][F][D]   per-frame value summaries (mean of the frame's T value vectors)
    DevPtr<double> rvsum;    // [U][C][D]   per-cluster sums of them (value representative = rvsum / n)
    // nested visual-semantic hierarchy (paper Sec. V-B, V-C)
    int Dv;
    DevPtr<double> vemb;     // [F][Dv]     visual embeddings of the frames (the visual level's states)
    DevPtr<double> vr;       // [P][Dv]     visual centroids
    DevPtr<double> vrn;      // [P]         their norms
    DevPtr<int> vn;          // [P]         their sizes in frames
    DevPtr<int> part;        // [F]         frame -> visual partition (shared by all units)
    DevPtr<double> pr;       // [U][P][D]   partition representatives in the unit's key space
    DevPtr<double> prn;      // [U][P]
    DevPtr<int> pn;          // [U][P]
    DevPtr<double> pscores;  // [U][P]      first-stage scores of the latest retrieval
    DevPtr<int> pids;        // [U][top_p]  partitions it kept
    DevPtr<int> n_pids;      // [U]
    DevPtr<int> tok_scratch; // [Hkv][F*T]  token-index expansion for the observer
    long long part_entries;
};

static_assert(sizeof(DeviceView) % 8 == 0, "loaded by words");

static_assert(offsetof(DeviceView, tier) == 64 && offsetof(DeviceView, scores) == 128 && offsetof(DeviceView, summ) == 192 &&
              offsetof(DeviceView, stage_k) == 256 && offsetof(DeviceView, nt_max) / 64 == 8 && offsetof(DeviceView, aug_ml) / 64 == 8, "lines of what decode reads");

// A kernel's view: the fields that it uses, by scalar loads.  A launch carries the address, which lies in registers when a wavefront starts (the build asks
// for that).  With the struct itself as an argument a launch of a few us is longer by 0.2 us and more, and so is the way to it.  What that is of a call is
// little, and the same for a question asked over and over / never before / with 1 GB read between the steps (us, with the struct -> so, runs
// within 0.5 %): a token through 28 layers (84 launches) 981 -> 961 / 990 -> 970 / 1030 -> 1009, four fp32 layers 129 -> 126 / 123 -> 121 / 130 -> 125, four with
// window and representatives 81.7 -> 81.3 / 84.0 -> 82.1 / 91.4 -> 89.4, one layer 19.3 -> 19.0 / 20.8 -> 20.8 / 25.7 -> 25.0.  768 frames one by one
// (784 launches) 5.20 -> 4.95 ms.
// LINES of it are fetched at once: the compiler loads a field where it is first used, which is one more trip to the L2 on a kernel's chain.
template <int... LINES>
__device__ __forceinline__ DeviceView device_view(const DeviceView *self) {
    typedef __attribute__((address_space(4))) const unsigned long long Word;
    constexpr int N = sizeof(DeviceView) / 8;
    const Word *w = (const Word *)(unsigned long long)self;
    unsigned long long a[N];
#pragma unroll
    for (int i = 0; i < N; ++i) a[i] = w[i];
    if constexpr (sizeof...(LINES) > 0) {
        const unsigned long long t = (0 | ... | a[LINES * 8]);
        asm volatile("" ::"s"(t));
    }
    DeviceView v;
    __builtin_memcpy(&v, a, sizeof v);
    return v;
}

struct HostTier;   // host_tier.hip
constexpr int kReadPieces = 4;      // pinned pieces that large read-backs go through

struct Ctx {
    mosaic_config cfg;
    DeviceView dv;
    hipStream_t stream;
    int device;
    int W;               // warm-up frames
    int iters;
    int impl;            // MOSAIC_ATTEND_VALU | MOSAIC_ATTEND_MFMA
    long long n_frames;  // ingested so far (host-side count)
    std::vector<long long> sel_epoch; // per layer: epoch at which the selection was made
    std::vector<int> sel_tq;
    long long epoch;     // bumped by ingest and reset
    int launch_epoch;    // numbers the launches that publish a selection inside the kernel (never 0)
    long long rv_epoch;  // epoch the value representatives were last computed at
    mosaic_stats stats;
    std::string err;
    bool views_written;   // the kernels' copies of dv are in the arena
    void *static_scratch; // device address, on this context's GPU, of the library's static partial buffer
    HostTier *host;      // non-null in the host tier
    // host tier: host-side views of the pinned arena
    char *h_k, *h_v;     // slab pools
    int *h_sel, *h_nsel; // page lists / counts staged for upload, [U][F] / [U]
    int *h_moves, *h_nmoves; // fetch work lists, [U][F][2] / [U]
    int *h_ids, *h_nids; // selections read back, [U][k] / [U]
    int *h_assign, *h_dest; // staged batch: assignments read back / slab positions, [U][SN]
    int *h_assign_full;      // maintainer: a unit's whole frame -> cluster map read back, [U][F]
    long long *h_cnt;        // ... its counters, [U][4]
    int *h_nbuf, *h_buf_frame, *h_buf_owner;   // ... its singleton buffer, [U] / [U][buf_max]
    int *h_resident;         // residency flags on their way to the device, [U][C]
    // ingest_overlap: the order-dependent part of batched ingest calls runs here, after `stored`;
    // `assigned` marks its end and the caller's stream waits for it before anything touches the index
    hipStream_t assign_stream;
    hipEvent_t stored, assigned;
    bool assign_pending;
    // large read-backs (null until the first one)
    char *read_buf;
    hipEvent_t read_done[kReadPieces];
    // profiling
    bool profile;
    std::vector<hipEvent_t> ev;      // pool of pairs, created by mosaic_profile_enable
    size_t ev_used;
    double prof_ms;                  // kernel time and launches folded out of the pool so far
    long long prof_n;
};

// ---- launchers (each checks its own launch; returns hipError_t) ----
// beyond: the pages go to a store far beyond the caches; e_in: the embeddings of these frames, of which the n_emb first are filed in the visual
// level's state array (nested hierarchy, warm-up)
hipError_t launch_store_summary(const DeviceView &dv, const void *k_in, const void *v_in,
                                int f0, int n_frames, bool beyond, const float *e_in, int n_emb, hipStream_t s);
// pages, summary, assignment and Eq. 3 of one frame in one launch (HBM tier, maintainer off,
// C <= 128, frame f beyond the warm-up)
hipError_t launch_ingest_one(const DeviceView &dv, const void *k_in, const void *v_in, int f, hipStream_t s);
hipError_t launch_assign_update(const DeviceView &dv, int f0, int f1, hipStream_t s);
hipError_t launch_lloyd(const DeviceView &dv, int n_frames, int iters, bool seed_from_warmup,
                        hipStream_t s);
// visual level: initial P-means over the first W embeddings / greedy assignment of frames f0..f1-1
hipError_t launch_visual_lloyd(const DeviceView &dv, int W, int iters, hipStream_t s);
// (e_in: fp32 embeddings of frames f0..f1-1, which the kernel also files in the state array)
hipError_t launch_visual_assign(const DeviceView &dv, const float *e_in, int f0, int f1, hipStream_t s);
// ... with the page stores of the same frames in the same launch (calls that it takes)
bool store_visual_assign_takes(const DeviceView &dv, int n_frames);
hipError_t launch_store_visual_assign(const DeviceView &dv, const void *k_in, const void *v_in, const float *e_in, int f0, int f1, bool beyond,
                                      hipStream_t s);
// per-unit partition representatives recomputed from the member lists (after a K-means run)
hipError_t launch_partition_reps(const DeviceView &dv, int n_frames, hipStream_t s);
// write_pages = false (host tier): only scores and ids; the page list comes from the host
hipError_t launch_retrieve(const DeviceView &dv, int u0, int n_units, const void *q, int Tq,
                           int n_frames, int score_mode, bool write_pages, hipStream_t s);
// deferred-split maintainer: singletons take part, residency and deferred splits follow the selection
hipError_t launch_retrieve_deferred(const DeviceView &dv, int u0, int n_units, const void *q, int Tq,
                                    int n_frames, int score_mode, hipStream_t s);
// the assignments of frames f0..f0+n-1 of every unit to rows, [U][n]
hipError_t launch_gather_assign(const DeviceView &dv, int *rows, int f0, int n, hipStream_t s);
// host tier: copy staged frames f0..f0+n-1 of every unit to host page dest[u][f - f0]
hipError_t launch_offload(const DeviceView &dv, const int *dest, int f0, int n, hipStream_t s);
// host tier: move the pages listed in moves[u0..u0+n_units) from the pinned slabs into the cache
hipError_t launch_fetch(const DeviceView &dv, int u0, int n_units, int max_moves, hipStream_t s);
hipError_t launch_expand_tok_idx(const DeviceView &dv, int u0, int n_units, hipStream_t s);
// n_splits = average splits per unit chosen by the caller (B = n_units * n_splits split
// workgroups are shared out by split_slot); partial entries needed = B * NT
// ev0/ev1 (may be null) receive the kernel's own start/stop timestamps
// shares (questions of more than one row tile): groups of equal shares of the launch's chunks and what a workgroup takes of them
// (even_share); partial entries needed = (groups + n_units - 1) * NT
struct Shares { int groups; bool walk; };
hipError_t launch_attend_prefill(const DeviceView &dv, int u0, int n_units, const unsigned short *q, int Tq,
                                 Shares shares, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
// bf16 pages on the vector ALU (MOSAIC_ATTEND_VALU)
hipError_t launch_attend_valu(const DeviceView &dv, int u0, int n_units, const void *q, int Tq,
                              int n_splits, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
// fp32 pages (fp32 matrix instruction)
hipError_t launch_attend_fp32(const DeviceView &dv, int u0, int n_units, const float *q, int Tq, int n_splits,
                              Shares shares, bool stream_kv, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
// stream_kv: the decode-shape kernels load K/V with the non-temporal hint (stores far beyond the caches)
hipError_t launch_attend_mfma(const DeviceView &dv, int u0, int n_units, const void *q, int Tq,
                              int n_splits, Shares shares, bool stream_kv, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
// uniform: every unit has exactly n_splits splits at slots unit * n_splits + split (fused decode step)
hipError_t launch_attend_combine(const DeviceView &dv, int u0, int n_units, int Tq, int n_splits,
                                 void *out, float *lse, hipStream_t s, bool uniform = false, Shares shares = {});
// selection + attention of one decode step of one layer in one launch with size-proportional splits: the
// first n_units workgroups select for one unit each and publish the result, all workgroups then share
// out the retrieved pages (one row tile, bf16, C <= 256).  epoch: a number no earlier launch on this
// context has used.  B = total workgroups (>= n_units)
hipError_t launch_decode_layer(const DeviceView &dv, int u0, int n_units, const void *q, int Tq, int B, int n_frames,
                               int score_mode, int epoch, bool stream_kv, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
// selection + attention of one decode step in one launch (one row tile, C <= 256, uniform splits)
hipError_t launch_decode_fused(const DeviceView &dv, int u0, int n_units, const void *q, int Tq, int n_splits,
                               int n_frames, int score_mode, bool stream_kv, hipStream_t s, hipEvent_t ev0,
                               hipEvent_t ev1);
// retrieval augmentation: per-cluster value sums of all units (after the clustering changed); the
// attention partial over the representatives is computed by extra workgroups of the attention launches
hipError_t launch_value_reps(const DeviceView &dv, int n_frames, hipStream_t s);

// A kernel launch that carries a HIP start/stop event pair when one is given (the events receive the
// kernel's own begin and end timestamps) and is a plain launch otherwise, which a caller may also
// record into a HIP graph.
template <typename K, typename... A>
inline void launch_timed(K kern, dim3 grid, dim3 block, size_t lds, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                         A... args) {
    if (ev0 || ev1) hipExtLaunchKernelGGL(kern, grid, block, (unsigned)lds, s, ev0, ev1, 0, args...);
    else hipLaunchKernelGGL(kern, grid, block, (unsigned)lds, s, args...);
}

// ---- small device helpers ----
__device__ __forceinline__ const char *k_page(const DeviceView &dv, int u, int p) {
    return dv.k_store + (size_t)u * dv.k_ustride + (size_t)p * dv.kpage;
}
__device__ __forceinline__ const char *v_page(const DeviceView &dv, int u, int p) {
    return dv.v_store + (size_t)u * dv.v_ustride + (size_t)p * dv.vpage;
}
__device__ __forceinline__ float bf16_to_f32(unsigned short h) {
    return __uint_as_float(((unsigned int)h) << 16);
}
__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f) {
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40); // NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}


// A score as the rankings order it.  What is not above the lowest number (no number at all, or minus infinity: a question that
// overflowed) counts as that, so that the live entries' ranks are distinct and an empty entry's minus infinity stays below them: a
// rank that two entries shared would leave another without one, and what lies there would be read as an id.
__device__ __forceinline__ double rank_score(double s) { return s > -1.7976931348623157e308 ? s : -1.7976931348623157e308; }

// Sum of N values (a power of two) in pairs: log2 N roundings on the way of each instead of up to N - 1.
template <int N> __device__ __forceinline__ float pair_sum(const float (&x)[N]) {
    float y[N];
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = x[i];
#pragma unroll
    for (int h = N / 2; h >= 1; h /= 2)
#pragma unroll
        for (int i = 0; i < h; ++i) y[i] += y[i + h];
    return y[0];
}

// ---------------------------------------------------------------------------
// Reductions over the 16 lanes of a DPP row (lanes 16k .. 16k + 15) with data-parallel
// primitives instead of LDS permutes: a butterfly over the lane-index masks 8, 7, 3, 1
// (row_ror:8, row_half_mirror, quad_perm [3,2,1,0], quad_perm [1,0,3,2]), which span all
// 16 lanes.  Every step adds a lane's partner symmetrically, so all 16 lanes end with the
// same bits.  About 80 cycles for a double against about 500 with ds_bpermute.
// ---------------------------------------------------------------------------
template <int CTRL> __device__ __forceinline__ int dpp_i32(int x) {
    // bound_ctrl on: a source lane that is out of range or switched off reads as 0, which is also what the old value 0
    // would leave, and the compiler need not clear the destination first (two instructions fewer per 64-bit step)
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ double dpp_f64(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = dpp_i32<CTRL>((int)b), hi = dpp_i32<CTRL>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}
constexpr int kDppXor8 = 0x128, kDppXor7 = 0x141, kDppXor3 = 0x1B, kDppXor1 = 0xB1;
__device__ __forceinline__ double row16_sum(double x) {
    x += dpp_f64<kDppXor8>(x);
    x += dpp_f64<kDppXor7>(x);
    x += dpp_f64<kDppXor3>(x);
    x += dpp_f64<kDppXor1>(x);
    return x;
}
// Sum over the 64 lanes of a wavefront (all lanes active), the same bits in every lane: the four rows'
// sums are read from their first lanes and added in a fixed order.
__device__ __forceinline__ double wave64_sum(double x) {
    x = row16_sum(x);
    const long long b = __double_as_longlong(x);
    const int lo = (int)b, hi = (int)(b >> 32);
    double r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int l = __builtin_amdgcn_readlane(lo, 16 * i), h = __builtin_amdgcn_readlane(hi, 16 * i);
        r[i] = __longlong_as_double(((long long)h << 32) | (long long)(unsigned int)l);
    }
    return (r[0] + r[1]) + (r[2] + r[3]);
}


// ---------------------------------------------------------------------------
// Load-balanced KV splits.  An attend launch has B split workgroups (per row
// block) for the n_units units of the call.  Units retrieve different numbers
// of tokens, so the splits are shared out in proportion to the selected page
// counts: unit i gets (n_sel_i > 0) + floor((B - n_units) * n_sel_i / total),
// capped at kMaxUnitSplits, contiguous workgroup ids, in unit order.  The attention
// kernels (by workgroup id) and the combine kernel (by unit) evaluate the same
// function of the same device-resident sizes, so they agree without any
// host round trip.  Every lane of the calling wavefront gets the result.
// ---------------------------------------------------------------------------
struct SplitSlot {
    int uc;      // unit within the call, -1: this workgroup has no work
    int split;   // split index within the unit
    int S;       // number of splits of the unit
    int base;    // first split slot of the unit (partials are indexed by slot)
    int n;       // the unit's retrieved size (n_sel), so that the caller need not load it again
};

// Agent-scope (write-through / cache-bypassing) accesses for values that one workgroup publishes and
// others of the SAME launch read: an ordinary store may sit in the writing XCD's L2 until the kernel ends.
// Workgroup barrier that orders LDS accesses only: does not wait for outstanding global loads and stores.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ void st_agent(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ int ld_agent(const int *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_agent(long long *p, long long v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ long long ld_agent(const long long *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

template <bool BY_UNIT>
__device__ __forceinline__ SplitSlot split_slot(const int *n_sel_call, int n_units, int B, int key) {
    const int lane = threadIdx.x % 64;
    if (n_units <= 8) {
        // A layer's few units (the per-layer decode chain, where this sits at the head of two launches' dependent
        // chains): sizes, shares and offsets as wave-uniform scalars read from the first lanes, one 32-bit
        // division per lane where the product fits, no cross-lane scans.  Same shares as the general path below.
        const int ns = lane < n_units ? n_sel_call[lane] : 0;
        long long total = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) total += __builtin_amdgcn_readlane(ns, i);
        int want = 0;
        if (ns > 0) {
            const long long prod = (long long)(B - n_units) * ns;      // total >= ns > 0 here
            want = 1 + (prod < (1ll << 32) && total < (1ll << 32) ? (int)((unsigned int)prod / (unsigned int)total)
                                                                  : (int)(prod / total));
            want = min(want, kMaxUnitSplits);
        }
        SplitSlot r{-1, 0, 0, 0, 0};
        int run = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int w = __builtin_amdgcn_readlane(want, i);
            const bool hit = BY_UNIT ? (i == key) : (key >= run && key < run + w);
            if (hit && r.uc < 0 && i < n_units) {
                r.uc = i; r.S = w; r.base = run; r.split = BY_UNIT ? 0 : key - run;
                r.n = __builtin_amdgcn_readlane(ns, i);
            }
            run += w;
        }
        return r;
    }
    long long total = 0;
    for (int i = lane; i < n_units; i += 64) total += n_sel_call[i];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) total += __shfl_xor(total, o, 64);
    SplitSlot r{-1, 0, 0, 0, 0};
    int run = 0;
    for (int i0 = 0; i0 < n_units; i0 += 64) {
        const int i = i0 + lane;
        const int ns = i < n_units ? n_sel_call[i] : 0;
        int want = 0;
        if (i < n_units && ns > 0) {
            want = 1 + (int)(((long long)(B - n_units) * ns) / (total > 0 ? total : 1));
            want = min(want, kMaxUnitSplits);
        }
        int incl = want;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        const int excl = run + incl - want;
        const bool hit = BY_UNIT ? (i == key) : (key >= excl && key < excl + want);
        const unsigned long long mask = __ballot(hit);
        if (mask) {
            const int src = __ffsll((long long)mask) - 1;
            r.uc = i0 + src;
            r.S = __shfl(want, src, 64);
            r.base = __shfl(excl, src, 64);
            r.n = __shfl(ns, src, 64);
            r.split = BY_UNIT ? 0 : key - r.base;
        }
        run += __shfl(incl, 63, 64);
    }
    return r;
}

// ---------------------------------------------------------------------------
// Equal shares, for questions of more than one row tile.  What the units of a launch retrieved is one sequence of chunks (32
// tokens of a page in the bf16 kernel, 16 tokens across pages in the fp32 one), in unit order; group g of G has chunks
// g * per .. (g + 1) * per - 1 of it, per = ceil(chunks / G), whichever units they belong to.  The partial of (unit i,
// group g) sits at slot g + i, which rises by at least one from each (unit, group) pair to the next, so that slots are distinct
// and there are at most G + n_units - 1 of them; unit i's are the S slots from base on.
// (Chunks of a launch fit 32 bits: each has at least 4 KB of pages in GPU memory.)
// A workgroup takes a group and walks over its units, or it takes one slot.  The attention kernels look up the group or the
// slot, the merge the unit; every lane of the wavefront gets the result.
// ---------------------------------------------------------------------------
// bf16: chunks stay inside a page (per = chunks of a page); fp32: a unit's tokens are one sequence (per = tokens of a page;
// max_frames * T fits in 32 bits)
template <bool FP32> struct ChunkSize {
    int per;
    __device__ __forceinline__ explicit ChunkSize(const DeviceView &dv) : per(FP32 ? dv.T : dv.chunks_per_page) {}
    __device__ __forceinline__ int of(int pages) const { return FP32 ? (pages * per + kGroup - 1) / kGroup : pages * per; }
};
enum ShareKey { kShareOfGroup, kShareOfSlot, kShareOfUnit };
struct EvenShare {
    int uc;        // unit within the call: the group's first, the slot's, or the one asked for; -1: there is none
    int before;    // chunks of the units before it
    int n;         // the unit's retrieved pages
    int chunks;    // its chunks
    int per;       // chunks per group
    int all;       // chunks of the launch
    __device__ __forceinline__ int base() const { return before / per + uc; }
    __device__ __forceinline__ int splits() const { return chunks > 0 ? (before + chunks - 1) / per - before / per + 1 : 0; }
};

template <ShareKey BY, bool FP32>
__device__ __forceinline__ EvenShare even_share(const int *n_sel_call, int n_units, ChunkSize<FP32> cs, int G, int key) {
    const int lane = threadIdx.x % 64;
    int total = 0;
    for (int i = lane; i < n_units; i += 64) total += cs.of(n_sel_call[i]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) total += __shfl_xor(total, o, 64);
    EvenShare r{-1, 0, 0, 0, 1, total};
    r.per = max(1, (int)((unsigned int)(total + G - 1) / (unsigned int)G));
    const long long want = (long long)key * r.per;          // the group's first chunk
    int run = 0;
    for (int i0 = 0; i0 < n_units; i0 += 64) {
        const int i = i0 + lane;
        const int pages = i < n_units ? n_sel_call[i] : 0, c = cs.of(pages);
        int incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        const int excl = run + incl - c;
        bool hit;
        if (BY == kShareOfUnit) hit = i == key;
        else if (BY == kShareOfGroup) hit = want >= excl && want < excl + c;
        else hit = c > 0 && key >= excl / r.per + i && key <= (excl + c - 1) / r.per + i;
        const unsigned long long mask = __ballot(hit);
        if (mask) {
            const int src = __ffsll((long long)mask) - 1;
            r.uc = i0 + src;
            r.before = __shfl(excl, src, 64);
            r.n = __shfl(pages, src, 64);
            r.chunks = __shfl(c, src, 64);
        }
        run += __shfl(incl, 63, 64);
    }
    return r;
}

// What one workgroup takes, unit by unit.  Wave-uniform values are moved to scalar registers (quotients are formed in vector
// registers).
template <bool FP32> struct ShareWalk {
    int uc, n;              // unit within the call, its pages
    int c0, c1;             // the range of the unit's chunks
    int base, S, split;     // its partials: first slot and number of the unit's, which of them this is
    int left, before, per, grp;
    __device__ __forceinline__ void enter(int chunks) {      // the unit (uc, n) from chunk c0 on, in group grp
        c1 = min(chunks, c0 + left);
        left -= c1 - c0;
        const int g0 = __builtin_amdgcn_readfirstlane(before / per);
        base = g0 + uc;
        S = __builtin_amdgcn_readfirstlane((before + chunks - 1) / per) - g0 + 1;
        split = grp - g0;
    }
    // walk: key is a group, else a slot.  false: nothing to do
    __device__ __forceinline__ bool start(const int *n_sel_call, int n_units, ChunkSize<FP32> cs, int G, int key, bool walk) {
        EvenShare sh;
        if (walk) sh = even_share<kShareOfGroup, FP32>(n_sel_call, n_units, cs, G, key);
        else sh = even_share<kShareOfSlot, FP32>(n_sel_call, n_units, cs, G, key);
        uc = __builtin_amdgcn_readfirstlane(sh.uc); n = __builtin_amdgcn_readfirstlane(sh.n);
        before = __builtin_amdgcn_readfirstlane(sh.before); per = __builtin_amdgcn_readfirstlane(sh.per);
        if (uc < 0) return false;
        grp = walk ? key : key - uc;
        c0 = max(grp * per - before, 0);                     // (grp * per is at most the launch's chunks)
        left = min((grp + 1) * (long long)per, (long long)__builtin_amdgcn_readfirstlane(sh.all)) - before - c0;
        enter(cs.of(n));
        if (!walk) left = 0;
        return true;
    }
    // the group's next unit; false: there is none
    __device__ __forceinline__ bool next(const int *n_sel_call, ChunkSize<FP32> cs) {
        if (left <= 0) return false;
        do {
            before += cs.of(n);
            n = __builtin_amdgcn_readfirstlane(n_sel_call[++uc]);
        } while (n == 0);                                    // (chunks are left, so a later unit has some)
        c0 = 0;
        enter(cs.of(n));
        return true;
    }
};

// Workgroup w of a launch of (group, row block) pairs, w = group * row blocks + row block, for block id `id`: workgroups go to
// the 8 XCDs round-robin by id and are dispatched in id order, so the pairs are dealt in eight contiguous runs.  A group's row
// blocks then share one XCD and its L2 (those at a run's end: two) and have neighbouring dispatch slots there, which keeps
// them together in time, so that the group's K/V is fetched from memory once and found in L2 by the rest; and any number of pairs
// fills the XCDs evenly.  -1: none.  The grid has 8 * ceil(pairs / 8) ids.
__device__ __forceinline__ int xcd_run(int id, int pairs) {
    const int per = (pairs + 7) / 8, seq = id / 8, w = id % 8 * per + seq;
    return seq < per && w < pairs ? w : -1;
}

} // namespace mosaic
