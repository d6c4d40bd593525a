// HIP kernels (gfx950, wave64) and the device-facing entry points of the C ABI.
//
// Pipeline of one rsdgc_compress call, all layers per launch.  "Candidate path": a layer whose
// keep ratio leaves room for it records only the centres whose score reaches a bound and ranks
// those; the other layers are ranked on a full score map.  The result is the same on both.
//   begin      zero histograms, bitmasks, counters, flags; per-layer state; for every layer on
//              the candidate path the bound predicted from the thresholds of the two calls before.
//              A launch of its own (k_begin) only where the tables are laid down: every call
//              clears what it has used and its emit sets the next call's states (NextCall)
//   first pass every tile of the layers that are always ranked on the full score map: v = r + g
//              (Eq. 12), NSI (Eqs. 6-10), score map, exact 12-bit histogram; during the first calls
//              with a workspace, in the same launch, one tile in 16 .. 64 of the candidate-path
//              layers that have no predicted bound: their score histogram gives a bound with
//              about 2 k_l centres expected above it (k_hint).  Not launched when it has no tiles.
//   capture    the main pass: v = r + g and NSI for every element of the candidate-path layers;
//              centres whose score reaches the bound are recorded per tile (no score map) and
//              counted in fine bins above the bound; with a second residual arena v is stored
//              there as it is formed; with one, in large plans, in the residual's place, and the
//              windows across the tiles' edges follow in a launch of their own (k_seams)
//   find0      first ranking digit of every layer; a layer whose bound caught fewer than k_l
//              centres, or overfilled a tile, falls back to the full map (a flag tells the
//              fallback kernels there is work)
//   fallback   score map + histogram of such layers (rare); the same launch as find0 where its
//              workgroups can look at every layer (k_find0_fallback)
//   select     gather: the candidates above each layer's threshold bucket are selected for certain
//              and mark their windows; the bucket's keys are copied to a list and their next digit
//              counted; finish: one workgroup per layer resolves the remaining digits
//              (Algorithm 1's ranking; Eq. 11's k_l) and keeps the threshold for the next calls
//   mark       the bucket's keys that reach the threshold set the bits of their p x p window
//              (Section III-C: whole neighbourhoods are kept); full-map layers: every centre
//              (small plans with every layer on the candidate path: find0 to mark are one launch, k_select)
//   count      kept elements per chunk and per group of chunks (no scan kernel: each consumer
//              adds up its own prefix from those): small plans count as they mark, large ones of few layers beside
//              the ranking, the others in a launch of its own, as all do with the centres, where their lists are wanted
//   emit       ordered (index, value) pairs and the residual update (Eq. 12): either only the
//              kept elements are touched (v is stored already; by workgroups or, on large plans, by
//              waves), or g and r are streamed again (one arena, smaller plans)
//
// Sections of this file, in order (each starts with a "// ---- name --" line):
//   begin            k_begin
//   work feed        WorkFeed: tiles handed to persistent workgroups through per-XCD counters
//   nsi              k_nsi<P, PASS, MOM, FEED>: the NSI passes, with or without Eq. 12's momentum; k_seams
//   ranking digits   block_find_digit, publish_threshold
//   hint .. finish   k_hint, k_find0, k_find0_fallback(_all), k_gather, k_filter, k_finish: bounds and
//                    the radix select
//   select           k_select: find0 to mark in one launch, small plans
//   mark             k_mark: p x p windows into the bitmask; k_mark_flat: block grids
//   count            k_count, chunk_prefix_wave0
//   emit             k_emit, k_emit_sparse, k_emit_waves, k_emit_centres
//   decompress       k_zero_layers, k_scatter (for_each_pair)
//   block reading    k_block_nsi, k_emit_blocks, k_scatter_blocks
//   apply            k_apply_ranges, k_apply_chunks, k_apply_single, k_apply_blocks (receiving side)
//   dynamic ratios   k_dyn_*
//   host side        launch helpers and the extern "C" entry points
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "rsdgc_internal.h"

using namespace rsdgc;

namespace {

thread_local char g_hip_error[256] = "";

int hip_fail(hipError_t e, const char *what) {
    std::snprintf(g_hip_error, sizeof(g_hip_error), "%s: %s", what, hipGetErrorString(e));
    return RSDGC_EHIP;
}
#define HIP_TRY(expr)                                        \
    do {                                                     \
        hipError_t e_ = (expr);                              \
        if (e_ != hipSuccess) return hip_fail(e_, #expr);    \
    } while (0)

// Composite ranking key  K = (score bits << 32) | ~index.  Scores are non-negative floats, so
// their bit pattern orders like the value; ~index makes the lower index the larger key; all
// keys of a layer are distinct.
constexpr uint32_t kNumCUs = 256;   // MI355X
__device__ __forceinline__ unsigned long long composite_key(uint32_t score_bits, uint32_t index) {
    return (static_cast<unsigned long long>(score_bits & 0x7fffffffu) << 32) |
           static_cast<unsigned long long>(~index);
}

// Entry e with dir[e].begin <= id < dir[e + 1].begin  (dir has n entries + a sentinel).
__device__ __forceinline__ uint32_t dir_lookup(const DirEntry *__restrict__ dir, uint32_t n,
                                               uint32_t id) {
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (dir[mid].begin <= id) lo = mid; else hi = mid;
    }
    return lo;
}

// The same from entry e, which lies at or before the wanted one: a workgroup's next item is often in
// the same layer or the next, but in a plan of many small layers it may lie hundreds of layers on --
// stepping there entry by entry is a chain of dependent loads that costs more than the tile itself.
__device__ __forceinline__ uint32_t dir_advance(const DirEntry *__restrict__ dir, uint32_t n, uint32_t e,
                                                uint32_t id) {
    if (id < dir[e + 1].begin) return e;
    ++e;
    if (id < dir[e + 1].begin) return e;
    return e + 1 + dir_lookup(dir + e + 1, n - (e + 1), id);    // (id < dir[n].begin, so e + 1 < n)
}

// Workgroups are handed to the 8 XCDs round-robin by id; give each XCD one contiguous
// range of tiles so that neighbouring tiles (which share halo rows/columns) meet in
// the same L2.
__device__ __forceinline__ uint32_t xcd_contiguous(uint32_t bid, uint32_t n) {
    const uint32_t xcd = bid & 7u, slot = bid >> 3;
    const uint32_t per = n >> 3, rem = n & 7u;
    return xcd * per + (xcd < rem ? xcd : rem) + slot;
}

// Inclusive scan over the NW * 64 threads of a workgroup.
template <int NW>
__device__ __forceinline__ uint32_t block_scan_incl_n(uint32_t v, uint32_t *wave_tot /*[NW]*/) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    if (lane == 63) wave_tot[wave] = v;
    __syncthreads();
    uint32_t add = 0;
#pragma unroll
    for (int w = 0; w < NW - 1; ++w)
        if (w < wave) add += wave_tot[w];
    const uint32_t r = v + add;
    __syncthreads();   // wave_tot may be reused by the caller
    return r;
}

// Position for one appended item per flagged lane: one atomic on the LDS counter per wave.
// Called by all 64 lanes of a wave; the result is meaningful for flagged lanes only.
__device__ __forceinline__ uint32_t wave_append(uint32_t *counter, bool flag) {
    const unsigned long long m = __ballot(flag);
    if (m == 0ull) return 0u;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t leader = static_cast<uint32_t>(__ffsll(static_cast<long long>(m))) - 1u;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, static_cast<uint32_t>(__popcll(m)));
    base = __shfl(base, static_cast<int>(leader), 64);
    return base + static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)));
}

// One more in bin b of a histogram in LDS for every flagged lane; the lanes whose bin is the first one's count with one atomic
// (masses of equal scores: 64 atomics on one address are served one after the other).
__device__ __forceinline__ void wave_count(uint32_t *h, uint32_t b, bool flag) {
    const unsigned long long m = __ballot(flag);
    if (m == 0ull) return;
    const uint32_t leader = static_cast<uint32_t>(__ffsll(static_cast<long long>(m))) - 1u;
    const uint32_t first = __builtin_amdgcn_readlane(b, leader);
    const unsigned long long same = __ballot(flag && b == first);
    if (flag && b != first) atomicAdd(&h[b], 1u);
    if ((threadIdx.x & 63u) == leader) atomicAdd(&h[first], static_cast<uint32_t>(__popcll(same)));
}

// Whether more than `limit` items have been appended to a stage in LDS (n: its counter): the same answer in every thread.
// The first barrier has all appends so far counted; the second keeps a wave that is already through from appending
// again before the last one has read the counter.
__device__ __forceinline__ bool staged_more_than(const uint32_t &n, uint32_t limit) {
    __syncthreads();
    const bool more = n > limit;
    __syncthreads();
    return more;
}

// Inclusive scan over the 256 threads of a workgroup (4 waves of 64).
__device__ __forceinline__ uint32_t block_scan_incl(uint32_t v, uint32_t *wave_tot /*[4]*/) {
    return block_scan_incl_n<4>(v, wave_tot);
}

// Safety margin (in log2 of the score) of a layer's first predicted bounds: the k-th largest of few
// scores moves more from call to call than that of many.
__device__ __forceinline__ float margin_init_log2(uint32_t k) {
    return fmaxf(kMarginInitLog2, 0.75f * rsqrtf(static_cast<float>(max(k, 1u))));
}

// ---------------------------------------------------------------- begin --
// When the plan's tables have been copied into a workspace, by whichever call comes first (k_begin): all workgroups
// but the last clear the histograms, counters and bitmasks; the last one writes every layer's initial selection state.
// After that every compress call leaves both as the next one needs them (prepare_next_call), so a call is the same
// whether it is enqueued or replayed from a graph, and whatever came before it.  A large layer gets its
// candidate bound here when the thresholds of its last two calls (kept in `pred`) lie close
// together.  While a residual builds up, the threshold keeps moving in one direction by steps
// that, on a logarithmic scale, shrink smoothly from call to call; so after a step d of
// log2(threshold) the next one is taken to lie between 0.6 d and 1.15 d, and the bound sits a
// margin below the lowest threshold that allows.  The margin doubles after a bound that lay too high
// and halves after one that lay too low (k_find0).
// The result of the call never depends on the bound -- only whether the layer has to be redone
// through the full map.  Without a usable history (first calls, after a failure, a threshold
// that jumps) the bound comes from a sample of this call's scores (k_hint) during the first
// calls with a workspace (`sampling`); later such a layer is ranked on the full map until its
// threshold has settled, and the call needs neither the sampled tiles nor k_hint.
// flags[0] tells the fallback kernels whether any large layer is on the full map.
// One layer's state; true: the layer starts on the full map for want of a bound.
__device__ __forceinline__ bool init_layer_state(const LayerDev *__restrict__ layers, SelState *__restrict__ state, int l,
                                                 PredState *__restrict__ pred /* nullable */, int sampling,
                                                 uint32_t last_path) {
    SelState s;
    const LayerDev L = layers[l];
    PredState ps = {};
    if (pred) ps = pred[l];              // (beside the layer's constants: with thousands of layers this chain is what the last kernel waits for)
    bool fallback_work = false;
    s.T = L.k == 0 ? ~0ull : 0ull;   // no key reaches ~0: nothing is selected when k = 0
    s.k_rem = L.k;
    s.done = L.k == 0 ? 1u : 0u;
    s.mode = L.k == 0 ? kModeSkip : (L.large ? kModeCandidates : kModeFullMap);
    s.hint_key = 0;
    s.overflow = 0;
    s.lo = 0;
    s.span = 0;
    s.predicted = last_path << kLastPathShift;
    if (pred && s.mode == kModeCandidates) {
        // after a failed bound the layer goes back to sampled bounds for a few calls -- where there
        // are any: past the calls that sample, the alternative would be the full map, and the
        // widened margin is tried at once
        const bool paused = ps.cooldown > 0 && (sampling || L.grid != 0u);
        // the call before failed: its threshold was a jump, not part of a trend -- the forecast
        // is that threshold itself
        const bool just_failed = ps.cooldown == kCooldownCalls;
        if (ps.cooldown > 0) ps.cooldown -= 1;
        ps.has_forecast = 0;
        bool predicted = false;
        if (ps.tau1 >= (1u << 23) && ps.tau2 >= (1u << 23)) {   // (both in the normal float32 range)
            const float l1 = __log2f(__uint_as_float(ps.tau1)), l2 = __log2f(__uint_as_float(ps.tau2));
            const float d = l1 - l2;
            const float dd = just_failed ? 0.f : fminf(fmaxf(d, -2.f * kTrendMaxLog2), kTrendMaxLog2);
            // the forecast is made in every call, used or not: how far the threshold then ends
            // below it is what sizes the margin (publish_threshold)
            ps.forecast = l1 + (dd > 0.f ? 0.6f * dd : 1.15f * dd);
            ps.has_forecast = 1;
            // (a threshold that jumps: sampled bounds while there are any; later the trend is
            // taken as far as it is trusted -- a bound that fails costs less than the full map)
            // (... except of a grid: its map costs it less than a bound that fails)
            if (!paused && (fabsf(d) <= kTrendMaxLog2 || (!sampling && !L.grid))) {   // (d, not dd: a jump is sampled)
                float margin = ps.margin > 0.f ? ps.margin : margin_init_log2(L.k);
                if (L.grid) margin = 2.f * margin + 0.03f;
                const float bound = exp2f(ps.forecast - margin);
                const uint32_t key = __float_as_uint(bound);
                if (key >= kPreF32MinKey && key <= kPreF32MaxKey) {   // (else: no bound, the full map)
                    s.hint_key = key;
                    predicted = true;
                }
            }
        }
        pred[l] = ps;
        if (predicted) {
            s.predicted |= 1u;
        } else if (!sampling) {
            s.mode = kModeFullMap;
            fallback_work = true;
        }
    }
    state[l] = s;
    return fallback_work;
}

// What the states hold before init_states writes them: nothing (fresh memory), what a compress call ends with, or the
// states of a call that has not been made.
enum StatesBefore : int { kStatesNone = 0, kStatesAfterCall = 1, kStatesBeforeCall = 2 };

// Every layer's state for the next call, by one workgroup of 256 threads.
__device__ __forceinline__ void init_states(const LayerDev *__restrict__ layers, SelState *__restrict__ state, int n_layers,
                                            PredState *__restrict__ pred, uint32_t *__restrict__ flags, int sampling,
                                            int before) {
    bool fallback_work = false;
    for (int l = threadIdx.x; l < n_layers; l += 256) {
        uint32_t last_path = 0;
        if (before != kStatesNone) {
            const SelState s = state[l];
            if (before == kStatesBeforeCall) last_path = s.predicted >> kLastPathShift;
            else last_path = s.mode == kModeCandidates && (s.predicted & 1u) ? 3u : s.mode;
        }
        fallback_work |= init_layer_state(layers, state, l, pred, sampling, last_path);
    }
    const int any = __syncthreads_or(fallback_work ? 1 : 0);
    if (threadIdx.x == 0) flags[0] = any ? 1u : 0u;
}

__global__ __launch_bounds__(256) void k_begin(uint4 *__restrict__ p, size_t n16,
                                               const LayerDev *__restrict__ layers,
                                               SelState *__restrict__ state, int n_layers,
                                               PredState *__restrict__ pred /* nullable */,
                                               uint32_t *__restrict__ flags, int sampling, int before) {
    if (blockIdx.x + 1 == gridDim.x) {
        init_states(layers, state, n_layers, pred, flags, sampling, before);
        return;
    }
    const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    const size_t stride = static_cast<size_t>(gridDim.x - 1) * 256;
    for (size_t j = i; j < n16; j += stride) p[j] = make_uint4(0, 0, 0, 0);
}

// What the last kernel of a call does for the next one, beside its own work: a launch of k_begin in front of every
// call cost 5 us on a small plan (of 76 on resnet18) and 8 us on VGG-19.  Every workgroup clears a share of the
// counters that no kernel of this call reads any more; one more workgroup (the grid's first: its chain of loads is
// longer than a chunk's) sets the layers' states.
struct NextCall {
    uint4 *zero[2];            // two runs of counters
    uint32_t n16[2];           // their lengths in 16-byte units
    const LayerDev *layers;
    SelState *state;
    PredState *pred;
    uint32_t *flags;
    int n_layers, sampling;    // sampling: whether the next call still samples bounds
};
// True: this workgroup was the extra one and is done.  (The others' chunk is blockIdx.x - 1.)
__device__ __forceinline__ bool prepare_next_call(const NextCall &nc) {
    if (blockIdx.x == 0) {
        init_states(nc.layers, nc.state, nc.n_layers, nc.pred, nc.flags, nc.sampling, kStatesAfterCall);
        return true;
    }
    const uint32_t stride = (gridDim.x - 1) * 256u;
#pragma unroll
    for (int r = 0; r < 2; ++r)
        for (uint32_t j = (blockIdx.x - 1) * 256u + threadIdx.x; j < nc.n16[r]; j += stride) nc.zero[r][j] = make_uint4(0, 0, 0, 0);
    return false;
}

// What one wave has written to LDS and reads back (its DS operations are carried out in order): keeps the compiler from
// moving the accesses of different lanes past each other.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// 16-byte store of data this call does not read again (the new residual / momentum arena):
// marked non-temporal so that it does not displace the halo rows and candidate slots that
// later tiles and kernels find in cache (measured: -12 us on the VGG-19 main pass).
__device__ __forceinline__ void store_streaming(float *__restrict__ dst, const float4 v) {
    typedef float vf4 __attribute__((ext_vector_type(4)));
    const vf4 vv = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(vv, reinterpret_cast<vf4 *>(dst));
}

// 16-byte load of data no other workgroup reads and this one reads once: marked non-temporal,
// so that it does not displace what is reused (measured: -8 % on the block-score pass).
__device__ __forceinline__ float4 load_streaming(const float *__restrict__ src) {
    typedef float vf4 __attribute__((ext_vector_type(4)));
    const vf4 t = __builtin_nontemporal_load(reinterpret_cast<const vf4 *>(src));
    return make_float4(t.x, t.y, t.z, t.w);
}

// A float that is the same in every lane, moved to a scalar register.
__device__ __forceinline__ float uniform_f32(float x) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// Eqs. 8-10 from the window sums sa = sum|w|, ss = sum w, sq = sum w^2 (n = p*p slots):
//   mean = sa / n,  std = sqrt(d) / n  with  d = n*sq - ss^2 = n^2 * variance,
//   NSI = alpha*mean + (1-alpha)*std = ca*sa + cb*sqrt(d).
// d is formed from two separately rounded products.  That form cancels: its absolute error
// is a few 1e-16 of n*sq, so the relative error of the standard deviation grows like
// 1e-16 * (1 + mean^2 / variance).  A window whose d falls below kCancelFrac * n*sq
// (|mean| beyond a thousand standard deviations: near-constant values on a large offset)
// is therefore evaluated again the way Eq. 10 is printed -- window_ssd below -- and only the
// others (relative error of the one-pass form below 3e-9) keep the one-pass value.
constexpr double kCancelFrac = 1.0 / 1048576.0;

// The main pass rules out the centres below the bound in float32 (half the registers of the same
// test in double, no conversions).  It must never rule out a centre that
// the evaluation in full would record, so every float32 quantity is bounded against the exact one.
// With u = 2^-24, n = p*p, exact window sums SA = sum|w|, SS = sum w, SQ = sum w^2, D = n SQ - SS^2
// (SA^2 <= n SQ, |SS| <= SA), and a bound B in [2^-40, 2^40] (nothing of weight under- or overflows):
//   sa = SA (1 + t), |t| <= (n-1) u          (non-negative terms)
//   ss is off by at most (n-1) u SA, so ss^2 <= SS^2 + (2n - 1.9) u * n SQ; sq >= SQ (1 - n u);
//   rest = B' - ca sa with B' = B * kBoundFactor = B (1 - 2^-22 - 2.04 n u), rounded down: at most the exact
//     B (1 - 2^-22) - ca SA whenever ca SA < 2 B, and negative otherwise;
//   e = A sq - (cb ss)^2, one fma of two rounded products, with A = cb^2 n (1 + kSlack) (1 + 2e-6) rounded up: the roundings
//     of cb, of both products and of sq and ss take away less than (3n + 3.5) u * cb^2 n SQ, and kSlack = 1.3 (3n + 3) u is more,
//     so e >= cb^2 D (1 + 1.9e-6) (as D <= n SQ);
//   the centre stays unless e < t^2 with t = max(rest, 0): a centre that reaches B has cb^2 D >= (B (1 - 2^-22) - ca SA)^2 >= t^2
//     exactly, or t = 0, and the roundings of e and t^2 are less than 1.9e-6.
// The comparison is written so that a NaN on either side keeps the centre (the maximum takes the 0), and an infinite sum does:
// such windows are left to the evaluation in full.  Squares of values below 2^-63 underflow; what is
// lost (below 2^-126 each) is far less than either slack for a bound of at least 2^-40.  Outside
// that range no bound is handed out: the layer is ranked on the full map (k_begin, k_hint).
// Seven operations.  With d and rest scaled apart and compared in two steps (twelve, and beside them the test of the matrix's
// edges, which is left to the evaluation in full now) the main pass took 234 us on 25088 x 4096 with p = 5, now 216; with p = 7 on 38 M
// elements 92.6, now 86.2; VGG-19, which the streaming bounds, 312 -> 307 on one step repeated and no less on a carried residual (315,
// 319), where it stores no v 255 -> 246.
template <int P> struct PreF32 {
    static constexpr float kSlack = 1.3f * (3.f * P * P + 3.f) * 5.9604645e-8f;
    static constexpr double kBoundFactor = 1.0 - 1.0 / 4194304.0 - 2.04 * (P * P) * 5.9604645e-8;
    __device__ static __forceinline__ float square_factor(double cb) {                       // A
        return __double2float_ru(cb * cb * static_cast<double>(P * P) * (1.0 + static_cast<double>(kSlack)) * (1.0 + 2e-6));
    }
    __device__ static __forceinline__ float bound(float b) { return __double2float_rd(static_cast<double>(b) * kBoundFactor); }        // B'
    // Whether the centre stays, from its window's sums.
    __device__ static __forceinline__ bool stays(float sa, float ss, float sq, float ca, float cb, float a, float b) {
        const float m = cb * ss, e = fmaf(-m, m, a * sq);
        const float t = fmaxf(fmaf(-ca, sa, b), 0.f);
        return !(e < t * t);
    }
};

// Sums over P neighbours of a row.
template <int P>
__device__ __forceinline__ void row_sums(const float *row, float &sa, float &ss, float &sq) {
    sa = fabsf(row[0]);
    ss = row[0];
    sq = row[0] * row[0];
#pragma unroll
    for (int j = 1; j < P; ++j) {
        sa += fabsf(row[j]);
        ss += row[j];
        sq = fmaf(row[j], row[j], sq);
    }
}
// Sums of the last P row sums of a column, row by row (P compile-time indices: all of it in registers).  Pairs and pairs of
// pairs are kept and shared by the windows: P = 5 takes three additions a row instead of four, P = 7 four instead of six (the main
// pass with p = 7 on 38 M elements: 86.2 us without, 84.9 with).
template <int P>
struct ColumnSums {
    static_assert(P == 3 || P == 5 || P == 7, "single elements have no windows");
    float s[8], p[8], c[8];               // of row i (at i % 8): its sum, with the row before, with the three before
    __device__ __forceinline__ void push(int i, float row) {
        s[i & 7] = row;
        if (i >= 1) p[i & 7] = s[(i - 1) & 7] + row;
        if (P == 7 && i >= 3) c[i & 7] = p[(i - 2) & 7] + p[i & 7];
    }
    __device__ __forceinline__ float window(int i) const {
        if (P == 3) return s[(i - 2) & 7] + p[i & 7];
        if (P == 5) return (p[(i - 3) & 7] + p[(i - 1) & 7]) + s[i & 7];
        return (c[(i - 3) & 7] + p[(i - 1) & 7]) + s[i & 7];
    }
};

// With v in place of the residual the main pass may not read what another workgroup's tile holds: its neighbours may have their
// v there already or not.  A workgroup takes kRun tiles at a time, one below the other where the layer's tiles divide so, and carries the
// last rows of one into the windows of the next; the windows that still reach into another tile are left to k_seams.
constexpr uint32_t kRun = 2;
// A layer's tile number `listed` in that order, number t of the launch.
struct RunTile {
    int trow, tcol;
    bool above, below;                     // whether the tile on that side is taken with it
    __device__ __forceinline__ RunTile(const LayerDev &L, uint32_t listed, uint32_t t) {
        const uint32_t band = listed / (kRun * L.tiles_x), rest = listed - band * kRun * L.tiles_x;
        const uint32_t rows = min(kRun, L.n_tiles / L.tiles_x - band * kRun), col = rest / rows, i = rest - col * rows;
        trow = static_cast<int>(band * kRun + i);
        tcol = static_cast<int>(col);
        above = i != 0u && t % kRun != 0u;
        below = i + 1u < rows && (t + 1u) % kRun != 0u;
    }
};
// The positions of such a tile that are left: along its edges, where there is another tile or -- the main pass ends H rows
// before it -- the matrix's lower edge.
template <int H>
struct TileSeams {
    bool top, bottom, left, right;
    __device__ __forceinline__ TileSeams(const RunTile &rt, int R, int C)
        : top(rt.trow > 0 && !rt.above), bottom(rt.trow * kTileRows + kTileRows - H < R && !rt.below), left(rt.tcol > 0),
          right((rt.tcol + 1) * kTileCols < C) {}
    __device__ __forceinline__ bool on_column(int col) const { return (col < H && left) || (col >= kTileCols - H && right); }
};

// Centres one tile can queue for full evaluation: twice the largest slot, and the positions beyond the matrix's edge whose windows
// reach into it (the test in the sweep does not ask where a position lies).
template <int P> constexpr int kQueueCap = 1024 + (P - 1) / 2 * (kTileCols + kTileRows);

__device__ __forceinline__ double var_n2_one_pass(double ss, double nsq) {
    return __dsub_rn(nsq, __dmul_rn(ss, ss));
}

// Eq. 10 as printed, for the rare window where the one-pass form cancels: the sum over the
// P x P window at `win` (LDS, row pitch `pitch`) of (w - m)^2, rows top to bottom, left to right.
// Equal windows give equal bits wherever they lie, and a constant window gives exactly 0
// (m = P*P*c / (P*P) is exact), which the ranking's tie rule relies on.  Loops are kept rolled:
// this is cold code inside an unrolled loop.
template <int P>
__device__ __forceinline__ double window_ssd(const float *win, int pitch, double m) {
    double acc = 0.0;
#pragma unroll 1
    for (int dx = 0; dx < P; ++dx) {
#pragma unroll 1
        for (int dy = 0; dy < P; ++dy) {
            const double e = static_cast<double>(win[dx * pitch + dy]) - m;
            acc += __dmul_rn(e, e);
        }
    }
    return acc;
}

// ca*sa + cb*sqrt(d).  The square root is one v_rsq_f64 seed, one coupled Newton step and one
// residual correction (about 1 ulp in double); the floor 1e-300 stands in for 0 and vanishes
// when the score is rounded to float32.
__device__ __forceinline__ double nsi_from_var(double sa, double d, double ca, double cb) {
    d = fmax(d, 1e-300);
    const double y = __builtin_amdgcn_rsq(d);
    double g = d * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    const double e = fma(-g, g, d);
    g = fma(e, h, g);
    return fma(cb, g, ca * sa);
}

// A window's score as float32 bits, from its sums; Eq. 10 again from the window where the one-pass variance cancels (never for
// P = 1, where it is 0 by definition).
template <int P>
__device__ __forceinline__ uint32_t score_from_sums(double sa, double ss, double sq, const float *win, int pitch, double ca, double cb) {
    const double n = static_cast<double>(P * P), nsq = __dmul_rn(n, sq);
    double d = var_n2_one_pass(ss, nsq);
    if (P > 1 && d < kCancelFrac * nsq) d = __dmul_rn(n, window_ssd<P>(win, pitch, ss / n));
    return __float_as_uint(static_cast<float>(nsi_from_var(sa, d, ca, cb))) & 0x7fffffffu;
}
// The score of one window in full: Eqs. 8-10 in double, the sums row by row.  (Rows kept rolled: few registers that way.)
template <int P>
__device__ __forceinline__ uint32_t window_score(const float *win, int pitch, double ca, double cb) {
    double sa = 0.0, ss = 0.0, sq = 0.0;
#pragma unroll 1
    for (int dx = 0; dx < P; ++dx) {
        const double w0 = static_cast<double>(win[dx * pitch]);
        double ra = fabs(w0), rs = w0, rq = w0 * w0;
#pragma unroll
        for (int j = 1; j < P; ++j) {
            const double wj = static_cast<double>(win[dx * pitch + j]);
            ra += fabs(wj);
            rs += wj;
            rq = fma(wj, wj, rq);
        }
        if (dx == 0) { sa = ra; ss = rs; sq = rq; }
        else { sa += ra; ss += rs; sq += rq; }
    }
    return score_from_sums<P>(sa, ss, sq, win, pitch, ca, cb);
}

// ----------------------------------------------------------- work feed --
// Hands the items of a launch (tiles) to its persistent workgroups.  With a fixed strided
// share per workgroup the workgroups drift apart (measured on the VGG-19 main pass: the first
// leaves at 240 us, the mean at 310, the last at 390); here every workgroup takes its next item
// from a counter when it is ready.
//
// Locality is kept: the items are cut into stretches of 8 * S consecutive items, part d of
// every stretch belongs to domain d (one per XCD: workgroups are handed to the XCDs
// round-robin by id), and a domain's counter walks its parts in order -- so at any moment an
// XCD's workgroups hold consecutive items (neighbouring tiles share halo rows in that XCD's
// L2), and a counter's cache line stays in that XCD's L2.  A workgroup leaves when its own
// domain is used up: taking from other domains was measured too (in ring order, or from the
// fullest), and the tickets it costs on other XCDs' counters outweigh the better balance.
//
// The ticket for the item after the current one is requested (one atomic by thread 0) when the
// current item starts and read when it ends, so its latency is hidden.
constexpr uint32_t kNoItem = 0xffffffffu;
constexpr int kFeedDomains = 8;
constexpr int kFeedStride = 32;          // uint32 between two counters (one 128-byte line each)
constexpr int kFeedSets = 16;            // counter sets per call: (pass, p-group) pairs

// Items of domain d: part d of every full stretch, and its share of the last, partial one.
__device__ __forceinline__ uint32_t feed_domain_items(uint32_t n_items, uint32_t shift, uint32_t d) {
    const uint32_t S = 1u << shift;
    const uint32_t full = n_items >> (shift + 3), rem = n_items & ((S << 3) - 1u);
    const uint32_t lo = d << shift;
    return (full << shift) + (rem > lo ? min(rem - lo, S) : 0u);
}

struct WorkFeed {
    uint32_t *ctr;        // the workgroup's domain counter (zero at launch)
    uint32_t items;       // items of that domain
    uint32_t shift, dom;
    uint32_t par;         // LDS slot of the next hand-over
    bool stashed;         // the requested ticket is already in that slot
    uint32_t pending;     // thread 0: the ticket requested last
    // (plain members whose values the compiler can follow through the loop: with the flags
    // packed into one word the main pass needed 15 more registers)

    // Thread 0 puts the requested ticket into LDS.  Reading it waits for the wave's memory
    // operations up to the request, and the compiler may make that a wait for everything
    // issued since.  So the item's code calls this after its loads have arrived and before
    // its first store; next() does it for items that never got there.
    __device__ __forceinline__ void stash(uint32_t *slot /*[2], LDS*/) {
        if (!stashed && threadIdx.x == 0) slot[par] = pending;
        stashed = true;
    }
    // Called by all threads of the workgroup (it contains a barrier); returns the next item or
    // kNoItem.
    __device__ __forceinline__ uint32_t next(uint32_t *slot) {
        if (!stashed && threadIdx.x == 0) slot[par] = pending;
        stashed = false;
        __syncthreads();
        const uint32_t t = __builtin_amdgcn_readfirstlane(slot[par]);   // the same in every lane: keep it scalar
        par ^= 1u;
        if (t >= items) return kNoItem;                 // uniform: the domain is used up
        if (threadIdx.x == 0) pending = atomicAdd(ctr, 1u);
        return ((t >> shift) * kFeedDomains + dom) * (1u << shift) + (t & ((1u << shift) - 1u));
    }
    // counters: the launch's kFeedDomains counters; log2_part: log2 S.
    __device__ __forceinline__ uint32_t first(uint32_t *__restrict__ counters, uint32_t n_items, uint32_t log2_part,
                                              uint32_t *slot) {
        dom = blockIdx.x % kFeedDomains;                // workgroups go to the XCDs round-robin by id
        shift = log2_part;
        items = feed_domain_items(n_items, shift, dom);
        ctr = counters + dom * kFeedStride;
        par = 0;
        stashed = false;
        pending = kNoItem;                              // an empty domain never touches its counter
        if (threadIdx.x == 0 && items != 0u) pending = atomicAdd(ctr, 1u);
        return next(slot);
    }
};

// ------------------------------------------------------------------ nsi --
// What one launch of the NSI kernel produces.
enum NsiPass : int {
    kPassMapOnly = 0,   // score map to a caller buffer (rsdgc_nsi)
    kPassFullMap = 1,   // score map + 12-bit histogram of the large layers that fell back to the full map
    kPassCapture = 2,   // candidates (score >= bound) recorded per tile, layers in candidate mode
    kPassSample = 3,    // first pass over the plan's tile list: 12-bit histogram of the sampled tiles
                        // of the large layers; score map + histogram of every tile of the others
    kPassCaptureInPlace = 4,    // kPassCapture where v replaces the residual: windows inside a tile only (the others: k_seams)
};
constexpr bool pass_captures(int pass) { return pass == kPassCapture || pass == kPassCaptureInPlace; }

struct NsiArgs {
    const LayerDev *layers;
    const DirEntry *dir;          // tile directory of the launch (kPassMapOnly, and with the work feed)
    uint32_t n_dir;
    uint32_t n_tiles;
    const SampleEntry *samples;   // the launch's tiles (kPassSample; the large layers' passes without the work feed)
    const float *grad;
    const float *resid;           // nullable: all-zero residual
    float *nsi_out;               // score map (kPassMapOnly, kPassFullMap; kPassSample: of the layers that are always ranked on it)
    float *v_out;                 // nullable: second residual arena that receives v = r + g (kPassCaptureInPlace: the residual's own)
    int v_in_place;               // the layers' v has replaced the residual where the main pass took them (kPassFullMap: it is read there)
    const float *mom;             // nullable: momentum arena u (Eq. 12, first line); then v = r + (m*u + g)
    float *mom_out;               // with mom: receives m*u + g wherever v_out receives v
    float m;                      // momentum factor
    const uint32_t *flags;        // [0] != 0: some large layer fell back to the full map
    uint32_t *hist;               // [n_layers][kHistBins]
    uint32_t *hist_s;             // [n_layers][kHistBins]  scores of the sampled tiles of the large layers; main pass: fine bins
    uint32_t *list_cnt;           // main pass: adds up a layer's candidates in word 1 of its shards' lines
    int n_layers;
    const SelState *state;
    SelState *state_rw;           // same array; the main pass sets the overflow flag
    uint32_t *slot_cnt;           // [n_tiles_all]
    unsigned long long *slot_ent; // per large layer n_tiles slots of slot_cap entries, from the layer's slot_off
    double ca, cb;                // alpha / p^2, (1 - alpha) / p^2: NSI = ca * sum|w| + cb * sqrt(p^2 * sum w^2 - (sum w)^2)
    uint4 *counts;                // main pass: chunk counters that it clears where k_select follows (no launch of k_find0 does)
    uint32_t n16;
    uint32_t *feed;               // work-feed counters of this launch (all but kPassMapOnly)
    uint32_t feed_shift;          // log2 of the items per domain and stretch
};

// Bucket that holds the k-th largest entry of a 4096-bucket histogram h (completed by an earlier
// launch), walking down from the top bucket.  One wave; every lane returns the same result
// (found = 0 when the histogram holds fewer than k entries).  Cold code inside hot kernels: its
// loops stay rolled so that it needs next to no registers.
struct WaveBucket {
    uint32_t bucket, above, count, found;
};
__device__ __forceinline__ WaveBucket wave_find_bucket(const uint32_t *__restrict__ h, uint32_t k) {
    const int lane = threadIdx.x & 63;
    constexpr int per = kHistBins / 64;
    const int hi = kHistBins - lane * per;              // lane 0 holds the top buckets
    uint32_t own = 0;
#pragma unroll 1
    for (int b = hi - 1; b >= hi - per; --b) own += h[b];
    uint32_t incl = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    const uint32_t excl = incl - own;
    WaveBucket r = {0u, 0u, 0u, 0u};
    const bool mine = excl < k && k <= incl;
    if (mine) {
        uint32_t acc = excl;
#pragma unroll 1
        for (int b = hi - 1; b >= hi - per; --b) {
            const uint32_t c = h[b];
            if (acc + c >= k) {
                r.bucket = static_cast<uint32_t>(b);
                r.above = acc;
                r.count = c;
                break;
            }
            acc += c;
        }
    }
    const unsigned long long who = __ballot(mine);
    if (who == 0ull) return r;
    const int src = __ffsll(static_cast<long long>(who)) - 1;
    r.bucket = __shfl(r.bucket, src, 64);
    r.above = __shfl(r.above, src, 64);
    r.count = __shfl(r.count, src, 64);
    r.found = 1u;
    return r;
}

// Where a workgroup adds the candidates it recorded of a layer: word 1 of one of the first kRecordedParts list shards' lines
// (several, as all workgroups of a launch end at about the same time).
constexpr uint32_t kRecordedParts = 4;
__device__ __forceinline__ uint32_t *recorded_slot(uint32_t *list_cnt, uint32_t layer, uint32_t wg) {
    return list_cnt + (static_cast<size_t>(layer) * kListShards + (wg % kRecordedParts)) * kListCntStride + 1;
}

// Whether a large layer is ranked on the full map in this call: it started so, or its bound failed -- fewer than k_l
// centres reach it, k_l or more lie in the open-ended top bin, or a tile slot overflowed.  k_find0's test, from what the
// main pass has left, for workgroups of its own launch (which may see the mode before or after k_find0 has changed it).
__device__ __forceinline__ bool layer_falls_back(const LayerDev *__restrict__ layers, const SelState *state, const uint32_t *__restrict__ hist_s,
                                                 uint32_t *list_cnt, uint32_t l) {
    const SelState *st = state + l;
    const uint32_t mode = st->mode, hint_key = st->hint_key, overflow = st->overflow;
    const uint32_t large = layers[l].large, k = layers[l].k;
    const uint32_t top = hist_s[static_cast<size_t>(l) * kHistBins + kFineBins - 1];
    uint32_t recorded = 0;
#pragma unroll
    for (uint32_t q = 0; q < kRecordedParts; ++q) recorded += *recorded_slot(list_cnt, l, q);
    if (large == 0u || mode == kModeSkip) return false;
    return mode == kModeFullMap || hint_key == 0u || overflow != 0u || recorded < k || top >= k;
}

// Beside them (below: k_seams) the main pass keeps the first and the last few columns of every tile row in the layer's part of the
// score map, which is free while the layer is on the candidate path: out of the matrix they would be a cache line each.
template <int P> constexpr int kSeamCols = P <= 5 ? 4 : 8;           // at least P - 1
template <int P>
__device__ __forceinline__ float *seam_columns(float *map, const LayerDev &L, int x, int tcol, int side) {
    return map + L.elem_off + (static_cast<size_t>(2 * tcol + side) * L.R + x) * kSeamCols<P>;
}

// Whether the main pass takes a layer with this candidate bound (0: none).  It stays as it is from the main pass to the emit.
__device__ __forceinline__ bool bound_in_range(uint32_t hint_key) { return hint_key >= kPreF32MinKey && hint_key <= kPreF32MaxKey; }

// Work unit: one 16 x 256 tile of one layer.  The tile of v = r + g plus a halo of
// h = (P-1)/2 rows and 4 columns (16-byte aligned) goes to LDS; each thread then walks
// down the 16 rows of one column, keeping per-row horizontal sums of |w|, w and w^2
// for the last P rows in registers.  Every score that is stored, counted or recorded is
// computed in double: the variance as (P^2 * sum w^2 - (sum w)^2) / P^4, or -- where that
// form cancels -- from the tile again as Eq. 10 prints it; either way equal windows get
// equal scores wherever they lie and a constant window gets a variance of exactly 0.  The
// main pass (capture) runs the sweep in float32 instead and only decides there which centres
// cannot reach the layer's bound (PreF32 above); the others it evaluates in double as said.
// The capture variants are held to five waves per SIMD for p <= 3 and four for p = 5, 7
// (what their registers allow without spilling; measured faster than one wave less), those with momentum to
// three: 485 us on VGG-19, with four, which 128 registers would allow p = 3, 497, with two 527.
//
// A workgroup takes tiles b, b + W, ... of the launch (W workgroups, laid out so that each XCD
// gets one contiguous part of every stretch of W tiles: neighbouring tiles share halo rows in
// one L2), or -- FEED -- whatever the launch's work feed hands it next.  Its LDS histogram is
// flushed to the layer's global histogram only when the layer changes or its tiles end, so
// a launch issues few same-address global atomics.
// MOM: with Eq. 12's momentum term (a.mom, a.mom_out, a.m).  FEED: the workgroups take their
// tiles from the launch's work feed instead of a fixed strided share.
template <int P, int PASS>
struct NsiShared {
    static constexpr bool kCapture = pass_captures(PASS);
    static constexpr int kBins = PASS == kPassFullMap || PASS == kPassSample ? kHistBins : (kCapture ? kFineBins : 1);
    __attribute__((aligned(16))) float tile[(kTileRows + P - 1) * (kTileCols + 8)];
    unsigned long long cand[kCapture ? kSlotCapMax : 1];
    uint32_t lhist[kBins];
    uint16_t queue[kCapture ? kQueueCap<P> : 1];
    uint32_t ncand, nqueue;
    uint32_t nabove;                      // kPassCaptureInPlace: candidates in the tile above
    uint32_t feed_slot[2];
};

// wg, n_wgs: the workgroup's number among those of this pass, and how many they are.  WITH_FIND0: the fallback pass
// in one launch with k_find0 -- it cannot wait for the flag and looks at the layers itself (at most 256 of them).
template <int P, int PASS, bool MOM, bool FEED, bool WITH_FIND0 = false>
__device__ __forceinline__ void nsi_pass(const NsiArgs &a, NsiShared<P, PASS> &sh, uint32_t wg, uint32_t n_wgs) {
    constexpr int H = (P - 1) / 2;
    constexpr int ROWS = kTileRows + 2 * H;
    constexpr int PADL = 4;
    constexpr int PITCH = kTileCols + 2 * PADL;   // 264 floats
    // One column per thread (two adjacent columns would share LDS reads, but the second set of row
    // sums costs 18 registers and a wave per SIMD).
    constexpr int RPT = kTileRows * kTileCols / 256;           // output rows per thread
    constexpr bool MAP = PASS == kPassMapOnly || PASS == kPassFullMap;
    constexpr bool CAPTURE = pass_captures(PASS), IN_PLACE = PASS == kPassCaptureInPlace;
    constexpr bool FULLHIST = PASS == kPassFullMap || PASS == kPassSample;
    constexpr bool STORE_V = PASS != kPassMapOnly;
    constexpr int NBINS = NsiShared<P, PASS>::kBins;
    float *const tile = sh.tile;
    uint32_t *const lhist = sh.lhist;
    unsigned long long *const cand = sh.cand;
    uint16_t *const queue = sh.queue;
    uint32_t &ncand = sh.ncand, &nqueue = sh.nqueue;
    uint32_t *const feed_slot = sh.feed_slot;

    const int tid = threadIdx.x;
    // the launch's work items (tiles, or sampled tiles): at any moment the resident workgroups
    // work on one compact stretch of tiles, so neighbouring tiles' halo rows are still in
    // cache; inside a stretch each XCD takes one contiguous part
    const uint32_t n_items = IN_PLACE ? (a.n_tiles + kRun - 1u) / kRun : a.n_tiles;
    const uint32_t stride = n_wgs;
    if (PASS == kPassFullMap) {            // no layer fell back: nothing to do
        if (WITH_FIND0) {
            if (!__syncthreads_or(tid < a.n_layers && layer_falls_back(a.layers, a.state, a.hist_s, a.list_cnt, tid))) return;
        } else if (a.flags[0] == 0u) {
            return;
        }
    }
    if (CAPTURE && !FEED)                  // (the last kernel of the call before still read them)
        for (uint32_t j = wg * 256u + tid; j < a.n16; j += n_wgs * 256u) a.counts[j] = make_uint4(0, 0, 0, 0);
    WorkFeed feed;
    uint32_t first;
    if (FEED) {
        first = feed.first(a.feed, n_items, a.feed_shift, feed_slot);
        if (first == kNoItem) return;      // uniform
    } else {
        first = xcd_contiguous(wg, n_wgs);
        if (first >= n_items) return;
    }

    if (NBINS > 1)
        for (int b = tid; b < NBINS; b += 256) lhist[b] = 0;
    if (CAPTURE && tid == 0) { ncand = 0; nqueue = 0; }
    if (IN_PLACE && tid == 0) sh.nabove = 0;
    if (IN_PLACE)                          // (no halo is loaded: the columns beside the tile's own stay as they are)
        for (int j = tid; j < ROWS * PITCH; j += 256) tile[j] = 0.f;
    __syncthreads();

    // Where the next tile is known beforehand its list entry is requested a tile ahead: a first tile costs one load where
    // the directory takes a bisection (161 layers: 34.2 -> 32.2 us; 21 layers: no difference).  With the work
    // feed the directory's neighbouring entry, usually cached, is the shorter way.
    constexpr bool LISTED = !FEED && PASS != kPassMapOnly && !IN_PLACE;
    uint32_t e = 0;                       // directory entry of the current layer
    SampleEntry ahead = {0u, 0u};
    if (LISTED) ahead = a.samples[first];
    else e = dir_lookup(a.dir, a.n_dir, IN_PLACE ? first * kRun : first);
    uint32_t cur_l = 0xffffffffu;         // layer whose counts sit in lhist
    uint32_t hint_key = 0;
    uint32_t *hist_base = CAPTURE ? a.hist_s : a.hist;         // first pass: a.hist_s for the sampled tiles of a large layer
    uint32_t recorded = 0;                // main pass: the workgroup's candidates of layer cur_l
    bool active = true;
    bool whole = true;                    // every tile of the layer is visited: v and the scores go out
    bool v_stored = false;                // kPassFullMap: the layer's residual holds v already
    LayerDev L;

    const double n = static_cast<double>(P * P);
    // (kernel arguments: the same in every lane, so they stay in scalar registers -- the scalar unit
    // has no floating point, a uniform value computed here would occupy vector registers)
    const double ca = a.ca, cb = a.cb;
    const float caf = uniform_f32(static_cast<float>(ca)), cbf = uniform_f32(static_cast<float>(cb));
    const float pre_a = uniform_f32(PreF32<P>::square_factor(cb));
    float bound_lof = 0.f;                // capture: a conservative form of the candidate bound (PreF32)
    static_assert(kTileCols * (kTileRows / RPT) == 256, "one thread per RPT rows of one column");
    const int c0 = tid % kTileCols, ty = tid / kTileCols;
    const int row_base = ty * RPT;

    // (IN_PLACE: an item is a run of tiles, of which t is one)
    uint32_t run = first;
    float carry[H > 0 ? 2 * H : 1] = {};  // ... the last rows of the tile above: the thread's column
    uint32_t n_above = 0;                 // ... and its candidates
    auto after = [&](uint32_t t) {
        if (IN_PLACE && (t + 1u) % kRun != 0u && t + 1u < a.n_tiles) return t + 1u;
        if (!IN_PLACE) return FEED ? feed.next(feed_slot) : t + stride;
        run = FEED ? feed.next(feed_slot) : run + stride;
        return FEED && run == kNoItem ? kNoItem : run * kRun;
    };
    for (uint32_t t = IN_PLACE ? first * kRun : first; FEED ? t != kNoItem : t < a.n_tiles; t = after(t)) {
        uint32_t l, local;
        if (LISTED) {
            l = ahead.layer;
            local = ahead.local_tile;
            if (t + stride < n_items) ahead = a.samples[t + stride];
        } else {
            e = dir_advance(a.dir, a.n_dir, e, t);
            l = a.dir[e].layer;
            local = t - a.dir[e].begin;
        }
        if (l != cur_l) {
            if (NBINS > 1 && cur_l != 0xffffffffu && active) {   // flush the finished layer's counts
                uint32_t *__restrict__ gh = hist_base + static_cast<size_t>(cur_l) * kHistBins;
                for (int b = tid; b < NBINS; b += 256) {
                    const uint32_t c = lhist[b];
                    if (c) { atomicAdd(&gh[b], c); lhist[b] = 0; }
                }
                if (CAPTURE && tid == 0 && recorded) atomicAdd(recorded_slot(a.list_cnt, cur_l, wg), recorded);
                recorded = 0;
                __syncthreads();
            }
            cur_l = l;
            L = a.layers[l];
            active = true;
            hint_key = 0;
            whole = PASS != kPassSample || L.large == 0u;
            if (PASS == kPassFullMap || CAPTURE || (PASS == kPassSample && !whole)) {
                const SelState st = a.state[l];
                if (PASS == kPassFullMap) active = WITH_FIND0 ? layer_falls_back(a.layers, a.state, a.hist_s, a.list_cnt, l) : st.mode == kModeFullMap && L.large != 0u;
                else if (PASS == kPassSample) active = st.mode == kModeCandidates && st.hint_key == 0u;   // no predicted bound
                else active = st.mode == kModeCandidates;
                if (PASS == kPassFullMap) v_stored = a.v_in_place && bound_in_range(st.hint_key);
                if (CAPTURE) {
                    hint_key = st.hint_key;
                    bound_lof = uniform_f32(PreF32<P>::bound(__uint_as_float(hint_key)));
                    // (k_begin and k_hint give no bound outside the range of the float32 test; should one
                    // arrive all the same, the layer is not captured and k_find0 sends it to the full map)
                    if (active && !bound_in_range(hint_key)) {
                        active = false;
                        if (tid == 0 && hint_key != 0u) a.state_rw[l].overflow = 1u;
                    }
                }
            }
            if (PASS == kPassSample) hist_base = whole ? a.hist : a.hist_s;
        }
        if (!active) {                    // skip the rest of this layer
            if (!FEED && !LISTED && !IN_PLACE) {
                const uint32_t nb = a.dir[e + 1].begin;          // first tile of the next layer
                t += (nb - t + stride - 1) / stride * stride - stride;   // loop increment adds the last stride
            }
            continue;
        }

        int trow = static_cast<int>(local / L.tiles_x);
        int tcol = static_cast<int>(local - static_cast<uint32_t>(trow) * L.tiles_x);
        bool above = false;               // IN_PLACE: the tile before was the one above
        float bound_above = bound_lof, bound_top = bound_lof, bound_rest = bound_lof;      // infinite where the windows are k_seams'
        const int R = static_cast<int>(L.R), C = static_cast<int>(L.C);
        if constexpr (IN_PLACE) {
            const RunTile rt(L, local, t);
            const TileSeams<H> seam(rt, R, C);
            trow = rt.trow;
            tcol = rt.tcol;
            local = static_cast<uint32_t>(trow) * L.tiles_x + static_cast<uint32_t>(tcol);
            above = rt.above;
            const float never = __uint_as_float(0x7f800000u);
            if (seam.on_column(c0)) bound_rest = never;
            bound_above = above ? bound_rest : never;
            bound_top = seam.top ? never : bound_rest;
#pragma unroll
            for (int i = 0; i < 2 * H; ++i) tile[i * PITCH + PADL + c0] = above ? carry[i] : 0.f;
        }
        const int x0 = trow * kTileRows, y0 = tcol * kTileCols;
        const float *__restrict__ g = a.grad + L.elem_off;
        const float *__restrict__ r = a.resid ? a.resid + L.elem_off : nullptr;

        // ---- load v = r + g for the tile and its halo; zero outside the matrix
        if ((C & 3) == 0) {
            // The tile's own 256 columns: wave w takes rows w, w + 4, ... of the tile and its row
            // halo, lane j the 16 bytes at column 4 j -- 1 KB per wave and row, and next to no
            // index arithmetic (a flat split of the tile into 16-byte pieces needs a division per
            // piece, which the compiler computes once and then keeps in a dozen registers).  The
            // column halo, H floats on either side of every row, is loaded as single floats by the
            // first 2 H ROWS threads.
            constexpr int ROW0 = IN_PLACE ? H : 0;             // rows loaded, from the halo's first on; rows further down that they lie in LDS
            constexpr int ROW1 = IN_PLACE ? H + kTileRows : ROWS, DOWN = IN_PLACE ? H : 0;
            constexpr int ITER = (ROW1 - ROW0 + 3) / 4;
            const int wave = tid >> 6, lane = tid & 63;
            const int ym = y0 + 4 * lane;
            const int hrow = H > 0 ? tid / (2 * H > 0 ? 2 * H : 1) : 0;
            const int hc = H > 0 ? tid - hrow * 2 * H : 0;              // 0 .. H-1 left of the tile, H .. 2H-1 right of it
            const int hy = hc < H ? y0 - 1 - hc : y0 + kTileCols + (hc - H);
            const int hx = x0 - H + hrow;
            const bool halo_thread = !IN_PLACE && H > 0 && tid < 2 * H * ROWS;
            const bool halo_in = halo_thread && hx >= 0 && hx < R && hy >= 0 && hy < C;
            const size_t hoff = halo_in ? static_cast<size_t>(hx) * C + hy : 0;
            float4 gv[ITER], rv[ITER];
            float gh = 0.f, rh = 0.f;
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int rr = ROW0 + 4 * it + wave;
                const int x = x0 - H + rr;
                gv[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                rv[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (rr < ROW1 && x >= 0 && x < R && ym < C) {
                    const size_t off = static_cast<size_t>(x) * C + ym;
                    if (IN_PLACE) {       // (no other workgroup reads them: with plain loads the pass takes 339 us on VGG-19, with these 288)
                        gv[it] = load_streaming(g + off);
                        rv[it] = load_streaming(r + off);
                        continue;
                    }
                    if (!(PASS == kPassFullMap && v_stored)) gv[it] = *reinterpret_cast<const float4 *>(g + off);
                    if (r) rv[it] = *reinterpret_cast<const float4 *>(r + off);
                }
            }
            if (halo_in) {
                if (!(PASS == kPassFullMap && v_stored)) gh = g[hoff];
                if (r) rh = r[hoff];
            }
            if (MOM) {                    // Eq. 12, first line: the gradient term becomes u = m*u + g
                const float *__restrict__ u = a.mom + L.elem_off;
                float4 uv[ITER];
                float uh = 0.f;
#pragma unroll
                for (int it = 0; it < ITER; ++it) {
                    const int rr = 4 * it + wave;
                    const int x = x0 - H + rr;
                    uv[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (rr < ROWS && x >= 0 && x < R && ym < C)
                        uv[it] = *reinterpret_cast<const float4 *>(u + static_cast<size_t>(x) * C + ym);
                }
                if (halo_in) uh = u[hoff];
                if (FEED) feed.stash(feed_slot);   // the loads are out, no store of this tile yet
                gh = __fmul_rn(a.m, uh) + gh;
#pragma unroll
                for (int it = 0; it < ITER; ++it) {
                    gv[it].x = __fmul_rn(a.m, uv[it].x) + gv[it].x;
                    gv[it].y = __fmul_rn(a.m, uv[it].y) + gv[it].y;
                    gv[it].z = __fmul_rn(a.m, uv[it].z) + gv[it].z;
                    gv[it].w = __fmul_rn(a.m, uv[it].w) + gv[it].w;
                    if (STORE_V && a.mom_out && whole) {   // the tile's own elements (not the halo) go out once
                        const int rr = 4 * it + wave;
                        const int x = x0 - H + rr;
                        if (rr >= H && rr < H + kTileRows && x < R && ym < C)
                            store_streaming(a.mom_out + L.elem_off + static_cast<size_t>(x) * C + ym, gv[it]);
                    }
                }
            }
            if (FEED) feed.stash(feed_slot);       // the loads are out, no store of this tile yet
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int rr = ROW0 + 4 * it + wave;
                if (rr < ROW1) {
                    float4 v;
                    v.x = rv[it].x + gv[it].x;
                    v.y = rv[it].y + gv[it].y;
                    v.z = rv[it].z + gv[it].z;
                    v.w = rv[it].w + gv[it].w;
                    *reinterpret_cast<float4 *>(&tile[(rr + DOWN) * PITCH + PADL + 4 * lane]) = v;
                    if (STORE_V && a.v_out && whole) {     // the tile's own elements (not the halo) go out once
                        const int x = x0 - H + rr;
                        if (rr >= H && rr < H + kTileRows && x < R && ym < C)
                            store_streaming(a.v_out + L.elem_off + static_cast<size_t>(x) * C + ym, v);
                        if (IN_PLACE && L.tiles_x > 1u && x < R && (lane < kSeamCols<P> / 4 || lane >= 64 - kSeamCols<P> / 4))
                            *reinterpret_cast<float4 *>(seam_columns<P>(a.nsi_out, L, x, tcol, lane < 32 ? 0 : 1) + 4 * lane % kSeamCols<P>) = v;
                    }
                }
            }
            if (halo_thread) tile[hrow * PITCH + (hc < H ? PADL - 1 - hc : PADL + kTileCols + (hc - H))] = rh + gh;
        } else {
            if (FEED) feed.stash(feed_slot);
            // rows that are no multiple of 16 bytes long: a wave takes whole rows, all of a row's floats requested before any is used
            // (split flat over the threads, every float waited for the one before and cost a division: 16 us for a tile of 22 rows)
            constexpr int N = (PITCH + 63) / 64;
            const int wave = tid >> 6;
#pragma unroll 1
            for (int rr = (IN_PLACE ? H : 0) + wave; rr < (IN_PLACE ? H + kTileRows : ROWS); rr += 4) {
                // (the columns' masks are worked out row by row: held over the rows they cost the pass its scalar registers, and
                // 4 of 234 us with p = 5 on 103 M elements whose rows never come here.  With the work feed 12 or 13
                // scalar registers are still spilled to vector ones; the loop that was here before, with none, was no faster
                // there: 242 against 240 us on one card)
                int lane = tid & 63;
                asm("" : "+v"(lane));
                const int x = x0 - H + rr;
                const size_t row = static_cast<size_t>(max(x, 0)) * C;
                float gq[N], rq[N], uq[MOM ? N : 1];
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    const int j = lane + 64 * q, y = y0 - PADL + j;
                    gq[q] = rq[q] = 0.f;
                    if (MOM) uq[q] = 0.f;
                    if (x >= 0 && x < R && j < PITCH && y >= 0 && y < C && (!IN_PLACE || (j >= PADL && j < PADL + kTileCols))) {
                        if (!(PASS == kPassFullMap && v_stored)) gq[q] = (g + row)[y];
                        if (r) rq[q] = (r + row)[y];
                        if (MOM) uq[q] = (a.mom + L.elem_off + row)[y];
                    }
                }
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    const int j = lane + 64 * q, y = y0 - PADL + j;
                    float v = 0.f;
                    if (x >= 0 && x < R && j < PITCH && y >= 0 && y < C && (!IN_PLACE || (j >= PADL && j < PADL + kTileCols))) {
                        const bool own = rr >= H && rr < H + kTileRows && j >= PADL && j < PADL + kTileCols;
                        float gu = gq[q];
                        if (MOM) {
                            gu = __fmul_rn(a.m, uq[q]) + gu;
                            if (STORE_V && a.mom_out && whole && own) (a.mom_out + L.elem_off + row)[y] = gu;
                        }
                        v = rq[q] + gu;
                        if (STORE_V && a.v_out && whole && own) (a.v_out + L.elem_off + row)[y] = v;
                        if (IN_PLACE && L.tiles_x > 1u) {
                            const int col = j - PADL;
                            if (col < kSeamCols<P>) seam_columns<P>(a.nsi_out, L, x, tcol, 0)[col] = v;
                            if (col >= kTileCols - kSeamCols<P>) seam_columns<P>(a.nsi_out, L, x, tcol, 1)[col - (kTileCols - kSeamCols<P>)] = v;
                        }
                    }
                    if (j < PITCH && (!IN_PLACE || (j >= PADL && j < PADL + kTileCols))) tile[(rr + (IN_PLACE ? H : 0)) * PITCH + j] = v;
                }
            }
        }
        __syncthreads();

        // ---- window statistics
        // (the column as the compiler cannot see through it: otherwise it forms the 16 queue
        // entries of the thread once, outside the loop over the tiles, and keeps them in registers)
        int c0q = c0;
        asm volatile("" : "+v"(c0q));
        if constexpr (CAPTURE) {
            // Only the centres that reach the bound are wanted, and about 99.5 % do not.  A test
            // without the square root rules those out:
            //   NSI >= B  <=>  cb*sqrt(d) >= B - ca*sa  <=>  cb^2 * d >= max(B - ca*sa, 0)^2
            // in float32, with the slacks of PreF32 (a window whose variance cancels is never ruled out
            // on a value that is too small).  Each thread walks down its column keeping the last P row
            // sums.  The few centres that remain are queued and evaluated in full after the sweep, one
            // per thread.
            ColumnSums<P> ca_, cs_, cq_;
#pragma unroll
            for (int i = 0; i < RPT + 2 * H; ++i) {
                {
                    float sa, ss, sq;
                    const float *row = &tile[(row_base + i) * PITCH + PADL + c0 - H];
                    row_sums<P>(row, sa, ss, sq);
                    if (IN_PLACE && i >= kTileRows) carry[i - kTileRows] = row[H];
                    ca_.push(i, sa);
                    cs_.push(i, ss);
                    cq_.push(i, sq);
                }
                if (i >= 2 * H) {
                    const int o = i - 2 * H;
                    const float lo = !IN_PLACE ? bound_lof : o < H ? bound_above : o < 2 * H ? bound_top : bound_rest;     // (in place: row o - H of the tile)
                    if (PreF32<P>::stays(ca_.window(i), cs_.window(i), cq_.window(i), caf, cbf, pre_a, lo)) {   // (outside the matrix too: the queue's turn to tell)
                        const uint32_t pos = atomicAdd(&nqueue, 1u);
                        if (pos < static_cast<uint32_t>(kQueueCap<P>))
                            queue[pos] = static_cast<uint16_t>((row_base + o) * kTileCols + c0q);
                    }
                }
            }
        } else {
        double hs_a[P], hs_s[P], hs_q[P];
#pragma unroll
        for (int i = 0; i < RPT + 2 * H; ++i) {
            const float *row = &tile[(row_base + i) * PITCH + PADL + c0 - H];
            double w[P];
#pragma unroll
            for (int j = 0; j < P; ++j) w[j] = static_cast<double>(row[j]);
            {
                double sa = fabs(w[0]), ss = w[0], sq = w[0] * w[0];
#pragma unroll
                for (int j = 1; j < P; ++j) {
                    sa += fabs(w[j]);
                    ss += w[j];
                    sq = fma(w[j], w[j], sq);
                }
                hs_a[i % P] = sa;
                hs_s[i % P] = ss;
                hs_q[i % P] = sq;
            }
            if (i >= 2 * H) {
                const int o = i - 2 * H;   // output row inside the thread's strip
                double sa = hs_a[o % P], ss = hs_s[o % P], sq = hs_q[o % P];
#pragma unroll
                for (int j = 1; j < P; ++j) {
                    sa += hs_a[(o + j) % P];
                    ss += hs_s[(o + j) % P];
                    sq += hs_q[(o + j) % P];
                }
                const double nsq = __dmul_rn(n, sq);
                double d = var_n2_one_pass(ss, nsq);
                const int x = x0 + row_base + o, y = y0 + c0;
                {
                    // the one-pass variance cancelled (rare; never for P = 1, where it is 0 by definition)
                    if (P > 1 && d < kCancelFrac * nsq)
                        d = __dmul_rn(n, window_ssd<P>(&tile[(row_base + o) * PITCH + PADL + c0 - H], PITCH, ss / n));
                    const float out = static_cast<float>(nsi_from_var(sa, d, ca, cb));
                    if (x < R && y < C) {
                        if (MAP || (PASS == kPassSample && whole))
                            a.nsi_out[static_cast<size_t>(L.elem_off) + static_cast<size_t>(x) * C + y] = out;
                        if (FULLHIST) atomicAdd(&lhist[(__float_as_uint(out) & 0x7fffffffu) >> kCoarseShift], 1u);
                    }
                }
            }
        }
        }
        __syncthreads();                  // the sweep is complete (the tile is still needed by the queue)

        if (CAPTURE) {
            // ---- the queued centres in full: the same sums in the same order as above, Eq. 10 again
            // from the tile where the one-pass variance cancels, score, and the record if it reaches
            // the bound
            const uint32_t nq = nqueue;
            if (nq > static_cast<uint32_t>(kQueueCap<P>) && tid == 0) a.state_rw[l].overflow = 1u;   // (more than any slot holds)
            for (uint32_t qi = tid; qi < min(nq, static_cast<uint32_t>(kQueueCap<P>)); qi += 256) {
                const int pos = queue[qi];
                const int wrow = pos / kTileCols, ocol = pos - wrow * kTileCols, orow = IN_PLACE ? wrow - H : wrow;
                if (x0 + orow >= R || y0 + ocol >= C) continue;
                if (IN_PLACE) {            // (a window whose sums are not finite is queued whatever the bound)
                    if ((orow < 0 && !above) || (orow >= 0 && orow < H && trow > 0 && !above) || (ocol < H && tcol > 0) || (ocol >= kTileCols - H && y0 + kTileCols < C)) continue;
                }
                const uint32_t key = window_score<P>(&tile[wrow * PITCH + PADL + ocol - H], PITCH, ca, cb);
                if (key >= hint_key) {
                    const uint32_t x = static_cast<uint32_t>(x0 + orow), y = static_cast<uint32_t>(y0 + ocol);
                    if (IN_PLACE && orow < 0) {
                        const uint32_t cp = n_above + atomicAdd(&sh.nabove, 1u);
                        if (cp < L.slot_cap)
                            a.slot_ent[L.slot_off + static_cast<size_t>(local - L.tiles_x) * L.slot_cap + cp] = composite_key(key, x * L.C + y);
                    } else {
                        const uint32_t cp = atomicAdd(&ncand, 1u);
                        if (cp < static_cast<uint32_t>(kSlotCapMax)) cand[cp] = composite_key(key, x * L.C + y);
                    }
                    // fine bins upwards from the bound; the last one is open-ended
                    const uint32_t rel = (key - hint_key) >> kFineShift;
                    atomicAdd(&lhist[min(rel, static_cast<uint32_t>(kFineBins - 1))], 1u);
                }
            }
            __syncthreads();              // all reads of the tile are complete, all records made
        }

        if (CAPTURE) {
            const uint32_t nc = ncand, cap = L.slot_cap;
            recorded += nc;
            if (IN_PLACE) {
                const uint32_t more = sh.nabove;
                recorded += more;
                if (tid == 0 && more != 0u) {
                    a.slot_cnt[L.tile_begin_all + local - L.tiles_x] = min(n_above + more, cap);
                    if (n_above + more > cap) a.state_rw[l].overflow = 1u;
                }
                n_above = nc;
            }
            unsigned long long *__restrict__ dst = a.slot_ent + L.slot_off + static_cast<size_t>(local) * cap;
            for (uint32_t i = tid; i < min(nc, cap); i += 256) dst[i] = cand[i];
            if (tid == 0) {
                a.slot_cnt[L.tile_begin_all + local] = min(nc, cap);
                if (nc > cap) a.state_rw[l].overflow = 1u;
            }
            __syncthreads();
            if (tid == 0) { ncand = 0; nqueue = 0; }
            if (IN_PLACE && tid == 0) sh.nabove = 0;
            // the next tile's first barrier orders this reset before any new append
        }
    }

    if (NBINS > 1 && cur_l != 0xffffffffu && active) {
        uint32_t *__restrict__ gh = hist_base + static_cast<size_t>(cur_l) * kHistBins;
        for (int b = tid; b < NBINS; b += 256) {
            const uint32_t c = lhist[b];
            if (c) atomicAdd(&gh[b], c);
        }
        if (CAPTURE && tid == 0 && recorded) atomicAdd(recorded_slot(a.list_cnt, cur_l, wg), recorded);
    }
}

template <int P, int PASS, bool MOM, bool FEED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pass_captures(PASS) && !MOM ? (P <= 3 ? 5 : 4) : 1, PASS == kPassCapture && MOM ? 3 : 8)))
void k_nsi(const NsiArgs a) {
    __shared__ NsiShared<P, PASS> sh;
    nsi_pass<P, PASS, MOM, FEED>(a, sh, blockIdx.x, gridDim.x);
}

// The windows across the tiles' edges where v replaces the residual (one arena).  VGG-19: main pass 257 us and an emit that forms v once
// more 271, now 288 (of which the columns it keeps for this pass about 8), this pass 48 and an emit of the kept elements 41; the call 572 -> 460 us.
// What bounds this pass is its chain of loads, LDS and the evaluation in double on four waves per SIMD; its loads alone take 28 us.  The main pass stores v in the arena it reads,
// so no workgroup may read what another's tile holds; it scores the windows inside its run of tiles, and this pass, after it, those
// that reach further, from v.  A wave takes the positions along a run's edges, so that a tile's slot stays one
// wave's: the 3 H rows around the upper and the lower edge, lane j the columns from 4 j on, and the columns around the sides from where
// the main pass has put them.  The next run's are requested before this one's are looked at; the four waves of a workgroup share
// nothing but the candidates' counts: bins for one layer, that of the launch's middle tile, a list for the others (a
// few hundred candidates a workgroup in all).  They go to memory at the end: an atomic that is on its way holds up the next
// run's loads (59.6 us where each of the others' candidates was added at once, of which a quarter of the elements had
// them).  Nothing is counted of a layer whose slots are overfilled: after a gradient four times as large, when every window reaches the
// bounds, the adds to one bin of each layer took 9.2 ms.
template <int P>
struct SeamWave {
    static constexpr int kH = (P - 1) / 2, kRows = 6 * kH, kRunRows = kRun * kTileRows;      // rows around the edges, the upper one's first
    static constexpr int kPitch = kTileCols + 8, kSidePitch = (3 * kH) | 1;
    __attribute__((aligned(16))) float rows[kRows * kPitch];
    float side[2][(kRunRows + 2 * kH) * kSidePitch];                     // H columns of the tile on that side, 2 H own (to the right: the other way round)
    uint16_t queue[2 * kH * (kTileCols + kRunRows)];                     // every position along the edges
    uint32_t ncand[kRun], nqueue;
};
template <int P>
struct SeamShared {
    static constexpr uint32_t kOthers = 704;
    SeamWave<P> wave[4];
    uint32_t lhist[kFineBins];             // counts of the launch's main layer
    uint32_t others[kOthers], n_others;    // the other layers' candidates: layer and bin
};
template <int P>
__global__ __launch_bounds__(256) void k_seams(const NsiArgs a) {
    constexpr int H = (P - 1) / 2, PADL = 4, PITCH = SeamWave<P>::kPitch, SP = SeamWave<P>::kSidePitch;
    constexpr int EDGE = 3 * H, NR = 2 * EDGE, W = kSeamCols<P>, NS = (NR * 2 * H + 63) / 64;
    static_assert(NR < kTileRows + 2 * H && kRun == 2u, "the rows around the two edges are different rows; two tiles' rows, a lane per row's four pieces");
    __shared__ SeamShared<P> shared;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    SeamWave<P> &sh = shared.wave[wave];
    const uint32_t n_runs = (a.n_tiles + kRun - 1u) / kRun, step = gridDim.x * 4u;
    const uint32_t hist_l = a.samples[a.n_tiles / 2u].layer;
    for (int b = threadIdx.x; b < kFineBins; b += 256) shared.lhist[b] = 0u;
    if (threadIdx.x == 0) shared.n_others = 0u;
    for (uint32_t i = lane; i < 2u * (kRun * kTileRows + 2 * H) * SP; i += 64) sh.side[0][i] = 0.f;    // (the rows above and below stay so)
    if (lane == 0) sh.ncand[0] = sh.ncand[1] = sh.nqueue = 0u;
    __syncthreads();

    // The next tiles, as requested: a run's two, or one of them.
    struct Unit {
        uint32_t t, tiles, slot;          // first tile; how many; the first one's slot (the second's: L.tiles_x further)
        int x0, y0;
        bool top, bottom, left, right;
    } u = {};
    LayerDev L;
    uint32_t l = 0xffffffffu, hint_key = 0, n0 = 0, n1 = 0;  // the layer that L is; candidates in the slots
    bool active = false;
    float4 f[NR], sd[2][W / 4];
    float hs[NS];
    auto row_of = [](int q, int height) { return q < EDGE ? q - H : height - NR + H + q; };  // rows around the edges in order
    auto request = [&](uint32_t t) {
        const SampleEntry at = a.samples[t];
        if (at.layer != l) {
            l = at.layer;
            L = a.layers[l];
            hint_key = a.state[l].hint_key;
            // (with a tile overfilled the layer is ranked on its map, and what is added here would only be counted, at worst for every window)
            active = __builtin_amdgcn_readfirstlane(a.state[l].mode == kModeCandidates && bound_in_range(hint_key) && a.state[l].overflow == 0u ? 1u : 0u) != 0u;
        }
        const RunTile rt(L, at.local_tile, t);
        const int R = static_cast<int>(L.R), C = static_cast<int>(L.C), tcol = rt.tcol;
        u.t = t;
        u.tiles = rt.below ? 2u : 1u;
        u.slot = static_cast<uint32_t>(rt.trow) * L.tiles_x + static_cast<uint32_t>(tcol);
        u.x0 = rt.trow * kTileRows;
        u.y0 = tcol * kTileCols;
        const int height = static_cast<int>(u.tiles) * kTileRows;
        u.top = rt.trow > 0;
        u.bottom = u.x0 + height - H < R;
        u.left = tcol > 0;
        u.right = u.y0 + kTileCols < C;
        if (!active) return;
        const float *v = a.v_out + L.elem_off;
        const int y = u.y0 + 4 * static_cast<int>(lane);
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int x = u.x0 + row_of(q, height);
            f[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!(q < EDGE ? u.top : u.bottom) || x < 0 || x >= R || y >= C) continue;
            const float *row = v + static_cast<size_t>(x) * C + y;
            if ((C & 3) == 0) {
                f[q] = *reinterpret_cast<const float4 *>(row);
            } else {
                f[q].x = row[0];
                if (y + 1 < C) f[q].y = row[1];
                if (y + 2 < C) f[q].z = row[2];
                if (y + 3 < C) f[q].w = row[3];
            }
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) {                       // the columns beside those rows
            const int e = static_cast<int>(lane) + 64 * i, q = e / (2 * H), c = e - q * 2 * H;
            const int x = u.x0 + row_of(q, height), hy = c < H ? u.y0 - 1 - c : u.y0 + kTileCols + (c - H);
            hs[i] = q < NR && x >= 0 && x < R && hy >= 0 && hy < C ? v[static_cast<size_t>(x) * C + hy] : 0.f;
        }
        const int which = static_cast<int>(lane & 3u);       // left tile's last columns, own first, own last, right tile's first
        const int c = which == 0 ? tcol - 1 : which == 3 ? tcol + 1 : tcol;
        const bool there = (u.left || u.right) && c >= 0 && c < static_cast<int>(L.tiles_x);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int row = k * kTileRows + static_cast<int>(lane >> 2), x = u.x0 + row;
#pragma unroll
            for (int i = 0; i < W / 4; ++i) {
                sd[k][i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (there && row < height && x < R)
                    sd[k][i] = *reinterpret_cast<const float4 *>(seam_columns<P>(a.nsi_out, L, x, c, which == 0 || which == 2 ? 1 : 0) + 4 * i);
            }
        }
        n0 = a.slot_cnt[L.tile_begin_all + u.slot];
        if (u.tiles == 2u) n1 = a.slot_cnt[L.tile_begin_all + u.slot + L.tiles_x];
    };

    const double ca = a.ca, cb = a.cb;
    const float caf = uniform_f32(static_cast<float>(ca)), cbf = uniform_f32(static_cast<float>(cb));
    const float pre_a = uniform_f32(PreF32<P>::square_factor(cb));
    uint32_t cur_l = 0xffffffffu, recorded = 0;              // the layer that was looked at last, and its candidates
    uint32_t run = xcd_contiguous(blockIdx.x, gridDim.x) * 4u + wave;
    uint32_t t = run < n_runs ? run * kRun : kNoItem;
    if (t != kNoItem) request(t);
    while (t != kNoItem) {                                   // the same in all lanes
        const Unit me = u;
        const uint32_t ml = l, key0 = hint_key, had0 = n0, had1 = n1, C32 = L.C, cap = L.slot_cap, tiles_x = L.tiles_x, cnt0 = L.tile_begin_all + me.slot;
        const int R = static_cast<int>(L.R), C = static_cast<int>(C32), height = static_cast<int>(me.tiles) * kTileRows;
        unsigned long long *__restrict__ dst = a.slot_ent + L.slot_off + static_cast<size_t>(me.slot) * cap;
        const bool on = active && (me.top || me.bottom || me.left || me.right);
        if (on) {
            wave_lds_order();
#pragma unroll
            for (int q = 0; q < NR; ++q) *reinterpret_cast<float4 *>(&sh.rows[q * PITCH + PADL + 4 * lane]) = f[q];
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const int e = static_cast<int>(lane) + 64 * i, q = e / (2 * H), c = e - q * 2 * H;
                if (q < NR) sh.rows[q * PITCH + PADL + (c < H ? -1 - c : kTileCols + (c - H))] = hs[i];
            }
            const int which = static_cast<int>(lane & 3u), first = which == 0 ? H - W : which == 1 ? H : which == 2 ? 2 * H - W : 2 * H;
            const int inside = C - me.y0 - (which == 1 ? 0 : kTileCols);         // (a tile's first columns beyond the matrix's edge are 0)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                float *to = &sh.side[which >> 1][(k * kTileRows + static_cast<int>(lane >> 2) + H) * SP];
#pragma unroll
                for (int i = 0; i < W / 4; ++i) {
                    const float e[4] = {sd[k][i].x, sd[k][i].y, sd[k][i].z, sd[k][i].w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int col = first + 4 * i + j;
                        if (col >= 0 && col < EDGE) to[col] = (which & 1) != 0 && 4 * i + j >= inside ? 0.f : e[j];
                    }
                }
            }
        }
        // the run's other tile, if it was not taken with this one; else the next run
        t = me.tiles == 1u && me.t % kRun == 0u && me.t + 1u < a.n_tiles ? me.t + 1u : kNoItem;
        if (t == kNoItem) {
            run += step;
            if (run < n_runs) t = run * kRun;
        }
        if (t != kNoItem) request(t);
        if (!on) continue;
        if (ml != cur_l) {
            if (lane == 0 && recorded) atomicAdd(recorded_slot(a.list_cnt, cur_l, wave), recorded);
            recorded = 0;
            cur_l = ml;
        }
        const float bound = uniform_f32(PreF32<P>::bound(__uint_as_float(key0)));
        wave_lds_order();

        auto on_row = [&](int row) { return (row < H && me.top) || (row >= height - H && me.bottom); };
        auto queue = [&](int row, int col) { sh.queue[atomicAdd(&sh.nqueue, 1u)] = static_cast<uint16_t>(row * kTileCols + col); };
#pragma unroll
        for (int edge = 0; edge < 2; ++edge) {               // four columns a lane
            if (edge == 0 ? !me.top : !me.bottom) continue;
            ColumnSums<P> ca_[4], cs_[4], cq_[4];
#pragma unroll
            for (int i = 0; i < EDGE; ++i) {
                const float4 *row = reinterpret_cast<const float4 *>(&sh.rows[(edge * EDGE + i) * PITCH + 4 * lane]);      // from 4 columns to the left on
                const float4 q0 = row[0], q1 = row[1], q2 = row[2];
                const float w[12] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y, q2.z, q2.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float sa, ss, sq;
                    row_sums<P>(w + PADL + c - H, sa, ss, sq);
                    ca_[c].push(i, sa);
                    cs_[c].push(i, ss);
                    cq_[c].push(i, sq);
                    if (i >= 2 * H && PreF32<P>::stays(ca_[c].window(i), cs_[c].window(i), cq_[c].window(i), caf, cbf, pre_a, bound))
                        queue((edge == 0 ? 0 : height - H) + i - 2 * H, 4 * static_cast<int>(lane) + c);
                }
            }
        }
        // along the sides, where they are not in the rows above
        auto side_window = [&](int row, int col) { return &sh.side[col < H ? 0 : 1][row * SP + (col < H ? col : col - (kTileCols - H))]; };
        if (me.left || me.right) {
            for (int i = static_cast<int>(lane); i < height * 2 * H; i += 64) {
                const int row = i / (2 * H), c = i - row * 2 * H, col = c < H ? c : kTileCols - 2 * H + c;
                if (on_row(row) || !(c < H ? me.left : me.right)) continue;
                const float *win = side_window(row, col);
                float sa = 0.f, ss = 0.f, sq = 0.f;
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    float ra, rs, rq;
                    row_sums<P>(win + k * SP, ra, rs, rq);
                    sa += ra;
                    ss += rs;
                    sq += rq;
                }
                if (PreF32<P>::stays(sa, ss, sq, caf, cbf, pre_a, bound)) queue(row, col);
            }
        }
        wave_lds_order();
        const uint32_t nq = sh.nqueue;
        for (uint32_t qi = lane; qi < nq; qi += 64) {        // in full, as in nsi_pass
            const int pos = sh.queue[qi], row = pos / kTileCols, col = pos - row * kTileCols;
            if (me.x0 + row >= R || me.y0 + col >= C) continue;
            const bool along = on_row(row);
            const float *win = along ? &sh.rows[(row < H && me.top ? row : EDGE + row - (height - H)) * PITCH + PADL + col - H] : side_window(row, col);
            const uint32_t key = window_score<P>(win, along ? PITCH : SP, ca, cb);
            if (key >= key0) {
                const bool second = row >= kTileRows;
                const uint32_t cp = (second ? had1 : had0) + atomicAdd(&sh.ncand[second ? 1 : 0], 1u);
                if (cp >= cap) continue;       // (overfilled: as above)
                dst[(second ? static_cast<size_t>(tiles_x) * cap : 0u) + cp] = composite_key(key, static_cast<uint32_t>(me.x0 + row) * C32 + static_cast<uint32_t>(me.y0 + col));
                const uint32_t bin = min((key - key0) >> kFineShift, static_cast<uint32_t>(kFineBins - 1));
                if (ml == hist_l) {
                    atomicAdd(&shared.lhist[bin], 1u);
                } else {
                    static_assert(kFineBins == 1 << 10, "a list entry's lower bits, under a layer's number (< 65536)");
                    const uint32_t at = atomicAdd(&shared.n_others, 1u);
                    if (at < shared.kOthers) shared.others[at] = ml << 10 | bin;
                    else atomicAdd(&a.hist_s[static_cast<size_t>(ml) * kHistBins + bin], 1u);
                }
            }
        }
        wave_lds_order();
        const uint32_t nc0 = sh.ncand[0], nc1 = sh.ncand[1];
        recorded += nc0 + nc1;
        if (lane == 0) {
            if (nc0 != 0u) a.slot_cnt[cnt0] = min(had0 + nc0, cap);
            if (nc1 != 0u) a.slot_cnt[cnt0 + tiles_x] = min(had1 + nc1, cap);
            if ((nc0 != 0u && had0 + nc0 > cap) || (nc1 != 0u && had1 + nc1 > cap)) a.state_rw[ml].overflow = 1u;
            sh.ncand[0] = sh.ncand[1] = sh.nqueue = 0u;
        }
    }
    if (lane == 0 && recorded) atomicAdd(recorded_slot(a.list_cnt, cur_l, wave), recorded);
    __syncthreads();
    uint32_t *__restrict__ gh = a.hist_s + static_cast<size_t>(hist_l) * kHistBins;
    for (int b = threadIdx.x; b < kFineBins; b += 256) {
        const uint32_t n = shared.lhist[b];
        if (n) atomicAdd(&gh[b], n);
    }
    for (uint32_t i = threadIdx.x; i < min(shared.n_others, shared.kOthers); i += 256)
        atomicAdd(&a.hist_s[static_cast<size_t>(shared.others[i] >> 10) * kHistBins + (shared.others[i] & (kFineBins - 1))], 1u);
}

// All sides' launches in one (the fallback pass of small plans): a range of workgroups each.
constexpr int kSides = (RSDGC_MAX_P + 1) / 2;
struct NsiAllArgs {
    NsiArgs side[kSides];                 // p = 1, 3, 5, 7
    uint32_t first_wg[kSides + 1];
};

// The main pass of layers whose neighbourhoods are single elements: Eqs. 8-10 leave NSI = alpha |v| there (sum|w| = |v|, the
// variance is exactly 0; nsi_from_var's floor for it vanishes in the rounding to float32), so there is no halo, no tile in LDS
// and no test in front of the score.  A workgroup takes tiles as in nsi_pass; what reaches the bound goes straight to the tile's
// slot.  FEED: the tiles come from the launch's work feed, under the rule of the other sides (fixed shares / by the feed: 134 M
// elements 415 / 399 us a call, VGG-19 434 / 412, 72 M 233 / 238, 34 M 126 / 139).
// What bounds it is the streaming of g, r and v.  Groups of layers with other neighbourhoods that are not too large (kRideTiles,
// kRideMost) ride along as workgroups of the same launch: alone, a side's launch takes 8 to 15 us however few its tiles are.
// ResNet-50 with all its vectors, p after the kernels' sides: four launches of 24.1, 23.4, 34.4 and 14.6 us before, now two of 30.3 and 37.2;
// the call, whose magnitudes no longer need the score map, 191.7 -> 138.0 us.  2048 x 1024 at 2 % 60.0 -> 38.9 us, 8192 x 4096 232.7 -> 136.8.
struct FlatShared {
    uint32_t lhist[kFineBins];
    uint32_t n[2];                        // candidates of the tile; the other one is being cleared
    uint32_t feed_slot[2];
};
template <bool MOM, bool FEED>
__device__ __forceinline__ void capture_flat(const NsiArgs &a, FlatShared &sh, uint32_t wg, uint32_t n_wgs) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (uint32_t j = wg * 256u + tid; j < a.n16; j += n_wgs * 256u) a.counts[j] = make_uint4(0, 0, 0, 0);
    WorkFeed feed;
    const uint32_t first = FEED ? feed.first(a.feed, a.n_tiles, a.feed_shift, sh.feed_slot) : xcd_contiguous(wg, n_wgs);
    if (FEED ? first == kNoItem : first >= a.n_tiles) return;        // uniform
    for (int b = tid; b < kFineBins; b += 256) sh.lhist[b] = 0u;
    if (tid < 2) sh.n[tid] = 0u;
    __syncthreads();
    uint32_t e = 0;                       // (as in nsi_pass)
    SampleEntry ahead = {0u, 0u};
    if (FEED) e = dir_lookup(a.dir, a.n_dir, first);
    else ahead = a.samples[first];
    uint32_t cur_l = 0xffffffffu, hint_key = 0, recorded = 0, par = 0;
    bool active = false;
    LayerDev L;
    const double ca = a.ca;
    auto flush = [&]() {                  // the finished layer's counts
        uint32_t *__restrict__ gh = a.hist_s + static_cast<size_t>(cur_l) * kHistBins;
        for (int b = tid; b < kFineBins; b += 256) {
            const uint32_t c = sh.lhist[b];
            if (c) { atomicAdd(&gh[b], c); sh.lhist[b] = 0u; }
        }
        if (tid == 0 && recorded) atomicAdd(recorded_slot(a.list_cnt, cur_l, wg), recorded);
        recorded = 0;
    };
    for (uint32_t t = first; FEED ? t != kNoItem : t < a.n_tiles; t = FEED ? feed.next(sh.feed_slot) : t + n_wgs) {
        if (FEED) e = dir_advance(a.dir, a.n_dir, e, t);
        const uint32_t l = FEED ? a.dir[e].layer : ahead.layer, local = FEED ? t - a.dir[e].begin : ahead.local_tile;
        if (!FEED && t + n_wgs < a.n_tiles) ahead = a.samples[t + n_wgs];
        if (l != cur_l) {
            if (active) {                 // uniform
                flush();
                __syncthreads();
            }
            cur_l = l;
            L = a.layers[l];
            const SelState st = a.state[l];
            active = st.mode == kModeCandidates;
            hint_key = st.hint_key;
            if (active && !bound_in_range(hint_key)) {                // (as in nsi_pass)
                active = false;
                if (tid == 0 && hint_key != 0u) a.state_rw[l].overflow = 1u;
            }
        }
        if (!active) continue;
        const int trow = static_cast<int>(local / L.tiles_x), tcol = static_cast<int>(local - static_cast<uint32_t>(trow) * L.tiles_x);
        const int R = static_cast<int>(L.R), C = static_cast<int>(L.C), x0 = trow * kTileRows, y0 = tcol * kTileCols;
        const float *__restrict__ g = a.grad + L.elem_off;
        const float *__restrict__ r = a.resid + L.elem_off;
        const float *__restrict__ u = MOM ? a.mom + L.elem_off : nullptr;
        const uint32_t cap = L.slot_cap;
        unsigned long long *__restrict__ dst = a.slot_ent + L.slot_off + static_cast<size_t>(local) * cap;
        auto record = [&](float v, bool in, uint32_t index) {        // by whole waves
            const uint32_t key = __float_as_uint(static_cast<float>(ca * static_cast<double>(fabsf(v)))) & 0x7fffffffu;
            const bool hit = in && key >= hint_key;
            const uint32_t pos = wave_append(&sh.n[par], hit);
            if (hit) {
                if (pos < cap) dst[pos] = composite_key(key, index);
                atomicAdd(&sh.lhist[min((key - hint_key) >> kFineShift, static_cast<uint32_t>(kFineBins - 1))], 1u);
            }
        };
        if ((C & 3) == 0) {               // wave w takes rows w, w + 4, ..., lane j the 16 bytes at column 4 j
            constexpr int N = kTileRows / 4;
            const int y = y0 + 4 * lane;
            float4 gv[N], rv[N], uv[MOM ? N : 1];
            bool in[N];
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const int x = x0 + 4 * q + wave;
                in[q] = x < R && y < C;
                gv[q] = rv[q] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (MOM) uv[q] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (in[q]) {
                    const size_t off = static_cast<size_t>(x) * C + y;
                    gv[q] = load_streaming(g + off);
                    rv[q] = load_streaming(r + off);
                    if (MOM) uv[q] = load_streaming(u + off);
                }
            }
            if (FEED) feed.stash(sh.feed_slot);
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const uint32_t at = static_cast<uint32_t>(x0 + 4 * q + wave) * L.C + static_cast<uint32_t>(y);
                if (MOM) {
                    gv[q] = make_float4(__fmul_rn(a.m, uv[q].x) + gv[q].x, __fmul_rn(a.m, uv[q].y) + gv[q].y,
                                        __fmul_rn(a.m, uv[q].z) + gv[q].z, __fmul_rn(a.m, uv[q].w) + gv[q].w);
                    if (in[q] && a.mom_out) store_streaming(a.mom_out + L.elem_off + at, gv[q]);
                }
                const float4 v = make_float4(rv[q].x + gv[q].x, rv[q].y + gv[q].y, rv[q].z + gv[q].z, rv[q].w + gv[q].w);
                if (in[q] && a.v_out) store_streaming(a.v_out + L.elem_off + at, v);
                record(v.x, in[q], at);
                record(v.y, in[q], at + 1u);
                record(v.z, in[q], at + 2u);
                record(v.w, in[q], at + 3u);
            }
        } else {
            if (FEED) feed.stash(sh.feed_slot);
#pragma unroll 1
            for (int q = 0; q < kTileRows; q += 4) {                 // four rows' elements of a column at a time
                float gq[4], rq[4], uq[MOM ? 4 : 1];
                const int y = y0 + tid;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gq[i] = rq[i] = 0.f;
                    if (MOM) uq[i] = 0.f;
                    if (x0 + q + i < R && y < C) {
                        const size_t off = static_cast<size_t>(x0 + q + i) * C + y;
                        gq[i] = g[off];
                        rq[i] = r[off];
                        if (MOM) uq[i] = u[off];
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = x0 + q + i < R && y < C;
                    const uint32_t at = static_cast<uint32_t>(x0 + q + i) * L.C + static_cast<uint32_t>(y);
                    if (MOM) {
                        gq[i] = __fmul_rn(a.m, uq[i]) + gq[i];
                        if (in && a.mom_out) a.mom_out[L.elem_off + at] = gq[i];
                    }
                    const float v = rq[i] + gq[i];
                    if (in && a.v_out) a.v_out[L.elem_off + at] = v;
                    record(v, in, at);
                }
            }
        }
        __syncthreads();                  // all of the tile's candidates are recorded
        if (tid == 0) {
            const uint32_t n = sh.n[par];
            recorded += n;
            a.slot_cnt[L.tile_begin_all + local] = min(n, cap);
            if (n > cap) a.state_rw[l].overflow = 1u;
            sh.n[par] = 0u;               // (used again after the next tile's barrier)
        }
        par ^= 1u;
    }
    if (active) flush();
}
template <bool MOM, bool FEED>
__global__ __launch_bounds__(256) void k_capture_flat(const NsiArgs a) {
    __shared__ FlatShared sh;
    capture_flat<MOM, FEED>(a, sh, blockIdx.x, gridDim.x);
}
// ... with the small groups of other sides: a range of workgroups each, theirs first (they take longest).
template <bool MOM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_capture_mixed(const NsiAllArgs a) {
    __shared__ union Shared {
        FlatShared flat;
        NsiShared<3, kPassCapture> s3;
        NsiShared<5, kPassCapture> s5;
        NsiShared<7, kPassCapture> s7;
        __device__ Shared() {}
    } sh;
    const uint32_t b = blockIdx.x;
    if (b < a.first_wg[1]) nsi_pass<7, kPassCapture, MOM, false>(a.side[3], sh.s7, b, a.first_wg[1]);
    else if (b < a.first_wg[2]) nsi_pass<5, kPassCapture, MOM, false>(a.side[2], sh.s5, b - a.first_wg[1], a.first_wg[2] - a.first_wg[1]);
    else if (b < a.first_wg[3]) nsi_pass<3, kPassCapture, MOM, false>(a.side[1], sh.s3, b - a.first_wg[2], a.first_wg[3] - a.first_wg[2]);
    else capture_flat<MOM, false>(a.side[0], sh.flat, b - a.first_wg[3], a.first_wg[4] - a.first_wg[3]);
}
constexpr uint32_t kRideTiles = 256;      // tiles of a side up to which it rides along: one round of workgroups ...
// ... or, up to kRideMost for all sides together and as many as there are of single elements, where none of the side's layers has more than
// kRideLayer of them: two launches one behind the other leave the chip half idle twice, but more workgroups add more counts to the one
// row of a large layer, and with more tiles the launch of all sides, at three waves per SIMD, takes longer than theirs.  The call in two launches / one,
// so many tiles of p = 3 beside about as many of single elements: 1024 in one layer 81 / 73 us, 1536 90.5 / 89.4, 2048 106 / 107, 2816 131 / 147,
// in two 131 / 123, in four 129 / 115, 3072 in 16 127 / 125, 3584 in 16 131 / 137; p = 5 1536 in one 91 / 87, 2816 130 / 137, in two 128 / 118, 3072
// in 16 125 / 123, 3584 135 / 138; p = 7 94 / 90, 133 / 140, 132 / 122, 131 / 126, 141 / 140; with momentum p = 3 1024 in one 93 / 85, 2816 in two
// 169 / 153, p = 7 2048 in one 131 / 139, 2816 in two 164 / 160.  ResNet-50 with all its vectors (2790 beside 2950) 230 / 214, with
// momentum 258 / 243.
constexpr uint32_t kRideMost = 3072, kRideLayer = 1536;

// ------------------------------------------------------- ranking digits --
// The k_l-th largest composite key of a layer (Algorithm 1's ranking, Eq. 11's k_l) is found
// digit by digit, most significant first:
//   first digit   where the k_l-th score lies, from a histogram over all scores of the layer:
//                 candidate path: kFineBins bins of 2^kFineShift score-bit values each, counted
//                 upwards from the candidate bound by the main pass; full-map path: the top 12
//                 bits of the score, counted by the pass that writes the map (k_find0);
//   second digit  the next kLevel1Bits bits inside that bucket; the bucket's keys are gathered
//                 into the layer's list on the way (k_gather, many workgroups per layer);
//   the rest      remaining score bits, then -- only if equal scores straddle the k_l-th rank --
//                 the bits of ~index, so that the lower index wins: one workgroup per layer, on
//                 the gathered keys (k_finish).
struct DigitResult {
    uint32_t digit, above, count, found;
};

// Digit that holds the k_rem-th largest key of a histogram of nb <= 4096 bins (LDS or global),
// counted from the top; every thread of the workgroup (NW waves) returns the same result.
// `found` is 0 when the histogram holds fewer than k_rem keys.
template <int NW>
__device__ __forceinline__ DigitResult block_find_digit(const uint32_t *h, int nb, uint32_t k_rem,
                                                        uint32_t *wave_tot /*[NW]*/, DigitResult *res) {
    const int tid = threadIdx.x;
    const int per = nb >= 256 ? nb >> 8 : 1;    // the first 256 threads own `per` bins each, top bins first
    if (tid == 0) res->found = 0;
    const int hi = nb - tid * per;              // bins [hi - per, hi), as far as they exist
    uint32_t own = 0;
    if (tid < 256)
        for (int b = hi - 1; b >= hi - per && b >= 0; --b) own += h[b];
    const uint32_t incl = block_scan_incl_n<NW>(own, wave_tot);
    const uint32_t excl = incl - own;
    if (tid < 256 && excl < k_rem && k_rem <= incl) {
        uint32_t acc = excl;
        for (int b = hi - 1; b >= hi - per && b >= 0; --b) {
            const uint32_t c = h[b];
            if (acc + c >= k_rem) {
                res->digit = static_cast<uint32_t>(b);
                res->above = acc;
                res->count = c;
                res->found = 1;
                break;
            }
            acc += c;
        }
    }
    __syncthreads();
    const DigitResult r = *res;
    __syncthreads();
    return r;
}

// A candidate-path layer's threshold of this call, kept for the next calls' bounds.  The margin of
// those bounds follows what the forecasts miss: it decays slowly towards its initial value, and a
// threshold that ends s below this call's forecast (used for the bound or not) widens it to at
// least 1.5 s + 0.01 -- so the layer learns how much its threshold jitters from call to call
// without a bound having to fail first.
__device__ __forceinline__ void publish_threshold(PredState *__restrict__ pred, uint32_t l, uint32_t large,
                                                  uint32_t k, unsigned long long T) {
    if (pred == nullptr || large == 0u) return;
    PredState ps = pred[l];
    const uint32_t tau = static_cast<uint32_t>(T >> 32);
    const float init = margin_init_log2(k);
    float margin = fmaxf(init, (ps.margin > 0.f ? ps.margin : init) * kMarginDecay);
    if (ps.has_forecast && tau >= (1u << 23)) {
        const float shortfall = ps.forecast - __log2f(__uint_as_float(tau));
        // (a shortfall beyond the widest margin is a jump of the gradient's scale, not jitter: no
        // margin would have covered it, and none is sized by it)
        if (shortfall > 0.f && shortfall <= kMarginMaxLog2) margin = fmaxf(margin, kMarginSafety * shortfall + 0.01f);
    }
    ps.margin = fminf(margin, kMarginMaxLog2);
    ps.tau2 = ps.tau1;
    ps.tau1 = tau;
    pred[l] = ps;
}

// Small plans: whoever sets mask bits also counts them -- the kept elements per 8192-element chunk
// and per group of kChunkGroup chunks, which the emit turns into output positions -- and the
// pass over the mask is not needed.  A call on a
// small plan is a chain of launches of a few microseconds each; on a large one the extra atomics of the gather
// cost more than a pass (measured: VGG-19 +12 us, ResNet-18 -7 us), so there the gather counts nothing: in a plan of few layers k_finish's launch counts
// what it has marked (CountShare), and only k_mark, which sets few bits, counts as it goes; in the others k_count goes over the finished mask
// (CountHow).  A mask word lies in one chunk: chunks are 256 words long and a layer starts at a word boundary.
struct CountCtx {
    uint32_t *chunk_cnt, *group_cnt;   // cleared by the find0 launch, or by the main pass where k_select follows; null: nothing is counted
    size_t word0;                      // the layer's first mask word
    uint32_t chunk_begin, cgroup_begin;
    uint32_t gstride;                  // words between two chunk groups' counters
};
__device__ __forceinline__ CountCtx count_ctx(const LayerDev &L, uint32_t *chunk_cnt, uint32_t *group_cnt, uint32_t gstride = kGroupCntStride) {
    return CountCtx{chunk_cnt, group_cnt, static_cast<size_t>(L.elem_off) >> 5, L.chunk_begin, L.cgroup_begin, gstride};
}
// n more kept elements in the layer's chunk number cl / in its chunk group number gl.  Many
// workgroups add to one group counter, so each has a cache line of its own (atomics on one line
// are served one after the other, 11 ns each).
__device__ __forceinline__ void count_add_chunk_only(const CountCtx &c, uint32_t cl, uint32_t n) {
    atomicAdd(&c.chunk_cnt[c.chunk_begin + cl], n);
}
__device__ __forceinline__ void count_add_group(const CountCtx &c, uint32_t gl, uint32_t n) {
    atomicAdd(&c.group_cnt[static_cast<size_t>(c.cgroup_begin + gl) * c.gstride], n);
}
__device__ __forceinline__ void count_add_chunk(const CountCtx &c, uint32_t cl, uint32_t n) {
    count_add_chunk_only(c, cl, n);
    count_add_group(c, cl / kChunkGroup, n);
}
// The first wave of a workgroup hands over what the workgroup counted in LDS for the 64 chunks from
// cl0 on (lane = chunk): one add per chunk that got something, and one per chunk group -- 64
// consecutive chunks lie in at most two.
__device__ __forceinline__ void count_flush_wave0(const CountCtx &c, uint32_t cl0, uint32_t n) {
    const uint32_t lane = threadIdx.x & 63u;
    if (n) count_add_chunk_only(c, cl0 + lane, n);
    const uint32_t g0 = cl0 / kChunkGroup;
    const bool first = (cl0 + lane) / kChunkGroup == g0;
    uint32_t a = first ? n : 0u, b = first ? 0u : n;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        a += __shfl_xor(a, d, 64);
        b += __shfl_xor(b, d, 64);
    }
    if (lane == 0) {
        if (a) count_add_group(c, g0, a);
        if (b) count_add_group(c, g0 + 1, b);
    }
}
// ORs bits into mask word w and (COUNT) counts those that were not set before.
template <bool COUNT>
__device__ __forceinline__ void or_counted(const CountCtx &c, uint32_t *__restrict__ mask, size_t w, uint32_t bits) {
    if (!COUNT) {
        atomicOr(&mask[w], bits);
        return;
    }
    const uint32_t old = atomicOr(&mask[w], bits);
    const uint32_t n = __popc(bits & ~old);
    if (n) count_add_chunk(c, static_cast<uint32_t>((w - c.word0) >> 8), n);
}

// A selected centre (flat index i inside its layer) ORs the bits of its p x p window into the
// mask -- Section III-C: whole neighbourhoods are kept -- and its own bit into the
// centre mask when centre lists are wanted; bits that were not set before are counted, on large plans, whose groups' counters share
// cache lines, a chunk group's in LDS (`groups`: as many of the layer's first ones as the array holds).  The words touched by different centres are nearly
// all distinct, which is the case global atomics handle well; all of a window's are on their way before the first one's old value
// is looked at.
struct WindowGeom {
    size_t elem_off;
    int R, C, h;
};
constexpr uint32_t kMarkGroups = 512;      // (2^28 elements)
enum MarkCount : int { kMarkOnly, kMarkCounts, kMarkCountsShared };       // no counts, counts, the groups' in LDS first
template <MarkCount HOW>
__device__ __forceinline__ void mark_window(const WindowGeom &g, const CountCtx &c, uint32_t *groups /*[kMarkGroups], LDS*/, uint32_t i,
                                            uint32_t *__restrict__ mask, uint32_t *__restrict__ cmask) {
    const int xc = static_cast<int>(i / static_cast<uint32_t>(g.C));
    const int yc = static_cast<int>(i - static_cast<uint32_t>(xc) * static_cast<uint32_t>(g.C));
    const int ylo = max(0, yc - g.h), nbits = min(g.C - 1, yc + g.h) - ylo + 1;
    const uint32_t bits = (1u << nbits) - 1u;
    size_t word[RSDGC_MAX_P];
    uint32_t lo[RSDGC_MAX_P], hi[RSDGC_MAX_P], old_lo[RSDGC_MAX_P], old_hi[RSDGC_MAX_P];
#pragma unroll
    for (int d = 0; d < RSDGC_MAX_P; ++d) {
        const int x = xc - g.h + d;
        lo[d] = hi[d] = old_lo[d] = old_hi[d] = 0u;
        word[d] = 0;
        if (d > 2 * g.h || x < 0 || x >= g.R) continue;
        const size_t pos = g.elem_off + static_cast<size_t>(x) * g.C + ylo;
        const uint32_t b = static_cast<uint32_t>(pos & 31);
        word[d] = pos >> 5;
        lo[d] = bits << b;
        old_lo[d] = atomicOr(&mask[word[d]], lo[d]);
        if (b + nbits > 32u) {
            hi[d] = bits >> (32u - b);
            old_hi[d] = atomicOr(&mask[word[d] + 1], hi[d]);
        }
    }
    auto count = [&](size_t w, uint32_t n) {
        if (n == 0u) return;
        const uint32_t cl = static_cast<uint32_t>((w - c.word0) >> 8), gl = cl / kChunkGroup;
        count_add_chunk_only(c, cl, n);
        if (HOW == kMarkCountsShared && gl < kMarkGroups) atomicAdd(&groups[gl], n);
        else count_add_group(c, gl, n);
    };
#pragma unroll
    for (int d = 0; d < RSDGC_MAX_P && HOW != kMarkOnly; ++d) {
        count(word[d], __popc(lo[d] & ~old_lo[d]));
        count(word[d] + 1, __popc(hi[d] & ~old_hi[d]));
    }
    if (cmask) {
        const size_t pos = g.elem_off + i;
        atomicOr(&cmask[pos >> 5], 1u << (pos & 31));
    }
}

// ----------------------------------------------------------------- hint --
// First calls with a workspace only: one workgroup per large layer that has no predicted bound
// turns the layer's sampled scores (12-bit histogram) into its candidate bound: the lower edge
// of the bucket at which the target count is reached from the top.  A layer whose sample gives
// none (too few scores, or the target only in bucket 0) goes to the full map.
__global__ __launch_bounds__(256) void k_hint(const LayerDev *__restrict__ layers,
                                              SelState *__restrict__ state,
                                              uint32_t *__restrict__ hist_s,
                                              uint32_t *__restrict__ flags) {
    __shared__ uint32_t wave_tot[4];
    __shared__ DigitResult res;
    const int l = blockIdx.x, tid = threadIdx.x;
    const SelState st = state[l];
    const uint32_t target = layers[l].hint_target;
    constexpr int per = kHistBins / 256;
    uint32_t *__restrict__ hs = hist_s + static_cast<size_t>(l) * kHistBins;
    const int hi = kHistBins - tid * per;          // thread 0 holds the top buckets
    uint32_t v[per];
    uint32_t own = 0;
#pragma unroll
    for (int j = 0; j < per; ++j) {                // (independent loads: one round trip)
        v[j] = hs[hi - 1 - j];
        own += v[j];
    }
    if (st.mode != kModeCandidates || st.hint_key != 0u) return;    // uniform
#pragma unroll
    for (int j = 0; j < per; ++j)                  // (the main pass counts its candidates here)
        if (v[j]) hs[hi - 1 - j] = 0u;
    if (tid == 0) res.found = 0;
    const uint32_t incl = block_scan_incl(own, wave_tot);
    const uint32_t excl = incl - own;
    if (excl < target && target <= incl) {
        uint32_t acc = excl;
#pragma unroll
        for (int j = 0; j < per; ++j) {
            if (acc < target && acc + v[j] >= target) {
                res.digit = static_cast<uint32_t>(hi - 1 - j);
                res.found = 1;
            }
            acc += v[j];
        }
    }
    __syncthreads();
    if (tid == 0) {
        const uint32_t key = res.found ? res.digit << kCoarseShift : 0u;
        if (key >= kPreF32MinKey && key <= kPreF32MaxKey) {      // (a bound the main pass can test in float32)
            state[l].hint_key = key;
        } else {
            state[l].mode = kModeFullMap;
            flags[0] = 1u;                 // the fallback pass has work
        }
    }
}

// ---------------------------------------------------------------- find0 --
// One workgroup per layer, after the NSI passes: the first ranking digit.  For a layer on the
// candidate path this is also the check of its bound: the recorded centres are usable only if
// no tile slot overflowed, at least k_l were recorded (then the k_l best of the layer are all
// among them) and the k_l-th does not lie in the open-ended top bin.  Otherwise the layer falls
// back to the full map in this call (a flag tells the fallback kernels that there is work), goes
// back to sampled bounds for the next few calls and widens the margin of its predictions.
struct Find0Args {
    const LayerDev *layers;
    SelState *state;
    const uint32_t *hist, *hist_s;
    uint32_t *flags;
    PredState *pred;           // nullable
    uint4 *counts;             // the chunk counters: cleared here for the kernels to come
    uint32_t n16;
    int n_layers;
};
// What a layer remembers of a bound that failed (st: its state, r: what the candidates' first digit gave).
__device__ __forceinline__ void bound_failed(PredState *__restrict__ pred, uint32_t l, uint32_t k, const SelState &st,
                                             const DigitResult &r) {
    PredState ps = pred[l];
    ps.cooldown = kCooldownCalls;
    if (st.predicted & 1u) {
        // the margin of the predicted bounds follows the way this one failed: too few centres above
        // it -- twice the margin; a tile with too many, or a threshold beyond the bins -- the bound
        // lay too low, and a wider margin would only repeat that: half of it, down to its start value
        const float init = margin_init_log2(k);
        const float m = ps.margin > 0.f ? ps.margin : init;
        const bool too_low = st.overflow != 0u || (r.found && r.digit == static_cast<uint32_t>(kFineBins - 1));
        ps.margin = too_low ? fmaxf(0.5f * m, init) : fminf(2.f * m, kMarginMaxLog2);
    }
    pred[l] = ps;
}

__device__ __forceinline__ void find0(const Find0Args &f, int l) {
    __shared__ uint32_t wave_tot[4];
    __shared__ DigitResult res;
    const int tid = threadIdx.x;
    // the chunk counters, which the last kernel of the call before still read
    for (uint32_t j = static_cast<uint32_t>(l) * 256u + tid; j < f.n16; j += static_cast<uint32_t>(f.n_layers) * 256u) f.counts[j] = make_uint4(0, 0, 0, 0);
    // state, layer constants and counts are requested together: one round trip to memory
    // instead of three (each costs this one-workgroup-per-layer kernel about 2 us)
    const SelState st = f.state[l];
    const uint32_t large = f.layers[l].large, grid = f.layers[l].grid;
    const bool cand = st.mode == kModeCandidates;                  // uniform
    const uint32_t *__restrict__ h = (cand ? f.hist_s : f.hist) + static_cast<size_t>(l) * kHistBins;
    const int nb = cand ? kFineBins : kHistBins, per = nb >> 8;
    const int hi = nb - tid * per;              // thread t owns bins [hi - per, hi): t = 0 holds the top bins
    constexpr int kMaxPer = kHistBins / 256;
    uint32_t v[kMaxPer];
    uint32_t own = 0;
#pragma unroll
    for (int j = 0; j < kMaxPer; ++j) {
        v[j] = j < per ? h[hi - 1 - j] : 0u;
        own += v[j];
    }
    if (st.done || st.mode == kModeSkip) return;
    // a large layer that is already on the full map (its sample gave no bound): its histogram
    // comes with the fallback pass, and the select pass finds its first digit (a block grid's has been counted by the block pass)
    if (st.mode == kModeFullMap && large != 0u && grid == 0u) return;
    if (tid == 0) res.found = 0;
    const uint32_t incl = block_scan_incl(own, wave_tot);
    const uint32_t excl = incl - own;
    if (excl < st.k_rem && st.k_rem <= incl) {
        uint32_t acc = excl;
        bool hit = false;
#pragma unroll
        for (int j = 0; j < kMaxPer; ++j) {
            if (!hit && j < per && acc + v[j] >= st.k_rem) {
                res.digit = static_cast<uint32_t>(hi - 1 - j);
                res.above = acc;
                res.count = v[j];
                res.found = 1;
                hit = true;
            }
            if (!hit) acc += v[j];
        }
    }
    __syncthreads();
    const DigitResult r = res;
    if (cand && (!r.found || st.overflow != 0u || r.digit == static_cast<uint32_t>(kFineBins - 1) ||
                 st.hint_key == 0u)) {
        if (tid == 0) {
            SelState ns = st;
            ns.mode = kModeFullMap;
            f.state[l] = ns;
            f.flags[0] = 1u;                 // the fallback pass has work
            bound_failed(f.pred, l, f.layers[l].k, st, r);
        }
        return;
    }
    if (tid == 0) {
        SelState ns = st;
        if (!r.found) {                    // fewer keys than k_l (cannot happen for finite input)
            ns.done = 1;
        } else {
            const uint32_t shift = cand ? kFineShift : kCoarseShift;
            ns.lo = (cand ? st.hint_key : 0u) + (r.digit << shift);
            ns.span = shift;
            ns.k_rem = st.k_rem - r.above;
            ns.T = static_cast<unsigned long long>(ns.lo) << 32;
            if (r.count == ns.k_rem) {     // whole bucket taken: the threshold is its lower edge
                ns.done = 1;
                publish_threshold(f.pred, l, large, f.layers[l].k, ns.T);
            }
        }
        f.state[l] = ns;
    }
}

__global__ __launch_bounds__(256) void k_find0(const Find0Args f) { find0(f, blockIdx.x); }

// k_find0 and the fallback pass in one launch (up to 256 layers): in nearly every call the pass finds nothing to do, and
// a launch that does nothing costs as much as k_find0's -- 4.7 us each.
template <int P, bool MOM>
__global__ __launch_bounds__(256) void k_find0_fallback(const Find0Args f, const NsiArgs a) {
    __shared__ NsiShared<P, kPassFullMap> sh;
    if (blockIdx.x < static_cast<uint32_t>(f.n_layers)) find0(f, blockIdx.x);
    else nsi_pass<P, kPassFullMap, MOM, false, true>(a, sh, blockIdx.x - f.n_layers, gridDim.x - f.n_layers);
}
template <bool MOM>
__global__ __launch_bounds__(256) void k_find0_fallback_all(const Find0Args f, const NsiAllArgs a) {
    __shared__ union Shared {
        NsiShared<1, kPassFullMap> s1;
        NsiShared<3, kPassFullMap> s3;
        NsiShared<5, kPassFullMap> s5;
        NsiShared<7, kPassFullMap> s7;
        __device__ Shared() {}
    } sh;
    if (blockIdx.x < static_cast<uint32_t>(f.n_layers)) {
        find0(f, blockIdx.x);
        return;
    }
    const uint32_t b = blockIdx.x - f.n_layers;
    if (b < a.first_wg[1]) nsi_pass<1, kPassFullMap, MOM, false, true>(a.side[0], sh.s1, b, a.first_wg[1]);
    else if (b < a.first_wg[2]) nsi_pass<3, kPassFullMap, MOM, false, true>(a.side[1], sh.s3, b - a.first_wg[1], a.first_wg[2] - a.first_wg[1]);
    else if (b < a.first_wg[3]) nsi_pass<5, kPassFullMap, MOM, false, true>(a.side[2], sh.s5, b - a.first_wg[2], a.first_wg[3] - a.first_wg[2]);
    else nsi_pass<7, kPassFullMap, MOM, false, true>(a.side[3], sh.s7, b - a.first_wg[3], a.first_wg[4] - a.first_wg[3]);
}

// --------------------------------------------------------------- gather --
// After the first digit: the keys of each layer's threshold bucket (score bits in
// [lo, lo + 2^span)) are copied into the layer's list and their next digit is histogrammed.
// Three kinds of workgroups share the launch:
//   [0, n_map_chunks)           a chunk each of the plan's list of 8192-element score-map chunks
//                               (layers that are always ranked on the full map);
//   [n_map_chunks, +n_slot_wgs) stride over the plan's list of slot groups (large layers,
//                               where they are still in candidate mode);
//   the last n_fb_wgs           only when some large layer fell back to the full map: they
//                               walk all chunks and take those of such layers (and find the
//                               first digit of such a layer themselves, from the histogram the
//                               fallback pass has counted).
// Matches of the fallback walk are staged in LDS and appended with one atomic per flush.
// The recorded candidates of a large layer are nearly all decided by the first digit already
// (its bins are fine: the threshold bucket holds a per cent or two of them): a candidate above
// the bucket is selected whatever the later digits say, so its window is marked here and now
// (k_mark marks the few that the bucket contributes); one in the bucket is appended to the
// list straight away, one atomic per wave, without staging or barriers.
// (In-kernel hand-over of a finished layer to "the last workgroup" was measured and dropped:
// the device-scope fences it needs write back the whole L2 of an XCD each time and cost more
// than the launch they save.)
constexpr int kStage = 2048;            // staged keys per workgroup (a round adds at most 1024)
// Small plans: a workgroup takes a quarter of a group.  Their gather is one short chain per workgroup -- entry, slots, marks,
// words -- on a chip that is mostly idle, and four workgroups get through it in less time than one.  The more groups there are,
// the more the words that neighbours share, and their atomics, weigh; where the line lies between 377 and 512 groups was not
// looked for.  By groups, whole / quarters: resnet18 13.7 / 10.1 us, 256 groups 16.8 / 12.4, resnet50 (377) 19.6 / 18.3, 512
// groups 18.4 / 20.7 and with p = 1 12.4 / 17.5.
constexpr int kSlotParts = 4;
constexpr uint32_t kSplitGroups = 512;  // groups from which a workgroup takes a whole one

constexpr uint32_t kWideGrid = 32768;       // block columns from which a grid's gather counts by row ...
constexpr uint32_t kWideSlots = 4;          // ... so many chunks of each
constexpr int kTileMaskWords = kTileRows * kTileCols / 32;    // mask words of one tile (rows of 8 words)
constexpr int kGatherCountSlots = 64;                          // chunks a group of tiles counts for in LDS (the rest: directly)

// The words of a group of tiles in LDS: a slot's rows are 8 words, and a slot's pitch is 8 words more than its tile, so that the
// words of a matrix row through eight slots lie in different banks.
constexpr int kSlotPitch = kTileMaskWords + 8;
template <int SLOTS>
struct GroupMarks {
    __attribute__((aligned(16))) uint32_t bits[SLOTS * kSlotPitch];   // mask words of the group of tiles being written
    uint32_t ccnt[kGatherCountSlots];             // bits set, per chunk from the group's first one on
    uint2 corner[SLOTS];                          // first row and column of every tile
};

struct GatherShared {
    union {
        unsigned long long ent[kStage];               // score-map roles: staged keys
        GroupMarks<kSlotGroup> marks;                 // slot role
    };
    uint32_t hist[kLevel1Bins];         // second-digit counts
    DigitResult res;
    uint32_t n;                         // staged keys
    uint32_t base;
    uint32_t wave_tot[4];
};

struct GatherLists {
    const DirEntry *chunk_dir;       // all chunks by layer (fallback walk)
    const ChunkInfo *chunks;         // ... each (block grids)
    const ChunkEntry *map_chunks;    // [n_map_chunks]
    const GroupEntry *cand_groups;   // [n_cand_groups]
    uint32_t n_layers, n_chunks, n_map_chunks, n_cand_groups;
    uint32_t n_slot_wgs;             // the remaining workgroups are fallback walkers
};

struct GatherArgs {
    const LayerDev *layers;
    const SelState *state;
    const uint32_t *keys;                 // score map
    const uint32_t *slot_cnt;
    const unsigned long long *slot_ent;
    uint32_t *list_cnt;
    unsigned long long *list_ent;
    const uint32_t *hist;                 // first-digit counts (fallback layers)
    uint32_t *hist1;                      // [n_layers][kLevel1Bins]
    const uint32_t *flags;
    uint32_t *mask, *cmask;               // kept-element bitmask; selected-centre bitmask (nullable)
    uint32_t *chunk_cnt, *group_cnt;      // kept elements per chunk / chunk group, counted as the bits are set
};

// Entries of a layer's list.  While a block grid is on the candidate path its tile slots lie in the upper half of it.
__device__ __forceinline__ uint32_t list_entries(const LayerDev &L, bool candidates) {
    return L.grid != 0u && candidates ? L.list_cap / 2u - 1u : L.list_cap;
}

// The list of the layer the workgroup is working on.
struct GatherList {
    uint32_t *cnt;                        // this workgroup's shard counter
    unsigned long long *ent;              // ... and region
    uint32_t cap;
};

// Appends the staged keys to the current layer's list.
__device__ __forceinline__ void gather_flush_keys(GatherShared &sh, const GatherList &gl) {
    __syncthreads();
    const uint32_t n = sh.n;
    if (n != 0) {                          // uniform
        if (threadIdx.x == 0) sh.base = atomicAdd(gl.cnt, n);
        __syncthreads();
        const uint32_t base = sh.base;
        for (uint32_t i = threadIdx.x; i < n; i += 256)
            if (base + i < gl.cap) gl.ent[base + i] = sh.ent[i];
        __syncthreads();
        if (threadIdx.x == 0) sh.n = 0;
    }
    __syncthreads();
}

// One round of at most 1024 appends (4 per thread) is about to start: make room for it.
__device__ __forceinline__ void gather_make_room(GatherShared &sh, const GatherList &gl) {
    if (staged_more_than(sh.n, static_cast<uint32_t>(kStage) - 1024u)) gather_flush_keys(sh, gl);
}

// Stages key K (of a flagged lane) and counts its second digit.  Called by whole waves.
__device__ __forceinline__ void gather_stage_key(GatherShared &sh, bool hit, unsigned long long K,
                                                 uint32_t lo, uint32_t shift1) {
    const uint32_t pos = wave_append(&sh.n, hit);
    if (hit) {
        sh.ent[pos] = K;
        atomicAdd(&sh.hist[(static_cast<uint32_t>(K >> 32) - lo) >> shift1], 1u);
    }
}

// A chunk of a layer that is ranked on the full map: always, or, a block grid, in this call.  All of a thread's 32 scores are requested before any is looked at, and
// places in the list are handed out once per chunk: what bounds this is the reading.  (Workgroups that strode over
// the chunks, a quarter of a chunk and two barriers at a time: 35.9 us for the 62 MB of VGG-19's block scores, now 30.4: an atomic per key on
// the second digit's counts is most of what is left.)
constexpr uint32_t kNoDigit = 0xffffffffu;      // the layer's state tells its first digit
__device__ __forceinline__ void gather_map_chunk(const GatherArgs &a, const ChunkEntry ce, GatherShared &sh, uint32_t digit) {
    constexpr int N = kChunk / 1024;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));         // (or places in a chunk are worked out once and kept over a workgroup's chunks, in scratch memory)
    const uint32_t *__restrict__ src = a.keys + ce.arena_off;
    uint4 q[N];
    if (ce.len == static_cast<uint32_t>(kChunk)) {
#pragma unroll
        for (int j = 0; j < N; ++j) q[j] = *reinterpret_cast<const uint4 *>(src + j * 1024 + 4 * tid);
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint32_t e = j * 1024 + 4 * tid;
            q[j] = make_uint4(0, 0, 0, 0);
            if (e < ce.len) q[j].x = src[e];
            if (e + 1 < ce.len) q[j].y = src[e + 1];
            if (e + 2 < ce.len) q[j].z = src[e + 2];
            if (e + 3 < ce.len) q[j].w = src[e + 3];
        }
    }
    const uint32_t l = ce.layer;
    const SelState st = a.state[l];
    const LayerDev &L = a.layers[l];
    const uint32_t shard = (ce.start / kChunk) % L.list_shards, cap = L.list_cap / L.list_shards;
    uint32_t *cnt = a.list_cnt + (static_cast<size_t>(l) * kListShards + shard) * kListCntStride;
    unsigned long long *ent = a.list_ent + L.list_off + static_cast<size_t>(shard) * cap;
    if (st.done || st.mode != kModeFullMap) return;                  // uniform
    for (int b = tid; b < kLevel1Bins; b += 256) sh.hist[b] = 0;
    __syncthreads();
    const uint32_t lo = digit != kNoDigit ? digit << kCoarseShift : st.lo, width = 1u << kCoarseShift;
    constexpr uint32_t shift1 = kCoarseShift - kLevel1Bits;
    uint32_t hits = 0;                    // a bit per score
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const uint32_t kk[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t rel = (kk[c] & 0x7fffffffu) - lo;
            if (rel < width && static_cast<uint32_t>(j * 1024 + 4 * tid + c) < ce.len) {
                hits |= 1u << (4 * j + c);
                atomicAdd(&sh.hist[rel >> shift1], 1u);
            }
        }
    }
    const uint32_t own = __popc(hits), incl = block_scan_incl(own, sh.wave_tot);
    if (tid == 255) sh.base = incl ? atomicAdd(cnt, incl) : 0u;
    __syncthreads();
    uint32_t pos = sh.base + incl - own;
    if (hits) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint32_t kk[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (hits & (1u << (4 * j + c))) {
                    if (pos < cap) ent[pos] = composite_key(kk[c], ce.start + j * 1024 + 4 * tid + c);
                    ++pos;
                }
        }
    }
    uint32_t *__restrict__ gh = a.hist1 + static_cast<size_t>(l) * kLevel1Bins;
    for (int b = tid; b < kLevel1Bins; b += 256) {
        const uint32_t c = sh.hist[b];
        if (c) atomicAdd(&gh[b], c);
    }
}

// A group of consecutive tile slots of a layer.  The workgroup builds the bits of its tiles in LDS, eight words per tile row,
// from the group's own candidates and writes them with plain stores, whole cache lines at a time -- except the mask words that others
// write too: those that windows of other groups' candidates can reach (the h rows along a tile's upper and lower edge, the first
// and last columns of the group's run of tiles), and, where a row is no multiple of 32 long, those that hold the
// end of one tile row and the beginning of another.  Those, and the bits that the group's
// windows set in other groups' tiles, are ORed into the (cleared) mask.  Words without a bit are not written.
// COUNT: the bits are counted as they are set (an OR tells which were new), per chunk, in LDS first: a group of tiles
// lies in a few chunks.
// Rows that are no whole mask words took a returning atomic for every row of every window before, one after the other: calls on
// 1448 x 1448 with p = 3 at 2 % 69.2 us, now 35.4, at 13 % 238.0, now 48.7; 999 x 1001 with p = 1 95.9, now 33.2; 20000 x 45 65.4, now 38.7.
// What bounds this is the number of instructions, a few hundred per wave: no division by anything but the tile's corner (once per
// tile), a window's rows addressed from the tile it starts in, and what crosses a tile's side edge in a second round that a wave
// only takes when one of its lanes needs it.  With the place of every row and word worked out by itself (1700 instructions per
// wave) k_gather took 29.9 us on VGG-19, now 24.2; 25088 x 4096 at 0.1 % with p = 5 21.0, now 14.6; ResNet-50 15.2, now 14.0.
struct GroupGeom {
    int h, C, R, tiles_x;
    int g0, gn;                           // the group's first tile inside the layer, and how many
    uint32_t cl0;                         // COUNT: first chunk that the group's windows can reach
    float inv_c;                          // a little below 1 / C
    uint32_t *mask;                       // the layer's first mask word
    CountCtx cctx;
};
__device__ __forceinline__ GroupGeom group_geom(const LayerDev &L, uint32_t g0, uint32_t gn, uint32_t *mask, const CountCtx &cctx) {
    GroupGeom q;
    q.h = (static_cast<int>(L.p) - 1) / 2;
    q.C = static_cast<int>(L.C);
    q.R = static_cast<int>(L.R);
    q.tiles_x = static_cast<int>(L.tiles_x);
    q.g0 = static_cast<int>(g0);
    q.gn = static_cast<int>(gn);
    q.cl0 = 0;
    q.inv_c = (1.f - 4.8e-7f) / static_cast<float>(L.C);
    q.mask = mask + (static_cast<size_t>(L.elem_off) >> 5);
    q.cctx = cctx;
    return q;
}
// Clears the words and writes the tiles' corners; a barrier has to follow.
template <int THREADS, int SLOTS>
__device__ __forceinline__ void group_clear(const GroupGeom &q, GroupMarks<SLOTS> &sh) {
    uint4 *b = reinterpret_cast<uint4 *>(sh.bits);
    for (int i = threadIdx.x; i < SLOTS * kSlotPitch / 4; i += THREADS) b[i] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < static_cast<uint32_t>(kGatherCountSlots)) sh.ccnt[threadIdx.x] = 0u;
    if (threadIdx.x < static_cast<uint32_t>(q.gn)) {
        const uint32_t local = static_cast<uint32_t>(q.g0) + threadIdx.x, tr = local / static_cast<uint32_t>(q.tiles_x);
        sh.corner[threadIdx.x] = make_uint2(tr * kTileRows, (local - tr * static_cast<uint32_t>(q.tiles_x)) * kTileCols);
    }
}
// First chunk that the group's windows can reach: that of the element h rows above and h columns left of the first tile's corner.
__device__ __forceinline__ uint32_t group_first_chunk(const GroupGeom &q, const uint2 corner) {
    return static_cast<uint32_t>((static_cast<size_t>(max(0, static_cast<int>(corner.x) - q.h)) * static_cast<uint32_t>(q.C) +
                                  static_cast<size_t>(max(0, static_cast<int>(corner.y) - q.h))) / kChunk);
}
template <int SLOTS>
__device__ __forceinline__ void group_count(const GroupGeom &q, GroupMarks<SLOTS> &sh, uint32_t word, uint32_t n) {
    const uint32_t slot = (word >> 8) - q.cl0;                       // (a chunk is 256 words)
    if (slot < static_cast<uint32_t>(kGatherCountSlots)) atomicAdd(&sh.ccnt[slot], n);
    else count_add_chunk(q.cctx, q.cl0 + slot, n);
}
// The window of the candidate with flat index i, which lies in the group's tile sidx.
template <bool COUNT, int SLOTS>
__device__ __forceinline__ void group_mark(const GroupGeom &q, GroupMarks<SLOTS> &sh_, int sidx, uint32_t i) {
    const uint2 corner = sh_.corner[sidx];
    const uint32_t C = static_cast<uint32_t>(q.C);
    const uint32_t d = i - (corner.x * C + corner.y);
    // row inside the tile (below 16): the product is exact or one too low (inv_c is 2^-21 low, the roundings add up to less)
    uint32_t dx = static_cast<uint32_t>(static_cast<float>(d) * q.inv_c);
    uint32_t dy = d - dx * C;
    if (dy >= C) { ++dx; dy -= C; }
    const int h = q.h;
    // the window's columns, counted from the tile's first one; at most one side lies in a neighbouring tile
    const int ya = max(static_cast<int>(dy) - h, -static_cast<int>(corner.y));
    const int yb = min(static_cast<int>(dy) + h, q.C - 1 - static_cast<int>(corner.y));
    const int oa = max(static_cast<int>(dx) - h, -static_cast<int>(corner.x));           // ... and rows
    const int ob = min(static_cast<int>(dx) + h, q.R - 1 - static_cast<int>(corner.x));
    const int side = ya < 0 ? -1 : yb >= kTileCols ? 1 : 0;
    int s = sidx, a = max(ya, 0), b = min(yb, kTileCols - 1);
#pragma unroll 1
    for (int part = 0;; ++part) {
        const uint32_t w0 = static_cast<uint32_t>(a) >> 5, b0 = static_cast<uint32_t>(a) & 31u;
        const uint32_t len = static_cast<uint32_t>(b - a + 1), run = (1u << len) - 1u;
        const uint32_t bits0 = run << b0, bits1 = b0 + len > 32u ? run >> (32u - b0) : 0u;
        const uint32_t col = corner.y + static_cast<uint32_t>((s - sidx) * kTileCols + a);
#pragma unroll 1
        for (int o = oa; o <= ob; ++o) {
            int t = s, row = o;
            if (o < 0) { t -= q.tiles_x; row += kTileRows; }
            if (o >= kTileRows) { t += q.tiles_x; row -= kTileRows; }
            if (static_cast<uint32_t>(t) < static_cast<uint32_t>(q.gn)) {
                uint32_t *w = sh_.bits + t * kSlotPitch + row * (kTileCols / 32) + w0;
                atomicOr(w, bits0);
                if (bits1) atomicOr(w + 1, bits1);
            } else {                      // another group's tile: straight into the mask
                const uint32_t pos = static_cast<uint32_t>(static_cast<int>(corner.x) + o) * C + col, word = pos >> 5, sh = pos & 31u;
                uint32_t *w = q.mask + word;
                const uint32_t over = sh + len > 32u ? run >> (32u - sh) : 0u;
                if (!COUNT) {
                    atomicOr(w, run << sh);
                    if (over) atomicOr(w + 1, over);
                } else {                  // ... and the new bits counted
#pragma unroll
                    for (uint32_t j = 0; j < 2u; ++j) {
                        const uint32_t bits = j == 0u ? run << sh : over;
                        if (bits == 0u) continue;
                        const uint32_t fresh = __popc(bits & ~atomicOr(w + j, bits));
                        if (fresh) group_count(q, sh_, word + j, fresh);
                    }
                }
            }
        }
        if (part != 0 || side == 0) break;
        s = sidx + side;
        a = side < 0 ? ya + kTileCols : 0;
        b = side < 0 ? kTileCols - 1 : yb - kTileCols;
    }
}
// The group's words, after a barrier.  Neighbouring tiles of one tile row are neighbours in memory: consecutive threads walk
// along a matrix row through the group's tiles, so a wave writes whole cache lines.  Thread ww of the eight of a tile row writes the
// mask word that begins with the last bits of the row's word ww - 1, if the row does not begin with a mask word; the last
// thread then has a ninth.
template <bool COUNT, int SLOTS>
__device__ __forceinline__ void group_put(const GroupGeom &q, GroupMarks<SLOTS> &sh, uint32_t at, uint32_t word, bool owned) {
    if (word == 0u) return;
    uint32_t *dst = q.mask + at;
    uint32_t fresh = word;
    if (owned) *dst = word;
    else if (COUNT) fresh = word & ~atomicOr(dst, word);
    else atomicOr(dst, word);
    if (COUNT && fresh) group_count(q, sh, at, __popc(fresh));
}
template <bool COUNT, int THREADS, int SLOTS>
__device__ __forceinline__ void group_write(const GroupGeom &q, GroupMarks<SLOTS> &sh) {
    constexpr uint32_t ROW = SLOTS * (kTileCols / 32);              // words of one row through the group
    const uint32_t tid = threadIdx.x, ww = tid & 7u;
    const int sidx = static_cast<int>((tid / 8u) % static_cast<uint32_t>(SLOTS));
    if (sidx < q.gn) {
        const uint2 corner = sh.corner[sidx];
        const int h = q.h, below = q.R - static_cast<int>(corner.x) - kTileRows;             // rows of the matrix below the tile
        const int cols = q.C - static_cast<int>(corner.y);                                   // ... columns from the tile's first on
        // the columns that no other group's candidates reach and that no other tile row shares a word with
        const int c_lo = sidx == 0 && corner.y > 0u ? h : 0;
        const int c_hi = cols <= kTileCols ? cols : sidx == q.gn - 1 ? kTileCols - h : kTileCols;
        for (uint32_t row = tid / ROW; row < static_cast<uint32_t>(kTileRows); row += THREADS / ROW) {
            const uint32_t *bits = sh.bits + sidx * kSlotPitch + row * (kTileCols / 32) + ww;
            const uint32_t pos = (corner.x + row) * static_cast<uint32_t>(q.C) + corner.y, shift = pos & 31u;
            const int rr = static_cast<int>(row), c0 = 32 * static_cast<int>(ww) - static_cast<int>(shift);      // the word's first column
            const bool inner = !((rr < h && corner.x > 0u) || (rr >= kTileRows - h && below > 0));
            uint32_t word = bits[0];
            if (shift) {                  // (uniform where rows are whole words: 0)
                if (ww == 7u) group_put<COUNT>(q, sh, (pos >> 5) + 8u, word >> (32u - shift), false);      // (it goes on beyond the tile)
                word <<= shift;
                if (ww != 0u) word |= bits[-1] >> (32u - shift);
            }
            group_put<COUNT>(q, sh, (pos >> 5) + ww, word, inner && c0 >= c_lo && c0 + 32 <= c_hi);
        }
    }
    static_assert(kGatherCountSlots == 64, "one lane of the first wave per counted chunk");
    if (COUNT) {
        __syncthreads();
        if (tid < 64) count_flush_wave0(q.cctx, q.cl0, sh.ccnt[tid]);
    }
}

// Held to five waves per SIMD.
template <bool COUNT, int PARTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PARTS == 0 ? 4 : 5, 8))) void k_gather(const GatherArgs a, const GatherLists gl) {
    __shared__ GatherShared sh;
    const int tid = threadIdx.x;
    constexpr bool BLOCKS = PARTS == 0;       // block grids: whole groups of slots, and single bits
    if (BLOCKS ? blockIdx.x - gl.n_map_chunks >= gl.n_slot_wgs : blockIdx.x < gl.n_map_chunks) {
        uint32_t c = blockIdx.x, stride = 1u, end = c + 1u;           // a listed chunk ...
        const bool listed = c < gl.n_map_chunks;
        if (!listed) {                    // ... or those of a grid that has no bound in this call
            if (a.flags[0] == 0u) return;
            c -= gl.n_map_chunks + gl.n_slot_wgs;
            stride = gridDim.x - gl.n_map_chunks - gl.n_slot_wgs;
            end = gl.n_chunks;
        }
        for (; c < end; c += stride) {
            ChunkEntry ce;
            uint32_t digit = kNoDigit;
            if (listed) {
                ce = gl.map_chunks[c];
            } else {
                const ChunkInfo ci = gl.chunks[c];
                const SelState &st = a.state[ci.layer];
                if (a.layers[ci.layer].large == 0u || st.mode != kModeFullMap) continue;      // uniform
                if (st.span == 0u && st.done == 0u) {      // its bound failed: the first digit, from the histogram that the rescoring has counted
                    const uint32_t k = a.layers[ci.layer].k;
                    if (tid < 64) {
                        const WaveBucket wb = wave_find_bucket(a.hist + static_cast<size_t>(ci.layer) * kHistBins, k);
                        if (tid == 0) sh.n = wb.found && wb.count != k - wb.above ? wb.bucket : kNoDigit;
                    }
                    __syncthreads();
                    digit = sh.n;
                    __syncthreads();
                    if (digit == kNoDigit) continue;       // nothing left to rank
                }
                ce = ChunkEntry{ci.layer, ci.start, ci.len, 0u, ci.arena_off};
            }
            gather_map_chunk(a, ce, sh, digit);
            if (!BLOCKS) break;
            __syncthreads();
        }
        return;
    }
    // role 1: listed slot groups, 2: fallback walk over all chunks
    const uint32_t wg = blockIdx.x - gl.n_map_chunks;
    const int role = BLOCKS || wg < gl.n_slot_wgs ? 1 : 2;
    const uint32_t first = role == 1 ? wg : wg - gl.n_slot_wgs;
    const uint32_t stride = role == 1 ? gl.n_slot_wgs : gridDim.x - gl.n_map_chunks - gl.n_slot_wgs;
    constexpr int SHARES = BLOCKS ? 1 : PARTS, SLOTS = kSlotGroup / SHARES;
    const uint32_t n_items = role == 1 ? gl.n_cand_groups * SHARES : gl.n_chunks;
    const DirEntry *__restrict__ dir = gl.chunk_dir;
    if (first >= n_items) return;
    if (role == 2 && a.flags[0] == 0u) return;
    // (role 1 counts its few bucket keys in the layer's histogram itself: clearing and flushing 2048 bins in LDS costs a
    // workgroup more than the two or three atomics)
    if (role != 1) {
        if (tid == 0) sh.n = 0;
        for (int b = tid; b < kLevel1Bins; b += 256) sh.hist[b] = 0;
        __syncthreads();
    }

    uint32_t e = role == 2 ? dir_lookup(dir, gl.n_layers, first) : 0u;
    uint32_t cur_l = 0xffffffffu;
    bool active = false;
    uint32_t lo = 0, width = 0, shift1 = 0;   // the current layer's bucket [lo, lo + width) and its second digit's shift
    uint32_t above = 0;                       // candidate layers: scores from here on are selected for certain
    LayerDev L;
    GatherList list = {nullptr, nullptr, 0u};

    for (uint32_t it = first; it < n_items; it += stride) {
        uint32_t l;
        GroupEntry ge = {};
        const unsigned long long *__restrict__ ent0 = nullptr;     // role 1: the group's first slot entry
        if (role == 1) {
            ge = gl.cand_groups[it / SHARES];
            l = ge.layer;
            const uint32_t s0 = (it % SHARES) * SLOTS;
            if (s0 >= ge.ntile) continue;
            ge.slot0 += s0;
            ge.ntile = static_cast<uint8_t>(min(static_cast<uint32_t>(ge.ntile) - s0, static_cast<uint32_t>(SLOTS)));
            ent0 = a.slot_ent + (((static_cast<uint64_t>(ge.ent0_high) << 32) | ge.ent0_low) << 1) + s0 * ge.slot_cap;
        } else {
            e = dir_advance(dir, gl.n_layers, e, it);
            l = dir[e].layer;
        }
        if (l != cur_l) {
            if (active && role != 1) {     // uniform: the finished layer's keys and counts go out
                gather_flush_keys(sh, list);
                uint32_t *__restrict__ gh = a.hist1 + static_cast<size_t>(cur_l) * kLevel1Bins;
                for (int b = tid; b < kLevel1Bins; b += 256) {
                    const uint32_t cc = sh.hist[b];
                    if (cc) { atomicAdd(&gh[b], cc); sh.hist[b] = 0; }
                }
                __syncthreads();
            }
            cur_l = l;
            L = a.layers[l];
            const SelState st = a.state[l];
            active = !st.done && st.mode == (role == 1 ? kModeCandidates : kModeFullMap);
            lo = st.lo;
            width = 1u << st.span;
            shift1 = st.span - kLevel1Bits;
            if (role == 1) {
                // candidates: everything at or above `above` is selected for certain.  A layer whose
                // first digit already settled the ranking (done) has its threshold at lo.
                active = st.mode == kModeCandidates;
                above = st.done ? static_cast<uint32_t>(st.T >> 32) : lo + width;
                if (st.done) width = 0;
            }
            if (role == 2) {
                active = st.mode == kModeFullMap && L.large != 0u;      // (the others are on the list)
                if (active) {              // uniform: first digit from the histogram of the fallback pass
                    if (tid < 64) {
                        const WaveBucket wb = wave_find_bucket(a.hist + static_cast<size_t>(l) * kHistBins, L.k);
                        if (tid == 0) sh.res = DigitResult{wb.bucket, wb.above, wb.count, wb.found};
                    }
                    __syncthreads();
                    const DigitResult r = sh.res;
                    __syncthreads();
                    lo = r.found ? r.digit << kCoarseShift : 0u;
                    width = 1u << kCoarseShift;
                    shift1 = kCoarseShift - kLevel1Bits;
                    if (!r.found || r.count == L.k - r.above) active = false;   // nothing left to rank
                }
            }
            // the workgroup's shard of the layer's list: its own counter (own cache line) and region
            const uint32_t shard = blockIdx.x % L.list_shards;
            list.cap = (BLOCKS ? list_entries(L, true) : L.list_cap) / L.list_shards;
            list.cnt = a.list_cnt + (static_cast<size_t>(l) * kListShards + shard) * kListCntStride;
            list.ent = a.list_ent + L.list_off + static_cast<size_t>(shard) * list.cap;
        }
        if (!active) {
            if (role == 2) {               // on to this workgroup's first chunk of the next layer
                const uint32_t nb = dir[e + 1].begin;
                it += (nb - it + stride - 1) / stride * stride - stride;
            }
            continue;
        }
        if (role != 1) {
            const uint32_t start = (it - L.chunk_begin) * kChunk, len = min(static_cast<uint32_t>(kChunk), L.G - start);
            const uint32_t *__restrict__ src = a.keys + L.elem_off + start;
            // half a chunk is requested before any of it is used
            constexpr int NQ = kChunk / 2048;
#pragma unroll 1
            for (uint32_t half = 0; half < 2u && half * (kChunk / 2) < len; ++half) {
                uint4 q[NQ];
#pragma unroll
                for (int j = 0; j < NQ; ++j) {
                    const uint32_t e4 = half * (kChunk / 2) + j * 1024 + 4 * tid;
                    q[j] = make_uint4(0, 0, 0, 0);
                    if (e4 + 3 < len) {
                        q[j] = *reinterpret_cast<const uint4 *>(src + e4);
                    } else if (e4 < len) {
                        q[j].x = src[e4];
                        if (e4 + 1 < len) q[j].y = src[e4 + 1];
                        if (e4 + 2 < len) q[j].z = src[e4 + 2];
                    }
                }
#pragma unroll
                for (int j = 0; j < NQ; ++j) {
                    const uint32_t e4 = half * (kChunk / 2) + j * 1024 + 4 * tid;
                    if (half * (kChunk / 2) + static_cast<uint32_t>(j) * 1024u >= len) break;       // uniform
                    gather_make_room(sh, list);
                    const uint32_t kk[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
#pragma unroll
                    for (uint32_t c = 0; c < 4; ++c) {
                        const bool hit = e4 + c < len && (kk[c] & 0x7fffffffu) - lo < width;
                        gather_stage_key(sh, hit, composite_key(kk[c], start + e4 + c), lo, shift1);
                    }
                }
            }
        } else if constexpr (BLOCKS) {
            // A block is one bit, and every bit is one key's: nothing is built in LDS but the counts.
            const uint32_t slot_cap = ge.slot_cap, sidx = tid / 16u, j0 = tid % 16u;
            const CountCtx cctx = count_ctx(L, a.chunk_cnt, a.group_cnt);
            uint32_t *const ccnt = sh.marks.ccnt;
            const unsigned long long *__restrict__ slot = ent0 + static_cast<size_t>(sidx) * slot_cap;
            unsigned long long K = 0;
            uint32_t cnt = 0;
            if (sidx < ge.ntile) {
                cnt = min(a.slot_cnt[ge.slot0 + sidx], slot_cap);
                if (j0 < slot_cap) K = slot[j0];
            }
            // the first chunk that the group's tiles reach into (of the tile row of its first one).  The rows of a wide grid lie many
            // chunks apart, but at most two tile rows are meant, and of a row at most two chunks: counted by row.
            const uint32_t tile0 = ge.slot0 - L.tile_begin_all, trow0 = tile0 / L.tiles_x, row0 = trow0 * kBlockTileRows;
            const uint32_t cl0 = static_cast<uint32_t>(static_cast<uint64_t>(row0) * L.C / kChunk);
            const bool wide = L.C >= kWideGrid;
            const uint32_t col0 = wide ? (tile0 - trow0 * L.tiles_x) * (L.C / L.tiles_x) : 0u;      // (not past the first tile's first column)
            auto row_chunk = [&](uint32_t row) { return (row * L.C + (row < row0 + kBlockTileRows ? col0 : 0u)) / kChunk; };
            if (COUNT) {
                if (it != first) __syncthreads();
                if (tid < kGatherCountSlots) ccnt[tid] = 0u;
                __syncthreads();
            }
            for (uint32_t j = j0; j < cnt; j += 16u) {
                const unsigned long long next = j + 16u < cnt ? slot[j + 16u] : 0ull;
                const uint32_t score = static_cast<uint32_t>(K >> 32);
                if (score >= above) {
                    const uint32_t i = ~static_cast<uint32_t>(K), cl = i / kChunk;
                    const size_t pos = static_cast<size_t>(L.elem_off) + i;
                    atomicOr(&a.mask[pos >> 5], 1u << (pos & 31));
                    if (COUNT) {
                        uint32_t at = cl - cl0;
                        if (wide) {
                            const uint32_t row = i / L.C, in_row = cl - row_chunk(row);
                            at = in_row < kWideSlots ? (row - row0) * kWideSlots + in_row : static_cast<uint32_t>(kGatherCountSlots);
                        }
                        if (at < static_cast<uint32_t>(kGatherCountSlots)) atomicAdd(&ccnt[at], 1u);
                        else count_add_chunk(cctx, cl, 1u);
                    }
                } else if (score - lo < width) {
                    const uint32_t pos = atomicAdd(list.cnt, 1u);
                    if (pos < list.cap) list.ent[pos] = K;
                    atomicAdd(&a.hist1[l * kLevel1Bins + ((score - lo) >> shift1)], 1u);
                }
                K = next;
            }
            if (COUNT) {
                __syncthreads();
                if (tid < kGatherCountSlots && !wide) count_flush_wave0(cctx, cl0, ccnt[tid]);
                else if (tid < kGatherCountSlots && ccnt[tid] != 0u) count_add_chunk(cctx, row_chunk(row0 + tid / kWideSlots) + tid % kWideSlots, ccnt[tid]);
            }
        } else {
            const uint32_t slot_cap = ge.slot_cap;
            const CountCtx cctx = count_ctx(L, a.chunk_cnt, a.group_cnt);
            GroupMarks<SLOTS> &marks = *reinterpret_cast<GroupMarks<SLOTS> *>(&sh.marks);      // (a quarter needs less)
            GroupGeom q = group_geom(L, ge.slot0 - L.tile_begin_all, ge.ntile, a.mask, cctx);
            // LPS lanes per tile slot; a round covers as many entries of each.  The first entries are requested
            // beside the slot's count (a slot always has them; past the count they hold anything)
            constexpr uint32_t LPS = 256 / SLOTS;
            const int sidx = tid / static_cast<int>(LPS);
            const uint32_t j0 = static_cast<uint32_t>(tid) % LPS;
            const unsigned long long *__restrict__ slot = ent0 + static_cast<size_t>(sidx) * slot_cap;
            unsigned long long K = 0;
            uint32_t cnt = 0;
            if (sidx < q.gn) {
                cnt = a.slot_cnt[ge.slot0 + static_cast<uint32_t>(sidx)];
                if (j0 < slot_cap) K = slot[j0];
                cnt = min(cnt, slot_cap);
            }
            if (it != first) __syncthreads();                // (the previous group's words are written)
            group_clear<256>(q, marks);
            __syncthreads();
            if (COUNT) q.cl0 = group_first_chunk(q, marks.corner[0]);
            for (uint32_t j = j0; j < cnt; j += LPS) {
                const unsigned long long next = j + LPS < cnt ? slot[j + LPS] : 0ull;        // (on its way while this one is marked)
                const uint32_t score = static_cast<uint32_t>(K >> 32);
                if (score >= above) {                        // selected for certain
                    const uint32_t i = ~static_cast<uint32_t>(K);
                    group_mark<COUNT>(q, marks, sidx, i);
                    if (a.cmask) {
                        const size_t pos = static_cast<size_t>(L.elem_off) + i;
                        atomicOr(&a.cmask[pos >> 5], 1u << (pos & 31));
                    }
                } else if (score - lo < width) {             // in the threshold bucket (never when the layer is done):
                    const uint32_t pos = atomicAdd(list.cnt, 1u);           // few of them, one atomic each
                    if (pos < list.cap) list.ent[pos] = K;
                    atomicAdd(&a.hist1[l * kLevel1Bins + ((score - lo) >> shift1)], 1u);
                }
                K = next;
            }
            __syncthreads();
            group_write<COUNT, 256>(q, marks);
        }
    }
    if (active && role != 1) {
        gather_flush_keys(sh, list);
        uint32_t *__restrict__ gh = a.hist1 + static_cast<size_t>(cur_l) * kLevel1Bins;
        for (int b = tid; b < kLevel1Bins; b += 256) {
            const uint32_t cc = sh.hist[b];
            if (cc) atomicAdd(&gh[b], cc);
        }
    }
}

// --------------------------------------------------------------- filter --
// Only for plans with large layers that are ranked on the full map (a block grid, a keep ratio
// too high for the candidate path): the threshold bucket of such a layer holds hundreds of
// thousands of keys, too many for the one workgroup of k_finish to go through.  kFilterSplit
// workgroups per layer find the second digit (each for itself, from the layer's complete
// histogram) and copy the keys of the list that share it -- a few hundred -- to the layer's
// second, small list, from which k_finish then works.
constexpr int kFilterSplit = 32;
constexpr int kFilterThreads = 1024;
constexpr int kList2Cap = 2048;          // == kStage: what k_finish can hold in LDS

// The layers come as a list (161 layers of which nine are meant: 5152 workgroups of 1024 threads that nearly all leave at once
// took 16 us); beyond kFilterLayers of them every layer gets its workgroups.
constexpr int kFilterLayers = 256;
struct FilterLayers {
    uint32_t listed;
    uint16_t id[kFilterLayers];
};

// The keys K of list[0, n) with K - base < 2^top into `stage` (as many as it holds; *nstage counts them all), by workgroup `sub` of nsub.
__device__ __forceinline__ void filter_keys(const unsigned long long *__restrict__ list, uint32_t n, uint32_t sub, uint32_t nsub, unsigned long long base,
                                            int top, unsigned long long *stage /*[kList2Cap], LDS*/, uint32_t *nstage /*LDS*/) {
    const uint32_t tid = threadIdx.x;
    if (tid == 0) *nstage = 0;
    __syncthreads();
    constexpr uint32_t U = 4;              // independent loads in flight per thread
    for (uint32_t i0 = sub * U * kFilterThreads; i0 < n; i0 += nsub * U * kFilterThreads) {
        unsigned long long K[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * kFilterThreads + tid;
            K[u] = i < n ? list[i] : 0ull;
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (i0 + u * kFilterThreads + tid < n && K[u] >= base && ((K[u] - base) >> top) == 0ull) {
                const uint32_t pos = atomicAdd(nstage, 1u);
                if (pos < static_cast<uint32_t>(kList2Cap)) stage[pos] = K[u];
            }
    }
    __syncthreads();
}

__global__ __launch_bounds__(kFilterThreads) void k_filter(const FilterLayers fl, const LayerDev *__restrict__ layers,
                                                           const SelState *__restrict__ state,
                                                           const uint32_t *__restrict__ hist1,
                                                           const uint32_t *__restrict__ list_cnt,
                                                           const unsigned long long *__restrict__ list_ent,
                                                           uint32_t *__restrict__ list2_cnt,
                                                           unsigned long long *__restrict__ list2_ent) {
    __shared__ uint32_t lh[kLevel1Bins];
    __shared__ unsigned long long stage[kList2Cap];
    __shared__ uint32_t wave_tot[kFilterThreads / 64];
    __shared__ DigitResult res;
    __shared__ uint32_t nstage, base_pos;
    const int part = blockIdx.x % kFilterSplit, tid = threadIdx.x;
    const int l = fl.listed ? fl.id[blockIdx.x / kFilterSplit] : blockIdx.x / kFilterSplit;
    // lane s of every wave reads shard s's counter (unused shards stay 0); issued with the other loads
    const uint32_t *__restrict__ cnt = list_cnt + static_cast<size_t>(l) * kListShards * kListCntStride;
    const uint32_t c = (tid & 63) < kListShards ? cnt[(tid & 63) * kListCntStride] : 0u;
    const SelState st = state[l];
    const LayerDev L = layers[l];
    for (int b = tid; b < kLevel1Bins; b += kFilterThreads) lh[b] = hist1[static_cast<size_t>(l) * kLevel1Bins + b];
    // (a large layer that fell back to the full map has its first digit found in the gather pass only:
    // k_finish goes through its list alone -- rare)
    if (st.done || st.mode != kModeFullMap || L.large != 0u) return;
    uint32_t total = c;
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) total += __shfl_xor(total, d, 64);
    total = __shfl(total, 0, 64);
    const uint32_t shards = L.list_shards, cap = L.list_cap / shards;
    if (total <= static_cast<uint32_t>(kList2Cap) || __syncthreads_or(c > cap)) return;   // small enough, or overflowed
    const DigitResult r = block_find_digit<kFilterThreads / 64>(lh, kLevel1Bins, st.k_rem, wave_tot, &res);
    if (!r.found || r.count == st.k_rem - r.above) return;       // nothing left to rank below this digit
    const uint32_t sh1 = st.span - kLevel1Bits;
    const unsigned long long base = (static_cast<unsigned long long>(st.lo) << 32) +
                                    (static_cast<unsigned long long>(r.digit) << (32 + sh1));
    const int top = 32 + static_cast<int>(sh1);
    // this workgroup's shard, and its share of that shard
    const uint32_t shard = part % shards, sub = part / shards, nsub = (kFilterSplit + shards - 1 - shard) / shards;
    const uint32_t n = __shfl(c, static_cast<int>(shard), 64);
    const unsigned long long *__restrict__ list = list_ent + L.list_off + static_cast<size_t>(shard) * cap;
    filter_keys(list, n, sub, nsub, base, top, stage, &nstage);
    const uint32_t m = nstage;
    if (m == 0) return;                    // uniform
    if (tid == 0) base_pos = atomicAdd(&list2_cnt[l], m);        // counts past the capacity too
    __syncthreads();
    const uint32_t b0 = base_pos;
    for (uint32_t i = tid; i < min(m, static_cast<uint32_t>(kList2Cap)); i += kFilterThreads)
        if (b0 + i < static_cast<uint32_t>(kList2Cap))
            list2_ent[static_cast<size_t>(l) * kList2Cap + b0 + i] = stage[i];
}

// --------------------------------------------------------------- finish --
// One workgroup (1024 threads) per layer finishes the ranking: second digit from the layer's
// histogram; if the k-th rank is still inside a bucket of several keys, the bucket's keys are
// staged in LDS from the layer's list and the remaining score bits and -- only if equal
// scores straddle the k-th rank -- the bits of ~index are resolved there, so that the lower
// index wins.  Slow but exact routes: if the bucket's keys do not fit the stage, each further
// digit streams the list again; if the list itself overflowed (a huge number of nearly equal
// scores, e.g. an all-zero layer), each digit streams the layer's keys from the score map or
// the tile slots.
// What one workgroup hands to others of the launch goes through these two, past the caches of an XCD, and wait_stores waits until
// it is out.  (A fence at device scope instead writes back and invalidates the XCD's whole L2, once per wave: a call with a failed
// bound on 1024 x 1024 took 284 us with fences where it took 106 without.)
template <typename T>
__device__ __forceinline__ void agent_store(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T agent_load(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }      // a wave's own stores and adds

constexpr int kFinishThreads = 1024;
constexpr int kFinishWaves = kFinishThreads / 64;

// Calls f(K) for every key of a layer's list.  `c` holds, in lane s of every wave, the number of
// keys in shard s.  The shards are walked side by side -- one load per shard in flight per
// thread -- rather than one after the other: a shard of a few hundred keys is one round trip to
// memory, and sixteen of them in a row were most of this kernel's time.
template <typename F>
__device__ __forceinline__ void for_each_list_key(const unsigned long long *__restrict__ list, uint32_t shards,
                                                  uint32_t cap, uint32_t c, F f) {
    uint32_t longest = c;
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) longest = max(longest, __shfl_xor(longest, d, 64));
    longest = __shfl(longest, 0, 64);
    for (uint32_t i = threadIdx.x; i < longest + threadIdx.x; i += kFinishThreads) {   // (the same trip count in every thread)
        unsigned long long K[kListShards];
        bool have[kListShards];
#pragma unroll
        for (int s = 0; s < kListShards; ++s) {
            have[s] = static_cast<uint32_t>(s) < shards && i < __shfl(c, s, 64);
            K[s] = have[s] ? list[static_cast<size_t>(s) * cap + i] : 0ull;
        }
#pragma unroll
        for (int s = 0; s < kListShards; ++s)
            if (have[s]) f(K[s]);
    }
}

// kCountBeside: the kept elements that the gather has marked, counted by workgroups of this launch
// beside the ranking, which leaves most of the chip idle; k_mark adds the few that the threshold buckets contribute.  Ranking, marks and
// a counting launch behind them / ranking with counts and marks that count: VGG-19 6.4 + 4.5 + 9.3 / 12.1 + 6.2 us, in one arena, where
// more keys lie in the buckets, 9.8 + 6.4 + 9.1 / 10.8 + 8.2, 25088 x 4096 with p = 5 the call 250.9 -> 247.5.  Not with more layers, which the
// ranking and the marks have workgroups enough for already, nor where most tiles are marked from the map (the rule: kBesideLayers).
struct CountShare {
    const CountGroup *groups;      // null: nothing is counted here
    uint32_t n_groups;
    const uint32_t *mask;
    uint32_t *chunk_cnt, *group_cnt;
    uint32_t gstride;
};
// By whole workgroups of NW waves; a wave takes four chunks, 16 lanes and 256 mask words each, four waves a CountGroup.
template <int NW>
__device__ __forceinline__ void count_chunks(const CountShare &cs, uint32_t wg, uint32_t *wave_tot /*[2 NW], LDS*/) {
    static_assert(kCountChunks == 16 && NW % 4 == 0, "four waves of four chunks");
    constexpr int N = kChunk / 32 / 32;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), which = wg * (NW / 4) + wave / 4u;
    uint32_t n = 0, group = 0;
    if (which < cs.n_groups) {
        const CountGroup gr = cs.groups[which];
        group = gr.group;
        const uint32_t chunk = wave % 4u * 4u + lane / 16u, first = chunk * (kChunk / 32);
        uint2 w[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {      // (a layer starts at a whole pair of words and is padded to one)
            const uint32_t i = first + 2u * (lane % 16u + 16u * j);
            w[j] = i < gr.n_words ? *reinterpret_cast<const uint2 *>(cs.mask + gr.word0 + i) : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) n += __popc(w[j].x) + __popc(w[j].y);
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
        if (lane % 16u == 0u && n != 0u) cs.chunk_cnt[gr.first_chunk + chunk] = n;      // (cleared by the find0 launch)
        n += __shfl_xor(n, 16, 64);
        n += __shfl_xor(n, 32, 64);
    }
    if (lane == 0u) {
        wave_tot[wave] = n;
        wave_tot[NW + wave] = group;
    }
    __syncthreads();
    if (threadIdx.x < static_cast<uint32_t>(NW / 4)) {
        n = wave_tot[4 * threadIdx.x] + wave_tot[4 * threadIdx.x + 1] + wave_tot[4 * threadIdx.x + 2] + wave_tot[4 * threadIdx.x + 3];
        if (n != 0u) atomicAdd(&cs.group_cnt[static_cast<size_t>(wave_tot[NW + 4 * threadIdx.x]) * cs.gstride], n);
    }
}

constexpr int kFinishCtl = 8;      // this word of a layer's last list shard's line: how many of its workgroups have picked their keys
// GRIDS (block plans that take the candidate path): in a call that ranks a large grid on its map -- it has no bound, or its bound failed -- the
// bucket's list is as long as those that k_filter is for.  But a launch that nearly every call has nothing to do for costs 4 us, so such a
// grid has kFilterSplit workgroups here instead: each picks the keys of its `part` of the list, and the last of them to be done with that
// (nobody waits for another) goes on to rank them.  With one workgroup per grid this kernel took 91 us on VGG-19 without bounds, where
// k_filter and k_finish took 7 + 9; now 13.
template <bool GRIDS>
__device__ __forceinline__ void finish_layer(int l, uint32_t part, const LayerDev *__restrict__ layers,
    SelState *__restrict__ state, const uint32_t *__restrict__ hist, const uint32_t *__restrict__ hist1, uint32_t *__restrict__ list_cnt,
    const unsigned long long *__restrict__ list_ent, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ slot_cnt,
    const unsigned long long *__restrict__ slot_ent, uint32_t *__restrict__ list2_cnt, unsigned long long *__restrict__ list2_ent,
    PredState *__restrict__ pred /* nullable */) {
    __shared__ uint32_t lh[kLevel1Bins];
    __shared__ unsigned long long sel[kStage];
    __shared__ uint32_t wave_tot[kFinishWaves];
    __shared__ DigitResult res;
    __shared__ uint32_t nstage, ticket;
    __shared__ unsigned long long rank_key;
    const int tid = threadIdx.x;
    if (tid == 0) rank_key = 0ull;
    // lane s of every wave reads shard s's counter (unused shards stay 0); issued with the other loads
    const uint32_t *cnt = list_cnt + static_cast<size_t>(l) * kListShards * kListCntStride;
    const uint32_t c = (tid & 63) < kListShards ? cnt[(tid & 63) * kListCntStride] : 0u;
    uint32_t n2 = GRIDS ? 0u : list2_cnt[l];     // keys that k_filter has already picked from a long list (0: none)
    const SelState st = state[l];
    const LayerDev L = layers[l];
    // (the state of a grid with several workgroups is written when all of them have read it)
    const bool several = GRIDS && L.G >= static_cast<uint32_t>(kBigMapLayer) && st.mode == kModeFullMap;
    if (part != 0u && !several) return;
    for (int b = tid; b < kLevel1Bins; b += kFinishThreads) lh[b] = hist1[static_cast<size_t>(l) * kLevel1Bins + b];
    if (st.done || st.mode == kModeSkip) return;
    __syncthreads();
    uint32_t lo = st.lo, span = st.span, k_rem = st.k_rem;
    // (a grid's last workgroup goes on; of every other layer its only one)
    auto is_last = [&]() {
        if (!several) return true;
        wait_stores();
        __syncthreads();
        if (tid == 0) ticket = atomicAdd(list_cnt + (static_cast<size_t>(l) * kListShards + kListShards - 1) * kListCntStride + kFinishCtl, 1u);
        __syncthreads();
        return ticket == static_cast<uint32_t>(kFilterSplit) - 1u;
    };
    if (st.mode == kModeFullMap && L.large != 0u && span == 0u) {
        // a large layer that fell back to the full map: its first digit, as the gather pass found it
        __shared__ uint32_t lh0[kHistBins];
        for (int b = tid; b < kHistBins; b += kFinishThreads) lh0[b] = hist[static_cast<size_t>(l) * kHistBins + b];
        __syncthreads();
        const DigitResult r0 = block_find_digit<kFinishWaves>(lh0, kHistBins, L.k, wave_tot, &res);
        lo = r0.found ? r0.digit << kCoarseShift : 0u;
        span = kCoarseShift;
        k_rem = r0.found ? L.k - r0.above : 0u;
        if (!r0.found || r0.count == k_rem) {      // nothing left to rank
            if (is_last() && tid == 0) {
                SelState ns = st;
                ns.T = static_cast<unsigned long long>(lo) << 32;
                ns.lo = lo;
                ns.span = span;
                ns.k_rem = k_rem;
                ns.done = 1;
                state[l] = ns;
                publish_threshold(pred, l, L.large, L.k, ns.T);
            }
            return;
        }
    }
    const uint32_t shards = L.list_shards, cap = (GRIDS ? list_entries(L, st.mode == kModeCandidates) : L.list_cap) / shards;
    const bool use_list = __syncthreads_and(c <= cap) != 0;      // every shard of the list fits
    DigitResult r = block_find_digit<kFinishWaves>(lh, kLevel1Bins, k_rem, wave_tot, &res);
    const uint32_t sh1 = span - kLevel1Bits;                     // score bits still open after this digit
    unsigned long long T = static_cast<unsigned long long>(lo) << 32;
    bool done = !r.found;                  // fewer keys than k_rem (cannot happen for finite input)
    if (r.found) {
        T += static_cast<unsigned long long>(r.digit) << (32 + sh1);
        k_rem -= r.above;
        done = r.count == k_rem;           // whole bucket taken: the threshold is its lower edge
    }
    if constexpr (GRIDS) {
        uint32_t total = c;
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) total += __shfl_xor(total, d, 64);
        total = __shfl(total, 0, 64);
        const bool long_list = several && !done && use_list && total > static_cast<uint32_t>(kStage);
        if (long_list) {                   // (as in k_filter)
            const uint32_t shard = part % shards, sub = part / shards, nsub = (kFilterSplit + shards - 1 - shard) / shards;
            filter_keys(list_ent + L.list_off + static_cast<size_t>(shard) * cap, __shfl(c, static_cast<int>(shard), 64), sub, nsub, T,
                        32 + static_cast<int>(sh1), sel, &nstage);
            const uint32_t m = nstage;
            __syncthreads();
            if (m != 0u) {                 // uniform
                if (tid == 0) nstage = atomicAdd(&list2_cnt[l], m);
                __syncthreads();
                const uint32_t b0 = nstage;
                for (uint32_t i = tid; i < min(m, static_cast<uint32_t>(kStage)); i += kFinishThreads)
                    if (b0 + i < static_cast<uint32_t>(kStage)) agent_store(&list2_ent[static_cast<size_t>(l) * kList2Cap + b0 + i], sel[i]);
                __syncthreads();           // (nstage is used again)
            }
        }
        if (!is_last()) return;            // uniform
        if (long_list) n2 = agent_load(&list2_cnt[l]);
    }
    if (!done) {
        // Keys still in question: K - T < 2^(32 + sh1).  Their remaining bits are ranked as the
        // number rel = K - T, most significant digit first.
        const unsigned long long base = T;
        const int top = 32 + static_cast<int>(sh1);
        const unsigned long long *__restrict__ list = list_ent + L.list_off;
        uint32_t nsel = 0xffffffffu;
        if (use_list && n2 != 0u && n2 <= static_cast<uint32_t>(kStage)) {   // already picked by k_filter
            for (uint32_t i = tid; i < n2; i += kFinishThreads)
                sel[i] = (GRIDS ? agent_load(&list2_ent[static_cast<size_t>(l) * kList2Cap + i]) : list2_ent[static_cast<size_t>(l) * kList2Cap + i]) - base;
            __syncthreads();
            nsel = n2;
        } else if (use_list) {             // stage the bucket's keys
            if (tid == 0) nstage = 0;
            __syncthreads();
            for_each_list_key(list, shards, cap, c, [&](unsigned long long K) {
                if (K >= base && ((K - base) >> top) == 0ull) {
                    const uint32_t pos = atomicAdd(&nstage, 1u);
                    if (pos < static_cast<uint32_t>(kStage)) sel[pos] = K - base;
                }
            });
            __syncthreads();
            nsel = nstage;
        }
        const bool staged = nsel <= static_cast<uint32_t>(kStage);
        unsigned long long Trel = 0;
        int shift_prev = top;
        if (nsel <= 64u) {
            // The usual case: a lane per key counts the larger ones (all keys differ); the one with k_rem - 1 of them is the
            // threshold.  (Digit by digit that took up to twenty barriers of sixteen waves: 11.4 us on VGG-19, now 9.7.)
            if (tid < 64) {
                const unsigned long long own = static_cast<uint32_t>(tid) < nsel ? sel[tid] : 0ull;
                uint32_t larger = 0;
                for (uint32_t j = 0; j < nsel; ++j) {
                    const unsigned long long o = static_cast<unsigned long long>(__builtin_amdgcn_readlane(static_cast<uint32_t>(own >> 32), j)) << 32 |
                                                 static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(own), j));
                    larger += o > own ? 1u : 0u;
                }
                if (static_cast<uint32_t>(tid) < nsel && larger == k_rem - 1u) rank_key = own;
            }
            __syncthreads();
            Trel = rank_key;               // (1 <= k_rem <= nsel: the digit's count, as histogram and list agree)
            k_rem = 1;
            done = true;
        }
#pragma unroll 1
        for (int lv = 0; lv < 4 && !done; ++lv) {
            const int shift = lv == 0 ? 32 : lv == 1 ? 21 : lv == 2 ? 10 : 0;
            const int nb = 1 << (shift_prev - shift);            // 2^sh1 (4 or 256), 2048, 2048, 1024
            __syncthreads();
            for (int b = tid; b < nb; b += kFinishThreads) lh[b] = 0;
            __syncthreads();
            const unsigned long long want = Trel >> shift_prev;
#define RSDGC_COUNT_KEY(K_)                                                                         \
    {                                                                                               \
        const unsigned long long k_ = (K_);                                                         \
        if (k_ >= base && ((k_ - base) >> shift_prev) == want)                                      \
            atomicAdd(&lh[static_cast<uint32_t>((k_ - base) >> shift) & (nb - 1)], 1u);             \
    }
            if (staged) {
                for (uint32_t i = tid; i < nsel; i += kFinishThreads) {
                    const unsigned long long rel = sel[i];
                    if ((rel >> shift_prev) == want) atomicAdd(&lh[static_cast<uint32_t>(rel >> shift) & (nb - 1)], 1u);
                }
            } else if (use_list) {
                for_each_list_key(list, shards, cap, c, [&](unsigned long long K) { RSDGC_COUNT_KEY(K) });
            } else if (st.mode == kModeFullMap) {
                const uint32_t *__restrict__ src = keys + L.elem_off;
                for (uint32_t i = tid; i < L.G; i += kFinishThreads) RSDGC_COUNT_KEY(composite_key(src[i], i))
            } else {
                for (uint32_t t = tid >> 8; t < L.n_tiles; t += kFinishThreads / 256) {
                    const uint32_t n = min(slot_cnt[L.tile_begin_all + t], L.slot_cap);
                    const unsigned long long *__restrict__ ent = slot_ent + L.slot_off + static_cast<size_t>(t) * L.slot_cap;
                    for (uint32_t i = tid & 255; i < n; i += 256) RSDGC_COUNT_KEY(ent[i])
                }
            }
#undef RSDGC_COUNT_KEY
            __syncthreads();
            r = block_find_digit<kFinishWaves>(lh, nb, k_rem, wave_tot, &res);
            if (!r.found) break;           // fewer keys than k_rem (cannot happen for finite input)
            Trel |= static_cast<unsigned long long>(r.digit) << shift;
            k_rem -= r.above;
            done = r.count == k_rem;       // whole bucket taken: lower digits stay 0
            shift_prev = shift;
        }
        T = base + Trel;
    }
    if (tid == 0) {
        SelState ns = st;
        ns.T = T;
        ns.k_rem = k_rem;
        ns.done = 1;
        ns.lo = lo;
        ns.span = span;
        state[l] = ns;
        publish_threshold(pred, l, L.large, L.k, T);
    }
}
__global__ __launch_bounds__(kFinishThreads) void k_finish(const LayerDev *__restrict__ layers, uint32_t n_layers, const CountShare cs,
    SelState *__restrict__ state, const uint32_t *__restrict__ hist, const uint32_t *__restrict__ hist1, uint32_t *__restrict__ list_cnt,
    const unsigned long long *__restrict__ list_ent, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ slot_cnt,
    const unsigned long long *__restrict__ slot_ent, uint32_t *__restrict__ list2_cnt, unsigned long long *__restrict__ list2_ent,
    PredState *__restrict__ pred /* nullable */) {
    if (blockIdx.x >= n_layers) {
        __shared__ uint32_t tot[2 * kFinishWaves];
        count_chunks<kFinishWaves>(cs, blockIdx.x - n_layers, tot);
        return;
    }
    finish_layer<false>(blockIdx.x, 0u, layers, state, hist, hist1, list_cnt, list_ent, keys, slot_cnt, slot_ent, list2_cnt, list2_ent, pred);
}
// Workgroups: the layers', those that count, then kFilterSplit - 1 more for each of the listed grids (the large ones).
__global__ __launch_bounds__(kFinishThreads) void k_finish_grids(const LayerDev *__restrict__ layers, uint32_t n_layers, const CountShare cs,
    SelState *__restrict__ state, const uint32_t *__restrict__ hist, const uint32_t *__restrict__ hist1, uint32_t *__restrict__ list_cnt,
    const unsigned long long *__restrict__ list_ent, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ slot_cnt,
    const unsigned long long *__restrict__ slot_ent, uint32_t *__restrict__ list2_cnt, unsigned long long *__restrict__ list2_ent,
    PredState *__restrict__ pred /* nullable */,
    const FilterLayers big, uint32_t n_count_wgs) {
    const uint32_t b = blockIdx.x, others = n_layers + n_count_wgs;
    if (b >= n_layers && b < others) {
        __shared__ uint32_t tot[2 * kFinishWaves];
        count_chunks<kFinishWaves>(cs, b - n_layers, tot);
        return;
    }
    const uint32_t more = b - others;
    const bool own = b < n_layers;
    finish_layer<true>(own ? static_cast<int>(b) : big.id[more / (kFilterSplit - 1)], own ? 0u : 1u + more % (kFilterSplit - 1), layers, state, hist,
                       hist1, list_cnt, list_ent, keys, slot_cnt, slot_ent, list2_cnt, list2_ent, pred);
}

// --------------------------------------------------------------- select --
// Small plans, every layer on the candidate path: what find0, gather, finish and mark do on others, in one launch, where each of
// those was a launch of 3 to 6 us for a microsecond's work.  A workgroup of 1024 threads per group of tile slots.  It reads the
// first digit off its layer's fine bins, then -- every group of a layer the same -- the threshold bucket's keys from all
// of the layer's slots (a few per tile: reading them again and again costs less than handing them over), ranks those in LDS, and
// marks the windows of its own tiles' candidates that reach the threshold.  Nothing passes between workgroups -- unless a layer's
// bound failed: such a layer is ranked on its full score map (select_failed).
// What bounds it is a chain of six or seven dependent loads.  Kernels, before / now (find0 to mark, four launches / k_select): 512 x 512
// 19.7 / 10.4 us, ResNet-18 25.0 / 14.0, ResNet-50 32.0 / 21.6; calls 31.2 -> 22.6, 63.8 -> 53.1, 108.2 -> 95.9 us.  (The 68 bytes
// of scratch belong to select_failed: without it the kernel takes as long.)
// The rule (build_tables): up to 4096 chunks, as for all that counts where it marks; a layer's slots' counts fit the threads
// (kSelectTiles); and its candidates, which all of its workgroups read, are few enough (kSelectMaxK).
constexpr int kSelectThreads = 1024;
constexpr int kSelectWaves = kSelectThreads / 64;
static_assert(kSelectThreads == kFineBins && kSelectWaves == kSlotGroup, "a bin per thread, a tile slot per wave");
constexpr int kSelectList = 2048;        // keys of a threshold bucket that are ranked in LDS
constexpr int kSelectRun = 4;            // a failed bound: tiles that a workgroup marks at a time

struct SelectArgs {
    const LayerDev *layers;
    const GroupEntry *groups;
    SelState *state;
    PredState *pred;
    const uint32_t *hist_s;
    const uint32_t *slot_cnt;
    const unsigned long long *slot_ent;
    uint32_t *mask, *cmask, *chunk_cnt, *group_cnt;
    // where a bound failed
    const float *grad, *resid, *mom;
    float *v_out, *mom_out;
    float m;
    uint32_t *map, *hist, *hist1, *list_cnt;
    unsigned long long *list_ent;
    double alpha;
    uint32_t n_layers, n_groups;          // workgroups from n_groups on: helpers
};
struct SelectShared {
    union {
        struct {
            union {
                GroupMarks<kSlotGroup> marks;
                GroupMarks<kSelectRun> run;           // a failed bound
            };
            unsigned long long key[kSelectList];      // the threshold bucket's keys, less its lower edge
            uint32_t lh[kLevel1Bins];
        };
        struct {                                      // a failed bound: a tile of v with its halo, the first digit's counts
            float tile[(kTileRows + RSDGC_MAX_P - 1) * (kTileCols + RSDGC_MAX_P - 1)];
            uint32_t hist[kHistBins];
        };
    };
    uint32_t wave_tot[kSelectWaves];
    DigitResult res;
    unsigned long long rank_key;
    uint32_t n, ticket;
};

// What is the same in every lane, moved to scalar registers: branches on it go round what they skip.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ DigitResult uniform_digit(const DigitResult &r) {
    return DigitResult{uniform_u32(r.digit), uniform_u32(r.above), uniform_u32(r.count), uniform_u32(r.found)};
}

// The recorded candidates of a layer, by the whole workgroup: a wave takes every 16th slot, a lane's count each, and goes through
// their entries 64 at a time, wherever one slot ends and the next begins (slots hold a few entries or many; with threads
// tied to slots the longest slot of every wave was a chain of loads: 5.4 of 18 us on ResNet-18, 9.5 of 23 on ResNet-50).
struct SlotScan {
    static constexpr int U = 4;           // entries of a lane on their way at once
    const unsigned long long *ents;
    uint32_t cap, wave;
    uint32_t incl, total;                 // entries of the wave's slots up to the lane's; of all of them
    __device__ __forceinline__ void set(const LayerDev &L, const unsigned long long *slot_ent, uint32_t count /* of slot wave + 16 lane */) {
        const uint32_t lane = threadIdx.x & 63u;
        wave = threadIdx.x >> 6;
        ents = slot_ent + L.slot_off;
        cap = L.slot_cap;
        incl = min(count, cap);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(incl, d, 64);
            if (lane >= static_cast<uint32_t>(d)) incl += o;
        }
        total = __builtin_amdgcn_readlane(incl, 63);
    }
    __device__ __forceinline__ void load(unsigned long long (&K)[U], uint32_t e0) const {
        const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            K[u] = 0ull;                  // (not a candidate's key: those have scores above 0)
            const uint32_t e = e0 + 64u * u + lane;
            uint32_t s = 0;               // slots (of the wave) that end at or before entry e
#pragma unroll
            for (uint32_t step = 32; step >= 1u; step >>= 1)
                if (__shfl(incl, static_cast<int>(s + step - 1u), 64) <= e) s += step;
            const uint32_t before = __shfl(incl, static_cast<int>(s) - 1, 64);
            if (e < total) K[u] = ents[(wave + 16u * s) * cap + (e - (s ? before : 0u))];
        }
    }
    template <typename F>
    __device__ __forceinline__ void rest(unsigned long long (&K)[U], F f) const {      // K: the entries from 0 on
#pragma unroll 1
        for (uint32_t e0 = 0;;) {
#pragma unroll
            for (int u = 0; u < U; ++u) f(K[u]);
            e0 += 64u * U;
            if (e0 >= total) break;       // (the whole wave)
            load(K, e0);
        }
    }
};

// block_find_digit for the nb bins of sh.lh: two a thread.
__device__ __forceinline__ DigitResult select_digit(SelectShared &sh, int nb, uint32_t k_rem) {
    static_assert(kLevel1Bins == 2 * kSelectThreads, "two bins a thread");
    const int hi = nb - 2 * static_cast<int>(threadIdx.x);
    const uint32_t v0 = hi > 0 ? sh.lh[hi - 1] : 0u, v1 = hi > 0 ? sh.lh[hi - 2] : 0u;      // (nb is even)
    if (threadIdx.x == 0) sh.res.found = 0u;
    const uint32_t incl = block_scan_incl_n<kSelectWaves>(v0 + v1, sh.wave_tot), excl = incl - v0 - v1;
    if (excl < k_rem && k_rem <= incl) {
        const bool top = excl + v0 >= k_rem;
        sh.res = DigitResult{static_cast<uint32_t>(hi - (top ? 1 : 2)), top ? excl : excl + v0, top ? v0 : v1, 1u};
    }
    __syncthreads();
    const DigitResult r = uniform_digit(sh.res);
    __syncthreads();
    return r;
}

// The k_rem-th largest of n numbers below 2^top: from sh.key, if they fit there, else scan(f) calls f for each of them (until what
// is left fits).
template <typename S>
__device__ __forceinline__ unsigned long long select_rank(SelectShared &sh, uint32_t n, uint32_t k_rem, int top, S scan) {
    const uint32_t tid = threadIdx.x;
    if (n <= 64u) {                       // a lane per number counts the larger ones (all differ)
        if (tid < 64u) {
            const unsigned long long own = tid < n ? sh.key[tid] : 0ull;
            uint32_t larger = 0;
            for (uint32_t j = 0; j < n; ++j) {
                const unsigned long long o = static_cast<unsigned long long>(__builtin_amdgcn_readlane(static_cast<uint32_t>(own >> 32), j)) << 32 |
                                             static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(own), j));
                larger += o > own ? 1u : 0u;
            }
            if (tid < n && larger == k_rem - 1u) sh.rank_key = own;
        }
        __syncthreads();
        return sh.rank_key;
    }
    unsigned long long T = 0;
#pragma unroll 1
    for (int left = top; left > 0;) {     // digit by digit: at most five, and nearly always one
        const int bits = min(left, kLevel1Bits), shift = left - bits, nb = 1 << bits;
        __syncthreads();
        for (int b = tid; b < nb; b += kSelectThreads) sh.lh[b] = 0u;
        __syncthreads();
        auto count = [&](unsigned long long rel) {
            wave_count(sh.lh, static_cast<uint32_t>(rel >> shift) & (nb - 1), rel >> left == T >> left);
        };
        if (n <= static_cast<uint32_t>(kSelectList)) {
            for (uint32_t i = tid; i < n; i += kSelectThreads) count(sh.key[i]);
        } else {
            scan(count);
        }
        __syncthreads();
        const DigitResult d = select_digit(sh, nb, k_rem);
        T |= static_cast<unsigned long long>(d.digit) << shift;
        k_rem -= d.above;
        if (d.count == k_rem) break;      // all of them: lower digits stay 0
        left = shift;
        if (n > static_cast<uint32_t>(kSelectList) && d.count <= static_cast<uint32_t>(kSelectList)) {
            if (tid == 0) sh.n = 0u;
            __syncthreads();
            scan([&](unsigned long long rel) {
                if (rel >> left != T >> left) return;
                const uint32_t pos = atomicAdd(&sh.n, 1u);
                if (pos < static_cast<uint32_t>(kSelectList)) sh.key[pos] = rel;
            });
            n = d.count;
        }
    }
    return T;
}

// A failed bound: the layer is ranked on its full score map, as the fallback kernels of other plans do it.  Four steps, each cut
// into shares: scores, map and first digit (a tile); the threshold bucket's keys and their second digit (a chunk); the
// ranking (one share); the marks (a run of tiles).  Shares are taken by tickets in order: by the workgroups of the layer's own
// groups, by those of other failed layers when theirs are done, and by workgroups that the launch of a plan of few groups has for
// nothing else (without a failed layer they leave after one look at the layers: no difference to the call).  A share waits until all
// shares of the step before are done.  Those have lower tickets: they were taken by workgroups that are running, which go through
// a ticket that they hold without waiting for anything but still lower ones -- so every wait ends, however few
// workgroups are on the GPU at a time.
// What bounds it is the scores' arithmetic, about 5 us of a CU for a tile, and, on small layers, some thirty dependent loads and
// atomics.  A call all of whose bounds fail, with the launches that this one replaced / with scores formed from global loads by the
// layer's own groups alone / now: 512 x 512 with p = 3 56 / 310 / 47 us, 1024 x 1024 with p = 1 68 / 276 / 62, p = 3 64 / 371 / 60,
// p = 7 70 / 911 / 69, 2048 x 2048 with p = 3 89 / 412 / 98, p = 7 97 / 952 / 119, ResNet-18 175 / 602 / 181, ResNet-50
// 352 / 1225 / 343; one all-zero layer of a million elements, whose ties have one workgroup go through the map
// again and again, 3000 / 4230 / 1590.
constexpr int kSelectCtl = 8;            // this word of the layer's last list shards' lines: the tickets, then the shares done of the first three steps
// Workgroups of the launch, if its groups are fewer: one per CU, two in a plan of many groups (and so of several layers: 512
// workgroups on the tickets of one layer of 4 M elements took 125 us a call, 256 of them 98, and 256 on ResNet-18 / 50 with all
// bounds failed 192 / 383, 512 of them 181 / 343).
__host__ __device__ constexpr uint32_t select_workgroups(uint32_t n_groups) { return n_groups < 128u ? kNumCUs : 2u * kNumCUs; }
static_assert(kHistBins == 4 * kSelectThreads && kChunk == 8 * kSelectThreads && kListShards == kSelectWaves && kTileRows * kTileCols == 4 * kSelectThreads,
              "bins, keys, shards and scores per thread");

__device__ __forceinline__ void select_shares_done(uint32_t *done, uint32_t n) {
    wait_stores();
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(done, n);
}
__device__ __forceinline__ void select_wait(uint32_t *done, uint32_t n) {
    if (threadIdx.x == 0)
        while (agent_load(done) < n) __builtin_amdgcn_s_sleep(8);
    __syncthreads();
    asm volatile("" ::: "memory");        // (nothing is read before)
}
// i: 0 the tickets, 1 .. 3 the shares done.  (A cache line each: who waits reads his again and again.)
__device__ __forceinline__ uint32_t *select_ctl(uint32_t *list_cnt, uint32_t l, int i) {
    return list_cnt + (static_cast<size_t>(l) * kListShards + kListShards - 1 - i) * kListCntStride + kSelectCtl;
}
// First ticket of each step, and the number of tickets.
struct SelectTickets {
    uint32_t keys, rank, marks, end;
};
__device__ __forceinline__ SelectTickets select_tickets(const LayerDev &L) {
    SelectTickets s;
    s.keys = L.n_tiles;
    s.rank = s.keys + L.n_chunks;
    s.marks = s.rank + 1u;
    s.end = s.marks + (L.n_tiles + kSelectRun - 1) / kSelectRun;
    return s;
}

// The kernel's arguments and a layer's constants, read anew where they are wanted, into scalar registers: this code shares its
// registers with a kernel that is held to 64 of them, and what was kept in scratch memory instead cost the calls that come here 40 us.
__device__ __forceinline__ const SelectArgs &select_args() {
    auto *p = (const __attribute__((address_space(4))) SelectArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const SelectArgs *)p;
}
__device__ __forceinline__ const LayerDev &select_layer(const SelectArgs &a, uint32_t l) {
    auto *p = (const __attribute__((address_space(4))) LayerDev *)(a.layers + l);
    asm volatile("" : "+s"(p));
    return *(const LayerDev *)p;
}

// The next ticket: requested by thread 0 while it works on the one before (behind that one's loads, or they would be waited for
// together); handed to all.
__device__ __forceinline__ uint32_t select_hand_over(SelectShared &sh, uint32_t ticket) {
    __syncthreads();
    if (threadIdx.x == 0) sh.ticket = ticket;
    __syncthreads();
    return uniform_u32(sh.ticket);
}
__device__ __forceinline__ uint32_t select_request(uint32_t *ctl) { return threadIdx.x == 0 ? atomicAdd(ctl, 1u) : 0u; }

// v, scores and first digit of a tile (sh.hist: the workgroup's counts).  Returns the next ticket.
template <int P>
__device__ __forceinline__ uint32_t select_map_tile(SelectShared &sh, uint32_t l, uint32_t local, uint32_t *ctl) {
    const SelectArgs &a = select_args();
    const LayerDev &L = select_layer(a, l);
    constexpr int H = (P - 1) / 2, ROWS = kTileRows + 2 * H, PITCH = kTileCols + 2 * H, N = (ROWS * PITCH + kSelectThreads - 1) / kSelectThreads;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));         // (or the places of a thread's pieces are worked out before the loop over the tiles, and spilled)
    const uint32_t trow = local / L.tiles_x;
    const int R = static_cast<int>(L.R), C = static_cast<int>(L.C);
    const int x0 = static_cast<int>(trow) * kTileRows, y0 = static_cast<int>(local - trow * L.tiles_x) * kTileCols;
    const float *__restrict__ g = a.grad + L.elem_off, *__restrict__ r = a.resid + L.elem_off;
    const float *__restrict__ u = a.mom ? a.mom + L.elem_off : nullptr;
    float gq[N], rq[N], uq[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {         // (all requested before any is used)
        const int i = tid + j * kSelectThreads, rr = i / PITCH, x = x0 - H + rr, y = y0 - H + (i - rr * PITCH);
        gq[j] = rq[j] = uq[j] = 0.f;
        if (i < ROWS * PITCH && x >= 0 && x < R && y >= 0 && y < C) {
            const size_t at = static_cast<size_t>(x) * C + y;
            gq[j] = g[at];
            rq[j] = r[at];
            if (u) uq[j] = u[at];
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int i = tid + j * kSelectThreads, rr = i / PITCH, cc = i - rr * PITCH, x = x0 - H + rr, y = y0 - H + cc;
        const bool in = i < ROWS * PITCH && x >= 0 && x < R && y >= 0 && y < C;
        const float gu = u ? __fmul_rn(a.m, uq[j]) + gq[j] : gq[j];
        const float v = in ? rq[j] + gu : 0.f;
        if (i < ROWS * PITCH) sh.tile[i] = v;
        // the tile's own elements (a layer that had no bound went through no pass that stores them)
        if (in && a.v_out && rr >= H && rr < H + kTileRows && cc >= H && cc < H + kTileCols) {
            const size_t at = static_cast<size_t>(L.elem_off) + static_cast<size_t>(x) * C + y;
            a.v_out[at] = v;
            if (a.mom_out) a.mom_out[at] = gu;
        }
    }
    __syncthreads();
    const uint32_t next = select_request(ctl);
    // a thread: four rows of a column; a row's sums go to the windows that it lies in, from the top row on
    constexpr int RPT = kTileRows * kTileCols / kSelectThreads;
    const double n = static_cast<double>(P * P);
    const int col = tid % kTileCols, row0 = tid / kTileCols * RPT, y = y0 + col;
    double sa[RPT], ss[RPT], sq[RPT];
#pragma unroll
    for (int o = 0; o < RPT; ++o) sa[o] = ss[o] = sq[o] = 0.0;
#pragma unroll 1
    for (int i = 0; i < RPT + 2 * H; ++i) {
        const float *row = &sh.tile[(row0 + i) * PITCH + col];
        const double w0 = static_cast<double>(row[0]);
        double ra = fabs(w0), rs = w0, rq = w0 * w0;
#pragma unroll
        for (int j = 1; j < P; ++j) {
            const double w = static_cast<double>(row[j]);
            ra += fabs(w);
            rs += w;
            rq = fma(w, w, rq);
        }
#pragma unroll
        for (int o = 0; o < RPT; ++o)
            if (i >= o && i < o + P) {    // (0 + a sum is the sum: scores come from no signed zero)
                sa[o] += ra;
                ss[o] += rs;
                sq[o] += rq;
            }
    }
#pragma unroll
    for (int o = 0; o < RPT; ++o) {
        const int x = x0 + row0 + o;
        const bool in = x < R && y < C;
        uint32_t key = 0;
        if (in) {
            key = score_from_sums<P>(sa[o], ss[o], sq[o], &sh.tile[(row0 + o) * PITCH + col], PITCH, a.alpha / n, (1.0 - a.alpha) / n);
            agent_store(a.map + static_cast<size_t>(L.elem_off) + static_cast<size_t>(x) * C + y, key);
        }
        wave_count(sh.hist, key >> kCoarseShift, in);
    }
    __syncthreads();                      // (the next tile's v goes where this one's lies)
    return next;
}

// First digit of a layer's full map, from the histogram that the first step has counted: thread 0 has the top bins.
__device__ __forceinline__ DigitResult select_map_digit(SelectShared &sh, const uint32_t *hist, uint32_t k) {
    const uint32_t tid = threadIdx.x;
    const unsigned long long *bins = reinterpret_cast<const unsigned long long *>(hist) + 2 * (kSelectThreads - 1 - tid);
    const unsigned long long q0 = agent_load(bins), q1 = agent_load(bins + 1);
    const uint32_t v[4] = {static_cast<uint32_t>(q1 >> 32), static_cast<uint32_t>(q1), static_cast<uint32_t>(q0 >> 32), static_cast<uint32_t>(q0)};
    const uint32_t own = v[0] + v[1] + v[2] + v[3];
    if (tid == 0) sh.res.found = 0u;
    const uint32_t incl = block_scan_incl_n<kSelectWaves>(own, sh.wave_tot);
    uint32_t acc = incl - own;
    if (acc < k && k <= incl) {
        bool hit = false;
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
            if (!hit && acc + v[j] >= k) {
                sh.res = DigitResult{kHistBins - 1 - 4 * tid - j, acc, v[j], 1u};
                hit = true;
            }
            acc += v[j];
        }
    }
    __syncthreads();
    const DigitResult r = uniform_digit(sh.res);
    __syncthreads();
    return r;
}

// Marks of a run of tiles, from the map.
__device__ __forceinline__ uint32_t select_mark_run(SelectShared &sh, uint32_t l, uint32_t run, unsigned long long T, uint32_t *ctl) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));         // (as in select_map_tile)
    const SelectArgs &a = select_args();
    const LayerDev &L = select_layer(a, l);
    const uint32_t g0 = run * kSelectRun, lane = tid & 63u, wave = tid >> 6;
    GroupGeom q = group_geom(L, g0, min(static_cast<uint32_t>(kSelectRun), L.n_tiles - g0), a.mask, count_ctx(L, a.chunk_cnt, a.group_cnt));
    group_clear<kSelectThreads>(q, sh.run);
    __syncthreads();
    q.cl0 = group_first_chunk(q, sh.run.corner[0]);
    constexpr uint32_t WAVES = kSelectWaves / kSelectRun, U = kTileRows * kTileCols / 64 / WAVES, PER_ROW = kTileCols / 64;     // a tile's waves; their elements per lane
    const uint32_t tile = wave / WAVES, e0 = wave % WAVES * U;
    uint32_t key[U], hits = 0;
    const bool have = static_cast<int>(tile) < q.gn;                 // (uniform in a wave; the first one's is there)
    const uint2 corner = have ? sh.run.corner[tile] : make_uint2(0u, 0u);
    if (have) {
        const uint32_t *map = a.map + L.elem_off;
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
            const uint32_t x = corner.x + (e0 + j) / PER_ROW, y = corner.y + (e0 + j) % PER_ROW * 64u + lane;
            key[j] = x < L.R && y < L.C ? agent_load(map + x * L.C + y) : 0u;
        }
    }
    const uint32_t next = select_request(ctl);
    if (have) {
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
            const uint32_t x = corner.x + (e0 + j) / PER_ROW, y = corner.y + (e0 + j) % PER_ROW * 64u + lane;
            hits |= x < L.R && y < L.C && composite_key(key[j], x * L.C + y) >= T ? 1u << j : 0u;
        }
        while (hits) {
            const uint32_t j = static_cast<uint32_t>(__ffs(hits)) - 1u;
            hits &= hits - 1u;
            const uint32_t i = (corner.x + (e0 + j) / PER_ROW) * L.C + corner.y + (e0 + j) % PER_ROW * 64u + lane;
            group_mark<true>(q, sh.run, static_cast<int>(tile), i);
            if (a.cmask) {
                const size_t pos = static_cast<size_t>(L.elem_off) + i;
                atomicOr(&a.cmask[pos >> 5], 1u << (pos & 31));
            }
        }
    }
    __syncthreads();
    group_write<true, kSelectThreads>(q, sh.run);
    return next;
}

// Takes shares of layer l until all are taken.
__device__ __forceinline__ void select_map_steps(SelectShared &sh, uint32_t l) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));         // (as in select_map_tile)
    const SelectArgs &a = select_args();
    const LayerDev &L = select_layer(a, l);
    uint32_t *ctl = select_ctl(a.list_cnt, l, 0);
    const SelectTickets s = select_tickets(L);
    uint32_t t = select_hand_over(sh, select_request(ctl));
    if (t < s.keys) {                     // scores and first digit
        for (int b = tid; b < kHistBins; b += kSelectThreads) sh.hist[b] = 0u;
        __syncthreads();
        uint32_t done = 0;
        do {
            uint32_t next;
            switch (L.p) {
                case 1: next = select_map_tile<1>(sh, l, t, ctl); break;
                case 3: next = select_map_tile<3>(sh, l, t, ctl); break;
                case 5: next = select_map_tile<5>(sh, l, t, ctl); break;
                default: next = select_map_tile<7>(sh, l, t, ctl); break;
            }
            ++done;
            t = select_hand_over(sh, next);
        } while (t < s.keys);
        uint32_t *hist = a.hist + static_cast<size_t>(l) * kHistBins;
        for (int b = tid; b < kHistBins; b += kSelectThreads)
            if (sh.hist[b]) atomicAdd(&hist[b], sh.hist[b]);
        select_shares_done(ctl - 1 * kListCntStride, done);
    }
    if (t < s.marks) {
        select_wait(ctl - 1 * kListCntStride, s.keys);
        const DigitResult r = select_map_digit(sh, a.hist + static_cast<size_t>(l) * kHistBins, L.k);
        const uint32_t lo = r.found ? r.digit << kCoarseShift : 0u;
        const bool open = r.found && r.count != L.k - r.above;       // else the whole bucket is taken
        const uint32_t *map = a.map + L.elem_off;
        uint32_t *list_cnt = a.list_cnt + static_cast<size_t>(l) * kListShards * kListCntStride;
        uint32_t *hist1 = a.hist1 + static_cast<size_t>(l) * kLevel1Bins;
        const uint32_t cap = L.list_cap / L.list_shards;
        constexpr int kShift1 = kCoarseShift - kLevel1Bits, kKeys = kChunk / kSelectThreads;
        if (t < s.rank) {                 // the bucket's keys and second digit
            for (int b = tid; b < kLevel1Bins; b += kSelectThreads) sh.lh[b] = 0u;
            __syncthreads();
            uint32_t done = 0;
            do {
                uint32_t next;
                if (!open) {
                    next = select_request(ctl);
                } else {
                    const uint32_t start = (t - s.keys) * kChunk + tid, shard = (t - s.keys) % L.list_shards;
                    uint32_t key[kKeys], hits = 0;
#pragma unroll
                    for (uint32_t j = 0; j < kKeys; ++j) {
                        const uint32_t i = start + j * kSelectThreads;
                        key[j] = i < L.G ? agent_load(map + i) : ~0u;            // (scores have no sign)
                    }
                    next = select_request(ctl);
#pragma unroll
                    for (uint32_t j = 0; j < kKeys; ++j) {
                        const bool hit = key[j] - lo < 1u << kCoarseShift;
                        hits |= hit ? 1u << j : 0u;
                        wave_count(sh.lh, (key[j] - lo) >> kShift1, hit);
                    }
                    const uint32_t own = __popc(hits), incl = block_scan_incl_n<kSelectWaves>(own, sh.wave_tot);
                    if (tid == kSelectThreads - 1u) sh.n = incl ? atomicAdd(list_cnt + shard * kListCntStride, incl) : 0u;
                    __syncthreads();
                    uint32_t pos = sh.n + incl - own;
                    unsigned long long *ent = a.list_ent + L.list_off + static_cast<size_t>(shard) * cap;
#pragma unroll
                    for (uint32_t j = 0; j < kKeys; ++j)
                        if (hits & (1u << j)) {
                            if (pos < cap) agent_store(ent + pos, composite_key(key[j], start + j * kSelectThreads));
                            ++pos;
                        }
                }
                ++done;
                t = select_hand_over(sh, next);
            } while (t < s.rank);
            for (int b = tid; b < kLevel1Bins; b += kSelectThreads)
                if (sh.lh[b]) atomicAdd(&hist1[b], sh.lh[b]);
            select_shares_done(ctl - 2 * kListCntStride, done);
        }
        if (t == s.rank) {                // the ranking
            select_wait(ctl - 2 * kListCntStride, L.n_chunks);
            unsigned long long T = static_cast<unsigned long long>(lo) << 32;
            if (open) {
                const uint32_t lane = tid & 63u, wave = tid >> 6;
                const uint32_t listed_n = lane < static_cast<uint32_t>(kListShards) ? agent_load(list_cnt + lane * kListCntStride) : 0u;
                for (int b = tid; b < kLevel1Bins; b += kSelectThreads) sh.lh[b] = agent_load(hist1 + b);
                if (tid == 0) sh.n = 0u;
                const bool listed = uniform_u32(__syncthreads_and(listed_n <= cap)) != 0u;         // every shard of the list fits
                uint32_t k_rem = L.k - r.above;
                const DigitResult d = select_digit(sh, kLevel1Bins, k_rem);
                k_rem -= d.above;
                T += static_cast<unsigned long long>(d.digit) << (32 + kShift1);
                if (d.count != k_rem) {
                    // f for every key with these two digits, less their value: from the list, a shard per wave, or from the map
                    const unsigned long long base = T;
                    const unsigned long long *ent = a.list_ent + L.list_off + static_cast<size_t>(wave) * cap;
                    const uint32_t n = listed ? __builtin_amdgcn_readlane(listed_n, uniform_u32(wave)) : L.G;
                    const uint32_t step = listed ? 64u : kSelectThreads, at = listed ? lane : tid;
                    auto scan = [&](auto f) {
                        constexpr int U = 8;
#pragma unroll 1
                        for (uint32_t i0 = at; i0 - at < n; i0 += U * step) {        // (the same trip count in every lane)
                            unsigned long long rel[U];
#pragma unroll
                            for (int j = 0; j < U; ++j) {
                                const uint32_t i = i0 + j * step;
                                rel[j] = ~0ull;
                                if (i < n) rel[j] = (listed ? agent_load(ent + i) : composite_key(agent_load(map + i), i)) - base;
                            }
#pragma unroll
                            for (int j = 0; j < U; ++j)
                                if (rel[j] >> (32 + kShift1) == 0ull) f(rel[j]);
                        }
                    };
                    if (d.count <= static_cast<uint32_t>(kSelectList)) {
                        scan([&](unsigned long long rel) {
                            const uint32_t pos = atomicAdd(&sh.n, 1u);
                            if (pos < static_cast<uint32_t>(kSelectList)) sh.key[pos] = rel;
                        });
                        __syncthreads();
                    }
                    T += select_rank(sh, d.count, k_rem, 32 + kShift1, scan);
                }
            }
            if (tid == 0) agent_store(&a.state[l].T, T);
            select_shares_done(ctl - 3 * kListCntStride, 1u);
            if (tid == 0) {               // (for the next calls)
                const SelState st = a.state[l];
                if (st.mode == kModeCandidates) {
                    const uint32_t top = a.hist_s[static_cast<size_t>(l) * kHistBins + kFineBins - 1];
                    bound_failed(a.pred, l, L.k, st, DigitResult{kFineBins - 1, 0u, 0u, top >= L.k ? 1u : 0u});
                }
                SelState ns = st;
                ns.mode = kModeFullMap;
                ns.T = T;
                ns.lo = lo;
                ns.span = kCoarseShift;
                ns.done = 1u;
                a.state[l] = ns;
                publish_threshold(a.pred, l, 1u, L.k, T);
            }
            t = select_hand_over(sh, select_request(ctl));
        }
    }
    if (t < s.end) {                      // the marks
        select_wait(ctl - 3 * kListCntStride, 1u);
        const unsigned long long T = agent_load(&a.state[l].T);
        do {
            const uint32_t next = select_mark_run(sh, l, t - s.marks, T, ctl);
            t = select_hand_over(sh, next);
        } while (t < s.end);
    }
}

__device__ __forceinline__ uint32_t select_failed_layers(const SelectArgs &a) {      // of the layers tid, tid + 1024, ...: a bit each
    static_assert(kInlineCountChunks <= 4u * kSelectThreads, "layers per thread");
    uint32_t failed = 0;
    for (uint32_t j = 0, c = threadIdx.x; c < a.n_layers; ++j, c += kSelectThreads)
        failed |= layer_falls_back(a.layers, a.state, a.hist_s, a.list_cnt, c) ? 1u << j : 0u;
    return failed;
}
// The workgroups of a failed layer's groups (that layer first) and those without a group: shares of any failed layer that has some left.
__device__ __forceinline__ void select_failed(SelectShared &sh) {
    const SelectArgs &a = select_args();
    uint32_t wg = blockIdx.x;
    asm volatile("" : "+s"(wg));          // (nothing of select_group's is held for this rare case)
    const uint32_t tid = threadIdx.x;
    const bool helper = wg >= a.n_groups;
    if (helper && !uniform_u32(__syncthreads_or(select_failed_layers(a) != 0u))) return;
    // (helpers come to the layers in proportion to their groups)
    const uint32_t first = uniform_u32(a.groups[helper ? (wg - a.n_groups) * a.n_groups / (gridDim.x - a.n_groups) : wg].layer);
    uint32_t l = helper ? ~0u : first;
    for (;;) {
        if (l == ~0u) {
            const uint32_t failed = select_failed_layers(a);
            __syncthreads();
            if (tid == 0) sh.n = ~0u;
            __syncthreads();
            for (uint32_t j = 0, c = tid; c < a.n_layers; ++j, c += kSelectThreads) {
                if (!(failed & (1u << j))) continue;
                if (agent_load(select_ctl(a.list_cnt, c, 0)) < select_tickets(a.layers[c]).end)
                    atomicMin(&sh.n, c >= first ? c - first : c + a.n_layers - first);
            }
            __syncthreads();
            const uint32_t next = uniform_u32(sh.n);
            __syncthreads();
            if (next == ~0u) return;
            l = first + next < a.n_layers ? first + next : first + next - a.n_layers;
        }
        select_map_steps(sh, l);
        l = ~0u;
    }
}

// A group of tile slots; false: its layer's bound failed, nothing is done.
__device__ __forceinline__ bool select_group(const SelectArgs &a, SelectShared &sh) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const GroupEntry ge = a.groups[blockIdx.x];
    const uint32_t l = ge.layer, cap = ge.slot_cap;
    const LayerDev L = a.layers[l];
    const SelState st = a.state[l];
    const uint32_t own_bin = a.hist_s[static_cast<size_t>(l) * kHistBins + (kFineBins - 1 - tid)];      // thread 0 has the top bin
    // the layer's slots, and the wave's own one of the group: its first entries beside its count (a slot always has them; past
    // the count they hold anything)
    const uint32_t count = wave + 16u * lane < L.n_tiles ? a.slot_cnt[L.tile_begin_all + wave + 16u * lane] : 0u;
    const unsigned long long *__restrict__ slot = a.slot_ent + (((static_cast<uint64_t>(ge.ent0_high) << 32) | ge.ent0_low) << 1) + wave * cap;
    uint32_t cnt = 0;
    unsigned long long own = 0;
    if (wave < ge.ntile) {
        cnt = a.slot_cnt[ge.slot0 + wave];
        if (lane < cap) own = slot[lane];
    }
    const CountCtx cctx = count_ctx(L, a.chunk_cnt, a.group_cnt);
    GroupGeom q = group_geom(L, ge.slot0 - L.tile_begin_all, ge.ntile, a.mask, cctx);
    group_clear<kSelectThreads>(q, sh.marks);
    if (tid == 0) {
        sh.res.found = 0u;
        sh.n = 0u;
    }
    SlotScan scan;
    scan.set(L, a.slot_ent, count);
    unsigned long long K[SlotScan::U];
    scan.load(K, 0u);                     // (they arrive while the digit is found)
    const uint32_t incl = block_scan_incl_n<kSelectWaves>(own_bin, sh.wave_tot), excl = incl - own_bin;
    if (excl < L.k && L.k <= incl) sh.res = DigitResult{kFineBins - 1 - tid, excl, own_bin, 1u};
    __syncthreads();
    const DigitResult r = uniform_digit(sh.res);
    // k_find0's test of the bound
    const bool failed = st.mode != kModeCandidates || st.hint_key == 0u || st.overflow != 0u || !r.found || r.digit == static_cast<uint32_t>(kFineBins - 1);
    if (uniform_u32(failed ? 1u : 0u)) return false;
    const uint32_t lo = st.hint_key + (r.digit << kFineShift), k_rem = L.k - r.above;
    const unsigned long long base = static_cast<unsigned long long>(lo) << 32;
    unsigned long long T = base;                     // (the whole bucket is taken: its lower edge)
    if (r.count != k_rem) {
        scan.rest(K, [&](unsigned long long key) {
            if (static_cast<uint32_t>(key >> 32) - lo < 1u << kFineShift) {
                const uint32_t pos = atomicAdd(&sh.n, 1u);
                if (pos < static_cast<uint32_t>(kSelectList)) sh.key[pos] = key - base;
            }
        });
        __syncthreads();
        T += select_rank(sh, uniform_u32(sh.n), k_rem, 32 + kFineShift, [&](auto f) {
            scan.load(K, 0u);
            scan.rest(K, [&](unsigned long long key) {
                if (static_cast<uint32_t>(key >> 32) - lo < 1u << kFineShift) f(key - base);
            });
        });
    }
    q.cl0 = group_first_chunk(q, sh.marks.corner[0]);
    cnt = min(cnt, cap);
    for (uint32_t j = lane; j < cnt; j += 64u) {
        if (j != lane) own = slot[j];
        if (own < T) continue;
        const uint32_t i = ~static_cast<uint32_t>(own);
        group_mark<true>(q, sh.marks, static_cast<int>(wave), i);
        if (a.cmask) {
            const size_t pos = static_cast<size_t>(L.elem_off) + i;
            atomicOr(&a.cmask[pos >> 5], 1u << (pos & 31));
        }
    }
    __syncthreads();
    group_write<true, kSelectThreads>(q, sh.marks);
    if (q.g0 == 0 && tid == 0) publish_threshold(a.pred, l, 1u, L.k, T);
    return true;
}

__global__ __launch_bounds__(kSelectThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_select(const SelectArgs a) {
    __shared__ SelectShared sh;
    if (blockIdx.x < a.n_groups && select_group(a, sh)) return;
    select_failed(sh);
}

// ----------------------------------------------------------------- mark --
// OR a 64-bit group of mask bits that starts at bit position pos into a bitmask whose
// words may be shared with other workgroups (rows that are not a multiple of 32 long).
__device__ __forceinline__ void or_bits_shared(uint32_t *__restrict__ mask, size_t pos,
                                               unsigned long long v) {
    if (!v) return;
    const size_t w = pos >> 5;
    const uint32_t b = static_cast<uint32_t>(pos & 31);
    const uint32_t p0 = static_cast<uint32_t>(v << b);
    const uint32_t p1 = static_cast<uint32_t>(b ? (v >> (32 - b)) : (v >> 32));
    const uint32_t p2 = b ? static_cast<uint32_t>(v >> (64 - b)) : 0u;
    if (p0) atomicOr(&mask[w], p0);
    if (p1) atomicOr(&mask[w + 1], p1);
    if (p2) atomicOr(&mask[w + 2], p2);
}
// Full-map layers: workgroups stride over the 16 x 256 tiles (the NSI tiling).  Every centre
// of a tile and of a halo of h rows / columns is compared with the layer's threshold; the
// per-row results become 64-bit ballot words in LDS, the p x p box dilation (Section III-C:
// whole neighbourhoods are kept) is done on those words with shifts and ORs, and the tile's
// mask words are written with plain stores (rows that are a multiple of 32 long) -- no
// global atomics on that path.
// The first n_bucket_wgs workgroups take the layers on the candidate path, one workgroup per
// layer and shard of the layer's threshold-bucket list: the recorded candidates above the bucket
// were marked by the gather pass, those of the bucket that reach the threshold are marked here,
// each ORing the bits of its window into the mask.  (One workgroup per layer doing this at the
// end of k_finish took 20 .. 75 us: the marks of a large layer are too many for one CU.)  The
// next n_list_wgs workgroups stride over the plan's list of tiles of the layers that are
// always ranked on the full map; the others run only when some large layer fell back to it,
// walk all tiles and take those of such layers.
// Large plans: several workgroups per shard, a key per thread (a window's marks are two round trips to memory: in one arena on
// VGG-19 12.2 us with one, 8.2 with four).
constexpr uint32_t mark_parts(MarkCount how) { return how == kMarkCountsShared ? 4u : 1u; }
constexpr int kMarkCountSlots = 64;   // chunks a tile counts for in LDS (more only for rows beyond 32 K elements: directly)

struct MarkArgs {
    const LayerDev *layers;
    const SelState *state;
    uint32_t n_bucket_wgs;           // n_layers * kListShards * mark_parts
    const uint32_t *list_cnt;
    const unsigned long long *list_ent;
    const uint32_t *slot_cnt;
    const unsigned long long *slot_ent;
    const DirEntry *dir;             // tiles of all layers in layer order (fallback walk)
    uint32_t n_layers, n_tiles;
    const SampleEntry *map_tiles;
    uint32_t n_map_tiles, n_list_wgs;
    const uint32_t *flags;
    const uint32_t *keys;            // score map
    uint32_t *mask, *cmask;
    uint32_t *chunk_cnt, *group_cnt; // kept elements per chunk / chunk group, counted as the bits are set
    uint32_t gstride;                // words between two groups' counters
    const float *grad;               // v replaces the residual: of the layers that the main pass did not take, here (nullable)
    float *resid;
};

template <MarkCount HOW>
__global__ __launch_bounds__(256) void k_mark(const MarkArgs m) {
    constexpr bool COUNT = HOW != kMarkOnly, SHARED = HOW == kMarkCountsShared;
    constexpr int MAXH = (RSDGC_MAX_P - 1) / 2;
    constexpr int NSEG = kTileCols / 64;       // 64-column segments of a tile row
    static_assert(kTileRows * NSEG == 64, "one lane of wave 0 per row segment");
    __shared__ unsigned long long bits[kTileRows + 2 * MAXH][NSEG + 2];   // [row][left, segments, right]
    __shared__ uint32_t ccnt[kMarkCountSlots];      // bits set by the tile, per chunk from the tile's first one on
    __shared__ uint32_t groups[SHARED ? kMarkGroups : 1];      // bits set by the bucket keys, per chunk group
    const LayerDev *__restrict__ layers = m.layers;
    const DirEntry *__restrict__ dir = m.dir;
    const SampleEntry *__restrict__ map_tiles = m.map_tiles;
    const SelState *__restrict__ state = m.state;
    const uint32_t *__restrict__ keys = m.keys;
    uint32_t *__restrict__ mask = m.mask;
    uint32_t *__restrict__ cmask = m.cmask;
    const uint32_t n_layers = m.n_layers;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x < m.n_bucket_wgs) {
        constexpr uint32_t PARTS = mark_parts(HOW);
        const uint32_t l = blockIdx.x / (kListShards * PARTS), shard = blockIdx.x % kListShards, part = blockIdx.x / kListShards % PARTS;
        const uint32_t *__restrict__ cnt = m.list_cnt + static_cast<size_t>(l) * kListShards * kListCntStride;
        const uint32_t c = static_cast<uint32_t>(lane) < kListShards ? cnt[lane * kListCntStride] : 0u;
        const SelState st = state[l];
        if (st.mode != kModeCandidates || st.span == 0u) return;      // (no bucket: nothing was ranked)
        const LayerDev Lc = layers[l];
        const unsigned long long Tc = st.T;
        const WindowGeom geom = {static_cast<size_t>(Lc.elem_off), static_cast<int>(Lc.R), static_cast<int>(Lc.C),
                                 (static_cast<int>(Lc.p) - 1) / 2};
        const uint32_t shards = Lc.list_shards, cap = Lc.list_cap / shards;
        if (shard >= shards) return;
        if (SHARED) {
            for (uint32_t b = tid; b < kMarkGroups; b += 256) groups[b] = 0u;
            __syncthreads();
        }
        const CountCtx cctx = count_ctx(Lc, m.chunk_cnt, m.group_cnt, m.gstride);
        if (__ballot(c > cap) == 0ull) {       // every shard fits: this workgroup takes its shard
            const uint32_t n = __shfl(c, static_cast<int>(shard), 64);
            const unsigned long long *__restrict__ keys = m.list_ent + Lc.list_off + static_cast<size_t>(shard) * cap;
            for (uint32_t i = part * 256u + tid; i < n; i += 256u * PARTS) {
                const unsigned long long K = keys[i];
                if (K >= Tc) mark_window<HOW>(geom, cctx, groups, ~static_cast<uint32_t>(K), mask, cmask);
            }
        } else {                               // the list overflowed: the bucket's keys are still in the tile slots
            const unsigned long long bucket_end = (static_cast<unsigned long long>(st.lo) + (1ull << st.span)) << 32;
            for (uint32_t t = shard + shards * part; t < Lc.n_tiles; t += shards * PARTS) {
                const uint32_t n = min(m.slot_cnt[Lc.tile_begin_all + t], Lc.slot_cap);
                const unsigned long long *__restrict__ ent = m.slot_ent + Lc.slot_off + static_cast<size_t>(t) * Lc.slot_cap;
                for (uint32_t i = tid; i < n; i += 256) {
                    const unsigned long long K = ent[i];
                    if (K >= Tc && K < bucket_end) mark_window<HOW>(geom, cctx, groups, ~static_cast<uint32_t>(K), mask, cmask);
                }
            }
        }
        if (SHARED) {
            __syncthreads();
            for (uint32_t b = tid; b < min(kMarkGroups, (Lc.n_chunks + kChunkGroup - 1) / kChunkGroup); b += 256)
                if (groups[b]) count_add_group(cctx, b, groups[b]);
        }
        return;
    }
    const uint32_t bid = blockIdx.x - m.n_bucket_wgs;
    const bool listed = bid < m.n_list_wgs;
    const uint32_t first = listed ? bid : bid - m.n_list_wgs;
    const uint32_t stride = listed ? m.n_list_wgs : gridDim.x - m.n_bucket_wgs - m.n_list_wgs;
    const uint32_t n_items = listed ? m.n_map_tiles : m.n_tiles;
    if (first >= n_items) return;
    if (!listed && m.flags[0] == 0u) return;
    if (COUNT && tid < kMarkCountSlots) ccnt[tid] = 0u;       // (the tile loop's barriers come before the first use)
    uint32_t e = listed ? 0u : dir_lookup(dir, n_layers, first);
    uint32_t cur_l = 0xffffffffu;
    bool active = false, form_v = false;
    unsigned long long T = 0;
    LayerDev L;
    for (uint32_t t = first; t < n_items; t += stride) {
        uint32_t l, local;
        if (listed) {
            const SampleEntry se = map_tiles[t];
            l = se.layer;
            local = se.local_tile;
        } else {
            e = dir_advance(dir, n_layers, e, t);
            l = dir[e].layer;
            local = t - dir[e].begin;
        }
        if (l != cur_l) {
            cur_l = l;
            L = layers[l];
            const SelState st = state[l];
            active = st.mode == kModeFullMap && (listed || L.large != 0u);
            T = st.T;
            form_v = m.resid != nullptr && !(L.large != 0u && bound_in_range(st.hint_key));
        }
        if (!active) {
            if (!listed) {
                const uint32_t nb = dir[e + 1].begin;
                t += (nb - t + stride - 1) / stride * stride - stride;
            }
            continue;
        }
        const int h = (static_cast<int>(L.p) - 1) / 2;
        const int rows_ext = kTileRows + 2 * h;
        const int trow = static_cast<int>(local / L.tiles_x);
        const int tcol = static_cast<int>(local - static_cast<uint32_t>(trow) * L.tiles_x);
        const int R = static_cast<int>(L.R), C = static_cast<int>(L.C);
        const int x0 = trow * kTileRows, y0 = tcol * kTileCols;
        const uint32_t *__restrict__ src = keys + L.elem_off;
        const CountCtx cctx = count_ctx(L, m.chunk_cnt, m.group_cnt, m.gstride);
        const uint32_t cl0 = static_cast<uint32_t>((static_cast<size_t>(x0) * C + y0) / kChunk);   // the tile's first chunk

        // wave w takes segment w of every row: all its keys are requested before any is compared
        static_assert(NSEG == 4, "one wave per 64-column segment");
        constexpr int kMaxRowsExt = kTileRows + 2 * MAXH;
        {
            const int y = y0 + 64 * wave + lane;
            uint32_t key[kMaxRowsExt];
#pragma unroll
            for (int rr = 0; rr < kMaxRowsExt; ++rr) {
                const int x = x0 - h + rr;
                key[rr] = 0;
                if (rr < rows_ext && x >= 0 && x < R && y < C)
                    key[rr] = src[static_cast<uint32_t>(x) * L.C + static_cast<uint32_t>(y)];
            }
#pragma unroll
            for (int rr = 0; rr < kMaxRowsExt; ++rr) {
                const int x = x0 - h + rr;
                bool flag = false;
                if (rr < rows_ext && x >= 0 && x < R && y < C) {
                    const uint32_t i = static_cast<uint32_t>(x) * L.C + static_cast<uint32_t>(y);
                    flag = composite_key(key[rr], i) >= T;
                }
                const unsigned long long w = __ballot(flag);
                if (lane == 0 && rr < rows_ext) bits[rr][1 + wave] = w;
            }
        }
        if (wave < 2 && lane < rows_ext) {      // halo columns: lane = row; wave 0 left, wave 1 right
            unsigned long long hw = 0;
            const int x = x0 - h + lane;
            if (x >= 0 && x < R) {
                for (int d = 1; d <= h; ++d) {
                    const int y = wave == 0 ? y0 - d : y0 + kTileCols + (d - 1);
                    if (y >= 0 && y < C) {
                        const uint32_t i = static_cast<uint32_t>(x) * L.C + static_cast<uint32_t>(y);
                        if (composite_key(src[i], i) >= T)
                            hw |= wave == 0 ? (1ull << (64 - d)) : (1ull << (d - 1));
                    }
                }
            }
            bits[lane][wave == 0 ? 0 : NSEG + 1] = hw;
        }
        __syncthreads();

        const int r = lane / NSEG, seg = lane % NSEG;    // wave 0: rows x segments = 64 items
        const int x = x0 + r, yb = y0 + 64 * seg;
        if (wave == 0 && x < R && yb < C) {
            unsigned long long acc = 0;
            for (int rr = r; rr <= r + 2 * h; ++rr) {
                const unsigned long long W = bits[rr][1 + seg], Lw = bits[rr][seg], Rw = bits[rr][2 + seg];
                unsigned long long hd = W;
                for (int d = 1; d <= h; ++d)
                    hd |= (W << d) | (Lw >> (64 - d)) | (W >> d) | (Rw << (64 - d));
                acc |= hd;
            }
            const int ncols = min(64, C - yb);
            const unsigned long long valid = ncols >= 64 ? ~0ull : ((1ull << ncols) - 1ull);
            acc &= valid;
            const unsigned long long own = bits[r + h][1 + seg];
            const size_t pos = static_cast<size_t>(L.elem_off) + static_cast<size_t>(x) * C + yb;
            if ((C & 31) == 0) {                     // the tile owns its mask words
                const size_t w = pos >> 5;
                mask[w] = static_cast<uint32_t>(acc);
                if (ncols > 32) mask[w + 1] = static_cast<uint32_t>(acc >> 32);
                if (cmask) {
                    cmask[w] = static_cast<uint32_t>(own);
                    if (ncols > 32) cmask[w + 1] = static_cast<uint32_t>(own >> 32);
                }
                // its bits, per chunk (the two words may lie in different chunks)
#pragma unroll
                for (int part = 0; part < 2; ++part) {
                    const uint32_t n = COUNT ? __popc(static_cast<uint32_t>(acc >> (32 * part))) : 0u;
                    if (n) {
                        const uint32_t slot = static_cast<uint32_t>((w + part - cctx.word0) >> 8) - cl0;
                        if (slot < static_cast<uint32_t>(kMarkCountSlots)) atomicAdd(&ccnt[slot], n);
                        else count_add_chunk(cctx, cl0 + slot, n);
                    }
                }
            } else if (!COUNT) {
                or_bits_shared(mask, pos, acc);
                if (cmask) or_bits_shared(cmask, pos, own);
            } else {                                 // shared words: an OR tells which bits were new
                const size_t w = pos >> 5;
                const uint32_t b = static_cast<uint32_t>(pos & 31);
                const uint32_t part[3] = {static_cast<uint32_t>(acc << b),
                                          static_cast<uint32_t>(b ? (acc >> (32 - b)) : (acc >> 32)),
                                          b ? static_cast<uint32_t>(acc >> (64 - b)) : 0u};
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    if (part[j] == 0u) continue;
                    const uint32_t n = __popc(part[j] & ~atomicOr(&mask[w + j], part[j]));
                    if (n) {
                        const uint32_t slot = static_cast<uint32_t>((w + j - cctx.word0) >> 8) - cl0;
                        if (slot < static_cast<uint32_t>(kMarkCountSlots)) atomicAdd(&ccnt[slot], n);
                        else count_add_chunk(cctx, cl0 + slot, n);
                    }
                }
                if (cmask) or_bits_shared(cmask, pos, own);
            }
        }
        if (form_v) {                           // the tile's own elements, each by one thread: nothing reads its neighbours any more
            float *__restrict__ res = m.resid + L.elem_off;
            const float *__restrict__ g = m.grad + L.elem_off;
            const int y = y0 + 4 * lane;
            for (int row = x0 + wave; row < min(x0 + kTileRows, R); row += 4) {
                const size_t at = static_cast<size_t>(row) * C + y;
                if ((C & 3) == 0 && y < C) {
                    const float4 rv = *reinterpret_cast<const float4 *>(res + at), gv = *reinterpret_cast<const float4 *>(g + at);
                    *reinterpret_cast<float4 *>(res + at) = make_float4(rv.x + gv.x, rv.y + gv.y, rv.z + gv.z, rv.w + gv.w);
                } else {
                    for (int q = 0; q < 4 && y + q < C; ++q) res[at + q] += g[at + q];
                }
            }
        }
        __syncthreads();                        // the ballot words are reused by the next tile
        static_assert(kMarkCountSlots == 64, "one lane of the first wave per counted chunk");
        if (COUNT && tid < 64) {
            count_flush_wave0(cctx, cl0, ccnt[tid]);
            ccnt[tid] = 0u;
        }
    }
}

// The mark of block grids (neighbourhoods of one "element").  Layers ranked on the full map: the mask is the comparison itself, so
// there is no tile and no halo.  One wave per kFlatKeys consecutive scores -- a ballot over 64 of them is two mask words --, no
// barrier, few registers: all waves of a plan as large as VGG-19 (62 MB of scores) are on their way at once.  28.5 us by tiles
// in k_mark, 16.0 us so, 14 since a workgroup adds its chunk's count at once.  Layers on the candidate path: the keys of the threshold bucket's list that reach the threshold, a bit
// each.  Counts as it marks, as k_mark does.  Workgroups, as there: the listed chunks, a layer's list shards, and those that walk all
// chunks if some layer is on its map in this call.
constexpr int kFlatKeys = 2048;
struct MarkFlatArgs {
    const LayerDev *layers;
    const SelState *state;
    const ChunkEntry *map_chunks;
    const ChunkInfo *chunks;
    uint32_t n_map_chunks, n_bucket_wgs, n_chunks;
    const uint32_t *list_cnt, *slot_cnt, *flags, *keys;
    const unsigned long long *list_ent, *slot_ent;
    uint32_t *mask, *chunk_cnt, *group_cnt;
    uint32_t gstride;
};
// A quarter of a chunk, by one wave: the blocks it marked.
__device__ __forceinline__ uint32_t mark_flat_quarter(const MarkFlatArgs &m, uint32_t layer, uint32_t chunk_start, uint32_t chunk_len, uint64_t arena_off) {
    constexpr uint32_t N = kFlatKeys / 64, PER = kChunk / kFlatKeys;
    static_assert(PER == 4 && N == 32, "four waves, a workgroup, per chunk");
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));        // (as in gather_map_chunk)
    const uint32_t first = wave * kFlatKeys;                 // inside the chunk
    if (first >= chunk_len) return 0u;
    const uint32_t len = min(chunk_len - first, static_cast<uint32_t>(kFlatKeys));
    const uint32_t *__restrict__ src = m.keys + arena_off + first;
    uint32_t key[N];
    if (len == static_cast<uint32_t>(kFlatKeys)) {
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) key[j] = (src + 64u * j)[lane];
    } else {
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) key[j] = src[min(64u * j + lane, len - 1u)];     // (not used past len)
    }
    const unsigned long long T = m.state[layer].T;           // (mode kModeFullMap: these layers select something)
    // K >= T, in two halves: a larger score, or the same at an index that is not higher
    const uint32_t tau = static_cast<uint32_t>(T >> 32), last = ~static_cast<uint32_t>(T);
    const uint32_t start = chunk_start + first;
    unsigned long long mine = 0;                             // lane j: the ballot of round j
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) {
        const uint32_t e = 64u * j + lane, k = key[j] & 0x7fffffffu;
        const unsigned long long w = __ballot(e < len && (k > tau || (k == tau && start + e <= last)));
        if (lane == j) mine = w;
    }
    // (chunks and layers start at whole pairs of words, and layers are padded to one)
    if (64u * lane < len) *reinterpret_cast<unsigned long long *>(m.mask + ((arena_off + first) >> 5) + 2 * lane) = mine;
    uint32_t n = lane < N ? static_cast<uint32_t>(__popcll(mine)) : 0u;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
    return n;
}
// A chunk, by a workgroup.
__device__ __forceinline__ void mark_flat_chunk(const MarkFlatArgs &m, uint32_t layer, uint32_t start, uint32_t len, uint64_t arena_off, uint32_t *tot /*[4], LDS*/) {
    const uint32_t n = mark_flat_quarter(m, layer, start, len, arena_off);
    const CountCtx cctx = count_ctx(m.layers[layer], m.chunk_cnt, m.group_cnt, m.gstride);
    if (len < static_cast<uint32_t>(kChunk)) {       // uniform (a short chunk, of which most plans have few: its waves need not meet)
        if ((threadIdx.x & 63u) == 0u && n != 0u) count_add_chunk(cctx, start / kChunk, n);
        return;
    }
    if ((threadIdx.x & 63u) == 0u) tot[threadIdx.x >> 6] = n;
    __syncthreads();
    const uint32_t all = tot[0] + tot[1] + tot[2] + tot[3];
    if (threadIdx.x == 0 && all != 0u) count_add_chunk(cctx, start / kChunk, all);
    __syncthreads();
}
__global__ __launch_bounds__(256) void k_mark_flat(const MarkFlatArgs m) {
    __shared__ uint32_t tot[4];
    const uint32_t tid = threadIdx.x, wg = blockIdx.x - m.n_map_chunks;
    const bool listed = blockIdx.x < m.n_map_chunks;
    if (!listed && wg < m.n_bucket_wgs) {  // (as in k_mark)
        const uint32_t l = wg / kListShards, shard = wg % kListShards, lane = tid & 63u;
        const uint32_t *__restrict__ cnt = m.list_cnt + static_cast<size_t>(l) * kListShards * kListCntStride;
        const uint32_t c = lane < kListShards ? cnt[lane * kListCntStride] : 0u;
        const SelState st = m.state[l];
        const LayerDev &L = m.layers[l];
        const uint32_t shards = L.list_shards, cap = list_entries(L, true) / shards;
        if (st.mode != kModeCandidates || st.span == 0u || shard >= shards) return;
        const CountCtx cctx = count_ctx(L, m.chunk_cnt, m.group_cnt, m.gstride);
        auto mark = [&](unsigned long long K) {
            const uint32_t i = ~static_cast<uint32_t>(K);
            const size_t pos = static_cast<size_t>(L.elem_off) + i;
            atomicOr(&m.mask[pos >> 5], 1u << (pos & 31));
            count_add_chunk(cctx, i / kChunk, 1u);
        };
        if (__ballot(c > cap) == 0ull) {
            const uint32_t n = __shfl(c, static_cast<int>(shard), 64);
            const unsigned long long *__restrict__ part = m.list_ent + L.list_off + static_cast<size_t>(shard) * cap;
            for (uint32_t i = tid; i < n; i += 256)
                if (part[i] >= st.T) mark(part[i]);
        } else {                           // the list overflowed: the bucket's keys are still in the tile slots
            const unsigned long long bucket_end = (static_cast<unsigned long long>(st.lo) + (1ull << st.span)) << 32;
            for (uint32_t t = shard; t < L.n_tiles; t += shards) {
                const uint32_t n = min(m.slot_cnt[L.tile_begin_all + t], L.slot_cap);
                const unsigned long long *__restrict__ ent = m.slot_ent + L.slot_off + static_cast<size_t>(t) * L.slot_cap;
                for (uint32_t i = tid; i < n; i += 256)
                    if (ent[i] >= st.T && ent[i] < bucket_end) mark(ent[i]);
            }
        }
        return;
    }
    if (!listed && m.flags[0] == 0u) return;
    const uint32_t stride = gridDim.x - m.n_map_chunks - m.n_bucket_wgs, end = listed ? blockIdx.x + 1u : m.n_chunks;
    for (uint32_t c = listed ? blockIdx.x : wg - m.n_bucket_wgs; c < end; c += listed ? 1u : stride) {
        ChunkEntry ce;
        if (listed) {
            ce = m.map_chunks[c];
        } else {
            const ChunkInfo ci = m.chunks[c];
            if (m.layers[ci.layer].large == 0u || m.state[ci.layer].mode != kModeFullMap) continue;      // uniform
            ce = ChunkEntry{ci.layer, ci.start, ci.len, 0u, ci.arena_off};
        }
        mark_flat_chunk(m, ce.layer, ce.start, ce.len, ce.arena_off, tot);
    }
}

// ---------------------------------------------------------------- count --
// Kept elements of the plans that count them here (kCountAfter; else `mask` is null), and selected centres where their lists are wanted, per
// chunk and per group of kChunkGroup chunks, from the finished masks.  One workgroup per kCountChunks = 16 chunks; 16 adjacent threads read the 256 mask words of one
// chunk (16 consecutive words each, as independent 8-byte loads) and add their popcounts with
// four shuffles.  A workgroup adds its total to its chunk group's with one atomic -- four per
// group (one atomic per chunk put 17 k of them on 9 cache lines and cost 18 us).
constexpr int kCountThreads = 16 * kCountChunks;

__global__ __launch_bounds__(kCountThreads) void k_count(const CountGroup *__restrict__ groups,
                                                         const uint32_t *__restrict__ mask,
                                                         const uint32_t *__restrict__ cmask,
                                                         uint32_t *__restrict__ chunk_cnt,
                                                         uint32_t *__restrict__ chunk_ccnt,
                                                         uint32_t *__restrict__ group_cnt,
                                                         uint32_t *__restrict__ group_ccnt, uint32_t gstride) {
    constexpr int kPerThread = kChunk / 32 / 16;    // 16 words
    static_assert(kCountChunks <= 64, "one lane of the first wave per chunk");
    __shared__ uint32_t lcnt[2][kCountChunks];
    const int tid = threadIdx.x;
    const CountGroup gr = groups[blockIdx.x];
    const uint32_t i0 = static_cast<uint32_t>(tid) * kPerThread;
    // (a layer starts at a multiple of 64 elements, so word0 and i0 are even: 8-byte loads)
    uint2 wa[kPerThread / 2], wb[kPerThread / 2];
#pragma unroll
    for (int j = 0; j < kPerThread / 2; ++j) {
        const uint32_t i = i0 + 2 * j;
        wa[j] = make_uint2(0u, 0u);
        wb[j] = make_uint2(0u, 0u);
        if (i + 1 < gr.n_words) {
            if (mask) wa[j] = *reinterpret_cast<const uint2 *>(mask + gr.word0 + i);
            if (cmask) wb[j] = *reinterpret_cast<const uint2 *>(cmask + gr.word0 + i);
        } else if (i < gr.n_words) {
            if (mask) wa[j].x = mask[gr.word0 + i];
            if (cmask) wb[j].x = cmask[gr.word0 + i];
        }
    }
    uint32_t a = 0, b = 0;
#pragma unroll
    for (int j = 0; j < kPerThread / 2; ++j) {
        a += __popc(wa[j].x) + __popc(wa[j].y);
        b += __popc(wb[j].x) + __popc(wb[j].y);
    }
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) {
        a += __shfl_xor(a, d, 64);
        b += __shfl_xor(b, d, 64);
    }
    if ((tid & 15) == 0) {
        lcnt[0][tid >> 4] = a;
        lcnt[1][tid >> 4] = b;
    }
    __syncthreads();
    if (tid < 64) {                        // the first wave: one lane per chunk
        a = tid < kCountChunks ? lcnt[0][tid] : 0u;
        b = tid < kCountChunks ? lcnt[1][tid] : 0u;
        if (static_cast<uint32_t>(tid) < gr.n_chunks) {
            if (mask) chunk_cnt[gr.first_chunk + tid] = a;
            if (cmask) chunk_ccnt[gr.first_chunk + tid] = b;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            a += __shfl_xor(a, d, 64);
            b += __shfl_xor(b, d, 64);
        }
        if (tid == 0) {                    // (the group totals are cleared by the find0 launch)
            if (mask && a) atomicAdd(&group_cnt[static_cast<size_t>(gr.group) * gstride], a);
            if (cmask && b) atomicAdd(&group_ccnt[static_cast<size_t>(gr.group) * gstride], b);
        }
    }
}

// The chunk's prefix -- kept elements of its layer before it -- is the sum of the totals of
// the layer's earlier chunk groups and of the earlier chunks of its own group: at most a few
// hundred values, so every consumer adds them up itself instead of waiting for a scan
// kernel.  The first wave does it (independent loads issued with the workgroup's other loads,
// one wave reduction) and leaves the sum in *s_prefix; the caller reads it after its next
// barrier.
__device__ __forceinline__ uint32_t chunk_prefix_by_wave(const ChunkInfo &ci, uint32_t c,
                                                         const uint32_t *__restrict__ chunk_cnt,
                                                         const uint32_t *__restrict__ group_cnt) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t g0 = ci.layer_first_group + lane, g1 = ci.group;
    const uint32_t cc = ci.group_first_chunk + lane;     // at most kChunkGroup - 1 = 63 of them
    uint32_t v[5];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = g0 + 64 * j < g1 ? group_cnt[static_cast<size_t>(g0 + 64 * j) * ci.gstride] : 0u;
    v[4] = cc < c ? chunk_cnt[cc] : 0u;
    uint32_t own = v[0] + v[1] + v[2] + v[3] + v[4];
    for (uint32_t g = g0 + 256; g < g1; g += 64) own += group_cnt[static_cast<size_t>(g) * ci.gstride];     // layers beyond 2^27 elements
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) own += __shfl_xor(own, d, 64);
    return own;                    // the same in every lane of the wave
}

__device__ __forceinline__ void chunk_prefix_wave0(const ChunkInfo &ci, uint32_t c,
                                                   const uint32_t *__restrict__ chunk_cnt,
                                                   const uint32_t *__restrict__ group_cnt,
                                                   uint32_t *s_prefix) {
    if (threadIdx.x >= 64) return;
    const uint32_t own = chunk_prefix_by_wave(ci, c, chunk_cnt, group_cnt);
    if (threadIdx.x == 0) *s_prefix = own;
}

// ----------------------------------------------------------------- emit --
// Streams g and r once more: v = r + g; kept elements go out in ascending index order at
// the position given by the chunk prefix plus the popcount of the mask bits before them;
// the residual becomes +0 where kept and v elsewhere.
__global__ __launch_bounds__(256) void k_emit(const LayerDev *__restrict__ layers,
                                              const ChunkInfo *__restrict__ chunk_info, const float *__restrict__ grad,
                                              float *__restrict__ resid,
                                              uint32_t *__restrict__ mask,
                                              const uint32_t *__restrict__ chunk_cnt,
                                              const uint32_t *__restrict__ group_cnt,
                                              uint32_t *__restrict__ out_idx,
                                              float *__restrict__ out_val,
                                              int32_t *__restrict__ out_counts, const NextCall nc) {
    if (prepare_next_call(nc)) return;
    __shared__ uint32_t wave_tot[4];
    __shared__ uint32_t s_word[256];
    __shared__ uint32_t s_pref[256];
    __shared__ uint32_t s_cbase;
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x - 1;
    const ChunkInfo ci = chunk_info[c];
    const LayerDev L = layers[ci.layer];
    const uint32_t start = ci.start, len = ci.len;
    const size_t base = ci.arena_off;
    const uint32_t nwords = (len + 31) >> 5;
    const uint32_t word = static_cast<uint32_t>(tid) < nwords ? mask[(base >> 5) + tid] : 0;
    const float *__restrict__ g = grad + base;
    float *__restrict__ r = resid + base;
    const bool whole = len == static_cast<uint32_t>(kChunk);
    // A whole chunk: every load is issued before the mask scan, so the scan's latency and the
    // loads overlap and each thread keeps 16 wide loads in flight.
    float4 gq[kChunk / 1024], rq[kChunk / 1024];
    if (whole) {
#pragma unroll
        for (int j = 0; j < kChunk / 1024; ++j) {
            gq[j] = load_streaming(g + j * 1024 + 4 * tid);
            rq[j] = load_streaming(r + j * 1024 + 4 * tid);
        }
    }
    chunk_prefix_wave0(ci, c, chunk_cnt, group_cnt, &s_cbase);
    if (word) mask[(base >> 5) + tid] = 0u;            // (every word is read by one thread: clear for the next call)
    const uint32_t cnt = __popc(word);
    s_word[tid] = word;
    const uint32_t incl = block_scan_incl(cnt, wave_tot);
    const uint32_t cbase = s_cbase;
    const size_t obase = static_cast<size_t>(L.out_off) + cbase;
    const uint32_t room = L.cap > cbase ? L.cap - cbase : 0u;   // never write past the segment
    s_pref[tid] = incl - cnt;
    if (ci.last && tid == 255) out_counts[ci.layer] = static_cast<int32_t>(cbase + incl);
    __syncthreads();
    if (whole) {
#pragma unroll
        for (int j = 0; j < kChunk / 1024; ++j) {
            const uint32_t e = j * 1024 + 4 * tid;
            const uint32_t w = s_word[e >> 5];
            const uint32_t sh = e & 31;
            const uint32_t bits = (w >> sh) & 0xfu;
            float v[4] = {rq[j].x + gq[j].x, rq[j].y + gq[j].y, rq[j].z + gq[j].z, rq[j].w + gq[j].w};
            if (bits) {
                uint32_t pos = s_pref[e >> 5] + __popc(w & ((1u << sh) - 1u));
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (bits & (1u << q)) {
                        if (pos < room) {
                            out_idx[obase + pos] = start + e + q;
                            out_val[obase + pos] = v[q];
                        }
                        ++pos;
                        v[q] = 0.f;
                    }
            }
            store_streaming(r + e, make_float4(v[0], v[1], v[2], v[3]));
        }
        return;
    }
#pragma unroll 2
    for (int j = 0; j < kChunk / 1024; ++j) {
        const uint32_t e = j * 1024 + 4 * tid;
        if (e >= len) break;
        const uint32_t w = s_word[e >> 5];
        const uint32_t sh = e & 31;
        const uint32_t bits = (w >> sh) & 0xfu;
        if (e + 3 < len) {
            const float4 gv = *reinterpret_cast<const float4 *>(g + e);
            const float4 rv = *reinterpret_cast<const float4 *>(r + e);
            float v[4] = {rv.x + gv.x, rv.y + gv.y, rv.z + gv.z, rv.w + gv.w};
            if (bits) {
                uint32_t pos = s_pref[e >> 5] + __popc(w & ((1u << sh) - 1u));
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (bits & (1u << q)) {
                        if (pos < room) {
                            out_idx[obase + pos] = start + e + q;
                            out_val[obase + pos] = v[q];
                        }
                        ++pos;
                        v[q] = 0.f;
                    }
            }
            *reinterpret_cast<float4 *>(r + e) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
            uint32_t pos = s_pref[e >> 5] + __popc(w & ((1u << sh) - 1u));
            for (uint32_t q = 0; q < 4 && e + q < len; ++q) {
                float v = r[e + q] + g[e + q];
                if (bits & (1u << q)) {
                    if (pos < room) {
                        out_idx[obase + pos] = start + e + q;
                        out_val[obase + pos] = v;
                    }
                    ++pos;
                    v = 0.f;
                }
                r[e + q] = v;
            }
        }
    }
}

// Two-buffer form of the emit: the NSI passes have already stored v = r + g in the second
// residual arena, so only the kept elements are touched -- their value goes out and the
// arena gets +0 there.  A chunk without kept elements costs one read of its mask words.  A
// layer with k_l = 0 went through no NSI pass; its v is formed here.
__global__ __launch_bounds__(256) void k_emit_sparse(const ChunkInfo *__restrict__ chunk_info,
                                                     const SelState *__restrict__ state,
                                                     const float *__restrict__ grad,
                                                     const float *__restrict__ resid_in,
                                                     float *__restrict__ v_arena,
                                                     const float *__restrict__ mom_in,
                                                     float *__restrict__ mom_arena, float m,
                                                     uint32_t *__restrict__ mask,
                                                     const uint32_t *__restrict__ chunk_cnt,
                                                     const uint32_t *__restrict__ group_cnt,
                                                     uint32_t *__restrict__ out_idx,
                                                     float *__restrict__ out_val,
                                                     int32_t *__restrict__ out_counts, const NextCall nc) {
    if (prepare_next_call(nc)) return;
    __shared__ uint32_t wave_tot[4];
    __shared__ uint16_t s_list[kChunk];
    __shared__ uint32_t s_total, s_cbase;
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x - 1;
    const ChunkInfo ci = chunk_info[c];
    const uint32_t start = ci.start, len = ci.len;
    const size_t base = ci.arena_off;
    float *__restrict__ v = v_arena + base;
    // the three loads that depend only on the chunk's entry go out together
    const uint32_t nwords = (len + 31) >> 5;
    uint32_t word = static_cast<uint32_t>(tid) < nwords ? mask[(base >> 5) + tid] : 0;
    // (k_l = 0: kModeSkip in this call's state and in the next call's, which the first workgroup is writing)
    const uint32_t mode = state[ci.layer].mode;
    chunk_prefix_wave0(ci, c, chunk_cnt, group_cnt, &s_cbase);
    if (word) mask[(base >> 5) + tid] = 0u;            // (every word is read by one thread: clear for the next call)
    if (mode == kModeSkip) {
        if (ci.last && tid == 0) out_counts[ci.layer] = 0;
        const float *__restrict__ g = grad + base;
        const float *__restrict__ r = resid_in + base;
        for (uint32_t e = 4 * tid; e < len; e += 1024) {
            for (uint32_t q = 0; q < 4 && e + q < len; ++q) {
                float gu = g[e + q];
                if (mom_in) {
                    gu = __fmul_rn(m, mom_in[base + e + q]) + gu;
                    mom_arena[base + e + q] = gu;
                }
                v[e + q] = r[e + q] + gu;
            }
        }
        return;
    }
    if (!__syncthreads_or(word != 0u) && !ci.last) return;      // uniform
    const uint32_t cbase = s_cbase;
    const uint32_t cnt = __popc(word);
    const uint32_t incl = block_scan_incl(cnt, wave_tot);
    // the chunk's kept elements, in ascending order, as offsets inside the chunk
    uint32_t pos = incl - cnt;
    while (word) {
        const uint32_t b = static_cast<uint32_t>(__ffs(word)) - 1u;
        word &= word - 1u;
        s_list[pos++] = static_cast<uint16_t>(32u * static_cast<uint32_t>(tid) + b);
    }
    if (tid == 255) {
        s_total = incl;
        if (ci.last) out_counts[ci.layer] = static_cast<int32_t>(cbase + incl);
    }
    __syncthreads();
    const uint32_t total = s_total;
    const size_t obase = static_cast<size_t>(ci.out_off) + cbase;
    const uint32_t room = ci.cap > cbase ? ci.cap - cbase : 0u;   // never write past the segment
    // one kept element per thread: independent loads, coalesced pair stores
    for (uint32_t i = tid; i < total; i += 256) {
        const uint32_t e = s_list[i];
        if (e >= len) break;                // (mask bits exist only for elements of the layer)
        const float val = v[e];
        if (i < room) {
            out_idx[obase + i] = start + e;
            out_val[obase + i] = val;
        }
        v[e] = 0.f;
        if (mom_arena) mom_arena[base + e] = 0.f;     // the momentum restarts where v was sent
    }
}

// The same for plans of many chunks: one wave per chunk, four chunks per workgroup, no barrier.  What bounds the emit there is
// the chain entry -> mask words and prefix -> values, so as many chunks as possible have to be on their way at once.  Workgroup /
// wave per chunk, both with the mask clearing: 25088 x 4096 at 0.1 % 16.0 / 9.3 us, 4.2 k chunks 12.9 / 10.6 at 2 % and 8.5 / 5.9
// at 0.1 %, VGG-19 (17 k chunks, 2 %) 42.8 / 37.7 us on a residual carried for dozens of calls and 40.8 / 30.7 where the kept
// elements lie closer (the same step again from one residual).  With momentum, whose kept elements are zeroed in two arenas,
// the carried residual has it the other way round, 51.4 / 55.7 us, the repeated step 40.5 / 28.2.  On a plan of few chunks a
// workgroup each has the shorter chain (ResNet-18's 1.4 k chunks: 6.3 / 7.6 us; 3.1 k chunks with dense ones among them:
// 14.5 / 16.9 us).  The line is that of the plans that count as they mark.
constexpr int kEmitList = 1024;            // kept elements of a chunk that a wave lists at a time

// The 128 mask bits that a lane of the wave holds of its chunk, and the kept elements before them.
struct ChunkBits {
    uint32_t w[4];
    uint32_t before, total;                // kept elements of the chunk before this lane's / in all
};
__device__ __forceinline__ ChunkBits chunk_bits(const uint2 lo, const uint2 hi) {
    const int lane = threadIdx.x & 63;
    ChunkBits b;
    b.w[0] = lo.x; b.w[1] = lo.y; b.w[2] = hi.x; b.w[3] = hi.y;
    const uint32_t own = __popc(lo.x) + __popc(lo.y) + __popc(hi.x) + __popc(hi.y);
    uint32_t incl = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    b.before = incl - own;
    b.total = __builtin_amdgcn_readlane(incl, 63);
    return b;
}

// Offsets inside the chunk of its kept elements number b0 .. b0 + n - 1 (n <= kEmitList), in ascending order, to list.
__device__ __forceinline__ void list_chunk_bits(const ChunkBits &b, uint32_t b0, uint32_t n, uint16_t *list) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t pos = b.before - b0;          // (may wrap below zero: not below n then)
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        uint32_t word = b.w[j];
        while (word) {
            const uint32_t bit = static_cast<uint32_t>(__ffs(word)) - 1u;
            word &= word - 1u;
            if (pos < n) list[pos] = static_cast<uint16_t>(128u * lane + 32u * j + bit);
            ++pos;
        }
    }
}

__global__ __launch_bounds__(256) void k_emit_waves(const ChunkInfo *__restrict__ chunk_info, uint32_t n_chunks,
                                                    const SelState *__restrict__ state,
                                                    const float *__restrict__ grad,
                                                    const float *__restrict__ resid_in,
                                                    float *__restrict__ v_arena,
                                                    const float *__restrict__ mom_in,
                                                    float *__restrict__ mom_arena, float m,
                                                    uint32_t *__restrict__ mask,
                                                    const uint32_t *__restrict__ chunk_cnt,
                                                    const uint32_t *__restrict__ group_cnt,
                                                    uint32_t *__restrict__ out_idx,
                                                    float *__restrict__ out_val,
                                                    int32_t *__restrict__ out_counts, const NextCall nc) {
    if (prepare_next_call(nc)) return;
    __shared__ uint16_t s_list[4][kEmitList];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint16_t *list = s_list[wave];
    const uint32_t c = __builtin_amdgcn_readfirstlane((blockIdx.x - 1) * 4u + wave);
    if (c >= n_chunks) return;
    const ChunkInfo ci = chunk_info[c];
    const uint32_t start = ci.start, len = ci.len;
    const size_t base = ci.arena_off;
    float *__restrict__ v = v_arena + base;
    // the loads that depend only on the chunk's entry go out together.  (A layer starts at a multiple of two words and is
    // padded to one: a pair whose first word exists may be read whole.)
    const uint32_t nwords = (len + 31) >> 5;
    uint2 *__restrict__ words = reinterpret_cast<uint2 *>(mask + (base >> 5)) + 2 * lane;
    uint2 lo = make_uint2(0u, 0u), hi = make_uint2(0u, 0u);
    if (4 * lane < nwords) lo = words[0];
    if (4 * lane + 2 < nwords) hi = words[1];
    // (k_l = 0: kModeSkip in this call's state and in the next call's, which the first workgroup is writing)
    const uint32_t mode = state[ci.layer].mode;
    const uint32_t cbase = chunk_prefix_by_wave(ci, c, chunk_cnt, group_cnt);
    // (every word is read by one lane: clear for the next call)
    if (lo.x | lo.y) words[0] = make_uint2(0u, 0u);
    if (hi.x | hi.y) words[1] = make_uint2(0u, 0u);
    if (mode == kModeSkip) {
        if (ci.last && lane == 0) out_counts[ci.layer] = 0;
        const float *__restrict__ g = grad + base;
        const float *__restrict__ r = resid_in + base;
        for (uint32_t e = 4 * lane; e < len; e += 256) {
            if (e + 3 < len) {
                float4 gu = load_streaming(g + e);
                const float4 rv = load_streaming(r + e);
                if (mom_in) {
                    const float4 u = load_streaming(mom_in + base + e);
                    gu = make_float4(__fmul_rn(m, u.x) + gu.x, __fmul_rn(m, u.y) + gu.y, __fmul_rn(m, u.z) + gu.z, __fmul_rn(m, u.w) + gu.w);
                    store_streaming(mom_arena + base + e, gu);
                }
                store_streaming(v + e, make_float4(rv.x + gu.x, rv.y + gu.y, rv.z + gu.z, rv.w + gu.w));
                continue;
            }
            for (uint32_t q = 0; q < 4 && e + q < len; ++q) {
                float gu = g[e + q];
                if (mom_in) {
                    gu = __fmul_rn(m, mom_in[base + e + q]) + gu;
                    mom_arena[base + e + q] = gu;
                }
                v[e + q] = r[e + q] + gu;
            }
        }
        return;
    }
    const ChunkBits bits = chunk_bits(lo, hi);
    if (ci.last && lane == 0) out_counts[ci.layer] = static_cast<int32_t>(cbase + bits.total);
    const size_t obase = static_cast<size_t>(ci.out_off) + cbase;
    const uint32_t room = ci.cap > cbase ? ci.cap - cbase : 0u;   // never write past the segment
    for (uint32_t b0 = 0; b0 < bits.total; b0 += kEmitList) {
        const uint32_t n = min(bits.total - b0, static_cast<uint32_t>(kEmitList));
        wave_lds_order();
        list_chunk_bits(bits, b0, n, list);
        wave_lds_order();
        constexpr int U = 4;               // kept elements of a lane on their way at once; coalesced pair stores
        for (uint32_t i0 = lane; i0 < n; i0 += 64 * U) {
            uint32_t e[U];
            float val[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                e[u] = i0 + 64 * u < n ? list[i0 + 64 * u] : 0xffffffffu;
                if (e[u] < len) val[u] = v[e[u]];            // (mask bits exist only for elements of the layer)
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (e[u] >= len) continue;
                const uint32_t i = b0 + i0 + 64 * u;
                if (i < room) {
                    out_idx[obase + i] = start + e[u];
                    out_val[obase + i] = val[u];
                }
                v[e[u]] = 0.f;
                if (mom_arena) mom_arena[base + e[u]] = 0.f;     // the momentum restarts where v was sent
            }
        }
    }
}

// Ascending list of the selected centres of every layer.
__global__ __launch_bounds__(256) void k_emit_centres(const LayerDev *__restrict__ layers,
                                                      const ChunkInfo *__restrict__ chunk_info,
                                                      uint32_t *__restrict__ cmask,
                                                      const uint32_t *__restrict__ chunk_ccnt,
                                                      const uint32_t *__restrict__ group_ccnt,
                                                      uint32_t *__restrict__ out_centre_idx,
                                                      int32_t *__restrict__ out_centre_counts) {
    __shared__ uint32_t wave_tot[4];
    __shared__ uint32_t s_cbase;
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x;
    const ChunkInfo ci = chunk_info[c];
    const LayerDev L = layers[ci.layer];
    const uint32_t start = ci.start;
    const size_t base = ci.arena_off;
    const uint32_t nwords = (ci.len + 31) >> 5;
    uint32_t word = static_cast<uint32_t>(tid) < nwords ? cmask[(base >> 5) + tid] : 0;
    chunk_prefix_wave0(ci, c, chunk_ccnt, group_ccnt, &s_cbase);
    if (word) cmask[(base >> 5) + tid] = 0u;           // (every word is read by one thread: clear for the next call)
    const uint32_t cnt = __popc(word);
    const uint32_t incl = block_scan_incl(cnt, wave_tot);
    const uint32_t cbase = s_cbase;
    if (ci.last && tid == 255 && out_centre_counts) out_centre_counts[ci.layer] = static_cast<int32_t>(cbase + incl);
    uint32_t rank = cbase + (incl - cnt);
    while (word) {
        const int b = __ffs(word) - 1;
        word &= word - 1;
        if (out_centre_idx && rank < L.k) out_centre_idx[static_cast<size_t>(L.centre_off) + rank] = start + 32u * tid + b;
        ++rank;
    }
}

// ----------------------------------------------------------- decompress --
// +0 into every element of every layer (the padding between layers is left alone): one chunk
// per workgroup, streaming 16-byte stores.  In a large arena each XCD writes one contiguous part: 103 -> 93 us for VGG-19's
// 559 MB (a fill of 16 bytes per thread that need not look up its chunk takes 83 us; without streaming stores 130 us here, and
// the scatter that follows 30 instead of 20 us).  Whole calls by parts / without, one layer of so many MB: 33: 11.0 / 10.5 us,
// 67: 17.1 / 15.8, 100: 22.9 / 22.9, 150: 32.9 / 33.4, 218: 45.8 / 47.8, 268: 54.4 / 56.9, 470: 91.2 / 98.8.
constexpr uint32_t kZeroByParts = 4096;   // chunks of an arena (134 MB) from which the XCDs take parts
__global__ __launch_bounds__(256) void k_zero_layers(const ChunkInfo *__restrict__ chunk_info, float *__restrict__ dense) {
    const int tid = threadIdx.x;
    const ChunkInfo ci = chunk_info[gridDim.x >= kZeroByParts ? xcd_contiguous(blockIdx.x, gridDim.x) : blockIdx.x];
    const uint32_t len = ci.len;
    float *__restrict__ d = dense + ci.arena_off;
#pragma unroll
    for (int j = 0; j < kChunk / 1024; ++j) {
        const uint32_t e = j * 1024 + 4 * tid;
        if (e >= len) break;
        if (e + 3 < len) {
            store_streaming(d + e, make_float4(0.f, 0.f, 0.f, 0.f));
        } else {
            for (uint32_t q = 0; q < 4 && e + q < len; ++q) d[e + q] = 0.f;
        }
    }
}

// Pairs of a layer in one message, whatever the message says.
__device__ __forceinline__ uint32_t pairs_in_segment(int32_t count, uint32_t cap) {
    return static_cast<uint32_t>(min(max(count, 0), static_cast<int32_t>(min(cap, 0x7fffffffu))));
}

// f(arena position, value) for the pairs of a message that are to be taken: one position per thread.  Nearly always a wave's 64
// positions lie in one layer's segment: the wave looks that up once, 64 layers at a time, and its constants stay in scalar
// registers.  (A binary search by every thread: 20.0 us for VGG-19's 2.3 M pairs, now 15.8; ResNet-18 with few pairs 3.2, now
// 3.4.  Four pairs per thread: 16.7 and 4.8, two: 15.1 and 3.6.)
template <typename F>
__device__ __forceinline__ void for_each_pair(const LayerDev *__restrict__ layers, int n_layers, long long capacity,
                                              const uint32_t *__restrict__ idx, const float *__restrict__ val,
                                              const int32_t *__restrict__ counts, F f) {
    const int lane = threadIdx.x & 63;
    const long long j0 = static_cast<long long>(blockIdx.x) * 256 + 64 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (j0 >= capacity) return;            // (the whole wave)
    const long long j = j0 + lane;
    // last layer of [lo, hi) whose segment starts at or before `at`, by the whole wave
    auto layer_of = [&](long long at, int lo, int hi) {
        while (hi - lo > 1) {
            const int step = (hi - lo + 63) >> 6, l = lo + lane * step;
            const bool starts = l < hi && layers[l].out_off <= at;          // (true in lane 0)
            lo += (__popcll(__ballot(starts)) - 1) * step;
            hi = min(hi, lo + step);
        }
        return lo;
    };
    const int lo = layer_of(j0, 0, n_layers);
    const LayerDev &L = layers[lo];
    const long long end = lo + 1 < n_layers ? layers[lo + 1].out_off : capacity;
    if (j0 + 64 <= end) {
        const uint32_t n = pairs_in_segment(counts[lo], L.cap), G = L.G;
        if (static_cast<uint32_t>(j - L.out_off) < n) {
            const uint32_t i = idx[j];
            const float v = val[j];
            if (i < G) f(static_cast<size_t>(L.elem_off) + i, v);           // (malformed message: the pair is ignored; G < 2^32)
        }
    } else {
        const int last = layer_of(min(j0 + 64, capacity) - 1, lo, n_layers);
        if (j >= capacity) return;
        int l = lo, hi = last + 1;
        while (hi - l > 1) {
            const int mid = (l + hi) >> 1;
            if (layers[mid].out_off <= j) l = mid; else hi = mid;
        }
        const long long q = j - layers[l].out_off;
        if (q >= counts[l] || q >= static_cast<long long>(layers[l].cap)) return;
        const uint32_t i = idx[j];
        if (i < layers[l].G) f(static_cast<size_t>(layers[l].elem_off) + i, val[j]);
    }
}

__global__ __launch_bounds__(256) void k_scatter(const LayerDev *__restrict__ layers, int n_layers,
                                                 long long capacity,
                                                 const uint32_t *__restrict__ idx,
                                                 const float *__restrict__ val,
                                                 const int32_t *__restrict__ counts,
                                                 float *__restrict__ dense, int accumulate) {
    for_each_pair(layers, n_layers, capacity, idx, val, counts, [&](size_t pos, float v) {
        if (accumulate) dense[pos] = dense[pos] + v; else dense[pos] = v;
    });
}

// --------------------------------------------------------- block reading --
// Non-overlapping p x p neighbourhoods (the other reading of Section III-C): one score per
// block.  `outer` are the element matrices, `inner` the block grids (one "element" per block).
// Work unit: a tile of 8 block rows by block_tile_cols(P) block columns of one layer.  Its
// elements are loaded with 16-byte loads (rows that are a multiple of 4 floats long), v = r + g
// goes to LDS and to the new residual arena (which may be r's own: no element is read by two
// tiles), then every thread takes blocks of the tile: Eqs. 8-10 in double over the p*p slots
// (zero outside the matrix, divisor p*p), score to the inner score map, 12-bit histogram.
// Persistent workgroups stride over the tiles; the histogram is flushed on layer change.
// CAPTURE (plans with a grid on the candidate path): of the grids that have a bound, predicted as in rsdgc_compress (none is ever sampled: without one
// a grid is ranked on its map), only the blocks that reach it are recorded, per tile, and counted in fine bins: the map is neither written
// nor read again by the gather and the mark, which have some 500 K keys to go through instead of 15.5 M scores.  VGG-19 at 2 %: this pass 296 /
// 294 us (it is as fast as it streams), find0 to mark 67 / 34, the call 423.5 -> 377.5; ResNet-18 67.1 -> 53.7, ResNet-50 92.8 -> 78.5, 6000 x 6000
// with p = 1 at 0.1 % 202 -> 130, 512 x 512 32.5 -> 28.1.  A call without bounds (the first with a workspace, after new ratios or while the
// threshold moves fast) takes what it does where no grid is on the candidate path: 398 / 393.  A variant of its own: on grids that stay on the map (300000 x 27) the code for the
// candidates, unused, took the pass from 63 to 69 us.
// FEED: tiles come from the launch's work feed (many tiles per workgroup) instead of a
// fixed strided share.  MOM: Eq. 12's first line on the way in -- u_new = m*u + g (one rounded
// multiply, one rounded add) takes g's place and goes to the new momentum arena (which, like
// the residual's, may be the old one).
struct BlockCapture {                  // what the candidate path adds: the bounds, and where the blocks that reach them are recorded
    SelState *state;
    uint32_t *hist_s, *list_cnt, *slot_cnt;
    unsigned long long *slot_ent;      // a slot per tile
};
// The score of the P x P block at `win` (LDS, row pitch `pitch`).  UNROLL: rows of it that are read together.
template <int P, int UNROLL>
__device__ __forceinline__ float block_score(const float *win, int pitch, double ca, double cb) {
    const double n = static_cast<double>(P * P);
    double sa = 0.0, ss = 0.0, sq = 0.0;
#pragma unroll UNROLL
    for (int dx = 0; dx < P; ++dx)
#pragma unroll
        for (int dy = 0; dy < P; ++dy) {
            const double w = static_cast<double>(win[dx * pitch + dy]);
            sa += fabs(w);
            ss += w;
            sq = fma(w, w, sq);
        }
    const double nsq = __dmul_rn(n, sq);
    double d = var_n2_one_pass(ss, nsq);
    if (P > 1 && d < kCancelFrac * nsq)          // the one-pass variance cancelled (rare)
        d = __dmul_rn(n, window_ssd<P>(win, pitch, ss / n));
    return static_cast<float>(nsi_from_var(sa, d, ca, cb));
}
template <int P, bool FEED, bool MOM, bool CAPTURE>
__global__ __launch_bounds__(256) void k_block_nsi(const LayerDev *__restrict__ outer,
                                                   const DirEntry *__restrict__ tile_dir,
                                                   uint32_t n_layers, uint32_t n_tiles,
                                                   const LayerDev *__restrict__ inner,
                                                   const float *__restrict__ grad,
                                                   const float *resid, float *v_out,
                                                   float *__restrict__ score_map,
                                                   uint32_t *__restrict__ hist, double alpha,
                                                   uint32_t *__restrict__ feed_ctr, uint32_t feed_shift,
                                                   const float *mom_in, float *mom_out, float m, const BlockCapture cp) {
    constexpr int BCT = block_tile_cols(P);
    constexpr int TR = kBlockTileRows * P, TC = BCT * P;      // tile in elements; TC is a multiple of 4
    constexpr int VEC_PER_ROW = TC / 4;
    constexpr int NVEC = TR * VEC_PER_ROW;
    constexpr int ITER = (NVEC + 255) / 256;
    constexpr int NBLK = kBlockTileRows * BCT;
    static_assert(TC % 4 == 0, "tile rows are whole 16-byte groups");
    __shared__ __attribute__((aligned(16))) float tile[TR * TC];
    __shared__ uint32_t lhist[kHistBins];
    __shared__ uint32_t feed_slot[2];
    __shared__ uint32_t ncand[2];          // candidates of the tile; the other one is being cleared
    const int tid = threadIdx.x;
    const uint32_t stride = gridDim.x;
    WorkFeed feed;
    uint32_t first;
    if (FEED) {
        first = feed.first(feed_ctr, n_tiles, feed_shift, feed_slot);
        if (first == kNoItem) return;      // uniform
    } else {
        first = blockIdx.x;
        if (first >= n_tiles) return;
    }
    for (int b = tid; b < kHistBins; b += 256) lhist[b] = 0;
    if (CAPTURE && tid < 2) ncand[tid] = 0;
    __syncthreads();
    const double ca = alpha / (P * P), cb = (1.0 - alpha) / (P * P);
    uint32_t e = dir_lookup(tile_dir, n_layers, first);
    uint32_t cur_l = 0xffffffffu, hint_key = 0, recorded = 0, par = 0;
    bool active = false, capture = false;              // capture: the layer's blocks are held against its bound
    LayerDev O, I;
    auto flush = [&]() {                               // the finished layer's counts
        uint32_t *__restrict__ gh = (CAPTURE && capture ? cp.hist_s : hist) + static_cast<size_t>(cur_l) * kHistBins;
        for (int b = tid; b < (CAPTURE && capture ? kFineBins : kHistBins); b += 256) {
            const uint32_t c = lhist[b];
            if (c) { atomicAdd(&gh[b], c); lhist[b] = 0; }
        }
        if (CAPTURE && tid == 0 && recorded) atomicAdd(recorded_slot(cp.list_cnt, cur_l, blockIdx.x), recorded);
        recorded = 0;
    };
    for (uint32_t t = first; FEED ? t != kNoItem : t < n_tiles;
         t = FEED ? feed.next(feed_slot) : t + stride) {
        e = dir_advance(tile_dir, n_layers, e, t);
        const uint32_t l = tile_dir[e].layer;
        if (l != cur_l) {
            if (active) {
                flush();
                __syncthreads();
            }
            cur_l = l;
            O = outer[l];
            I = inner[l];
            active = static_cast<int>(O.p) == P;       // another launch takes the other neighbourhood sides
            if (CAPTURE) hint_key = cp.state[l].hint_key;
            capture = CAPTURE && active && I.large != 0u && cp.state[l].mode == kModeCandidates && bound_in_range(hint_key);
        }
        if (!active) {
            if (!FEED) {
                const uint32_t nb = tile_dir[e + 1].begin;
                t += (nb - t + stride - 1) / stride * stride - stride;
            }
            continue;
        }
        const uint32_t local = t - tile_dir[e].begin;
        const int trow = static_cast<int>(local / O.tiles_x);
        const int tcol = static_cast<int>(local - static_cast<uint32_t>(trow) * O.tiles_x);
        const int R = static_cast<int>(O.R), C = static_cast<int>(O.C);
        const int x0 = trow * TR, y0 = tcol * TC;
        const float *__restrict__ g = grad + O.elem_off;
        const float *r = resid + O.elem_off;           // may be the same arena as vo
        float *vo = v_out + O.elem_off;
        const float *ui = MOM ? mom_in + O.elem_off : nullptr;     // may be the same arena as uo
        float *uo = MOM ? mom_out + O.elem_off : nullptr;
        if ((C & 3) == 0) {
            float4 gv[ITER], rv[ITER], uv[MOM ? ITER : 1];
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int s = tid + it * 256;
                const int rr = s / VEC_PER_ROW, j4 = s - rr * VEC_PER_ROW;
                const int x = x0 + rr, y = y0 + 4 * j4;
                gv[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                rv[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (MOM) uv[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (s < NVEC && x < R && y < C) {
                    const size_t off = static_cast<size_t>(x) * C + y;
                    gv[it] = load_streaming(g + off);       // blocks share no element
                    rv[it] = load_streaming(r + off);
                    if (MOM) uv[it] = load_streaming(ui + off);
                }
            }
            if (FEED) feed.stash(feed_slot);      // the loads are out, no store of this tile yet
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int s = tid + it * 256;
                if (s < NVEC) {
                    const int rr = s / VEC_PER_ROW, j4 = s - rr * VEC_PER_ROW;
                    const int x = x0 + rr, y = y0 + 4 * j4;
                    const bool inside = x < R && y < C;
                    if (MOM) {
                        gv[it].x = __fmul_rn(m, uv[it].x) + gv[it].x;
                        gv[it].y = __fmul_rn(m, uv[it].y) + gv[it].y;
                        gv[it].z = __fmul_rn(m, uv[it].z) + gv[it].z;
                        gv[it].w = __fmul_rn(m, uv[it].w) + gv[it].w;
                        if (inside) store_streaming(uo + static_cast<size_t>(x) * C + y, gv[it]);
                    }
                    const float4 v = make_float4(rv[it].x + gv[it].x, rv[it].y + gv[it].y,
                                                 rv[it].z + gv[it].z, rv[it].w + gv[it].w);
                    *reinterpret_cast<float4 *>(&tile[s * 4]) = v;          // s*4 == rr*TC + 4*j4
                    if (inside) store_streaming(vo + static_cast<size_t>(x) * C + y, v);
                }
            }
        } else {
            // (whole rows per wave, all of a row's floats requested together, as in the NSI passes)
            constexpr int N = (TC + 63) / 64;
            const int wave = tid >> 6, lane = tid & 63;
#pragma unroll 1
            for (int rr = wave; rr < TR; rr += 4) {
                const int x = x0 + rr;
                const size_t row = static_cast<size_t>(x) * C;
                float gq[N], rq[N], uq[MOM ? N : 1];
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    const int j = lane + 64 * q, y = y0 + j;
                    gq[q] = rq[q] = 0.f;
                    if (MOM) uq[q] = 0.f;
                    if (x < R && j < TC && y < C) {
                        gq[q] = (g + row)[y];
                        rq[q] = (r + row)[y];
                        if (MOM) uq[q] = (ui + row)[y];
                    }
                }
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    const int j = lane + 64 * q, y = y0 + j;
                    float v = 0.f;
                    if (x < R && j < TC && y < C) {
                        float gu = gq[q];
                        if (MOM) {
                            gu = __fmul_rn(m, uq[q]) + gu;
                            (uo + row)[y] = gu;
                        }
                        v = rq[q] + gu;
                        (vo + row)[y] = v;
                    }
                    if (j < TC) tile[rr * TC + j] = v;
                }
            }
        }
        __syncthreads();
        const uint32_t BR = I.R, BC = I.C;
#pragma unroll
        for (int q = tid; q < NBLK; q += 256) {
            const int br = q / BCT, bc = q - br * BCT;
            const uint32_t bx = static_cast<uint32_t>(trow * kBlockTileRows + br);
            const uint32_t by = static_cast<uint32_t>(tcol * BCT + bc);
            if (bx < BR && by < BC) {
                const float score = block_score<P, P>(&tile[(br * P) * TC + bc * P], TC, ca, cb);
                const uint32_t key = __float_as_uint(score) & 0x7fffffffu;
                if (!CAPTURE || !capture) {
                    score_map[I.elem_off + static_cast<size_t>(bx) * BC + by] = score;
                    atomicAdd(&lhist[key >> kCoarseShift], 1u);
                } else if (key >= hint_key) {
                    const uint32_t pos = atomicAdd(&ncand[par], 1u);
                    if (pos < I.slot_cap) cp.slot_ent[I.slot_off + static_cast<size_t>(local) * I.slot_cap + pos] = composite_key(key, bx * BC + by);
                    atomicAdd(&lhist[min((key - hint_key) >> kFineShift, static_cast<uint32_t>(kFineBins - 1))], 1u);
                }
            }
        }
        __syncthreads();                               // the tile is reused by the next item
        if (CAPTURE && capture) {
            if (tid == 0) {
                const uint32_t nc = ncand[par];
                recorded += nc;
                cp.slot_cnt[I.tile_begin_all + local] = min(nc, I.slot_cap);
                if (nc > I.slot_cap) cp.state[l].overflow = 1u;
                ncand[par] = 0u;                       // (used again after the next tile's barrier)
            }
            par ^= 1u;
        }
    }
    if (active) flush();
}

// A grid whose bound failed, or whose tile overfilled its slot: it is ranked on its full map, and its blocks' scores are formed once more, from v,
// which the pass above has stored.  Workgroups stride over the tiles; in one launch with k_find0: they look at the layers themselves.
// P: the largest side of the plan, which sizes the tile in LDS.  VGG-19 with every bound failed: 202 us here (380 where a thread read its block from
// v, p floats from its neighbour's), the call 614, where a call that ranks them all on their maps takes 424.  (The scores stored by the
// pass in every call, and only counted here, made that 505 and the calls whose bounds hold 383 instead of 377.)
struct BlockRescore {
    const LayerDev *outer, *inner;
    const DirEntry *tile_dir;
    uint32_t n_tiles;
    const float *v;
    float *score_map;
    uint32_t *hist, *list_cnt;
    double alpha;
};
template <int P> constexpr int kBlockTileElems = kBlockTileRows * P * P * block_tile_cols(P);
static_assert(kBlockTileElems<1> <= kBlockTileElems<3> && kBlockTileElems<3> <= kBlockTileElems<5> && kBlockTileElems<5> <= kBlockTileElems<7>,
              "the largest side's tile holds any other's");
template <int P>
__device__ __forceinline__ void rescore_tile(const BlockRescore &r, const LayerDev &O, const LayerDev &I, uint32_t local, float *tile /*[kBlockTileElems], LDS*/,
                                             uint32_t *lhist) {
    constexpr int BCT = block_tile_cols(P), TC = BCT * P, TR = kBlockTileRows * P;
    const uint32_t tid = threadIdx.x, trow = local / O.tiles_x, tcol = local - trow * O.tiles_x, x0 = trow * TR, y0 = tcol * TC;
    const double ca = r.alpha / (P * P), cb = (1.0 - r.alpha) / (P * P);
    const float *__restrict__ v = r.v + O.elem_off;
    if constexpr (P == 1) {               // (elements in a row: a chunk by the workgroup of the tile of the same number, of which there are more)
        constexpr uint32_t N = kChunk / 256;
        if (local >= I.n_chunks) return;
        const uint32_t start = local * kChunk, len = min(static_cast<uint32_t>(kChunk), I.G - start);
        float e[N];
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) e[j] = v[start + min(256 * j + tid, len - 1u)];
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) {
            if (256 * j + tid >= len) break;
            const float score = block_score<1, 1>(&e[j], 1, ca, cb);
            r.score_map[I.elem_off + start + 256 * j + tid] = score;
            atomicAdd(&lhist[(__float_as_uint(score) & 0x7fffffffu) >> kCoarseShift], 1u);
        }
        return;
    }
    if ((O.C & 3u) == 0u) {
        constexpr uint32_t V = TC / 4, N = (TR * V + 255) / 256;
        float4 e[N];
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) {
            const uint32_t i = tid + 256 * j, row = i / V, y = y0 + 4 * (i - row * V);
            e[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (row < TR && x0 + row < O.R && y < O.C) e[j] = *reinterpret_cast<const float4 *>(v + static_cast<size_t>(x0 + row) * O.C + y);
        }
#pragma unroll
        for (uint32_t j = 0; j < N; ++j)
            if (tid + 256 * j < TR * V) *reinterpret_cast<float4 *>(&tile[4 * (tid + 256 * j)]) = e[j];
    } else {
        constexpr uint32_t N = (TC + 63) / 64;         // (whole rows per wave, as in the pass)
#pragma unroll 1
        for (uint32_t row = tid >> 6; row < TR; row += 4) {
            float e[N];
#pragma unroll
            for (uint32_t j = 0; j < N; ++j) {
                const uint32_t y = y0 + tid % 64 + 64 * j;
                e[j] = x0 + row < O.R && y < O.C ? (v + static_cast<size_t>(x0 + row) * O.C)[y] : 0.f;
            }
#pragma unroll
            for (uint32_t j = 0; j < N; ++j)
                if (tid % 64 + 64 * j < TC) tile[row * TC + tid % 64 + 64 * j] = e[j];
        }
    }
    __syncthreads();
    for (uint32_t q = tid; q < kBlockTileRows * BCT; q += 256) {
        const uint32_t br = q / BCT, bc = q - br * BCT, bx = trow * kBlockTileRows + br, by = tcol * BCT + bc;
        if (bx >= I.R || by >= I.C) continue;
        const float score = block_score<P, P <= 3 ? P : 1>(&tile[br * P * TC + bc * P], TC, ca, cb);
        r.score_map[I.elem_off + static_cast<size_t>(bx) * I.C + by] = score;
        atomicAdd(&lhist[(__float_as_uint(score) & 0x7fffffffu) >> kCoarseShift], 1u);
    }
    __syncthreads();
}
template <int P>
__global__ __launch_bounds__(256) void k_find0_blocks(const Find0Args f, const BlockRescore r) {
    __shared__ uint32_t lhist[kHistBins];
    __shared__ __attribute__((aligned(16))) float tile[kBlockTileElems<P>];
    const uint32_t n_layers = static_cast<uint32_t>(f.n_layers);
    if (blockIdx.x < n_layers) {
        find0(f, blockIdx.x);
        return;
    }
    auto failed = [&](uint32_t l) {                    // (without a bound the pass above has written the map)
        if (r.inner[l].large == 0u || !bound_in_range(f.state[l].hint_key)) return false;
        return layer_falls_back(r.inner, f.state, f.hist_s, r.list_cnt, l);
    };
    const uint32_t tid = threadIdx.x;
    static_assert(kGridLayers <= 256, "a layer per thread");
    if (!__syncthreads_or(tid < n_layers && failed(tid))) return;
    for (uint32_t b = tid; b < static_cast<uint32_t>(kHistBins); b += 256) lhist[b] = 0u;
    __syncthreads();
    uint32_t e = 0, cur_l = 0xffffffffu;
    bool active = false;
    auto flush = [&]() {
        uint32_t *__restrict__ gh = r.hist + static_cast<size_t>(cur_l) * kHistBins;
        for (uint32_t b = tid; b < static_cast<uint32_t>(kHistBins); b += 256) {
            const uint32_t c = lhist[b];
            if (c) { atomicAdd(&gh[b], c); lhist[b] = 0u; }
        }
    };
    const uint32_t stride = gridDim.x - n_layers;
    for (uint32_t t = blockIdx.x - n_layers; t < r.n_tiles; t += stride) {
        e = dir_advance(r.tile_dir, n_layers, e, t);
        if (r.tile_dir[e].layer != cur_l) {
            __syncthreads();
            if (active) flush();
            __syncthreads();
            cur_l = r.tile_dir[e].layer;
            active = failed(cur_l);
        }
        if (!active) {                                 // on to this workgroup's first tile of the next layer
            const uint32_t nb = r.tile_dir[e + 1].begin;
            t += (nb - t + stride - 1) / stride * stride - stride;
            continue;
        }
        const LayerDev &O = r.outer[cur_l], &I = r.inner[cur_l];
        const uint32_t local = t - r.tile_dir[e].begin;
        if (P == 7 && O.p == 7u) rescore_tile<7>(r, O, I, local, tile, lhist);
        else if (P >= 5 && O.p == 5u) rescore_tile<5>(r, O, I, local, tile, lhist);
        else if (P >= 3 && O.p == 3u) rescore_tile<3>(r, O, I, local, tile, lhist);
        else rescore_tile<1>(r, O, I, local, tile, lhist);
    }
    __syncthreads();
    if (active) flush();
}

// The kept blocks of a chunk, kEmitBlocks at a time: first their places (one division per block, not one per slot), then one
// thread per (kept block, slot), four slots of a thread on their way at once, contiguous value stores.  (Slot after slot,
// each with its own divisions: 48 us on VGG-19, now 41 us.)
constexpr uint32_t kEmitBlocks = 512;
template <int P>
__device__ __forceinline__ void emit_blocks_of_chunk(const LayerDev &O, uint32_t BC, const ChunkInfo &ci, uint32_t cbase,
                                                     uint32_t total, const uint16_t *s_list, uint2 *s_place /*[kEmitBlocks]*/,
                                                     float *__restrict__ v_arena, float *__restrict__ u_arena,
                                                     uint32_t *__restrict__ out_blocks, float *__restrict__ out_val) {
    constexpr uint32_t PP = P * P, U = 4;
    const uint32_t R = O.R, C = O.C, k = O.k;
    float *__restrict__ v = v_arena + O.elem_off;
    float *__restrict__ u = u_arena ? u_arena + O.elem_off : nullptr;
    float *__restrict__ out = out_val + static_cast<size_t>(O.out_off) + static_cast<size_t>(cbase) * PP;
    uint32_t *__restrict__ out_b = out_blocks + static_cast<size_t>(O.centre_off) + cbase;
    // (never past the layer's segment; mask bits exist only for blocks of the grid)
    const uint32_t n = min(total, k > cbase ? k - cbase : 0u);
    for (uint32_t b0 = 0; b0 < n; b0 += kEmitBlocks) {
        const uint32_t nb = min(n - b0, kEmitBlocks);
        for (uint32_t i = threadIdx.x; i < nb; i += 256) {
            const uint32_t b = ci.start + s_list[b0 + i];
            const uint32_t bx = b / BC, by = b - bx * BC;
            out_b[b0 + i] = b;
            // place of the first slot, and how many of the block's rows and columns lie inside the matrix
            s_place[i] = make_uint2(bx * P * C + by * P, min(R - bx * P, static_cast<uint32_t>(P)) << 8 | min(C - by * P, static_cast<uint32_t>(P)));
        }
        __syncthreads();
        for (uint32_t i0 = threadIdx.x; i0 < nb * PP; i0 += 256 * U) {
            uint32_t off[U];
            bool in[U];
            float val[U];
#pragma unroll
            for (uint32_t q = 0; q < U; ++q) {
                const uint32_t i = i0 + 256 * q;
                in[q] = false;
                val[q] = 0.f;
                if (i < nb * PP) {
                    const uint32_t kb = i / PP, sl = i - kb * PP, dx = sl / P, dy = sl - dx * P;
                    const uint2 place = s_place[kb];
                    in[q] = dx < (place.y >> 8) && dy < (place.y & 255u);
                    off[q] = place.x + dx * C + dy;           // (below R * C where it is inside)
                    if (in[q]) val[q] = v[off[q]];
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < U; ++q) {
                const uint32_t i = i0 + 256 * q;
                if (i < nb * PP) out[b0 * PP + i] = val[q];   // (a layer's value segment is counted in 32 bits)
                if (in[q]) {
                    v[off[q]] = 0.f;
                    if (u) u[off[q]] = 0.f;
                }
            }
        }
        __syncthreads();
    }
}

// Kept blocks of one chunk of a layer's grid, in ascending order: block index to the index
// list, the block's p*p values (row-major, +0 for slots outside the matrix) to the value
// list, +0 into the new residual (and into the new momentum, when the call carries one).
__global__ __launch_bounds__(256) void k_emit_blocks(const LayerDev *__restrict__ outer,
                                                     const ChunkInfo *__restrict__ inner_chunks,
                                                     uint32_t *__restrict__ mask,
                                                     const uint32_t *__restrict__ chunk_cnt,
                                                     const uint32_t *__restrict__ group_cnt,
                                                     const LayerDev *__restrict__ inner,
                                                     float *__restrict__ v_arena,
                                                     float *__restrict__ u_arena /* nullable */,
                                                     uint32_t *__restrict__ out_blocks,
                                                     float *__restrict__ out_val,
                                                     int32_t *__restrict__ out_counts, const NextCall nc) {
    if (prepare_next_call(nc)) return;
    __shared__ uint32_t wave_tot[4];
    __shared__ uint16_t s_list[kChunk];
    __shared__ uint2 s_place[kEmitBlocks];
    __shared__ uint32_t s_total, s_cbase;
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x - 1;
    const ChunkInfo ci = inner_chunks[c];
    const uint32_t nwords = (ci.len + 31) >> 5;
    uint32_t word = static_cast<uint32_t>(tid) < nwords ? mask[(ci.arena_off >> 5) + tid] : 0;
    chunk_prefix_wave0(ci, c, chunk_cnt, group_cnt, &s_cbase);
    if (word) mask[(ci.arena_off >> 5) + tid] = 0u;   // (every word is read by one thread: clear for the next call)
    if (!__syncthreads_or(word != 0u) && !ci.last) return;      // uniform
    const uint32_t cbase = s_cbase;
    const uint32_t cnt = __popc(word);
    const uint32_t incl = block_scan_incl(cnt, wave_tot);
    uint32_t pos = incl - cnt;
    while (word) {
        const uint32_t b = static_cast<uint32_t>(__ffs(word)) - 1u;
        word &= word - 1u;
        s_list[pos++] = static_cast<uint16_t>(32u * static_cast<uint32_t>(tid) + b);
    }
    if (tid == 255) {
        s_total = incl;
        if (ci.last) out_counts[ci.layer] = static_cast<int32_t>(cbase + incl);
    }
    __syncthreads();
    const uint32_t total = s_total;
    const LayerDev &O = outer[ci.layer];
    const uint32_t BC = inner[ci.layer].C;
    switch (O.p) {
        case 1: emit_blocks_of_chunk<1>(O, BC, ci, cbase, total, s_list, s_place, v_arena, u_arena, out_blocks, out_val); break;
        case 3: emit_blocks_of_chunk<3>(O, BC, ci, cbase, total, s_list, s_place, v_arena, u_arena, out_blocks, out_val); break;
        case 5: emit_blocks_of_chunk<5>(O, BC, ci, cbase, total, s_list, s_place, v_arena, u_arena, out_blocks, out_val); break;
        default: emit_blocks_of_chunk<7>(O, BC, ci, cbase, total, s_list, s_place, v_arena, u_arena, out_blocks, out_val); break;
    }
}

// Inverse: one thread per kept block of a message.
__global__ __launch_bounds__(256) void k_scatter_blocks(const LayerDev *__restrict__ outer, int n_layers,
                                                        long long capacity,
                                                        const uint32_t *__restrict__ blocks,
                                                        const float *__restrict__ val,
                                                        const int32_t *__restrict__ counts,
                                                        float *__restrict__ dense, int accumulate) {
    const long long j = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
    if (j >= capacity) return;
    int lo = 0, hi = n_layers;            // last layer whose block segment starts at or before j
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (outer[mid].centre_off <= j) lo = mid; else hi = mid;
    }
    const LayerDev O = outer[lo];
    const long long q = j - O.centre_off;
    if (q >= counts[lo] || q >= static_cast<long long>(O.k)) return;
    const int P = static_cast<int>(O.p), R = static_cast<int>(O.R), C = static_cast<int>(O.C);
    const uint32_t BC = (O.C + O.p - 1) / O.p, BR = (O.R + O.p - 1) / O.p;
    const uint32_t b = blocks[j];
    if (b >= BR * BC) return;             // malformed message: ignore the block
    const int bx = static_cast<int>(b / BC), by = static_cast<int>(b - static_cast<uint32_t>(bx) * BC);
    const float *__restrict__ src = val + static_cast<size_t>(O.out_off) + static_cast<size_t>(q) * (P * P);
    float *__restrict__ d = dense + O.elem_off;
    for (int dx = 0; dx < P; ++dx)
        for (int dy = 0; dy < P; ++dy) {
            const int x = bx * P + dx, y = by * P + dy;
            if (x < R && y < C) {
                const size_t off = static_cast<size_t>(x) * C + y;
                if (accumulate) d[off] = d[off] + src[dx * P + dy]; else d[off] = src[dx * P + dy];
            }
        }
}

// ---------------------------------------------------------------- apply --
// Eq. 12, third line: w <- w - eta * (sum over the nodes' messages).  No dense accumulator: the
// messages are index-sorted per layer (rsdgc_compress writes them so), so the pairs that fall into
// one stretch of kApplySpan elements of a layer are one contiguous stretch of every message.  A first
// kernel finds where those begin (one search per message and stretch, all in parallel); the second
// takes one stretch per workgroup, sums the messages' values in an LDS array in the order given --
// message after message, a barrier between them, plain float32 adds starting from +0 -- and updates
// the weights whose sum is not +0.  One message needs none of this: every pair is applied on its own.
struct ApplyMsgs {
    const uint32_t *idx[RSDGC_MAX_MSGS];
    const float *val[RSDGC_MAX_MSGS];
    const int32_t *counts[RSDGC_MAX_MSGS];
};
// Half a chunk: 16 KB of LDS, so that a CU holds eight workgroups (a whole chunk left it four, and
// what a workgroup waits for is latency).
constexpr int kApplySpan = kChunk / 2;
constexpr int kApplyAhead = 2;            // pairs of a message that a lane requests before any is added: 128 a message

// First position in a[0, n) whose value is not below x (a ascending).  Seven probes a round instead
// of one: the rounds are dependent loads, about 1 us each, and there are a third as many of them.
// Any content of a gives a position in [0, n] and reads inside it.
__device__ __forceinline__ uint32_t lower_bound_wide(const uint32_t *__restrict__ a, uint32_t n, uint32_t x) {
    uint32_t lo = 0, len = n;             // the answer lies in [lo, lo + len]
    while (len >= 8u) {
        const uint32_t step = len >> 3;
        uint32_t c = 0;
#pragma unroll
        for (uint32_t i = 1; i < 8u; ++i) c += a[lo + i * step - 1u] < x ? 1u : 0u;
        lo += c * step;
        len = c == 7u ? len - 7u * step : step - 1u;
    }
    uint32_t c = 0;
#pragma unroll
    for (uint32_t i = 0; i < 7u; ++i) c += i < len && a[lo + min(i, len - 1u)] < x ? 1u : 0u;
    return lo + c;
}

// First position in a[0, n) whose value is not below x (a ascending).
__device__ __forceinline__ uint32_t lower_bound_u32(const uint32_t *__restrict__ a, uint32_t n, uint32_t x) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// starts[k * 2 n_chunks + 2 c + s]: first pair of message k in its layer's segment that falls into
// half s of chunk c, or later (a short last chunk's second half: the number of pairs).
// VGG-19, eight messages: 22 us with two binary searches per chunk, 20 us for twice the stretches; filling the
// table on one pass over the indices took 30 us.
__global__ __launch_bounds__(256) void k_apply_ranges(const ChunkInfo *__restrict__ chunk_info,
                                                      uint32_t n_chunks, int n_msgs, const ApplyMsgs msgs,
                                                      uint32_t *__restrict__ starts) {
    const uint64_t t = static_cast<uint64_t>(blockIdx.x) * 256u + threadIdx.x;
    const uint64_t per = 2ull * n_chunks;
    if (t >= per * static_cast<uint32_t>(n_msgs)) return;
    const uint32_t k = static_cast<uint32_t>(t / per), cs = static_cast<uint32_t>(t - k * per);
    const ChunkInfo ci = chunk_info[cs >> 1];
    const uint32_t n = pairs_in_segment(msgs.counts[k][ci.layer], ci.cap);
    // (no index of the layer reaches start + len in its last chunk: the search would end at n)
    starts[t] = lower_bound_wide(msgs.idx[k] + ci.out_off, n, ci.start + (cs & 1u) * kApplySpan);
}

// One workgroup per half chunk; every wave requests the pairs of its messages before any is added (one load
// latency for all eight instead of one each), and the weights are updated by all threads side by side, 16 bytes
// read by each where any of the four sums is not +0 (a thread that walked the bits of a touched-map word had ten
// dependent updates in a row).  Written are the named ones only: another stream may be at work on the others.  Moved on
// VGG-19 with eight messages: 560 MB for 340 MB of pairs and weights -- windows of p elements reach 60 % of the weights'
// 64-byte lines.  A call there 306 us before, now 207 us; 224 us where four single weights are written however many
// are named, and 225 us where neighbouring lanes read and write single neighbouring weights.  Measured and not taken: every
// thread requesting a pair of every message (178 us: the waves issue four times the instructions); one stretch
// of 1024 elements per wave without barriers (175 us, and eight times the ranges to find); of 2048 (240 us: half
// the waves); persistent waves with a cursor into every message (296 us), or software-pipelined (213 us: 153 registers).
__global__ __launch_bounds__(256) void k_apply_chunks(const ChunkInfo *__restrict__ chunk_info, uint32_t n_chunks,
                                                      int n_msgs, const ApplyMsgs msgs,
                                                      const uint32_t *__restrict__ starts,
                                                      float *__restrict__ weights, float eta) {
    __shared__ __attribute__((aligned(16))) float acc[kApplySpan];
    __shared__ uint32_t s_rng[RSDGC_MAX_MSGS][2];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x >> 1, s = blockIdx.x & 1u;
    const ChunkInfo ci = chunk_info[c];
    const uint32_t first = s * kApplySpan;             // the stretch inside the chunk: [first, end)
    if (first >= ci.len) return;
    const uint32_t end = min(ci.len, first + kApplySpan), len = end - first;
    bool mine = false;
    if (tid < n_msgs) {
        const uint32_t *__restrict__ st = starts + static_cast<size_t>(tid) * 2u * n_chunks + 2u * c + s;
        const uint32_t a = st[0], b = ci.last && end == ci.len ? pairs_in_segment(msgs.counts[tid][ci.layer], ci.cap) : st[1];
        s_rng[tid][0] = a;
        s_rng[tid][1] = b;
        mine = a < b;
    }
    if (!__syncthreads_or(mine)) return;               // no message names an element of this stretch
#pragma unroll
    for (int j = 0; j < kApplySpan / 1024; ++j) *reinterpret_cast<float4 *>(&acc[j * 1024 + 4 * tid]) = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    const uint32_t base = ci.start + first;
    const int lane = tid & 63, wave = tid >> 6;
    for (int k0 = 0; k0 < n_msgs; k0 += 8) {           // wave w takes messages k0 + w and k0 + 4 + w of a batch of eight
        uint32_t rel[2][kApplyAhead];
        float val[2][kApplyAhead];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int k = k0 + 4 * m + wave;
            const uint32_t a = k < n_msgs ? s_rng[k][0] : 0u, b = k < n_msgs ? s_rng[k][1] : 0u;
            const int kc = min(k, n_msgs - 1);
#pragma unroll
            for (int q = 0; q < kApplyAhead; ++q) {
                rel[m][q] = 0xffffffffu;
                val[m][q] = 0.f;
                const uint32_t j = a + 64u * q + lane;
                if (j < b) {
                    rel[m][q] = msgs.idx[kc][ci.out_off + j] - base;
                    val[m][q] = msgs.val[kc][ci.out_off + j];
                }
            }
        }
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {               // the sum, message by message, in the order given
            const int k = k0 + kk;
            if (k >= n_msgs) break;                    // uniform
            if (wave == (kk & 3)) {
#pragma unroll
                for (int q = 0; q < kApplyAhead; ++q)
                    if (rel[kk >> 2][q] < len) acc[rel[kk >> 2][q]] = acc[rel[kk >> 2][q]] + val[kk >> 2][q];   // (always, for a sorted message)
                const uint32_t b = s_rng[k][1];
                for (uint32_t j = s_rng[k][0] + 64u * kApplyAhead + lane; j < b; j += 64u) {
                    const uint32_t rj = msgs.idx[k][ci.out_off + j] - base;
                    if (rj < len) acc[rj] = acc[rj] + msgs.val[k][ci.out_off + j];
                }
            }
            __syncthreads();
        }
    }
    float *__restrict__ w = weights + ci.arena_off + first;
    float4 sum[kApplySpan / 1024], old[kApplySpan / 1024];
    bool any[kApplySpan / 1024];
#pragma unroll
    for (int j = 0; j < kApplySpan / 1024; ++j) {
        const uint32_t e = j * 1024 + 4 * tid;
        sum[j] = *reinterpret_cast<const float4 *>(&acc[e]);
        any[j] = (__float_as_uint(sum[j].x) | __float_as_uint(sum[j].y) | __float_as_uint(sum[j].z) | __float_as_uint(sum[j].w)) != 0u;
        if (any[j] && e + 3 < len) old[j] = *reinterpret_cast<const float4 *>(w + e);
    }
#pragma unroll
    for (int j = 0; j < kApplySpan / 1024; ++j) {
        const uint32_t e = j * 1024 + 4 * tid;
        if (!any[j]) continue;
        const float t[4] = {sum[j].x, sum[j].y, sum[j].z, sum[j].w};
        if (e + 3 < len) {
            const float v[4] = {old[j].x - __fmul_rn(eta, t[0]), old[j].y - __fmul_rn(eta, t[1]),
                                old[j].z - __fmul_rn(eta, t[2]), old[j].w - __fmul_rn(eta, t[3])};
            if (__float_as_uint(t[0]) != 0u && __float_as_uint(t[1]) != 0u && __float_as_uint(t[2]) != 0u && __float_as_uint(t[3]) != 0u) {
                *reinterpret_cast<float4 *>(w + e) = make_float4(v[0], v[1], v[2], v[3]);
            } else {                       // (a weight that no message names is not written)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (__float_as_uint(t[q]) != 0u) w[e + q] = v[q];
            }
        } else {
            for (uint32_t q = 0; q < 4 && e + q < len; ++q)
                if (__float_as_uint(t[q]) != 0u) w[e + q] = w[e + q] - __fmul_rn(eta, t[q]);
        }
    }
}

// One message: every pair on its own.
__global__ __launch_bounds__(256) void k_apply_single(const LayerDev *__restrict__ layers, int n_layers,
                                                      long long capacity, const uint32_t *__restrict__ idx,
                                                      const float *__restrict__ val,
                                                      const int32_t *__restrict__ counts,
                                                      float *__restrict__ weights, float eta) {
    for_each_pair(layers, n_layers, capacity, idx, val, counts, [&](size_t pos, float v) {
        const float sum = 0.f + v;        // (the sum of one message, formed like any other: +0 + val)
        if (__float_as_uint(sum) != 0u) weights[pos] = weights[pos] - __fmul_rn(eta, sum);
    });
}

// Block messages (the block reading): one thread per kept block of every message.  The block
// belongs to the lowest-numbered message that names it (the others find it there by binary
// search in the layer's ascending block list and step aside); its owner looks the block up in
// the later messages, adds their values slot by slot in message order -- plain float32 adds
// starting from +0, as for element messages -- and updates the block's slots inside the matrix.
// No atomics, no scratch memory.
template <int P>
__device__ __forceinline__ void apply_block(const LayerDev &O, int layer, uint32_t b, int k, uint32_t q,
                                            int n_msgs, const ApplyMsgs &msgs,
                                            float *__restrict__ weights, float eta) {
    float sum[P * P];
    {
        const float *__restrict__ src = msgs.val[k] + O.out_off + static_cast<size_t>(q) * (P * P);
#pragma unroll
        for (int s = 0; s < P * P; ++s) sum[s] = 0.f + src[s];
    }
    for (int k2 = k + 1; k2 < n_msgs; ++k2) {
        const uint32_t n2 = static_cast<uint32_t>(min(max(msgs.counts[k2][layer], 0), static_cast<int32_t>(O.k)));
        const uint32_t *__restrict__ seg = msgs.idx[k2] + O.centre_off;
        const uint32_t pos = lower_bound_u32(seg, n2, b);
        if (pos < n2 && seg[pos] == b) {
            const float *__restrict__ src = msgs.val[k2] + O.out_off + static_cast<size_t>(pos) * (P * P);
#pragma unroll
            for (int s = 0; s < P * P; ++s) sum[s] = sum[s] + src[s];
        }
    }
    const int R = static_cast<int>(O.R), C = static_cast<int>(O.C);
    const uint32_t BC = (O.C + P - 1) / P;
    const int bx = static_cast<int>(b / BC), by = static_cast<int>(b - static_cast<uint32_t>(bx) * BC);
#pragma unroll
    for (int dx = 0; dx < P; ++dx)
#pragma unroll
        for (int dy = 0; dy < P; ++dy) {
            const int x = bx * P + dx, y = by * P + dy;
            if (x < R && y < C) {
                const size_t pos = static_cast<size_t>(O.elem_off) + static_cast<size_t>(x) * C + y;
                const float t = sum[dx * P + dy];
                if (__float_as_uint(t) != 0u) weights[pos] = weights[pos] - __fmul_rn(eta, t);
            }
        }
}

__global__ __launch_bounds__(256) void k_apply_blocks(const LayerDev *__restrict__ outer, int n_layers,
                                                      long long capacity, int n_msgs, const ApplyMsgs msgs,
                                                      float *__restrict__ weights, float eta) {
    const long long j = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
    if (j >= capacity) return;
    const int k = blockIdx.y;
    int lo = 0, hi = n_layers;            // last layer whose block segment starts at or before j
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (outer[mid].centre_off <= j) lo = mid; else hi = mid;
    }
    const LayerDev O = outer[lo];
    const long long q = j - O.centre_off;
    if (q >= msgs.counts[k][lo] || q >= static_cast<long long>(O.k)) return;
    const uint32_t BC = (O.C + O.p - 1) / O.p, BR = (O.R + O.p - 1) / O.p;
    const uint32_t b = msgs.idx[k][j];
    if (b >= BR * BC) return;             // malformed message: ignore the block
    for (int k2 = 0; k2 < k; ++k2) {      // an earlier message that names the block owns it
        const uint32_t n2 = static_cast<uint32_t>(min(max(msgs.counts[k2][lo], 0), static_cast<int32_t>(O.k)));
        const uint32_t *__restrict__ seg = msgs.idx[k2] + O.centre_off;
        const uint32_t pos = lower_bound_u32(seg, n2, b);
        if (pos < n2 && seg[pos] == b) return;
    }
    switch (O.p) {
        case 1: apply_block<1>(O, lo, b, k, static_cast<uint32_t>(q), n_msgs, msgs, weights, eta); break;
        case 3: apply_block<3>(O, lo, b, k, static_cast<uint32_t>(q), n_msgs, msgs, weights, eta); break;
        case 5: apply_block<5>(O, lo, b, k, static_cast<uint32_t>(q), n_msgs, msgs, weights, eta); break;
        default: apply_block<7>(O, lo, b, k, static_cast<uint32_t>(q), n_msgs, msgs, weights, eta); break;
    }
}

// ------------------------------------------------------- dynamic ratios --
// Section III-B, Eqs. 3-5: one ranking of mu = |w| over all layers; the K top-ranked weights
// survive and a layer's keep ratio is its share of survivors.  Keys are the 31-bit patterns of |w|.
// Large networks: a sample of the weights brackets the K-th largest key, and ONE pass over the
// weights counts per layer what lies above the bracket and lists what lies inside it (a per cent
// or less); the rest is decided on the list.  When the sample misled (the K-th key lies outside the
// bracket, or far more weights in it than expected) the call goes on with the general path: the
// K-th largest key by a radix select over three streaming passes (12 + 10 + 9 bits), a
// fourth pass counting per layer the keys above and at the threshold.

// f(key) for the len keys at src (16-byte aligned), by a workgroup: a whole chunk's loads go out together.
template <typename F>
__device__ __forceinline__ void dyn_for_each_key(const uint32_t *__restrict__ src, uint32_t len, F f) {
    typedef uint32_t vu4 __attribute__((ext_vector_type(4)));       // (read once per pass: streamed)
    constexpr int N = kChunk / 1024;
    const int tid = threadIdx.x;
    if (len == static_cast<uint32_t>(kChunk)) {
        vu4 q[N];
#pragma unroll
        for (int j = 0; j < N; ++j) q[j] = __builtin_nontemporal_load(reinterpret_cast<const vu4 *>(src + j * 1024 + 4 * tid));
#pragma unroll
        for (int j = 0; j < N; ++j) {
            f(q[j].x & 0x7fffffffu);
            f(q[j].y & 0x7fffffffu);
            f(q[j].z & 0x7fffffffu);
            f(q[j].w & 0x7fffffffu);
        }
    } else {
        for (uint32_t e = tid; e < len; e += 256) f(src[e] & 0x7fffffffu);
    }
}

constexpr int kDynSampleBits = 13;                       // the sample's histogram: top 13 of the 31 key bits (3 % steps)
constexpr int kDynSampleBins = 1 << kDynSampleBits;
constexpr int kDynSubBins = 2048;                        // bins of the bracket
constexpr uint32_t kDynFinalCap = 4096;                  // keys of one such bin that the last kernel can hold
constexpr int kDynMaxLayers = 4096;                      // layers that the list's counters cover (LDS)
constexpr uint32_t kDynStage = 1024;                     // listed keys a workgroup of the main pass holds back
constexpr uint32_t kDynSamplePieces = 4;                 // 64-byte pieces sampled per chunk: one weight in 128
constexpr int64_t kDynSplitMin = 1 << 20;                // weights from which the one-pass form is taken
constexpr int kDynThreads = 512;                         // the main pass: threads of a workgroup
constexpr uint32_t kDynWorkgroups = 2;                   // ... and workgroups per CU
constexpr uint32_t kDynSampleThreads = 1024;

// State of the one-pass form (cleared by k_dyn_sample).
struct DynSplit {
    unsigned long long above;  // keys above the bracket, all layers
    uint32_t lo, hi;           // the bracket: lo <= key < hi
    uint32_t sub_shift;        // its bins are 2^sub_shift keys wide
    uint32_t bad;              // the sample's bracket is not used
    uint32_t n_list, n_final;  // keys listed; of those, keys in the bin that holds the K-th
};
struct DynSplitArgs {
    DynSplit *state;
    uint32_t *sample_hist;     // [kDynSampleBins]
    uint32_t *sub_hist;        // [kDynSubBins]
    uint32_t *cnt;             // [n_layers][2]
    uint2 *final_list;         // [kDynFinalCap]  (key, layer)
    uint2 *list;               // [list_cap]
    uint32_t list_cap, n_layers;
    unsigned long long K, n_weights;
    uint32_t *out;             // [n_layers][2]  the counts, in host memory
};

// The sample's histogram, for a call that finds it as something else left it (k_dyn_list leaves it clear; a launch in front of every call cost
// 4 us).
__global__ __launch_bounds__(256) void k_dyn_clear(const DynSplitArgs a) {
    a.sample_hist[blockIdx.x * 256u + threadIdx.x] = 0u;
}

// Histogram of a sample: kDynSamplePieces pieces of 16 weights per chunk, at places given by a hash; a short chunk
// gives each of its pieces with the probability of its share of a whole one.  A chain of three loads and the counts' way out
// bound it: as many threads as a workgroup can have (with 256 the kernel took 11.9 us on VGG-19's 140 M weights, with 1024 8.9), and
// several of a thread's pieces requested at once.
__global__ __launch_bounds__(kDynSampleThreads) void k_dyn_sample(const ChunkInfo *__restrict__ chunk_info, uint32_t n_chunks,
                                                                  const uint32_t *__restrict__ w, const DynSplitArgs a) {
    __shared__ uint32_t lhist[kDynSampleBins];
    constexpr uint32_t kPieces = kDynSampleThreads / 16;      // a round's
    const int tid = threadIdx.x;
    for (int b = tid; b < kDynSampleBins; b += kDynSampleThreads) lhist[b] = 0u;
    {                                      // what the passes that follow count in
        const uint32_t i = blockIdx.x * kDynSampleThreads + threadIdx.x, all = gridDim.x * kDynSampleThreads;
        if (i == 0) *a.state = DynSplit{0ull, 0u, 0u, 0u, 0u, 0u, 0u};
        for (uint32_t b = i; b < kDynSubBins; b += all) a.sub_hist[b] = 0u;
        for (uint32_t b = i; b < 2u * a.n_layers; b += all) a.cnt[b] = 0u;
    }
    __syncthreads();
    const uint32_t n_pieces = n_chunks * kDynSamplePieces, stride = gridDim.x * kPieces;
    // pieces in flight per 16 threads: the chain entry -> weight -> bin is what this kernel waits for (a call with 2 / 4 / 8 of them:
    // 12 M weights 69.2 / 69.4 / 70.5 us, 100 M 121.0 / 120.6 / 122.1, 140 M 167.3 / 166.7 / 167.6, 400 M 316.2 / 313.4 / 314.0)
    constexpr int U = 4;
    for (uint32_t i0 = blockIdx.x * kPieces; i0 < n_pieces; i0 += U * stride) {
        uint64_t at[U];
        bool have[U];
        uint32_t key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * stride + (tid >> 4);
            const ChunkInfo &ci = chunk_info[min(i, n_pieces - 1u) / kDynSamplePieces];
            const uint32_t len = ci.len, h = (i + 1u) * 2654435761u;
            const uint32_t e = (((h * 40503u) >> 8) % ((len + 15u) / 16u)) * 16u + (tid & 15u);
            have[u] = i < n_pieces && (h >> 19) < len && e < len;       // (13 bits: 0 .. kChunk - 1)
            at[u] = ci.arena_off + min(e, len - 1u);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = w[at[u]] & 0x7fffffffu;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (have[u]) atomicAdd(&lhist[key[u] >> (31 - kDynSampleBits)], 1u);
    }
    __syncthreads();
    for (int b = tid; b < kDynSampleBins; b += kDynSampleThreads) {
        const uint32_t c = lhist[b];
        if (c) atomicAdd(&a.sample_hist[b], c);
    }
}

// Keys inside the bracket, held back by a workgroup of the main pass.
struct DynStage {
    uint2 ent[kDynStage];
    uint32_t n, base;
};
__device__ __forceinline__ void dyn_stage_key(DynStage &sh, const DynSplitArgs &a, uint2 entry) {
    const uint32_t pos = atomicAdd(&sh.n, 1u);
    if (pos < kDynStage) {
        sh.ent[pos] = entry;
    } else {                               // (a chunk full of such keys)
        const uint32_t g = atomicAdd(&a.state->n_list, 1u);
        if (g < a.list_cap) a.list[g] = entry;
    }
}
__device__ __forceinline__ void dyn_flush_stage(DynStage &sh, const DynSplitArgs &a) {
    __syncthreads();
    const uint32_t n = min(sh.n, kDynStage);
    if (threadIdx.x == 0 && n) sh.base = atomicAdd(&a.state->n_list, n);
    __syncthreads();
    if (threadIdx.x < 256u)
        for (uint32_t i = threadIdx.x; i < n; i += 256)
            if (sh.base + i < a.list_cap) a.list[sh.base + i] = sh.ent[i];
    __syncthreads();
    if (threadIdx.x == 0) sh.n = 0u;
    __syncthreads();
}
// After a chunk: a stage that is half full is emptied.
__device__ __forceinline__ void dyn_make_room(DynStage &sh, const DynSplitArgs &a) {
    if (staged_more_than(sh.n, kDynStage / 2)) dyn_flush_stage(sh, a);
}

// q[j] of N values in registers, j of the thread's own: by halvings, not by way of memory.
template <int N>
__device__ __forceinline__ uint32_t dyn_pick(const uint32_t (&q)[N], uint32_t j) {
    if constexpr (N == 1) {
        return q[0];
    } else {
        uint32_t m[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const uint32_t x = q[2 * i], y = q[2 * i + 1];
            m[i] = j & 1u ? y : x;
        }
        return dyn_pick<N / 2>(m, j >> 1);
    }
}

// The main pass.  Every workgroup reads the bracket off the sample's histogram (the same one in each): the K-th key's
// rank in the sample, give or take eight standard deviations of it, on the safe side of the bin edges.  Then it strides over
// the chunks; reading 4 bytes per weight is what bounds it.  A thread notes which of its keys lie inside the bracket and takes
// those afterwards: with a branch per key a wave went through the stage's returning atomics a dozen times a chunk, for two
// or three keys of a lane at most.  Every workgroup costs about 14 ns for the bracket and its counts at the end: half as many
// threads twice as often take 4 us longer, four workgroups per CU 3 us, 1024 threads 3 us; looking at the stage every fourth
// chunk only 1 us, and requesting the next chunk's keys while one is gone through 4 us.
// VGG-19 (139.7 M weights): four passes of 104 .. 281 us and 23 us of finding at first; 124 us with a branch per key and 2048
// workgroups of 256; now 109 us (a read of as much that does nothing else takes 80 to 84)
// and 23 us around it; a call, with its wait, 706 us at first, 180, 165, with the counts written to the host and no clearing launch 149.  11.5 M
// weights 78 -> 66, 49 M 89 -> 77.
__global__ __launch_bounds__(kDynThreads) void k_dyn_split(const ChunkInfo *__restrict__ chunk_info, uint32_t n_chunks,
                                                           const uint32_t *__restrict__ w, const DynSplitArgs a) {
    __shared__ uint32_t sub[kDynSubBins];
    __shared__ DynStage stage;
    __shared__ uint32_t wave_tot[kDynThreads / 64];
    __shared__ uint32_t s_above, s_sampled, s_hi_bin, s_lo_bin, s_cum_hi, s_cum_lo;
    const int tid = threadIdx.x;
    for (int b = tid; b < kDynSubBins; b += kDynThreads) sub[b] = 0u;
    if (tid == 0) {
        s_above = stage.n = 0u;
        s_hi_bin = kDynSampleBins;         // (nothing is certainly above)
        s_lo_bin = 0u;
        s_cum_hi = 0u;
    }
    {
        constexpr int per = kDynSampleBins / kDynThreads;
        const int top = kDynSampleBins - tid * per;          // thread 0 holds the top bins
        uint32_t v[per], own = 0;
#pragma unroll
        for (int j = 0; j < per / 4; ++j) {
            const uint4 q = *reinterpret_cast<const uint4 *>(a.sample_hist + top - 4 * (j + 1));
            v[4 * j] = q.w; v[4 * j + 1] = q.z; v[4 * j + 2] = q.y; v[4 * j + 3] = q.x;
            own += q.x + q.y + q.z + q.w;
        }
        const uint32_t incl = block_scan_incl_n<kDynThreads / 64>(own, wave_tot);
        if (tid == kDynThreads - 1) { s_sampled = incl; s_cum_lo = incl; }
        __syncthreads();
        const uint32_t S = s_sampled;
        const float q = static_cast<float>(static_cast<double>(a.K) / static_cast<double>(a.n_weights));
        const float r = q * static_cast<float>(S), slack = 8.f * sqrtf(r * (1.f - q)) + 16.f;
        // bins are certainly above while the sample holds at most r - slack keys from their lower edge on; the bracket
        // ends with the bin at which it holds r + slack
        const float upper = r - slack, lower = r + slack;
        uint32_t acc = incl - own;
#pragma unroll
        for (int j = 0; j < per; ++j) {
            const uint32_t before = acc;
            acc += v[j];
            if (static_cast<float>(acc) > upper && static_cast<float>(before) <= upper) { s_hi_bin = top - j; s_cum_hi = before; }
            if (static_cast<float>(acc) >= lower && static_cast<float>(before) < lower) { s_lo_bin = top - 1 - j; s_cum_lo = acc; }
        }
        __syncthreads();
        // far more keys in the bracket than a continuous distribution has there: the general path
        if (S == 0u || s_cum_lo - s_cum_hi > S / 16u) {      // uniform, and the same in every workgroup
            if (blockIdx.x == 0 && tid == 0) a.state->bad = 1u;
            return;
        }
    }
    const uint32_t lo = s_lo_bin << (31 - kDynSampleBits);
    const uint32_t hi = min(s_hi_bin << (31 - kDynSampleBits), 0x80000000u);
    const uint32_t width = hi - lo;
    uint32_t sub_shift = 0;
    while (((width - 1u) >> sub_shift) >= static_cast<uint32_t>(kDynSubBins)) ++sub_shift;
    if (blockIdx.x == 0 && tid == 0) {
        a.state->lo = lo;
        a.state->hi = hi;
        a.state->sub_shift = sub_shift;
    }
    uint32_t cur_l = 0xffffffffu, above = 0, above_wave = 0; // this thread's count for cur_l, and its wave's
    unsigned long long above_all = 0;                        // thread 0: the workgroup's, all layers
    auto flush_layer = [&]() {
        if ((tid & 63) == 0) above += above_wave;
        if (above) atomicAdd(&s_above, above);
        above = above_wave = 0;
        __syncthreads();
        if (tid == 0 && s_above) {
            atomicAdd(&a.cnt[2 * cur_l], s_above);
            above_all += s_above;
            s_above = 0u;
        }
        __syncthreads();
    };
    typedef uint32_t vu4 __attribute__((ext_vector_type(4)));       // (read once: streamed)
    auto take = [&](uint32_t key) {                          // a key inside the bracket
        atomicAdd(&sub[(key - lo) >> sub_shift], 1u);
        dyn_stage_key(stage, a, make_uint2(key, cur_l));
    };
    // (each XCD reads one contiguous part of a round of chunks: 132 -> 124 us on VGG-19.  A chunk's entry is requested a chunk ahead)
    uint32_t c = xcd_contiguous(blockIdx.x, gridDim.x);
    ChunkInfo next = chunk_info[min(c, n_chunks - 1u)];
    for (; c < n_chunks; c += gridDim.x) {
        const ChunkInfo ci = next;
        next = chunk_info[min(c + gridDim.x, n_chunks - 1u)];
        if (ci.layer != cur_l) {                             // uniform
            if (cur_l != 0xffffffffu) flush_layer();
            cur_l = ci.layer;
        }
        const uint32_t *__restrict__ src = w + ci.arena_off;
        if (ci.len == static_cast<uint32_t>(kChunk)) {
            constexpr int N = kChunk / kDynThreads;          // keys of a thread
            uint32_t q[N];
#pragma unroll
            for (int j = 0; j < N; j += 4) {
                const vu4 v = __builtin_nontemporal_load(reinterpret_cast<const vu4 *>(src + j * kDynThreads + 4 * tid));
                q[j] = v.x; q[j + 1] = v.y; q[j + 2] = v.z; q[j + 3] = v.w;
            }
            uint32_t hits = 0;                               // key j: bit N - 1 - j
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const uint32_t key = q[j] & 0x7fffffffu;
                const bool over = key >= hi;
                above_wave += static_cast<uint32_t>(__popcll(__ballot(over)));       // (counted by the scalar unit)
                hits += hits + (key >= lo && !over ? 1u : 0u);
            }
            while (hits) {                                   // two or three rounds of a wave
                const uint32_t j = static_cast<uint32_t>(__ffs(hits)) - 1u;
                hits &= hits - 1u;
                take(dyn_pick<N>(q, N - 1u - j) & 0x7fffffffu);
            }
        } else {
            for (uint32_t e = tid; e < ci.len; e += kDynThreads) {
                const uint32_t key = src[e] & 0x7fffffffu;
                if (key >= hi) ++above;
                else if (key >= lo) take(key);
            }
        }
        dyn_make_room(stage, a);
    }
    if (cur_l != 0xffffffffu) flush_layer();
    dyn_flush_stage(stage, a);
    if (tid == 0 && above_all) atomicAdd(&a.state->above, above_all);
    for (int b = tid; b < kDynSubBins; b += kDynThreads) {
        const uint32_t c = sub[b];
        if (c) atomicAdd(&a.sub_hist[b], c);
    }
}

// The bracket's bin that holds the K-th key, and the keys still to take inside it; all 256 or more
// threads of the workgroup return the same (found = 0: the K-th key is not in the bracket).
template <int NW>
__device__ __forceinline__ DigitResult dyn_sub_bin(const DynSplitArgs &a, uint32_t *lh /*[kDynSubBins]*/,
                                                   uint32_t *wave_tot, DigitResult *res) {
    for (int b = threadIdx.x; b < kDynSubBins; b += NW * 64) lh[b] = a.sub_hist[b];
    __syncthreads();
    const DynSplit st = *a.state;
    DigitResult none = {0u, 0u, 0u, 0u};
    if (st.bad || st.above >= a.K || st.n_list > a.list_cap || a.K - st.above > st.n_list) return none;      // uniform
    return block_find_digit<NW>(lh, kDynSubBins, static_cast<uint32_t>(a.K - st.above), wave_tot, res);
}

// The listed keys of the bins above that one, per layer; those inside it go to the final list.
__global__ __launch_bounds__(256) void k_dyn_list(const DynSplitArgs a) {
    __shared__ uint32_t lh[kDynSubBins];
    __shared__ uint32_t cnt[kDynMaxLayers];
    __shared__ uint32_t wave_tot[4];
    __shared__ DigitResult res;
    for (uint32_t b = blockIdx.x * 256u + threadIdx.x; b < kDynSampleBins; b += gridDim.x * 256u) a.sample_hist[b] = 0u;       // (for the next call)
    const DigitResult r = dyn_sub_bin<4>(a, lh, wave_tot, &res);
    if (!r.found) return;                                    // uniform
    for (uint32_t i = threadIdx.x; i < a.n_layers; i += 256) cnt[i] = 0u;
    __syncthreads();
    const DynSplit st = *a.state;
    constexpr uint32_t U = 4;
    const uint32_t stride = gridDim.x * 256u;
    for (uint32_t i0 = blockIdx.x * 256u + threadIdx.x; i0 < st.n_list; i0 += U * stride) {
        uint2 k[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) k[u] = a.list[min(i0 + u * stride, st.n_list - 1u)];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (i0 + u * stride >= st.n_list) break;
            const uint32_t bin = (k[u].x - st.lo) >> st.sub_shift;
            if (bin > r.digit) {
                atomicAdd(&cnt[k[u].y], 1u);
            } else if (bin == r.digit) {
                const uint32_t pos = atomicAdd(&a.state->n_final, 1u);
                if (pos < kDynFinalCap) a.final_list[pos] = k[u];
            }
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < a.n_layers; i += 256)
        if (cnt[i]) atomicAdd(&a.cnt[2 * i], cnt[i]);
}

// One workgroup: the K-th key itself, then the final list's keys above and at it per layer, and all counts to the host (a copy
// behind the kernel, to memory that is not pinned, cost the call 10 us).  out[0] = ~0 tells the host that the sample's bracket did not serve.
__global__ __launch_bounds__(1024) void k_dyn_last(const DynSplitArgs a) {
    __shared__ uint32_t lh[kDynSubBins];
    __shared__ uint2 keys[kDynFinalCap];
    __shared__ uint32_t cnt[2 * kDynMaxLayers];
    __shared__ uint32_t wave_tot[16];
    __shared__ DigitResult res;
    const uint32_t tid = threadIdx.x;
    const DigitResult r = dyn_sub_bin<16>(a, lh, wave_tot, &res);
    const DynSplit st = *a.state;
    if (!r.found || st.n_final > kDynFinalCap) {             // uniform
        if (tid == 0) a.out[0] = 0xffffffffu;
        return;
    }
    const uint32_t n = st.n_final;
    for (uint32_t i = tid; i < n; i += 1024) keys[i] = a.final_list[i];
    for (uint32_t i = tid; i < 2u * a.n_layers; i += 1024) cnt[i] = a.cnt[i];
    const uint32_t base = st.lo + (r.digit << st.sub_shift);
    uint32_t k_rem = static_cast<uint32_t>(a.K - st.above) - r.above;        // >= 1, <= n
    uint32_t T = 0;                                          // key - base, digit by digit: at most 11 bits each
    for (int left = static_cast<int>(st.sub_shift); left > 0;) {
        const int bits = min(left, 11), shift = left - bits, nb = 1 << bits;
        __syncthreads();
        for (int b = tid; b < nb; b += 1024) lh[b] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < n; i += 1024) {
            const uint32_t rel = keys[i].x - base;
            if ((rel >> left) == (T >> left)) atomicAdd(&lh[(rel >> shift) & (nb - 1)], 1u);
        }
        __syncthreads();
        const DigitResult d = block_find_digit<16>(lh, nb, k_rem, wave_tot, &res);
        T |= d.digit << shift;
        k_rem -= d.above;
        left = shift;
    }
    __syncthreads();
    for (uint32_t i = tid; i < n; i += 1024) {
        const uint32_t rel = keys[i].x - base;
        if (rel > T) atomicAdd(&cnt[2 * keys[i].y], 1u);
        else if (rel == T) atomicAdd(&cnt[2 * keys[i].y + 1], 1u);
    }
    __syncthreads();
    for (uint32_t i = tid; i < 2u * a.n_layers; i += 1024) a.out[i] = cnt[i];
}

// ---- the general path
__global__ __launch_bounds__(256) void k_dyn_init(DynState *__restrict__ state,
                                                  unsigned long long *__restrict__ hist,
                                                  uint32_t *__restrict__ cnt, uint32_t n_cnt,
                                                  unsigned long long K) {
    const int tid = threadIdx.x;
    if (tid == 0) {
        DynState s;
        s.k_rem = K;
        s.prefix = 0;
        s.pad_ = 0;
        *state = s;
    }
    for (int b = tid; b < kHistBins; b += 256) hist[b] = 0ull;
    for (uint32_t i = tid; i < n_cnt; i += 256) cnt[i] = 0u;
}

// Histogram of the digit (key >> shift) & (2^bits - 1) over the keys whose higher bits
// (key >> prev_shift) equal the resolved prefix.  Persistent workgroups stride over the
// 8192-element chunks (padding between layers is never read).
__global__ __launch_bounds__(256) void k_dyn_hist(const ChunkInfo *__restrict__ chunk_info,
                                                  uint32_t n_chunks, const uint32_t *__restrict__ w,
                                                  const DynState *__restrict__ state, int shift,
                                                  int bits, int prev_shift,
                                                  unsigned long long *__restrict__ hist) {
    __shared__ uint32_t lhist[kHistBins];
    const int tid = threadIdx.x;
    const int nb = 1 << bits;
    for (int b = tid; b < nb; b += 256) lhist[b] = 0;
    __syncthreads();
    const uint32_t prefix = state->prefix;
    const uint32_t dmask = static_cast<uint32_t>(nb - 1);
    for (uint32_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const ChunkInfo ci = chunk_info[c];
        const uint32_t *__restrict__ src = w + ci.arena_off;
        for (uint32_t e = 4 * tid; e < ci.len; e += 1024) {
            uint32_t kk[4] = {0, 0, 0, 0};
            uint32_t nv = min(4u, ci.len - e);
            if (nv == 4) {
                typedef uint32_t vu4 __attribute__((ext_vector_type(4)));   // read once per pass: streamed
                const vu4 qq = __builtin_nontemporal_load(reinterpret_cast<const vu4 *>(src + e));
                const uint4 q = make_uint4(qq.x, qq.y, qq.z, qq.w);
                kk[0] = q.x; kk[1] = q.y; kk[2] = q.z; kk[3] = q.w;
            } else {
                for (uint32_t q = 0; q < nv; ++q) kk[q] = src[e + q];
            }
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t key = kk[q] & 0x7fffffffu;
                if (q < nv && (prev_shift >= 31 || (key >> prev_shift) == prefix))
                    atomicAdd(&lhist[(key >> shift) & dmask], 1u);
            }
        }
    }
    __syncthreads();
    for (int b = tid; b < nb; b += 256) {
        const uint32_t c = lhist[b];
        if (c) atomicAdd(&hist[b], static_cast<unsigned long long>(c));
    }
}

// One workgroup: the digit that holds the k_rem-th largest key; clears the histogram.
__global__ __launch_bounds__(256) void k_dyn_find(DynState *__restrict__ state,
                                                  unsigned long long *__restrict__ hist, int bits) {
    __shared__ unsigned long long tot[256];
    const int tid = threadIdx.x;
    const int nb = 1 << bits, per = nb >> 8;   // bits >= 8
    const DynState st = *state;
    const int hi = nb - tid * per;             // thread t owns bins [hi - per, hi): t = 0 holds the top bins
    unsigned long long own = 0;
    for (int b = hi - 1; b >= hi - per; --b) own += hist[b];
    tot[tid] = own;
    __syncthreads();
    if (tid == 0) {                            // 256 partial sums: a serial walk is short enough
        unsigned long long acc = 0;
        int t = 0;
        while (t < 255 && acc + tot[t] < st.k_rem) acc += tot[t++];
        const int h2 = nb - t * per;
        int digit = h2 - per;
        for (int b = h2 - 1; b >= h2 - per; --b) {
            const unsigned long long c = hist[b];
            if (acc + c >= st.k_rem) { digit = b; break; }
            acc += c;
        }
        DynState ns = st;
        ns.prefix = (st.prefix << bits) | static_cast<uint32_t>(digit);
        ns.k_rem = st.k_rem - acc;
        *state = ns;
    }
    __syncthreads();
    for (int b = tid; b < nb; b += 256) hist[b] = 0ull;
}

// Per layer: keys above the threshold and keys equal to it.  Persistent workgroups; the
// counts of a layer are added to its two counters once per workgroup.
__global__ __launch_bounds__(256) void k_dyn_count(const ChunkInfo *__restrict__ chunk_info,
                                                   uint32_t n_chunks, const uint32_t *__restrict__ w,
                                                   const DynState *__restrict__ state,
                                                   uint32_t *__restrict__ cnt /*[n_layers][2]*/) {
    __shared__ uint32_t s_gt, s_eq;
    const int tid = threadIdx.x;
    const uint32_t T = state->prefix;          // all 31 bits are resolved
    if (tid == 0) { s_gt = 0; s_eq = 0; }
    __syncthreads();
    uint32_t cur_l = 0xffffffffu;
    uint32_t gt = 0, eq = 0;                   // this thread's counts for cur_l
    for (uint32_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const ChunkInfo ci = chunk_info[c];
        if (ci.layer != cur_l) {               // uniform
            if (cur_l != 0xffffffffu) {
                if (gt) atomicAdd(&s_gt, gt);
                if (eq) atomicAdd(&s_eq, eq);
                __syncthreads();
                if (tid == 0) {
                    if (s_gt) atomicAdd(&cnt[2 * cur_l], s_gt);
                    if (s_eq) atomicAdd(&cnt[2 * cur_l + 1], s_eq);
                    s_gt = 0; s_eq = 0;
                }
                __syncthreads();
                gt = eq = 0;
            }
            cur_l = ci.layer;
        }
        dyn_for_each_key(w + ci.arena_off, ci.len, [&](uint32_t key) {
            gt += key > T ? 1u : 0u;
            eq += key == T ? 1u : 0u;
        });
    }
    if (cur_l != 0xffffffffu) {
        if (gt) atomicAdd(&s_gt, gt);
        if (eq) atomicAdd(&s_eq, eq);
        __syncthreads();
        if (tid == 0) {
            if (s_gt) atomicAdd(&cnt[2 * cur_l], s_gt);
            if (s_eq) atomicAdd(&cnt[2 * cur_l + 1], s_eq);
        }
    }
}

// ------------------------------------------------------------ host side --
// Everything a compress call expects of the workspace beside the tables.  Recorded into a graph it prepares nothing
// yet (the graph may never be launched, or only after an eager call): ws_ready stays false then, and every call up to
// the next eager one brings its own preparation.
int prepare_workspace(rsdgc_plan_s *plan, char *ws, bool sampling, StatesBefore before, hipStream_t stream) {
    const WsLayout &w = plan->ws;
    const bool block_grid = !plan->k_override.empty();     // no centre lists
    const size_t n16 = ((block_grid ? w.cmask : w.zero_end) - w.zero_begin) / 16;
    const unsigned blocks = static_cast<unsigned>(std::min<size_t>((n16 + 255) / 256, 4096));
    hipLaunchKernelGGL(k_begin, dim3(blocks + 1), dim3(256), 0, stream,
                       reinterpret_cast<uint4 *>(ws + w.zero_begin), n16,
                       reinterpret_cast<const LayerDev *>(ws + w.layers), reinterpret_cast<SelState *>(ws + w.state),
                       plan->n_layers, reinterpret_cast<PredState *>(ws + w.pred),
                       reinterpret_cast<uint32_t *>(ws + w.flags), sampling ? 1 : 0, static_cast<int>(before));
    HIP_TRY(hipGetLastError());
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(stream, &capture));
    plan->ws_ready = capture == hipStreamCaptureStatusNone;
    return RSDGC_OK;
}

int upload_tables(rsdgc_plan_s *plan, void *workspace, hipStream_t stream) {
    if (plan->uploaded_ws == workspace && plan->uploaded_version == plan->version) return RSDGC_OK;
    // (new ratios or another path, the same memory: the paths of the last call are still asked for there)
    const StatesBefore before = plan->uploaded_ws == workspace && plan->ws_ready ? kStatesBeforeCall : kStatesNone;
    plan->uploaded_ws = nullptr;           // (until all of it is enqueued)
    plan->ws_ready = false;
    HIP_TRY(hipMemcpyAsync(workspace, plan->table.data(), plan->ws.table_bytes,
                           hipMemcpyHostToDevice, stream));
    plan->calls_since_upload = 0;
    plan->dyn_clear = false;
    // Whatever call lays the tables down prepares the rest too: what comes next may be the replay of a graph that was
    // recorded on a prepared workspace.  (A block plan has its tables only; the selection runs on the inner plan's.)
    if (!plan->blocks) {
        const int rc = prepare_workspace(plan, static_cast<char *>(workspace), plan->any_large && plan->k_override.empty(), before, stream);
        if (rc != RSDGC_OK) return rc;
    }
    plan->uploaded_ws = workspace;
    plan->uploaded_version = plan->version;
    return RSDGC_OK;
}

// Workgroups of 256 threads of `kernel` that the whole device keeps resident at once: a
// persistent launch of exactly this many workgroups runs as a single balanced wave.
template <typename K>
uint32_t resident_workgroups(K kernel) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess || per_cu < 1)
        per_cu = 2;
    return kNumCUs * static_cast<uint32_t>(per_cu);
}

constexpr uint32_t kFeedTiles = 16u * kNumCUs * 4u;       // tiles from which a launch hands them out by the work feed

// One launch of the NSI kernel per neighbourhood side.  kPassSample runs over the sampled
// tiles of the large layers, every other pass over all tiles (workgroups of layers that
// are in another mode leave at once).
struct Momentum {                 // Eq. 12's momentum term; all null / 0 without it
    const float *in = nullptr;
    float *out = nullptr;
    float m = 0.f;
};

template <int PASS>
int launch_nsi(const rsdgc_plan_s *plan, char *ws, const float *grad, const float *resid,
               float *nsi_out, float *v_out, const Momentum &mom, hipStream_t stream,
               bool with_sampled_tiles = true, const Find0Args *find0_args = nullptr, uint4 *counts = nullptr, uint32_t n16 = 0,
               bool v_in_place = false) {
    constexpr bool kCaptures = pass_captures(PASS);
    NsiArgs a;
    a.v_in_place = v_in_place ? 1 : 0;
    a.counts = counts;
    a.n16 = n16;
    a.list_cnt = reinterpret_cast<uint32_t *>(ws + plan->ws.list_cnt);
    a.n_layers = plan->n_layers;
    a.v_out = v_out;
    a.mom = mom.in;
    a.mom_out = mom.out;
    a.m = mom.m;
    a.flags = reinterpret_cast<const uint32_t *>(ws + plan->ws.flags);
    a.hist_s = reinterpret_cast<uint32_t *>(ws + plan->ws.hist_s);
    a.layers = reinterpret_cast<const LayerDev *>(ws + plan->ws.layers);
    a.grad = grad;
    a.resid = resid;
    a.nsi_out = nsi_out;
    a.hist = reinterpret_cast<uint32_t *>(ws + plan->ws.hist);
    a.state = reinterpret_cast<const SelState *>(ws + plan->ws.state);
    a.state_rw = reinterpret_cast<SelState *>(ws + plan->ws.state);
    a.slot_cnt = reinterpret_cast<uint32_t *>(ws + plan->ws.slot_cnt);
    a.slot_ent = reinterpret_cast<unsigned long long *>(ws + plan->ws.slot_ent);
    a.ca = a.cb = 0.0;                 // set per neighbourhood side below
    const DirEntry *tile_dir = reinterpret_cast<const DirEntry *>(ws + plan->ws.tile_dir);
    const DirEntry *large_dir = reinterpret_cast<const DirEntry *>(ws + plan->ws.large_dir);
    // the main pass and its fallback concern the large layers only: they walk those layers' tiles
    constexpr bool kLargeOnly = kCaptures || PASS == kPassFullMap;
    const SampleEntry *samples = reinterpret_cast<const SampleEntry *>(ws + plan->ws.samples);
    const SampleEntry *large_tiles = reinterpret_cast<const SampleEntry *>(ws + plan->ws.map_tiles);
    uint32_t *feed = reinterpret_cast<uint32_t *>(ws + plan->ws.feed);
    int group_index = 0;
    // several sides in a small plan: one launch, where each of them would find nothing to do in nearly every call (all sides get
    // the registers of the largest, which the main pass would feel)
    const bool together = PASS == kPassFullMap && find0_args && plan->groups.size() > 1 && plan->n_tiles_all < kFeedTiles;
    NsiAllArgs all = {};
    uint32_t all_items = 0, ridden = 0;
    // the main pass of single elements has a kernel of its own, which takes small groups of other sides along
    uint32_t n_flat = 0;
    for (const PGroup &g : plan->groups)
        if (kCaptures && g.p == 1) n_flat = g.n_large_tiles;
    const bool flat_fed = plan->work_feed != RSDGC_FEED_OFF && (plan->work_feed == RSDGC_FEED_ON || n_flat >= kFeedTiles);     // (as below; then alone)
    for (const PGroup &g : plan->groups) {
        // this launch's work-feed counters (left clear by the call before)
        const int pass_index = PASS == kPassSample ? 0 : kCaptures ? 1 : 2;
        a.feed = feed + static_cast<size_t>((pass_index * 4 + group_index++) % kFeedSets) * kFeedDomains * kFeedStride;
        a.ca = plan->alpha / static_cast<double>(g.p * g.p);
        a.cb = (1.0 - plan->alpha) / static_cast<double>(g.p * g.p);
        a.dir = kLargeOnly ? large_dir + g.large_dir_begin : tile_dir + g.dir_begin;
        a.n_dir = kLargeOnly ? g.large_dir_count : g.dir_count;
        a.n_tiles = g.n_tiles;
        a.samples = kLargeOnly ? large_tiles + g.large_list_begin : samples + g.sample_begin;
        // work items of this launch and the number of workgroups that share them
        // (the first pass without the sampled tiles: only the layers that are always ranked on the full map)
        const uint32_t items = PASS == kPassSample ? (with_sampled_tiles ? g.n_samples : g.n_map_samples)
                                                   : kLargeOnly ? g.n_large_tiles : g.n_tiles;
        if (items == 0) continue;
        a.n_tiles = items;
        a.feed_shift = 7;                  // 128 items per domain and stretch: one per resident workgroup of an XCD
        const uint32_t shares = PASS == kPassCaptureInPlace ? (items + kRun - 1) / kRun : items;       // what the workgroups take at a time
        while (a.feed_shift > 0 && (static_cast<uint32_t>(kFeedDomains) << a.feed_shift) > shares) --a.feed_shift;
        const bool rides = items <= kRideTiles || (ridden + items <= std::min(n_flat, kRideMost) && g.most_large_tiles <= kRideLayer);
        if (together || (n_flat != 0u && (g.p == 1 || (rides && !flat_fed && PASS != kPassCaptureInPlace)))) {
            if (g.p != 1) ridden += items;
            all.side[g.p / 2] = a;
            all_items += items;
            continue;
        }
        const dim3 block(256);
        switch (g.p) {
#define RSDGC_NSI_LAUNCH(PP, MM, FF)                                                        \
    {                                                                                       \
        static const uint32_t resident = resident_workgroups(k_nsi<PP, PASS, MM, FF>);      \
        /* fixed shares: as many workgroups as give every one the same number of tiles    \
           (2786 tiles on 1280 resident workgroups take three rounds either way; 929       \
           workgroups of three tiles each leave the CUs less crowded in all three) */      \
        const uint32_t rounds = (shares + resident - 1) / resident;                         \
        const dim3 grid(FF ? std::min<uint32_t>(shares, resident) : (shares + rounds - 1) / rounds); \
        if (PASS == kPassFullMap && find0_args) {                                           \
            hipLaunchKernelGGL((k_find0_fallback<PP, MM>), dim3(grid.x + find0_args->n_layers), block, 0, stream, *find0_args, a); \
            find0_args = nullptr;          /* (the other sides' launches, if any, go by the flag) */ \
        } else                                                                              \
            hipLaunchKernelGGL((k_nsi<PP, PASS, MM, FF>), grid, block, 0, stream, a);       \
        if constexpr (PASS == kPassCaptureInPlace) {                                        \
            static const uint32_t seam_wgs = resident_workgroups(k_seams<PP>);              \
            hipLaunchKernelGGL(k_seams<PP>, dim3(std::min<uint32_t>((shares + 3) / 4, seam_wgs)), block, 0, stream, a); \
        }                                                                                   \
    }
#define RSDGC_NSI_CASE(PP)                                                                  \
    case PP: {                                                                              \
        /* the work feed pays when a workgroup gets many tiles (its start and its end cost  \
           a few round trips to the counters); built for the main pass */                   \
        constexpr bool kFeedBuilt = kCaptures;                                              \
        const bool fed = kFeedBuilt && plan->work_feed != RSDGC_FEED_OFF &&                 \
                         (plan->work_feed == RSDGC_FEED_ON || items >= kFeedTiles);         \
        constexpr bool kMomBuilt = PASS != kPassCaptureInPlace;   /* (no momentum with one arena) */ \
        if (mom.in) {                                                                       \
            if (fed) RSDGC_NSI_LAUNCH(PP, kMomBuilt, kFeedBuilt)                            \
            else RSDGC_NSI_LAUNCH(PP, kMomBuilt, false)                                     \
        } else {                                                                            \
            if (fed) RSDGC_NSI_LAUNCH(PP, false, kFeedBuilt)                                \
            else RSDGC_NSI_LAUNCH(PP, false, false)                                         \
        }                                                                                   \
        break;                                                                              \
    }
            case 1:
                if constexpr (!kCaptures) {
                    switch (1) { RSDGC_NSI_CASE(1) }
                }
                break;
            RSDGC_NSI_CASE(3)
            RSDGC_NSI_CASE(5)
            RSDGC_NSI_CASE(7)
#undef RSDGC_NSI_CASE
#undef RSDGC_NSI_LAUNCH
            default: return RSDGC_EINVAL;
        }
        HIP_TRY(hipGetLastError());
    }
    if (n_flat != 0u) {
        const bool alone = all_items == n_flat;
        static const uint32_t resident[2][2] = {{resident_workgroups(k_capture_mixed<false>), resident_workgroups(k_capture_mixed<true>)},
                                                {resident_workgroups(k_capture_flat<false, false>), resident_workgroups(k_capture_flat<true, false>)}};
        static const uint32_t resident_fed[2] = {resident_workgroups(k_capture_flat<false, true>), resident_workgroups(k_capture_flat<true, true>)};
        const uint32_t most = resident[alone ? 1 : 0][mom.in ? 1 : 0];
        const uint32_t rounds = (n_flat + most - 1) / most, n_wgs = (n_flat + rounds - 1) / rounds;        // (shares as below)
        if (flat_fed) {
            const dim3 grid(std::min(n_flat, resident_fed[mom.in ? 1 : 0]));
            if (mom.in) hipLaunchKernelGGL((k_capture_flat<true, true>), grid, dim3(256), 0, stream, all.side[0]);
            else hipLaunchKernelGGL((k_capture_flat<false, true>), grid, dim3(256), 0, stream, all.side[0]);
        } else if (alone) {
            if (mom.in) hipLaunchKernelGGL((k_capture_flat<true, false>), dim3(n_wgs), dim3(256), 0, stream, all.side[0]);
            else hipLaunchKernelGGL((k_capture_flat<false, false>), dim3(n_wgs), dim3(256), 0, stream, all.side[0]);
        } else {
            for (int i = 1; i < kSides; ++i) all.first_wg[i] = all.first_wg[i - 1] + all.side[kSides - i].n_tiles;   // a tile each
            all.first_wg[kSides] = all.first_wg[kSides - 1] + n_wgs;
            if (mom.in) hipLaunchKernelGGL(k_capture_mixed<true>, dim3(all.first_wg[kSides]), dim3(256), 0, stream, all);
            else hipLaunchKernelGGL(k_capture_mixed<false>, dim3(all.first_wg[kSides]), dim3(256), 0, stream, all);
        }
        HIP_TRY(hipGetLastError());
    }
    if (together) {
        const uint32_t resident = kNumCUs * 2u;
        const uint32_t rounds = std::max<uint32_t>(1u, (all_items + resident - 1) / resident);
        for (int i = 0; i < kSides; ++i)
            all.first_wg[i + 1] = all.first_wg[i] + (all.side[i].n_tiles + rounds - 1) / rounds;
        const dim3 grid(all.first_wg[kSides] + find0_args->n_layers);
        if (mom.in) hipLaunchKernelGGL(k_find0_fallback_all<true>, grid, dim3(256), 0, stream, *find0_args, all);
        else hipLaunchKernelGGL(k_find0_fallback_all<false>, grid, dim3(256), 0, stream, *find0_args, all);
        HIP_TRY(hipGetLastError());
    }
    return RSDGC_OK;
}

// Records the event that closes `stage` (and opens the next) when profiling is on.
struct StageMarks {
    rsdgc_plan_s *plan;
    hipStream_t stream;
    int base;   // index of this call's first event, -1 when not recording
    StageMarks(rsdgc_plan_s *p, hipStream_t s) : plan(p), stream(s), base(-1) {
        if (!p->prof_events.empty() && p->prof_calls < p->prof_max_calls) {
            base = p->prof_calls * (RSDGC_N_STAGES + 1);
            ++p->prof_calls;
            (void)hipEventRecord(static_cast<hipEvent_t>(p->prof_events[base]), s);
        }
    }
    void close(int stage) {
        if (base >= 0)
            (void)hipEventRecord(static_cast<hipEvent_t>(plan->prof_events[base + stage + 1]), stream);
    }
};

bool aligned256(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

extern "C" {

const char *rsdgc_last_hip_error(void) { return g_hip_error; }

// The counts from finished masks: the kept elements' (nullable), the centres' (nullable), or both in one launch.
static void launch_count(const rsdgc_plan_s *plan, char *ws, const uint32_t *mask, const uint32_t *cmask, hipStream_t stream) {
    if (!mask && !cmask) return;
    const WsLayout &w = plan->ws;
    const CountGroup *groups = reinterpret_cast<const CountGroup *>(ws + w.count_groups);
    hipLaunchKernelGGL(k_count, dim3(plan->n_count_groups), dim3(kCountThreads), 0, stream, groups, mask, cmask,
                       reinterpret_cast<uint32_t *>(ws + w.chunk_cnt), reinterpret_cast<uint32_t *>(ws + w.chunk_ccnt),
                       reinterpret_cast<uint32_t *>(ws + w.group_cnt), reinterpret_cast<uint32_t *>(ws + w.group_ccnt),
                       static_cast<uint32_t>(group_cnt_stride(plan->count_how)));
}

// The part of a compress call between the NSI passes and the emit: radix select of every
// layer's threshold, marking of the kept elements, kept counts per chunk and chunk group.
static int select_mark_count(rsdgc_plan_s *plan, char *ws, bool want_centres, StageMarks &marks,
                             PredState *pred, hipStream_t stream, const float *grad = nullptr, float *v_in_place = nullptr) {
    const WsLayout &w = plan->ws;
    const int L = plan->n_layers;
    const uint32_t n_chunks = plan->n_chunks;
    const LayerDev *layers = reinterpret_cast<const LayerDev *>(ws + w.layers);
    const DirEntry *chunk_dir = reinterpret_cast<const DirEntry *>(ws + w.chunk_dir);
    SelState *state = reinterpret_cast<SelState *>(ws + w.state);
    const uint32_t *hist = reinterpret_cast<const uint32_t *>(ws + w.hist);
    uint32_t *flags = reinterpret_cast<uint32_t *>(ws + w.flags);
    uint32_t *chunk_cnt = reinterpret_cast<uint32_t *>(ws + w.chunk_cnt);
    uint32_t *mask = reinterpret_cast<uint32_t *>(ws + w.mask);
    uint32_t *cmask = want_centres ? reinterpret_cast<uint32_t *>(ws + w.cmask) : nullptr;
    float *nsi = reinterpret_cast<float *>(ws + w.nsi);
    const bool inline_count = plan->count_how == kCountMarked;
    const uint32_t gstride = group_cnt_stride(plan->count_how);
    const GroupEntry *cand_groups = reinterpret_cast<const GroupEntry *>(ws + w.cand_groups);
    const uint32_t n_cand_groups = static_cast<uint32_t>(plan->cand_groups.size());
    const uint32_t *slot_cnt = reinterpret_cast<const uint32_t *>(ws + w.slot_cnt);
    const unsigned long long *slot_ent = reinterpret_cast<const unsigned long long *>(ws + w.slot_ent);
    // the keys of each layer's threshold bucket are gathered, then one workgroup per layer finishes
    // the ranking on them
    {
        GatherArgs a;
        a.layers = layers;
        a.state = state;
        a.keys = reinterpret_cast<const uint32_t *>(nsi);
        a.slot_cnt = slot_cnt;
        a.slot_ent = slot_ent;
        a.list_cnt = reinterpret_cast<uint32_t *>(ws + w.list_cnt);
        a.list_ent = reinterpret_cast<unsigned long long *>(ws + w.list_ent);
        a.hist = hist;
        a.hist1 = reinterpret_cast<uint32_t *>(ws + w.hist1);
        a.flags = flags;
        a.mask = mask;
        a.cmask = cmask;
        a.chunk_cnt = inline_count ? chunk_cnt : nullptr;
        a.group_cnt = inline_count ? reinterpret_cast<uint32_t *>(ws + w.group_cnt) : nullptr;
        GatherLists gl;
        gl.chunk_dir = chunk_dir;
        gl.chunks = reinterpret_cast<const ChunkInfo *>(ws + w.chunk_info);
        gl.map_chunks = reinterpret_cast<const ChunkEntry *>(ws + w.map_chunks);
        gl.cand_groups = cand_groups;
        gl.n_layers = static_cast<uint32_t>(L);
        gl.n_chunks = n_chunks;
        gl.n_map_chunks = static_cast<uint32_t>(plan->map_chunks.size());
        gl.n_cand_groups = n_cand_groups;
        const bool blocks = !plan->k_override.empty() && plan->any_large, split = !blocks && inline_count && n_cand_groups < kSplitGroups;
        gl.n_slot_wgs = std::min<uint32_t>(n_cand_groups * (split ? kSlotParts : 1u), kNumCUs * 8u);
        const uint32_t n_fb_wgs = plan->any_large ? std::min<uint32_t>(n_chunks, kNumCUs * (blocks ? 32u : 2u)) : 0u;
        if (gl.n_map_chunks + gl.n_slot_wgs + n_fb_wgs > 0)
        {
            const dim3 grid(gl.n_map_chunks + gl.n_slot_wgs + n_fb_wgs);
            if (blocks && inline_count) hipLaunchKernelGGL((k_gather<true, 0>), grid, dim3(256), 0, stream, a, gl);
            else if (blocks) hipLaunchKernelGGL((k_gather<false, 0>), grid, dim3(256), 0, stream, a, gl);
            else if (split) hipLaunchKernelGGL((k_gather<true, kSlotParts>), grid, dim3(256), 0, stream, a, gl);
            else if (inline_count) hipLaunchKernelGGL((k_gather<true, 1>), grid, dim3(256), 0, stream, a, gl);
            else hipLaunchKernelGGL((k_gather<false, 1>), grid, dim3(256), 0, stream, a, gl);
        }
        uint32_t *list2_cnt = reinterpret_cast<uint32_t *>(ws + w.list2_cnt);
        unsigned long long *list2_ent = reinterpret_cast<unsigned long long *>(ws + w.list2_ent);
        FilterLayers fl = {};
        const size_t n_big = plan->big_map_layers.size();
        fl.listed = n_big <= static_cast<size_t>(kFilterLayers);
        if (fl.listed) std::copy(plan->big_map_layers.begin(), plan->big_map_layers.end(), fl.id);
        if (n_big != 0u && !blocks) {           // long threshold-bucket lists: many workgroups pick the keys k_finish needs
            hipLaunchKernelGGL(k_filter, dim3((fl.listed ? static_cast<uint32_t>(n_big) : static_cast<uint32_t>(L)) * kFilterSplit),
                               dim3(kFilterThreads), 0, stream, fl, layers, state, a.hist1, a.list_cnt, a.list_ent, list2_cnt, list2_ent);
        }
        CountShare cs = {};
        if (plan->count_how == kCountBeside && plan->any_large) {
            cs.groups = reinterpret_cast<const CountGroup *>(ws + w.count_groups);
            cs.n_groups = plan->n_count_groups;
            cs.mask = mask;
            cs.chunk_cnt = chunk_cnt;
            cs.group_cnt = reinterpret_cast<uint32_t *>(ws + w.group_cnt);
            cs.gstride = gstride;
        }
        const uint32_t count_wgs = (cs.n_groups * 4u + kFinishWaves - 1u) / kFinishWaves;
        const unsigned finish_wgs = static_cast<unsigned>(L) + count_wgs;
        if (blocks)                            // (at most kGridLayers of them)
            hipLaunchKernelGGL(k_finish_grids, dim3(finish_wgs + static_cast<unsigned>(n_big) * (kFilterSplit - 1)), dim3(kFinishThreads), 0, stream,
                               layers, static_cast<uint32_t>(L), cs, state, hist, a.hist1, a.list_cnt, a.list_ent, a.keys, slot_cnt, slot_ent,
                               list2_cnt, list2_ent, pred, fl, count_wgs);
        else
            hipLaunchKernelGGL(k_finish, dim3(finish_wgs), dim3(kFinishThreads), 0, stream, layers, static_cast<uint32_t>(L), cs, state, hist, a.hist1,
                               a.list_cnt, a.list_ent, a.keys, slot_cnt, slot_ent, list2_cnt, list2_ent, pred);
    }
    HIP_TRY(hipGetLastError());
    marks.close(4);

    {
        MarkArgs m;
        m.layers = layers;
        m.state = state;
        m.grad = grad;
        m.resid = v_in_place;
        m.dir = reinterpret_cast<const DirEntry *>(ws + w.all_tile_dir);
        m.n_layers = static_cast<uint32_t>(L);
        m.n_tiles = plan->n_tiles_all;
        m.map_tiles = reinterpret_cast<const SampleEntry *>(ws + w.map_tiles);
        m.n_map_tiles = plan->n_map_tiles;
        m.n_list_wgs = std::min<uint32_t>(m.n_map_tiles, kNumCUs * 8u);
        m.flags = flags;
        m.keys = reinterpret_cast<const uint32_t *>(nsi);
        m.mask = mask;
        m.cmask = cmask;
        m.chunk_cnt = chunk_cnt;
        m.group_cnt = reinterpret_cast<uint32_t *>(ws + w.group_cnt);
        m.gstride = gstride;
        const uint32_t n_fb_wgs = plan->any_large ? std::min<uint32_t>(plan->n_tiles_all, kNumCUs * 4u) : 0u;
        const MarkCount how = inline_count ? kMarkCounts : plan->count_how == kCountBeside ? kMarkCountsShared : kMarkOnly;
        m.n_bucket_wgs = plan->any_large ? static_cast<uint32_t>(L) * kListShards * mark_parts(how) : 0u;
        m.list_cnt = reinterpret_cast<const uint32_t *>(ws + w.list_cnt);
        m.list_ent = reinterpret_cast<const unsigned long long *>(ws + w.list_ent);
        m.slot_cnt = slot_cnt;
        m.slot_ent = slot_ent;
        const uint32_t n_wgs = m.n_bucket_wgs + m.n_list_wgs + n_fb_wgs;
        if (!plan->k_override.empty()) {                   // a block grid: no windows, no centre masks
            MarkFlatArgs b;
            b.layers = layers;
            b.state = state;
            b.map_chunks = reinterpret_cast<const ChunkEntry *>(ws + w.map_chunks);
            b.chunks = reinterpret_cast<const ChunkInfo *>(ws + w.chunk_info);
            b.n_map_chunks = static_cast<uint32_t>(plan->map_chunks.size());
            b.n_bucket_wgs = plan->any_large ? static_cast<uint32_t>(L) * kListShards : 0u;
            b.n_chunks = n_chunks;
            b.list_cnt = m.list_cnt;
            b.slot_cnt = slot_cnt;
            b.flags = flags;
            b.keys = m.keys;
            b.list_ent = m.list_ent;
            b.slot_ent = slot_ent;
            b.mask = mask;
            b.chunk_cnt = m.chunk_cnt;
            b.group_cnt = m.group_cnt;
            b.gstride = gstride;
            const uint32_t n = b.n_map_chunks + b.n_bucket_wgs + (plan->any_large ? std::min<uint32_t>(n_chunks, kNumCUs * 32u) : 0u);
            if (n != 0u) hipLaunchKernelGGL(k_mark_flat, dim3(n), dim3(256), 0, stream, b);
        } else if (n_wgs > 0) {
            if (how == kMarkOnly) hipLaunchKernelGGL(k_mark<kMarkOnly>, dim3(n_wgs), dim3(256), 0, stream, m);
            else if (how == kMarkCounts) hipLaunchKernelGGL(k_mark<kMarkCounts>, dim3(n_wgs), dim3(256), 0, stream, m);
            else hipLaunchKernelGGL(k_mark<kMarkCountsShared>, dim3(n_wgs), dim3(256), 0, stream, m);
        }
    }
    marks.close(5);
    launch_count(plan, ws, plan->count_how == kCountAfter && plan->k_override.empty() ? mask : nullptr, cmask, stream);
    marks.close(6);
    return RSDGC_OK;
}

// Small plans: everything between the main pass and the emit in one launch (and the centres' counts in another, if wanted).
static int launch_select(rsdgc_plan_s *plan, char *ws, const float *grad, const float *residual, float *v_out, const Momentum &mom,
                         bool want_centres, StageMarks &marks, hipStream_t stream) {
    const WsLayout &w = plan->ws;
    SelectArgs a;
    a.layers = reinterpret_cast<const LayerDev *>(ws + w.layers);
    a.groups = reinterpret_cast<const GroupEntry *>(ws + w.cand_groups);
    a.state = reinterpret_cast<SelState *>(ws + w.state);
    a.pred = reinterpret_cast<PredState *>(ws + w.pred);
    a.hist_s = reinterpret_cast<const uint32_t *>(ws + w.hist_s);
    a.slot_cnt = reinterpret_cast<const uint32_t *>(ws + w.slot_cnt);
    a.slot_ent = reinterpret_cast<const unsigned long long *>(ws + w.slot_ent);
    a.mask = reinterpret_cast<uint32_t *>(ws + w.mask);
    a.cmask = want_centres ? reinterpret_cast<uint32_t *>(ws + w.cmask) : nullptr;
    a.chunk_cnt = reinterpret_cast<uint32_t *>(ws + w.chunk_cnt);
    a.group_cnt = reinterpret_cast<uint32_t *>(ws + w.group_cnt);
    a.grad = grad;
    a.resid = residual;
    a.mom = mom.in;
    a.v_out = v_out;
    a.mom_out = mom.out;
    a.m = mom.m;
    a.map = reinterpret_cast<uint32_t *>(ws + w.nsi);
    a.hist = reinterpret_cast<uint32_t *>(ws + w.hist);
    a.hist1 = reinterpret_cast<uint32_t *>(ws + w.hist1);
    a.list_cnt = reinterpret_cast<uint32_t *>(ws + w.list_cnt);
    a.list_ent = reinterpret_cast<unsigned long long *>(ws + w.list_ent);
    a.alpha = plan->alpha;
    a.n_layers = static_cast<uint32_t>(plan->n_layers);
    a.n_groups = static_cast<uint32_t>(plan->cand_groups.size());
    uint32_t n_tiles = 0;
    for (const PGroup &g : plan->groups) n_tiles += g.n_large_tiles;
    const uint32_t n_wgs = std::max(a.n_groups, std::min(a.n_groups + n_tiles, select_workgroups(a.n_groups)));
    hipLaunchKernelGGL(k_select, dim3(n_wgs), dim3(kSelectThreads), 0, stream, a);
    marks.close(4);
    marks.close(5);
    launch_count(plan, ws, nullptr, a.cmask, stream);
    HIP_TRY(hipGetLastError());
    marks.close(6);
    return RSDGC_OK;
}

// What the last kernel of a call with this plan clears and sets for the next (sampling: whether that one samples bounds).
static NextCall next_call(const rsdgc_plan_s *plan, char *ws, const LayerDev *layers, SelState *state, PredState *pred,
                          bool sampling) {
    const WsLayout &w = plan->ws;
    NextCall nc;
    nc.zero[0] = reinterpret_cast<uint4 *>(ws + w.hist);
    nc.n16[0] = static_cast<uint32_t>((w.chunk_cnt - w.hist) / 16);
    nc.zero[1] = reinterpret_cast<uint4 *>(ws + w.list_cnt);
    nc.n16[1] = static_cast<uint32_t>((w.mask - w.list_cnt) / 16);
    nc.layers = layers;
    nc.state = state;
    nc.pred = pred;
    nc.flags = reinterpret_cast<uint32_t *>(ws + w.flags);
    nc.n_layers = plan->n_layers;
    nc.sampling = sampling ? 1 : 0;
    return nc;
}

// Plans whose layers' candidates a workgroup can read through: everything up to the emit in one launch.
static bool selects_in_one_launch(const rsdgc_plan_s *plan) {
    bool one = plan->one_select && plan->work_feed != RSDGC_FEED_ON;
    for (const PGroup &g : plan->groups) one = one && g.n_large_tiles < kFeedTiles;      // (no feed for the main pass)
    return one;
}
// One arena: whether the main pass puts v in the residual's place as it goes.
static bool replaces_residual(const rsdgc_plan_s *plan) { return plan->any_large && plan->v_in_place && !selects_in_one_launch(plan); }

int32_t rsdgc_replaces_residual(const rsdgc_plan_t *plan) { return !plan ? -1 : plan->blocks || replaces_residual(plan) ? 1 : 0; }

static int compress_impl(rsdgc_plan_t *plan, const float *grad, const Momentum &mom,
                         const float *residual, float *residual_out, uint32_t *out_idx,
                         float *out_val, int32_t *out_counts, uint32_t *out_centre_idx,
                         int32_t *out_centre_counts, void *workspace, void *stream_) {
    if (!plan || !grad || !residual || !residual_out || !out_idx || !out_val || !out_counts || !workspace)
        return RSDGC_EINVAL;
    if (plan->blocks) return RSDGC_EINVAL;              // a block plan goes with rsdgc_compress_blocks
    if (!aligned256(workspace) || !aligned16(grad) || !aligned16(residual) || !aligned16(residual_out))
        return RSDGC_EINVAL;
    const bool in_place = residual_out == residual;
    if (!in_place) {    // two arenas: they must not overlap, and the new one must not be the gradient
        const uintptr_t bytes = static_cast<uintptr_t>(plan->total_elems) * sizeof(float);
        const uintptr_t o = reinterpret_cast<uintptr_t>(residual_out);
        const uintptr_t r = reinterpret_cast<uintptr_t>(residual), g = reinterpret_cast<uintptr_t>(grad);
        if ((o < r + bytes && r < o + bytes) || (o < g + bytes && g < o + bytes)) return RSDGC_EINVAL;
    }
    float *v_out = in_place ? nullptr : residual_out;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    char *ws = static_cast<char *>(workspace);
    const WsLayout &w = plan->ws;
    const int L = plan->n_layers;
    const uint32_t n_chunks = plan->n_chunks;
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    // the first calls with a workspace (the thresholds have no history yet, or still move fast) may
    // take candidate bounds from a sample of the call's own scores
    const bool sampling = plan->any_large && plan->calls_since_upload < kSamplingCalls;
    if (plan->calls_since_upload < kSamplingCalls) ++plan->calls_since_upload;

    const LayerDev *layers = reinterpret_cast<const LayerDev *>(ws + w.layers);
    SelState *state = reinterpret_cast<SelState *>(ws + w.state);
    uint32_t *hist = reinterpret_cast<uint32_t *>(ws + w.hist);
    uint32_t *flags = reinterpret_cast<uint32_t *>(ws + w.flags);
    PredState *pred = reinterpret_cast<PredState *>(ws + w.pred);
    uint32_t *chunk_cnt = reinterpret_cast<uint32_t *>(ws + w.chunk_cnt);
    uint32_t *chunk_ccnt = reinterpret_cast<uint32_t *>(ws + w.chunk_ccnt);
    const uint32_t *group_cnt = reinterpret_cast<const uint32_t *>(ws + w.group_cnt);
    uint32_t *mask = reinterpret_cast<uint32_t *>(ws + w.mask);
    const bool want_centres = out_centre_idx || out_centre_counts;
    uint32_t *cmask = want_centres ? reinterpret_cast<uint32_t *>(ws + w.cmask) : nullptr;
    float *nsi = reinterpret_cast<float *>(ws + w.nsi);

    const bool one_select = selects_in_one_launch(plan);
    const bool v_in_place = in_place && replaces_residual(plan);

    StageMarks marks(plan, stream);
    if (!plan->ws_ready) {                 // the call before failed half way
        rc = prepare_workspace(plan, ws, sampling, kStatesNone, stream);
        if (rc != RSDGC_OK) return rc;
    }
    const bool ready = plan->ws_ready;     // (false: prepared by the graph that is being recorded)
    plan->ws_ready = false;                // (until all of this call is enqueued)
    const NextCall nc = next_call(plan, ws, layers, state, pred, plan->any_large && plan->calls_since_upload < kSamplingCalls);
    marks.close(0);

    // first pass: every tile of the layers ranked on the full map (scores, histogram, v) and, where a
    // large layer has no predicted bound, its sampled tiles (histogram only) share one launch.
    // (Running it on a second stream beside the main pass, which does not depend on it once the
    // bounds are predicted, was measured: the two event waits cost more than the overlap gains.)
    rc = launch_nsi<kPassSample>(plan, ws, grad, residual, nsi, v_out, mom, stream, sampling);
    if (rc != RSDGC_OK) return rc;
    if (sampling)
        hipLaunchKernelGGL(k_hint, dim3(L), dim3(256), 0, stream, layers, state,
                           reinterpret_cast<uint32_t *>(ws + w.hist_s), flags);
    marks.close(1);
    uint4 *counts = reinterpret_cast<uint4 *>(ws + w.chunk_cnt);
    const uint32_t counts_n16 = static_cast<uint32_t>((w.list_cnt - w.chunk_cnt) / 16);
    if (v_in_place) {
        rc = launch_nsi<kPassCaptureInPlace>(plan, ws, grad, residual, nsi, residual_out, mom, stream);
        if (rc != RSDGC_OK) return rc;
    } else if (plan->any_large) {
        rc = launch_nsi<kPassCapture>(plan, ws, grad, residual, nsi, v_out, mom, stream, true, nullptr, counts, one_select ? counts_n16 : 0u);
        if (rc != RSDGC_OK) return rc;
    }
    marks.close(2);
    if (one_select) {
        marks.close(3);
        rc = launch_select(plan, ws, grad, residual, v_out, mom, want_centres, marks, stream);
        if (rc != RSDGC_OK) return rc;
    } else {
        Find0Args f;
        f.layers = layers;
        f.state = state;
        f.hist = hist;
        f.hist_s = reinterpret_cast<const uint32_t *>(ws + w.hist_s);
        f.flags = flags;
        f.pred = pred;
        f.counts = counts;
        f.n16 = counts_n16;
        f.n_layers = L;
        // large layers whose candidate bound failed (rare): the workgroups find nothing to do otherwise.  Up to 256 layers they look
        // for such layers themselves, in one launch with k_find0.
        const bool one_launch = plan->any_large && L <= 256;
        if (!one_launch) hipLaunchKernelGGL(k_find0, dim3(L), dim3(256), 0, stream, f);
        if (plan->any_large) {
            rc = launch_nsi<kPassFullMap>(plan, ws, grad, residual, nsi, v_out, mom, stream, true, one_launch ? &f : nullptr, nullptr, 0u, v_in_place);
            if (rc != RSDGC_OK) return rc;
        }
        marks.close(3);

        rc = select_mark_count(plan, ws, want_centres, marks, pred, stream, grad, v_in_place ? residual_out : nullptr);
        if (rc != RSDGC_OK) return rc;
    }
    const ChunkInfo *chunk_info = reinterpret_cast<const ChunkInfo *>(ws + w.chunk_info);
    if (in_place && !v_in_place)
        hipLaunchKernelGGL(k_emit, dim3(n_chunks + 1), dim3(256), 0, stream, layers, chunk_info, grad,
                           residual_out, mask, chunk_cnt, group_cnt, out_idx, out_val, out_counts, nc);
    else if (n_chunks > kInlineCountChunks)
        hipLaunchKernelGGL(k_emit_waves, dim3((n_chunks + 3) / 4 + 1), dim3(256), 0, stream, chunk_info, n_chunks, state, grad,
                           residual, residual_out, mom.in, mom.out, mom.m, mask, chunk_cnt, group_cnt, out_idx,
                           out_val, out_counts, nc);
    else
        hipLaunchKernelGGL(k_emit_sparse, dim3(n_chunks + 1), dim3(256), 0, stream, chunk_info, state, grad,
                           residual, residual_out, mom.in, mom.out, mom.m, mask, chunk_cnt, group_cnt, out_idx,
                           out_val, out_counts, nc);
    marks.close(7);
    if (want_centres)                      // the list, the counts, or both
        hipLaunchKernelGGL(k_emit_centres, dim3(n_chunks), dim3(256), 0, stream, layers, chunk_info,
                           cmask, chunk_ccnt, reinterpret_cast<const uint32_t *>(ws + w.group_ccnt), out_centre_idx,
                           out_centre_counts);
    marks.close(8);
    HIP_TRY(hipGetLastError());
    plan->ws_ready = ready;
    return RSDGC_OK;
}

int rsdgc_compress(rsdgc_plan_t *plan, const float *grad, const float *residual,
                   float *residual_out, uint32_t *out_idx, float *out_val, int32_t *out_counts,
                   uint32_t *out_centre_idx, int32_t *out_centre_counts, void *workspace,
                   void *stream) {
    return compress_impl(plan, grad, Momentum{}, residual, residual_out, out_idx, out_val, out_counts,
                         out_centre_idx, out_centre_counts, workspace, stream);
}

// Workspace of rsdgc_compress_static: one array per GPU, part of the library's code object, so
// that the call needs no device allocation.  It lives as long as the process; every
// rsdgc_compress_static call on a GPU uses that GPU's copy, so two of them must not overlap in
// time on one GPU.  In host code the array's name is not a device address: the address is
// asked for once per device (hipGetSymbolAddress) and only that pointer is handed to kernels
// and copies.
static __device__ __align__(256) unsigned char scratch[RSDGC_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 64;
struct ScratchSlot {
    void *ptr = nullptr;            // device address of `scratch` on this device
    uint64_t owner_serial = 0;      // plan (and its version) whose tables the array holds now
    uint64_t owner_version = 0;
};
ScratchSlot g_scratch[kMaxDevices];
std::mutex g_scratch_mutex;
}  // namespace

int rsdgc_compress_static(rsdgc_plan_t *plan, const float *grad, const float *residual,
                          float *residual_out, uint32_t *out_idx, float *out_val, int32_t *out_counts,
                          uint32_t *out_centre_idx, int32_t *out_centre_counts, void *stream) {
    if (!plan || plan->blocks) return RSDGC_EINVAL;
    if (plan->ws.total > static_cast<size_t>(RSDGC_STATIC_WORKSPACE_BYTES)) {
        std::snprintf(g_hip_error, sizeof(g_hip_error),
                      "rsdgc_compress_static: the plan needs %zu bytes of workspace, the built-in one has %zu",
                      plan->ws.total, static_cast<size_t>(RSDGC_STATIC_WORKSPACE_BYTES));
        return RSDGC_ETOOBIG;
    }
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return RSDGC_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    ScratchSlot &slot = g_scratch[dev];
    if (!slot.ptr) {                       // once per device, with that device current
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || !aligned256(p)) return hip_fail(hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
        slot.ptr = p;
    }
    // the array keeps what the last call left: when that was another plan (or other ratios), this
    // plan's tables are laid down again and everything else a call expects is cleared and set with them
    if (slot.owner_serial != plan->serial || slot.owner_version != plan->version) plan->uploaded_ws = nullptr;
    const int rc = compress_impl(plan, grad, Momentum{}, residual, residual_out, out_idx, out_val,
                                 out_counts, out_centre_idx, out_centre_counts, slot.ptr, stream);
    if (rc == RSDGC_OK) {
        slot.owner_serial = plan->serial;
        slot.owner_version = plan->version;
    } else {
        slot.owner_serial = 0;
    }
    return rc;
}

int rsdgc_compress_momentum(rsdgc_plan_t *plan, const float *grad, const float *momentum,
                            float *momentum_out, float m, const float *residual,
                            float *residual_out, uint32_t *out_idx, float *out_val,
                            int32_t *out_counts, uint32_t *out_centre_idx,
                            int32_t *out_centre_counts, void *workspace, void *stream) {
    if (!plan || !grad || !momentum || !momentum_out || !residual || !residual_out) return RSDGC_EINVAL;
    if (!(m >= 0.f && m <= 1.f)) return RSDGC_EINVAL;                       // false for NaN
    if (!aligned16(momentum) || !aligned16(momentum_out)) return RSDGC_EINVAL;
    // five arenas, pairwise disjoint: both new arenas are written while the three inputs are still read
    const uintptr_t bytes = static_cast<uintptr_t>(plan->total_elems) * sizeof(float);
    const uintptr_t p[5] = {reinterpret_cast<uintptr_t>(grad), reinterpret_cast<uintptr_t>(momentum),
                            reinterpret_cast<uintptr_t>(residual), reinterpret_cast<uintptr_t>(momentum_out),
                            reinterpret_cast<uintptr_t>(residual_out)};
    for (int i = 0; i < 5; ++i)
        for (int j = (i < 3 ? 3 : i + 1); j < 5; ++j)
            if (p[i] < p[j] + bytes && p[j] < p[i] + bytes) return RSDGC_EINVAL;
    Momentum mom;
    mom.in = momentum;
    mom.out = momentum_out;
    mom.m = m;
    return compress_impl(plan, grad, mom, residual, residual_out, out_idx, out_val, out_counts,
                         out_centre_idx, out_centre_counts, workspace, stream);
}

// Two arenas of the plan's size overlap unless they are the same one.
static bool arenas_clash(const void *a, const void *b, uintptr_t bytes, bool same_allowed) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    if (x == y) return !same_allowed;
    return x < y + bytes && y < x + bytes;
}

static int compress_blocks_impl(rsdgc_plan_t *plan, const float *grad, const Momentum &mom,
                                const float *residual, float *residual_out, uint32_t *out_block_idx,
                                float *out_val, int32_t *out_counts, void *workspace, void *stream_) {
    if (!plan || !plan->blocks || !grad || !residual || !residual_out || !out_block_idx || !out_val ||
        !out_counts || !workspace)
        return RSDGC_EINVAL;
    if (!aligned256(workspace) || !aligned16(grad) || !aligned16(residual) || !aligned16(residual_out))
        return RSDGC_EINVAL;
    {
        // an output arena may be its own input (no element is read by two tiles) and nothing else
        const uintptr_t bytes = static_cast<uintptr_t>(plan->total_elems) * sizeof(float);
        if (arenas_clash(residual_out, residual, bytes, true) || arenas_clash(residual_out, grad, bytes, false))
            return RSDGC_EINVAL;
        if (mom.in) {
            if (!mom.out || !aligned16(mom.in) || !aligned16(mom.out)) return RSDGC_EINVAL;
            if (arenas_clash(mom.out, mom.in, bytes, true) || arenas_clash(mom.out, grad, bytes, false) ||
                arenas_clash(mom.out, residual, bytes, false) || arenas_clash(mom.out, residual_out, bytes, false) ||
                arenas_clash(mom.in, residual_out, bytes, false))
                return RSDGC_EINVAL;
        }
    }
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    char *ws_outer = static_cast<char *>(workspace);
    rsdgc_plan_s *in = plan->inner;
    char *ws = ws_outer + plan->ws.table_bytes;        // the inner plan's workspace
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    rc = upload_tables(in, ws, stream);
    if (rc != RSDGC_OK) return rc;
    const WsLayout &w = in->ws;
    const int L = in->n_layers;
    const LayerDev *outer = reinterpret_cast<const LayerDev *>(ws_outer + plan->ws.layers);
    const LayerDev *inner = reinterpret_cast<const LayerDev *>(ws + w.layers);
    const ChunkInfo *inner_chunks = reinterpret_cast<const ChunkInfo *>(ws + w.chunk_info);
    SelState *state = reinterpret_cast<SelState *>(ws + w.state);
    uint32_t *hist = reinterpret_cast<uint32_t *>(ws + w.hist);
    uint32_t *mask = reinterpret_cast<uint32_t *>(ws + w.mask);
    uint32_t *chunk_cnt = reinterpret_cast<uint32_t *>(ws + w.chunk_cnt);
    const uint32_t *group_cnt = reinterpret_cast<const uint32_t *>(ws + w.group_cnt);
    float *score_map = reinterpret_cast<float *>(ws + w.nsi);
    StageMarks marks(in, stream);                      // (the inner plan never records events)
    if (!in->ws_ready) {                   // the call before failed half way
        rc = prepare_workspace(in, ws, false, kStatesNone, stream);
        if (rc != RSDGC_OK) return rc;
    }
    const bool ready = in->ws_ready;       // (false: prepared by the graph that is being recorded)
    in->ws_ready = false;                  // (until all of this call is enqueued)
    PredState *pred = reinterpret_cast<PredState *>(ws + w.pred);
    const NextCall nc = next_call(in, ws, inner, state, pred, false);
    const BlockCapture cp = {state, reinterpret_cast<uint32_t *>(ws + w.hist_s), reinterpret_cast<uint32_t *>(ws + w.list_cnt),
                             reinterpret_cast<uint32_t *>(ws + w.slot_cnt), reinterpret_cast<unsigned long long *>(ws + w.slot_ent)};
    bool have[RSDGC_MAX_P + 1] = {};
    for (int l = 0; l < L; ++l) have[plan->p[l]] = true;
    // the work feed (counters in the inner plan's workspace, cleared above) pays when a
    // workgroup gets many tiles
    uint32_t *feed = reinterpret_cast<uint32_t *>(ws + w.feed);
    const bool fed = plan->work_feed != RSDGC_FEED_OFF &&
                     (plan->work_feed == RSDGC_FEED_ON || plan->n_tiles_all >= 16u * kNumCUs * 4u);
    uint32_t feed_shift = 7;
    while (feed_shift > 0 && (static_cast<uint32_t>(kFeedDomains) << feed_shift) > plan->n_tiles_all) --feed_shift;
    for (int pp = 1; pp <= RSDGC_MAX_P; pp += 2) {
        if (!have[pp]) continue;
        switch (pp) {
#define RSDGC_BLOCK_LAUNCH(PP, FF, MM, CC)                                                       \
    {                                                                                            \
        static const uint32_t resident = resident_workgroups(k_block_nsi<PP, FF, MM, CC>);           \
        hipLaunchKernelGGL((k_block_nsi<PP, FF, MM, CC>), dim3(std::min<uint32_t>(plan->n_tiles_all, resident)), \
                           dim3(256), 0, stream, outer,                                          \
                           reinterpret_cast<const DirEntry *>(ws_outer + plan->ws.all_tile_dir), \
                           static_cast<uint32_t>(L), plan->n_tiles_all, inner, grad, residual,   \
                           residual_out, score_map, hist, plan->alpha,                           \
                           feed + static_cast<size_t>(PP / 2) * kFeedDomains * kFeedStride,      \
                           feed_shift, mom.in, mom.out, mom.m, cp);                              \
    }
#define RSDGC_BLOCK_PICK(PP, FF, MM)                                                             \
    {                                                                                            \
        if (in->any_large) RSDGC_BLOCK_LAUNCH(PP, FF, MM, true)                                  \
        else RSDGC_BLOCK_LAUNCH(PP, FF, MM, false)                                               \
    }
#define RSDGC_BLOCK_CASE(PP)                                                                     \
    case PP: {                                                                                   \
        if (mom.in) {                                                                            \
            if (fed) RSDGC_BLOCK_PICK(PP, true, true)                                            \
            else RSDGC_BLOCK_PICK(PP, false, true)                                               \
        } else {                                                                                 \
            if (fed) RSDGC_BLOCK_PICK(PP, true, false)                                           \
            else RSDGC_BLOCK_PICK(PP, false, false)                                              \
        }                                                                                        \
        break;                                                                                   \
    }
            RSDGC_BLOCK_CASE(1)
            RSDGC_BLOCK_CASE(3)
            RSDGC_BLOCK_CASE(5)
            RSDGC_BLOCK_CASE(7)
#undef RSDGC_BLOCK_CASE
#undef RSDGC_BLOCK_PICK
#undef RSDGC_BLOCK_LAUNCH
        }
    }
    HIP_TRY(hipGetLastError());
    const Find0Args f = {inner, state, hist, cp.hist_s, reinterpret_cast<uint32_t *>(ws + w.flags), pred,
                         reinterpret_cast<uint4 *>(ws + w.chunk_cnt), static_cast<uint32_t>((w.list_cnt - w.chunk_cnt) / 16), L};
    if (!in->any_large) hipLaunchKernelGGL(k_find0, dim3(L), dim3(256), 0, stream, f);
    if (in->any_large) {
        const BlockRescore r = {outer, inner, reinterpret_cast<const DirEntry *>(ws_outer + plan->ws.all_tile_dir), plan->n_tiles_all, residual_out,
                                score_map, hist, cp.list_cnt, plan->alpha};
        const dim3 grid(L + std::min<uint32_t>(plan->n_tiles_all, kNumCUs * 8u));
        if (have[7]) hipLaunchKernelGGL(k_find0_blocks<7>, grid, dim3(256), 0, stream, f, r);
        else if (have[5]) hipLaunchKernelGGL(k_find0_blocks<5>, grid, dim3(256), 0, stream, f, r);
        else if (have[3]) hipLaunchKernelGGL(k_find0_blocks<3>, grid, dim3(256), 0, stream, f, r);
        else hipLaunchKernelGGL(k_find0_blocks<1>, grid, dim3(256), 0, stream, f, r);
    }
    rc = select_mark_count(in, ws, false, marks, pred, stream);
    if (rc != RSDGC_OK) return rc;
    hipLaunchKernelGGL(k_emit_blocks, dim3(in->n_chunks + 1), dim3(256), 0, stream, outer, inner_chunks, mask,
                       chunk_cnt, group_cnt, inner, residual_out, mom.out, out_block_idx, out_val, out_counts, nc);
    HIP_TRY(hipGetLastError());
    in->ws_ready = ready;
    return RSDGC_OK;
}

int rsdgc_compress_blocks(rsdgc_plan_t *plan, const float *grad, const float *residual,
                          float *residual_out, uint32_t *out_block_idx, float *out_val,
                          int32_t *out_counts, void *workspace, void *stream) {
    return compress_blocks_impl(plan, grad, Momentum(), residual, residual_out, out_block_idx, out_val,
                                out_counts, workspace, stream);
}

int rsdgc_compress_blocks_momentum(rsdgc_plan_t *plan, const float *grad, const float *momentum,
                                   float *momentum_out, float m, const float *residual,
                                   float *residual_out, uint32_t *out_block_idx, float *out_val,
                                   int32_t *out_counts, void *workspace, void *stream) {
    if (!momentum || !momentum_out || !(m >= 0.f && m <= 1.f)) return RSDGC_EINVAL;
    Momentum mom;
    mom.in = momentum;
    mom.out = momentum_out;
    mom.m = m;
    return compress_blocks_impl(plan, grad, mom, residual, residual_out, out_block_idx, out_val,
                                out_counts, workspace, stream);
}

int rsdgc_decompress_blocks(rsdgc_plan_t *plan, const uint32_t *block_idx, const float *val,
                            const int32_t *counts, float *dense, int accumulate, void *workspace,
                            void *stream_) {
    if (!plan || !plan->blocks || !block_idx || !val || !counts || !dense || !workspace) return RSDGC_EINVAL;
    if (!aligned256(workspace) || !aligned16(dense)) return RSDGC_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    char *ws = static_cast<char *>(workspace);
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    const LayerDev *outer = reinterpret_cast<const LayerDev *>(ws + plan->ws.layers);
    if (!accumulate)
        hipLaunchKernelGGL(k_zero_layers, dim3(plan->n_chunks), dim3(256), 0, stream,
                           reinterpret_cast<const ChunkInfo *>(ws + plan->ws.chunk_info), dense);
    if (plan->centre_capacity > 0) {
        const unsigned blocks = static_cast<unsigned>((plan->centre_capacity + 255) / 256);
        hipLaunchKernelGGL(k_scatter_blocks, dim3(blocks), dim3(256), 0, stream, outer, plan->n_layers,
                           static_cast<long long>(plan->centre_capacity), block_idx, val, counts, dense,
                           accumulate);
    }
    HIP_TRY(hipGetLastError());
    return RSDGC_OK;
}

int rsdgc_apply(rsdgc_plan_t *plan, int32_t n_msgs, const uint32_t *const *idx,
                const float *const *val, const int32_t *const *counts, float *weights, float eta,
                void *workspace, void *stream_) {
    if (!plan || plan->blocks || !idx || !val || !counts || !weights || !workspace) return RSDGC_EINVAL;
    if (n_msgs < 1 || n_msgs > RSDGC_MAX_MSGS || !(eta == eta)) return RSDGC_EINVAL;
    if (!aligned256(workspace) || !aligned16(weights)) return RSDGC_EINVAL;
    for (int k = 0; k < n_msgs; ++k)
        if (!idx[k] || !val[k] || !counts[k]) return RSDGC_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    char *ws = static_cast<char *>(workspace);
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    const LayerDev *layers = reinterpret_cast<const LayerDev *>(ws + plan->ws.layers);
    if (plan->out_capacity == 0) return RSDGC_OK;      // no message can hold a pair
    if (n_msgs == 1) {
        const unsigned blocks = static_cast<unsigned>((plan->out_capacity + 255) / 256);
        hipLaunchKernelGGL(k_apply_single, dim3(blocks), dim3(256), 0, stream, layers, plan->n_layers,
                           static_cast<long long>(plan->out_capacity), idx[0], val[0], counts[0], weights, eta);
        HIP_TRY(hipGetLastError());
        return RSDGC_OK;
    }
    ApplyMsgs m;
    std::memset(&m, 0, sizeof(m));
    for (int k = 0; k < n_msgs; ++k) {
        m.idx[k] = idx[k];
        m.val[k] = val[k];
        m.counts[k] = counts[k];
    }
    const ChunkInfo *chunk_info = reinterpret_cast<const ChunkInfo *>(ws + plan->ws.chunk_info);
    uint32_t *starts = reinterpret_cast<uint32_t *>(ws + plan->ws.apply_starts);
    const uint32_t n_chunks = plan->n_chunks;
    const unsigned range_blocks = static_cast<unsigned>((2ull * n_chunks * static_cast<unsigned>(n_msgs) + 255) / 256);
    hipLaunchKernelGGL(k_apply_ranges, dim3(range_blocks), dim3(256), 0, stream, chunk_info, n_chunks, n_msgs, m, starts);
    hipLaunchKernelGGL(k_apply_chunks, dim3(2 * n_chunks), dim3(256), 0, stream, chunk_info, n_chunks, n_msgs, m,
                       starts, weights, eta);
    HIP_TRY(hipGetLastError());
    return RSDGC_OK;
}

int rsdgc_apply_blocks(rsdgc_plan_t *plan, int32_t n_msgs, const uint32_t *const *block_idx,
                       const float *const *val, const int32_t *const *counts, float *weights, float eta,
                       void *workspace, void *stream_) {
    if (!plan || !plan->blocks || !block_idx || !val || !counts || !weights || !workspace) return RSDGC_EINVAL;
    if (n_msgs < 1 || n_msgs > RSDGC_MAX_MSGS || !(eta == eta)) return RSDGC_EINVAL;
    if (!aligned256(workspace) || !aligned16(weights)) return RSDGC_EINVAL;
    for (int k = 0; k < n_msgs; ++k)
        if (!block_idx[k] || !val[k] || !counts[k]) return RSDGC_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    char *ws = static_cast<char *>(workspace);
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    const LayerDev *outer = reinterpret_cast<const LayerDev *>(ws + plan->ws.layers);
    if (plan->centre_capacity == 0) return RSDGC_OK;   // no message can hold a block
    const unsigned blocks = static_cast<unsigned>((plan->centre_capacity + 255) / 256);
    ApplyMsgs m;
    std::memset(&m, 0, sizeof(m));
    for (int k = 0; k < n_msgs; ++k) {
        m.idx[k] = block_idx[k];
        m.val[k] = val[k];
        m.counts[k] = counts[k];
    }
    hipLaunchKernelGGL(k_apply_blocks, dim3(blocks, static_cast<unsigned>(n_msgs)), dim3(256), 0, stream, outer,
                       plan->n_layers, static_cast<long long>(plan->centre_capacity), n_msgs, m, weights, eta);
    HIP_TRY(hipGetLastError());
    return RSDGC_OK;
}

// The plan's host memory for the counts of rsdgc_dynamic_ratios (null: there is none to be had).
static uint32_t *pinned_counts(rsdgc_plan_s *plan) {
    if (!plan->dyn_out) {
        void *p = nullptr;
        if (hipHostMalloc(&p, 2 * sizeof(uint32_t) * static_cast<size_t>(plan->n_layers), hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        plan->dyn_out = static_cast<uint32_t *>(p);
        plan->dyn_free = [](void *q) { (void)hipHostFree(q); };
    }
    return plan->dyn_out;
}

int rsdgc_dynamic_ratios(rsdgc_plan_t *plan, const float *weights, double global_ratio,
                         double *ratios_out, void *workspace, void *stream_) {
    if (!plan || plan->blocks || !weights || !ratios_out || !workspace) return RSDGC_EINVAL;
    if (!(global_ratio >= 0.0 && global_ratio <= 1.0)) return RSDGC_EINVAL;     // false for NaN
    if (!aligned256(workspace) || !aligned16(weights)) return RSDGC_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const int L = plan->n_layers;
    double n_real = 0.0;
    for (int l = 0; l < L; ++l) n_real += static_cast<double>(plan->layers[l].G);
    double kf = std::ceil(global_ratio * n_real);       // survivors of the ranking (Eq. 4)
    kf = std::min(std::max(kf, 0.0), n_real);
    const unsigned long long K = static_cast<unsigned long long>(kf);
    if (K == 0ull || kf == n_real) {                    // nothing or everything survives
        for (int l = 0; l < L; ++l) ratios_out[l] = K == 0ull ? 0.0 : 1.0;
        return RSDGC_OK;
    }
    char *ws = static_cast<char *>(workspace);
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    const WsLayout &w = plan->ws;
    DynState *state = reinterpret_cast<DynState *>(ws + w.dyn);
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(ws + w.dyn + 256);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(ws + w.dyn + 256 + sizeof(unsigned long long) * kHistBins);
    const ChunkInfo *chunk_info = reinterpret_cast<const ChunkInfo *>(ws + w.chunk_info);
    const uint32_t *keys = reinterpret_cast<const uint32_t *>(weights);
    const uint32_t n_chunks = plan->n_chunks;
    std::vector<uint32_t> host;
    try {
        host.resize(2 * static_cast<size_t>(L));
    } catch (const std::bad_alloc &) {
        return RSDGC_ENOMEM;
    }
    auto read_counts = [&]() -> int {
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipMemcpyAsync(host.data(), cnt, sizeof(uint32_t) * host.size(), hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        return RSDGC_OK;
    };
    const uint32_t grid = std::min<uint32_t>(n_chunks, kNumCUs * 4u);
    // One pass, where it is the better one: from a million weights on (below, both forms are a chain of launches), and with a
    // counter per layer in LDS.  Its lists lie where a compress call keeps its score map.
    bool counted = false;
    plan->dyn_passes = 0;
    if (n_real >= static_cast<double>(kDynSplitMin) && L <= kDynMaxLayers && pinned_counts(plan)) {
        DynSplitArgs a;
        a.out = plan->dyn_out;
        char *area = ws + w.nsi;
        a.state = reinterpret_cast<DynSplit *>(ws + w.dyn);
        a.sample_hist = reinterpret_cast<uint32_t *>(hist);
        a.cnt = cnt;
        a.sub_hist = reinterpret_cast<uint32_t *>(area);
        a.final_list = reinterpret_cast<uint2 *>(area + sizeof(uint32_t) * kDynSubBins);
        a.list = a.final_list + kDynFinalCap;
        const size_t bytes = sizeof(float) * static_cast<size_t>(plan->total_elems) - sizeof(uint32_t) * kDynSubBins - sizeof(uint2) * kDynFinalCap;
        a.list_cap = static_cast<uint32_t>(std::min<size_t>(bytes / sizeof(uint2), 0x7fffffffu));
        a.n_layers = static_cast<uint32_t>(L);
        a.K = K;
        a.n_weights = static_cast<unsigned long long>(n_real);
        const bool clear = plan->dyn_clear;
        plan->dyn_clear = false;                          // (until all of this call is enqueued)
        if (!clear) hipLaunchKernelGGL(k_dyn_clear, dim3(kDynSampleBins / 256), dim3(256), 0, stream, a);
        const uint32_t sample_wgs = (16u * n_chunks * kDynSamplePieces + kDynSampleThreads - 1u) / kDynSampleThreads;
        hipLaunchKernelGGL(k_dyn_sample, dim3(std::min<uint32_t>(sample_wgs, kNumCUs)), dim3(kDynSampleThreads), 0, stream, chunk_info, n_chunks, keys, a);
        hipLaunchKernelGGL(k_dyn_split, dim3(std::min<uint32_t>(n_chunks, kNumCUs * kDynWorkgroups)), dim3(kDynThreads), 0, stream, chunk_info, n_chunks, keys, a);
        hipLaunchKernelGGL(k_dyn_list, dim3(kNumCUs), dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_dyn_last, dim3(1), dim3(1024), 0, stream, a);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipStreamSynchronize(stream));
        std::copy(a.out, a.out + host.size(), host.begin());
        counted = host[0] != 0xffffffffu;                 // (no layer has that many weights: rows * cols < 2^32)
        plan->dyn_clear = counted;                        // (the general path counts in the same place)
        plan->dyn_passes = 1;
    }
    if (!counted) {
        plan->dyn_passes += 4;
        plan->dyn_clear = false;
        hipLaunchKernelGGL(k_dyn_init, dim3(1), dim3(256), 0, stream, state, hist, cnt,
                           static_cast<uint32_t>(2 * L), K);
        int prev_shift = 31;
        for (int lv = 0; lv < 3; ++lv) {                    // 12 + 10 + 9 bits of the 31-bit key
            const int bits = lv == 0 ? 12 : lv == 1 ? 10 : 9, shift = lv == 0 ? 19 : lv == 1 ? 9 : 0;
            hipLaunchKernelGGL(k_dyn_hist, dim3(grid), dim3(256), 0, stream, chunk_info, n_chunks, keys,
                               state, shift, bits, prev_shift, hist);
            hipLaunchKernelGGL(k_dyn_find, dim3(1), dim3(256), 0, stream, state, hist, bits);
            prev_shift = shift;
        }
        hipLaunchKernelGGL(k_dyn_count, dim3(grid), dim3(256), 0, stream, chunk_info, n_chunks, keys, state, cnt);
        rc = read_counts();
        if (rc != RSDGC_OK) return rc;
    }
    // survivors per layer: everything above the threshold, then the keys equal to it in layer order
    unsigned long long above = 0, equal = 0;
    for (int l = 0; l < L; ++l) { above += host[2 * l]; equal += host[2 * l + 1]; }
    if (above > K || above + equal < K) {
        std::snprintf(g_hip_error, sizeof(g_hip_error), "rsdgc_dynamic_ratios: inconsistent counts");
        return RSDGC_EHIP;
    }
    unsigned long long remaining = K - above;
    for (int l = 0; l < L; ++l) {
        const unsigned long long take = std::min<unsigned long long>(host[2 * l + 1], remaining);
        remaining -= take;
        ratios_out[l] = static_cast<double>(host[2 * l] + take) / static_cast<double>(plan->layers[l].G);   // Eq. 5
    }
    return RSDGC_OK;
}

static int last_paths(const rsdgc_plan_s *plan, const char *states, int32_t *paths, void *stream_) {
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    std::vector<SelState> host;
    try {
        host.resize(plan->n_layers);
    } catch (const std::bad_alloc &) {
        return RSDGC_ENOMEM;
    }
    HIP_TRY(hipStreamSynchronize(stream));
    HIP_TRY(hipMemcpy(host.data(), states, sizeof(SelState) * plan->n_layers, hipMemcpyDeviceToHost));
    for (int l = 0; l < plan->n_layers; ++l)
        paths[l] = static_cast<int32_t>(host[l].predicted >> kLastPathShift);
    return RSDGC_OK;
}

int rsdgc_last_paths(rsdgc_plan_t *plan, const void *workspace, int32_t *paths, void *stream) {
    if (!plan || plan->blocks || !workspace || !paths) return RSDGC_EINVAL;
    return last_paths(plan, static_cast<const char *>(workspace) + plan->ws.state, paths, stream);
}

int rsdgc_last_paths_blocks(rsdgc_plan_t *plan, const void *workspace, int32_t *paths, void *stream) {
    if (!plan || !plan->blocks || !workspace || !paths) return RSDGC_EINVAL;
    // (the grids' states, in the inner plan's workspace)
    return last_paths(plan, static_cast<const char *>(workspace) + plan->ws.table_bytes + plan->inner->ws.state, paths, stream);
}

static void destroy_events(rsdgc_plan_s *plan) {
    for (void *e : plan->prof_events) (void)hipEventDestroy(static_cast<hipEvent_t>(e));
    plan->prof_events.clear();
    plan->prof_max_calls = plan->prof_calls = 0;
}

int rsdgc_profile_begin(rsdgc_plan_t *plan, int32_t max_calls) {
    if (!plan || max_calls < 1 || max_calls > 4096) return RSDGC_EINVAL;
    destroy_events(plan);
    const int n = max_calls * (RSDGC_N_STAGES + 1);
    try {
        plan->prof_events.reserve(n);
    } catch (const std::bad_alloc &) {
        return RSDGC_ENOMEM;
    }
    for (int i = 0; i < n; ++i) {
        hipEvent_t e;
        hipError_t err = hipEventCreate(&e);
        if (err != hipSuccess) {
            destroy_events(plan);
            return hip_fail(err, "hipEventCreate");
        }
        plan->prof_events.push_back(e);
    }
    plan->prof_max_calls = max_calls;
    plan->prof_calls = 0;
    return RSDGC_OK;
}

int rsdgc_profile_end(rsdgc_plan_t *plan, double *stage_ms, int32_t *n_calls) {
    if (!plan || !stage_ms || !n_calls) return RSDGC_EINVAL;
    for (int s = 0; s < RSDGC_N_STAGES; ++s) stage_ms[s] = 0.0;
    *n_calls = plan->prof_calls;
    int rc = RSDGC_OK;
    for (int c = 0; c < plan->prof_calls && rc == RSDGC_OK; ++c) {
        const int base = c * (RSDGC_N_STAGES + 1);
        hipError_t err = hipEventSynchronize(static_cast<hipEvent_t>(plan->prof_events[base + RSDGC_N_STAGES]));
        if (err != hipSuccess) { rc = hip_fail(err, "hipEventSynchronize"); break; }
        for (int s = 0; s < RSDGC_N_STAGES; ++s) {
            float ms = 0.f;
            err = hipEventElapsedTime(&ms, static_cast<hipEvent_t>(plan->prof_events[base + s]),
                                      static_cast<hipEvent_t>(plan->prof_events[base + s + 1]));
            if (err != hipSuccess) { rc = hip_fail(err, "hipEventElapsedTime"); break; }
            stage_ms[s] += ms;
        }
    }
    if (rc == RSDGC_OK && plan->prof_calls > 0)
        for (int s = 0; s < RSDGC_N_STAGES; ++s) stage_ms[s] /= plan->prof_calls;
    destroy_events(plan);
    return rc;
}

const char *rsdgc_stage_name(int32_t stage) {
    static const char *names[RSDGC_N_STAGES] = {"clear", "first_pass", "capture", "find0_fallback", "select",
                                                "mark", "count_scan", "emit", "centres"};
    return (stage >= 0 && stage < RSDGC_N_STAGES) ? names[stage] : "";
}

int rsdgc_nsi(rsdgc_plan_t *plan, const float *grad, const float *residual, float *nsi_out,
              void *workspace, void *stream_) {
    if (!plan || plan->blocks || !grad || !nsi_out || !workspace) return RSDGC_EINVAL;
    if (!aligned256(workspace) || !aligned16(grad) || !aligned16(nsi_out) ||
        (residual && !aligned16(residual)))
        return RSDGC_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    return launch_nsi<kPassMapOnly>(plan, static_cast<char *>(workspace), grad, residual, nsi_out,
                                    nullptr, Momentum{}, stream);
}

int rsdgc_decompress(rsdgc_plan_t *plan, const uint32_t *idx, const float *val,
                     const int32_t *counts, float *dense, int accumulate, void *workspace,
                     void *stream_) {
    if (!plan || plan->blocks || !idx || !val || !counts || !dense || !workspace) return RSDGC_EINVAL;
    if (!aligned256(workspace) || !aligned16(dense)) return RSDGC_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    char *ws = static_cast<char *>(workspace);
    int rc = upload_tables(plan, workspace, stream);
    if (rc != RSDGC_OK) return rc;
    const LayerDev *layers = reinterpret_cast<const LayerDev *>(ws + plan->ws.layers);
    if (!accumulate)
        hipLaunchKernelGGL(k_zero_layers, dim3(plan->n_chunks), dim3(256), 0, stream,
                           reinterpret_cast<const ChunkInfo *>(ws + plan->ws.chunk_info), dense);
    if (plan->out_capacity > 0) {
        const unsigned blocks = static_cast<unsigned>((plan->out_capacity + 255) / 256);
        hipLaunchKernelGGL(k_scatter, dim3(blocks), dim3(256), 0, stream, layers, plan->n_layers,
                           static_cast<long long>(plan->out_capacity), idx, val, counts, dense,
                           accumulate);
    }
    HIP_TRY(hipGetLastError());
    return RSDGC_OK;
}

}  // extern "C"
