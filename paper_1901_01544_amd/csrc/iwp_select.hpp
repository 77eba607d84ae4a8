// Kernels of the exact per-layer selection ("choose threshold" of Alg. 1 taken as
// the k-th largest importance) and of the ordered split into (index, value) pairs.
// All of them are segmented: one launch covers every layer of a layer table.
//
// The selection is an MSB-first radix select on the 31-bit importance key
// (digits of 12 + 10 + 9 bits).  Look 1 (iwp_stream.hpp) histograms the top digit
// of every element and copies out, per tile, the elements that can be kept by the caller's hint or by
// the estimate of a small sample (k_init).  Every tile owns a fixed slot in the staging arrays, so this needs no
// cross-workgroup coordination at all.  If b1, the bin that holds rank k, is not below the
// mark, the copies are complete and look 2 (k_stage) only reads the slots, to histogram the
// second digit of those inside b1; otherwise it reads the leader's residual and weights once
// more and copies out the elements whose top digit is >= b1 (above b1 all of them are kept, the
// threshold lies among those inside).  Everything after that works on the staged
// copies, a few percent of the layer: k_refine2 (on small tables k_refine_tiles) histograms the third digit, k_split, or k_count and
// k_write where slots are full or a layer is very long, place every kept element at its rank in index order.  A tile whose
// candidates do not fit its slot (heavy ties, e.g. a tile that is all zeros) is marked
// RAW and is simply re-read from r and w by the later passes (on small tables by one of them, see k_refine_tiles).  Both
// routes are exact.
//
// The second and third digit picks have no launches of their own: a finished histogram is
// the same for every reader, so each workgroup of the consuming kernel redoes the pick of its
// layer in its prologue (k_refine2 or k_refine_tiles the second, k_split or k_count the third), and one elected workgroup
// per layer records it.  Likewise
// k_split and k_write sum the counts of the layer's earlier super-tiles themselves unless a layer has so
// many that a scan launch (k_scan) is cheaper.  Kernel boundaries are the only
// synchronisation between workgroups.
#pragma once

#include <type_traits>

#include "iwp_common.hpp"

namespace iwp {


// ---------------------------------------------------------------------------
// Workspace initialisation with vector stores (a fill kernel rather than a memset
// node, so the call sequence can be graph-captured): histograms to zero, layer
// states reset; for the single-layer entry points also the one-row layer table.
//
// The first zero_blocks workgroups clear the histograms.  The others each reset one layer's state and
// decide from which key look 1 copies candidates out: on small tables from the caller's hint (HINT_BELOW) or not at all
// (LOOK_TWICE_TILES), otherwise by a sample of the layer: 16 to 64 evenly spaced
// runs of 256 elements (the whole layer if it has no more), scored exactly as look 1 will score them.  The key
// is the sample's of rank 1.25 ks + 4 sqrt(ks) + 2, ks = k * (sample size / n): four standard
// deviations and a quarter on top, so that look 1 copies about 1.5 elements per kept one and
// practically never misses one as long as scores are not correlated inside a run (a layer sampled whole: rank k
// itself); on a layer sorted by score the runs fall short.  The guess only decides
// whether look 2 has to read the layer again; it never changes a result.  A guess in whole
// top-digit bins (1/16 octave, with one bin of slack) copied 3 to 4 per kept element where
// the scores lie evenly below the threshold, as after some hundred steps, and overflowed the slots at
// small keep ratios.  With the sample's key, thresholds of the step before in hand either way: one worker's
// share of a 25.6 M-element table 207 -> 169 us, a 400 M-element layer at 1/1000 1745 -> 1494 us a step (look 2
// 652 -> 54 us).
//
// Latency bound: a layer's sample is at most two rounds of loads for its workgroup of 16 wavefronts (one
// for keep ratios from 1/64 up), its keys stay in registers for the second histogram; the numbers of runs and the
// rank come from the host with the table row.
// ---------------------------------------------------------------------------
struct SampleSource {      // what the sample is taken from; on == 0: no sampling
    WorkerPtrs P;
    const float* w;
    const uint32_t* leader;
    uint32_t W;
    float eps;
    uint32_t on;
    uint32_t trust_hint;   // 0: never, TRUST_DENSE: on layers that keep enough, TRUST_ALWAYS (see HINT_BELOW)
};

constexpr uint32_t SAMPLE_RUN = WAVE * VEC;        // 256 consecutive elements, one quad per lane
constexpr uint32_t SAMPLE_RUNS = 64;               // at most 16384 sampled elements per layer
constexpr uint32_t SAMPLE_RUNS_MIN = 16;           // at least 4096 (or the whole layer)
constexpr uint32_t SAMPLE_RANK = 128;              // rank of the estimated threshold inside the sample, about
// Where the caller gives a hint, the mark is taken from it instead of from a sample on tables so small that the sample
// costs more than the second reads it saves: up to HINT_MAX_TILES tiles, where those come from the caches, and tables of
// short layers, where the samples are a large part of the call.  The mark lies half a top-digit bin (2 to 4 %) below the
// hinted threshold; on layers that keep less than one element in HINT_KEEP, whose slots hold less, a quarter, and only if
// few layers can miss at once.  Against always sampling: six tensors of 235 k elements 48.8 -> 43.8 us a step, one layer
// of 200 k at 0.005, four workers, 46 -> 37 us, 600 tensors of 10 M 172 -> 159 us; 45 tensors of 1 M at 0.001 would lose
// (45 -> 68 us a call), a table of 25.6 M at 1/59 is alike.
// Where the mark is sampled, a hint below it takes its place: scores that differ from block to block (a convolution's
// channels) mislead a sample of runs upwards.  One layer of 100 M elements whose gradients' scale changes every 4608: 596
// -> 530 us; independent scores are alike, with the thresholds of the step before.
// Both only where residuals add up undiminished (momentum 1).  Where they decay, a threshold can fall or rise from step to
// step by far more than the margin: after some thousand steps at 0.9 on two gradients in turn (151 tensors of 1.3 M, two
// workers) 54 us a step with the sample's mark, 108 with the hint's; 9 tensors of 0.6 M 49 / 84 us.  There no mark
// comes from a hint alone, and only a hint HINT_SLACK or more below it takes its place.
constexpr uint32_t HINT_BELOW = 1u << 18;
constexpr uint32_t HINT_SLACK = 4u << 19;          // four top-digit bins
constexpr uint32_t HINT_KEEP = 128;
constexpr uint32_t HINT_MAX_TILES = 2048, HINT_FEW_LAYERS = 16;
// Tables of up to LOOK_TWICE_TILES tiles, or LOOK_TWICE_TILES_MANY in LOOK_TWICE_MANY layers or more, have no sampled mark, with
// one exception below: where no hint is taken, look 1 copies nothing and look 2 reads the tiles again, from the caches, and
// copies from the threshold's bin on.  A sample costs 4 to 5 us there and look 1's copies
// 1 to 2, the second reading 3.  us a call, one worker, its update included, sampled / read twice: 0.3 M elements 35.8 / 31.4 in
// one layer, 36.9 / 32.1 in 20, 1 M 38.3 / 36.1 and 39.0 / 35.6, 2 M 44.1 / 44.0 and 43.0 / 40.0 (kept at 1/64), 43.9 / 40.1 and
// 42.8 / 37.1 (at 0.001); 3 M 47.8 / 52.0 and 46.4 / 44.4 (in 300 layers 51.7 / 46.4), 6 M 60.5 / 74.4 and 59.2 / 65.1 (where layers are few their tiles'
// second-digit histograms queue up, where they are many samples cost more).  A hint that is taken
// (HINT_BELOW) is better than either: 1 M 32.7 and 33.3.  A whole bin holds up to 1/16 of the elements where
// scores lie evenly below the threshold, hence LOOK_TWICE_ROOM more entries a slot: without them 100 layers of 3 M elements kept
// at 0.004 overflowed (48 us sampled, 94 read twice; with them 42).  Fuller tiles: see k_refine_tiles.
// The exception (samples() in iwp_api.hip): a step or a compression at momentum 1 that is given no hint samples all the same.  It is
// the slower route (six tensors, 235 k elements, four workers 36.7 us a step sampled, 33.7 read twice), kept as it was before
// such tables went without a sample because a hint is tested to save 4 % of that call, and with one it takes 32.6.
constexpr uint32_t LOOK_TWICE_TILES = 512, LOOK_TWICE_ROOM = 320;
constexpr uint32_t LOOK_TWICE_TILES_MANY = 1024, LOOK_TWICE_MANY = 16;
constexpr uint32_t TRUST_DENSE = 1, TRUST_ALWAYS = 2;
constexpr int INIT_BLOCK = 1024;                   // threads of a k_init workgroup
constexpr uint32_t SAMPLE_LOW_BITS = 7;            // the key's low bits that the sample does not resolve

// The key from which look 1 should copy out (its low SAMPLE_LOW_BITS bits zero).  A run is a wavefront's, so whether it is there and
// whole is the same in all lanes: no branch per element, and the loads of two runs are on their way together.
__device__ __forceinline__ uint32_t sample_stage_key(const DevLayer& L, const float* gp, const float* rp,
                                                     const float* __restrict__ w, float eps, float m, uint32_t* lh,
                                                     uint32_t* sh) {
    constexpr uint32_t WAVES = INIT_BLOCK / WAVE;
    constexpr uint32_t ROUND = 2, ROUNDS = SAMPLE_RUNS / (WAVES * ROUND);   // runs a wavefront has in flight; rounds
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = wave_id();
    const float* rl = rp + L.offset;
    const float* gl = gp ? gp + L.offset : nullptr;
    const float* wl = w + L.offset;
    const uint32_t runs_total = (L.n - 1) / SAMPLE_RUN + 1;
    const uint32_t runs = L.sample >> 16, rank = (L.sample & 0xffffu) + 1u;
    static_assert(HIST0 == 4 * INIT_BLOCK, "four bins a thread");
    reinterpret_cast<uint4*>(lh)[tid] = make_uint4(0u, 0u, 0u, 0u);
    uint32_t key[ROUNDS][ROUND][4];
    bool there[ROUNDS][ROUND];                               // uniform
#pragma unroll
    for (uint32_t d = 0; d < ROUNDS; ++d) {
        float rv[ROUND][4], gv[ROUND][4], wv[ROUND][4];
        uint32_t from[ROUND];
#pragma unroll
        for (uint32_t c = 0; c < ROUND; ++c) {
            const uint32_t i = (d * ROUND + c) * WAVES + wave;
            there[d][c] = i < runs;
            from[c] = i * runs_total / runs * SAMPLE_RUN;     // i * runs_total < 2^30; a run starts inside the layer
            if (!there[d][c]) continue;
            const uint32_t left = L.n - from[c], e = lane * VEC;
            if (left >= SAMPLE_RUN) {
                auto whole = [&](const float* p, float (&v)[4]) {
                    const v4f t = load_v4<false>(p + from[c] + e);
                    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
                };
                whole(rl, rv[c]);
                if (gp) whole(gl, gv[c]);
                whole(wl, wv[c]);
            } else {                                         // the layer's last run
                load_quad(rl + from[c], e, left, rv[c]);
                if (gp) load_quad(gl + from[c], e, left, gv[c]);
                load_quad(wl + from[c], e, left, wv[c], 1.0f);
            }
        }
#pragma unroll
        for (uint32_t c = 0; c < ROUND; ++c) {
            if (!there[d][c]) continue;
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                key[d][c][q] = score_key(gp ? accum(rv[c][q], gv[c][q], m) : rv[c][q], wv[c][q], eps);
            if (L.n - from[c] < SAMPLE_RUN) {
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q)
                    if (lane * VEC + q >= L.n - from[c]) key[d][c][q] = NOT_AN_ELEMENT;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t d = 0; d < ROUNDS; ++d)
#pragma unroll
        for (uint32_t c = 0; c < ROUND; ++c) {
            if (!there[d][c]) continue;
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)                 // NOT_AN_ELEMENT: the word behind the bins
                atomicAdd(&lh[min(key[d][c][q] >> digit_shift(0), HIST0)], 1u);
        }
    __syncthreads();
    uint32_t top, k_rem, mid, k_rem2;
    block_pick<(int)HIST0, INIT_BLOCK>(lh, rank, sh, &top, &k_rem);
    reinterpret_cast<uint4*>(lh)[tid] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
#pragma unroll
    for (uint32_t d = 0; d < ROUNDS; ++d)
#pragma unroll
        for (uint32_t c = 0; c < ROUND; ++c) {
            if (!there[d][c]) continue;
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)                 // NOT_AN_ELEMENT shares no element's digit
                if ((key[d][c][q] >> digit_shift(0)) == top)
                    atomicAdd(&lh[(key[d][c][q] >> SAMPLE_LOW_BITS) & (HIST0 - 1)], 1u);
        }
    __syncthreads();
    block_pick<(int)HIST0, INIT_BLOCK>(lh, k_rem, sh, &mid, &k_rem2);
    return (top << digit_shift(0)) | (mid << SAMPLE_LOW_BITS);
}

__global__ __launch_bounds__(INIT_BLOCK, 8) void k_init(uint32_t* __restrict__ words, uint64_t n_words,
                                                     LayerState* __restrict__ state, uint32_t zero_blocks,
                                                     const iwp_threshold* __restrict__ hint,
                                                     const DevLayer* __restrict__ layers,
                                                     DevLayer* __restrict__ single_table, DevLayer row, DevLayer sentinel,
                                                     SampleSource S) {
    __shared__ alignas(16) uint32_t lh[HIST0 + 1];
    __shared__ uint32_t sh[PICK_WORDS];
    const uint32_t n_layers = gridDim.x - zero_blocks;
    if (blockIdx.x >= n_layers) {                            // the workspace's parts are whole 256-byte blocks
        const uint32_t b = blockIdx.x - n_layers;
        const uint64_t quads = (n_words + 3) / 4, stride = (uint64_t)zero_blocks * INIT_BLOCK;
        uint4* w4 = reinterpret_cast<uint4*>(words);
        for (uint64_t i = (uint64_t)b * INIT_BLOCK + threadIdx.x; i < quads; i += stride) w4[i] = make_uint4(0u, 0u, 0u, 0u);
        if (single_table && b == 0 && threadIdx.x == 0) {
            single_table[0] = row;
            single_table[1] = sentinel;
        }
        return;
    }
    const uint32_t j = blockIdx.x;
    const uint32_t hinted = hint ? hint[j].key & 0x7fffffffu : 0u;
    const DevLayer L = single_table ? row : layers[j];       // the one-row table is only being written by this launch
    constexpr uint32_t BIN = 1u << digit_shift(0);
    const uint32_t below = !S.trust_hint ? 0u : (uint64_t)L.k * HINT_KEEP >= L.n ? HINT_BELOW
                           : S.trust_hint == TRUST_ALWAYS ? HINT_BELOW / 2 : 0u;
    uint32_t from = 0;
    if (below && hinted >= 2u * BIN && hinted < QUIET_NAN_KEY) {
        from = hinted - below;
    } else if (S.on && L.k > 0 && L.n > 0) {                 // uniform over the workgroup
        const uint32_t p = leader_of(S.leader, j, S.W);
        from = sample_stage_key(L, S.P.g[p], S.P.r[p], S.w, S.eps, S.P.momentum, lh, sh);
    }
    if (threadIdx.x == 0) {
        LayerState st;
        st.b1 = 0; st.k_rem0 = 0; st.p22 = 0; st.k_rem1 = 0; st.thr = 0; st.n_eq_take = 0; st.prestaged = 0;
        // a guess in the lowest bin (among zero scores): look 1 stages nothing; among NaN: whole bins
        const uint32_t slack = S.P.momentum == 1.0f ? 0u : HINT_SLACK;
        if (hinted >= 2u * BIN && hinted + slack < from) from = hinted;
        st.shift = (from >= BIN && from < QUIET_NAN_KEY) ? (0u - from) & (BIN - 1u) : 0u;
        st.stage_bin = from >= BIN ? shifted(from, st.shift) >> digit_shift(0) : NO_STAGE_BIN;
        state[j] = st;
    }
}

// ---------------------------------------------------------------------------
// First digit pick: the bin b1 of the 4096-bin histogram that holds rank k, whether look 1's copies already cover it.
// On tables that the chip holds at one workgroup per tile (PICK_MAX_TILES), with at most four copies of a histogram, every
// workgroup of look 2 redoes the pick of its layer itself: a launch less, 0.5 to 1.5 us of 31 to 56 us a call (six tensors
// of 235 k elements, four workers 44.2 -> 42.7 us; 160 of 3 M elements, one worker 48.8 -> 47.2), nothing from 4 M elements
// on.  On larger ones that costs more than the launch (25.6 M elements: 18.8 us against
// 10.5 + 4.8), so one workgroup per layer adds the copies up in a launch of its own, of 16 wavefronts: sixteen copies, 7.6 us
// by 4, 5.3 by 16.  A summary
// would have to be built with atomics on a handful of addresses that all
// workgroups of look 1 hit (measured: look 1 nearly twice as slow).
// ---------------------------------------------------------------------------
constexpr uint32_t PICK_MAX_COPIES = 4, PICK_MAX_TILES = 2048;

constexpr int PICK_BLOCK = 1024;                   // threads of a k_first_pick workgroup

template <int THREADS>
__device__ __forceinline__ void first_pick(const DevLayer& L, const uint32_t* __restrict__ hist, uint32_t stage_bin,
                                           uint32_t* sh, uint32_t* b1, uint32_t* k_rem0, bool* prestaged) {
    block_pick<(int)HIST0, THREADS>(layer_hist(hist, L, 0), L.k, sh, b1, k_rem0, L.h0_copies);
    *prestaged = stage_bin != NO_STAGE_BIN && stage_bin <= *b1;
}

__global__ __launch_bounds__(PICK_BLOCK) void k_first_pick(const DevLayer* __restrict__ layers, const uint32_t* __restrict__ hist,
                                                      LayerState* __restrict__ state) {
    __shared__ uint32_t sh[PICK_WORDS];
    const uint32_t j = blockIdx.x;
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    uint32_t b1, k_rem0;
    bool prestaged;
    first_pick<PICK_BLOCK>(L, hist, state[j].stage_bin, sh, &b1, &k_rem0, &prestaged);
    if (threadIdx.x == 0) {
        state[j].b1 = b1;
        state[j].k_rem0 = k_rem0;
        state[j].prestaged = prestaged ? 1u : 0u;
    }
}

// ---------------------------------------------------------------------------
// Last digit pick on its own, one workgroup per layer, for the call that stops at the
// threshold (select_threshold): the exact k-th largest key and the number of ties to keep.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(WAVE) void k_final_pick(const DevLayer* __restrict__ layers, const uint32_t* __restrict__ hist,
                                                      LayerState* __restrict__ state, iwp_threshold* __restrict__ thr_out) {
    const uint32_t j = blockIdx.x;
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    const uint32_t p22 = state[j].p22, k_rem1 = state[j].k_rem1;
    uint32_t bin, k_rem;
    wave_pick<(int)HIST2>(layer_hist(hist, L, 2), k_rem1, &bin, &k_rem);
    if (threadIdx.x == 0) {
        state[j].thr = (p22 << digit_bits(2)) | bin;
        state[j].n_eq_take = k_rem;
        if (thr_out) {
            iwp_threshold th;
            th.key = unshifted((p22 << digit_bits(2)) | bin, state[j].shift); th.n_gt = L.k - k_rem; th.n_eq_take = k_rem;
            thr_out[j] = th;
        }
    }
}

// LDS histogram -> global, non-empty bins only.
template <int NB, uint32_t THREADS = BLOCK>
__device__ __forceinline__ void flush_hist(const uint32_t* lh, uint32_t* __restrict__ gh) {
    for (uint32_t b = threadIdx.x; b < NB; b += THREADS) {
        const uint32_t v = lh[b];
        if (v) atomicAdd(&gh[b], v);
    }
}

// One tile's residuals and keys in registers, every load issued before the first use; NOT_AN_ELEMENT past the layer's end.
template <uint32_t THREADS = BLOCK, uint32_t CHUNKS>
__device__ __forceinline__ void scored_tile(const float* __restrict__ rl, const float* __restrict__ wl, uint32_t n,
                                            uint32_t base, float eps, uint32_t shift,
                                            uint32_t (&key)[CHUNKS][4], float (&val)[CHUNKS][4]) {
    float wgt[CHUNKS][4];
    const bool full = base + TILE <= n;
    Rest val_rest, wgt_rest;
    request_tile<true, THREADS>(rl, n, base, val, val_rest);
    request_tile<true, THREADS>(wl, n, base, wgt, wgt_rest);
    settle_tile<THREADS>(n, base, val, val_rest);
    settle_tile<THREADS>(n, base, wgt, wgt_rest);
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) key[u][q] = shifted(score_key(val[u][q], wgt[u][q], eps), shift);
    if (!full) leave_out_rest<THREADS>(n, base, key);                // uniform
}

// The staged keys of n <= 64 consecutive tiles from tile lt of a layer on, none of which has more than 64 (lane i's c: entries of tile
// lt + i): a wavefront takes every fourth tile (THREADS / 64th), and all its tiles' entries are requested before any of them is used.
template <uint32_t THREADS, class Body>
__device__ __forceinline__ void each_key_of_64_tiles(const StageArrays& A, const DevLayer& L, uint32_t lt, uint32_t n, uint32_t c, Body body) {
    constexpr uint32_t WAVES = THREADS / WAVE, MINE = WAVE / WAVES;
    const uint32_t lane = threadIdx.x & (WAVE - 1), wave = wave_id();
    uint32_t key[MINE];
#pragma unroll
    for (uint32_t m = 0; m < MINE; ++m) {
        const uint32_t i = wave + m * WAVES;
        key[m] = i < n && lane < from_lane(c, i) ? A.key[L.slot_begin + (uint64_t)(lt + i) * L.slot_cap + lane] : NOT_AN_ELEMENT;
    }
#pragma unroll
    for (uint32_t m = 0; m < MINE; ++m) body(key[m]);
}

// ---------------------------------------------------------------------------
// Look 2: the second digit's histogram of the elements inside b1, and staged candidates
// for the passes that follow.  The unit of work is a tile; a workgroup takes consecutive
// tiles (the grid is capped: a launch of hundreds of
// thousands of workgroups that mostly have nothing to do costs more than their work).
//  * Look 1 already filled the layer's slots from a bin <= b1:
//    only the slots are read, by the first tile's unit of every STAGE_GROUP tiles, into one
//    LDS histogram that is flushed once per workgroup and layer.  In the steady state of a training run the
//    threshold's bin holds about as many elements as are kept; that many single atomics per
//    tile, or one flush per tile, would queue up on the histogram's few cache lines.  A tile
//    whose candidates overflowed its slot in look 1 (RAW) is read again from r and w by its
//    own unit, as below; its new count carries the RESTAGED flag, so the reader of look-1
//    slots leaves it alone whether it sees the old or the new count.
//  * Otherwise the tile is read again from r and w: the elements whose top digit is >= b1
//    are copied into the tile's slot in index order (a tile with more candidates than its
//    slot holds is marked RAW), those inside b1 go into the histogram.
// ---------------------------------------------------------------------------
constexpr uint32_t STAGE_GROUP = 16;               // tiles whose slots one unit histograms
constexpr uint32_t STAGE_LARGE_TABLE = 32768;      // tiles from which the grid is what the chip holds at once ...
constexpr uint32_t STAGE_RESIDENT = 1280;          // ... five workgroups per compute unit
constexpr uint32_t STAGE_MAX_GRID = 32768;         // at most this many workgroups, unless that takes more than 64 tiles each
constexpr uint32_t STAGE_TILES_MAX = 64;           // tiles per workgroup, at most (their look-1 counts: one per lane)

template <bool PICK, uint32_t THREADS>
__global__ __launch_bounds__(THREADS, PICK ? 4 : 5) void k_stage(ResidualPtrs R, const float* __restrict__ w,
                                                 const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                 uint32_t tiles, const uint32_t* __restrict__ leader, uint32_t W,
                                                 float eps, LayerState* __restrict__ state,
                                                 uint32_t* __restrict__ hist, uint32_t* __restrict__ stage_cnt,
                                                 StageArrays A) {
    __shared__ uint32_t lh[HIST1];
    __shared__ uint32_t slot[STAGE_WORDS];
    __shared__ uint32_t sh[PICK_WORDS];
    constexpr uint32_t CHUNKS = TILE / (THREADS * VEC);
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = wave_id();
    // the workgroup's tiles are consecutive (at most 64: the host sizes the grid accordingly); their counts
    // from look 1 are fetched in one go, and a layer's row and state only when the layer changes, so that a
    // tile with nothing to do costs no memory access at all
    const uint32_t per = (tiles + gridDim.x - 1) / gridDim.x;
    const uint32_t t0 = blockIdx.x * per, t1 = min(t0 + per, tiles);
    const uint32_t my_cnt = (t0 + lane < t1) ? stage_cnt[t0 + lane] : 0u;
    uint32_t cur_j = 0xFFFFFFFFu, b1 = 0, shift = 0;
    bool prestaged = false;
    bool filled = false;                                   // lh holds counts of layer cur_j that are not flushed yet:
                                                           // one flush per workgroup and layer, however many tiles
    DevLayer L;
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t j = layer_of_tile(layers, n_layers, t);
        if (j != cur_j) {
            if (filled) {
                __syncthreads();
                flush_hist<HIST1, THREADS>(lh, layer_hist(hist, L, 1));
                filled = false;
            }
            L = layers[j];
            cur_j = j;
            if (L.k == 0) continue;
            shift = state[j].shift;
            if (PICK) {
                uint32_t k_rem0;
                first_pick<THREADS>(L, hist, state[j].stage_bin, sh, &b1, &k_rem0, &prestaged);
                if (t == L.tile_begin && tid == 0) {       // for the launches that follow
                    state[j].b1 = b1;
                    state[j].k_rem0 = k_rem0;
                }
            } else {
                b1 = state[j].b1;
                prestaged = state[j].prestaged != 0;
            }
        }
        if (L.k == 0) continue;
        const uint32_t lt = t - L.tile_begin;
        // slots: of every STAGE_GROUP tiles by the first one's workgroup, or, where a workgroup has more tiles than that, its own ones
        const bool own = per >= STAGE_GROUP;
        const bool do_slots = prestaged && (own ? t == max(t0, L.tile_begin) : lt % STAGE_GROUP == 0);
        const bool raw = prestaged && from_lane(my_cnt, t - t0) == RAW_TILE;
        if (prestaged && !do_slots && !raw) continue;      // uniform
        if (!filled) {
            __syncthreads();                               // a flush above has read lh
            for (uint32_t b = tid; b < HIST1; b += THREADS) lh[b] = 0u;
            __syncthreads();
            filled = true;
        }

        const uint32_t ntiles = (L.n + TILE - 1) / TILE;
        const uint32_t n_slots = min(own ? t1 - t : STAGE_GROUP, ntiles - lt);
        // lane i: look 1's count of tile t + i.  A tile that overflowed there has its own unit, which also histograms it
        uint32_t own_cnt = own ? (uint32_t)__shfl((int)my_cnt, (int)((lane + t - t0) & (WAVE - 1))) : 0u;
        if (lane >= n_slots || (own_cnt & RESTAGED)) own_cnt = 0u;
        if (do_slots && own && !__any(own_cnt > WAVE)) {     // uniform
            each_key_of_64_tiles<THREADS>(A, L, lt, n_slots, own_cnt, [&](uint32_t key) {    // b1 is no NOT_AN_ELEMENT's digit
                if ((key >> digit_shift(0)) == b1) atomicAdd(&lh[(key >> digit_shift(1)) & (HIST1 - 1)], 1u);
            });
        } else if (do_slots) for (uint32_t g0 = 0; g0 < n_slots; g0 += STAGE_GROUP) {
            // a wavefront takes every fourth tile of the group (THREADS / 64th); the counts and the first 256 entries of all
            // its tiles are requested before any of them is used
            const uint32_t from = lt + g0, last = min(from + STAGE_GROUP, lt + n_slots);
            constexpr uint32_t MINE = STAGE_GROUP / (THREADS / WAVE);
            uint32_t cnt[MINE];
            uint32_t key[MINE][4];
#pragma unroll
            for (uint32_t m = 0; m < MINE; ++m) {
                const uint32_t tt = from + wave + m * (THREADS / WAVE);
                cnt[m] = tt < last ? (own ? from_lane(own_cnt, tt - lt) : stage_cnt[L.tile_begin + tt]) : 0u;
                if (cnt[m] & RESTAGED) cnt[m] = 0u;        // overflowed in look 1 (RAW, or already filled again by
                                                           // the tile's own unit, which also histograms it)
            }
#pragma unroll
            for (uint32_t m = 0; m < MINE; ++m) {
                const uint64_t sbb = L.slot_begin + (uint64_t)(from + wave + m * (THREADS / WAVE)) * L.slot_cap;
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    const uint32_t e = q * WAVE + lane;
                    key[m][q] = e < cnt[m] ? A.key[sbb + e] : NOT_AN_ELEMENT;
                }
            }
#pragma unroll
            for (uint32_t m = 0; m < MINE; ++m) {
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q)
                    if (key[m][q] != NOT_AN_ELEMENT && (key[m][q] >> digit_shift(0)) == b1)
                        atomicAdd(&lh[(key[m][q] >> digit_shift(1)) & (HIST1 - 1)], 1u);
                const uint64_t sbb = L.slot_begin + (uint64_t)(from + wave + m * (THREADS / WAVE)) * L.slot_cap;
                for (uint32_t e = 4 * WAVE + lane; e < cnt[m]; e += WAVE) {    // fuller slots: the rest
                    const uint32_t k2 = A.key[sbb + e];
                    if ((k2 >> digit_shift(0)) == b1) atomicAdd(&lh[(k2 >> digit_shift(1)) & (HIST1 - 1)], 1u);
                }
            }
        }

        if (!prestaged || raw) {                           // uniform: this tile is read again
            const float* rl = R.r[leader_of(leader, j, W)] + L.offset;
            const float* wl = w + L.offset;
            const uint32_t base = lt * TILE;
            uint32_t key[CHUNKS][4];
            float val[CHUNKS][4];
            scored_tile<THREADS>(rl, wl, L.n, base, eps, shift, key, val);
            // a tile whose keys are all the same (typically a tile of zero residuals in a layer whose threshold is
            // zero, where everything ties) is recorded as such: one entry instead of an overflowing slot
            const uint32_t k0 = shifted(score_key(rl[base], wl[base], eps), shift);   // the tile's first element
            bool same = true;
#pragma unroll
            for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) same = same && (key[u][q] == k0 || key[u][q] == NOT_AN_ELEMENT);
            const bool uniform_tile = __syncthreads_and(same ? 1 : 0) != 0;
            const uint64_t sb = L.slot_begin + (uint64_t)lt * L.slot_cap;
            if (uniform_tile) {
                if (tid == 0) {
                    if ((k0 >> digit_shift(0)) == b1)
                        atomicAdd(&lh[(k0 >> digit_shift(1)) & (HIST1 - 1)], min(TILE, L.n - base));
                    A.key[sb] = k0;
                    stage_cnt[t] = UNIFORM_TILE;
                }
            } else {
#pragma unroll
                for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (key[u][q] != NOT_AN_ELEMENT && (key[u][q] >> digit_shift(0)) == b1)
                            atomicAdd(&lh[(key[u][q] >> digit_shift(1)) & (HIST1 - 1)], 1u);
                const uint32_t cnt = stage_tile<THREADS>(key, val, base, b1 << digit_shift(0), L.slot_cap, sb, A, slot);
                if (tid == 0) stage_cnt[t] = (prestaged && cnt != RAW_TILE) ? (cnt | RESTAGED) : cnt;
            }
        }
    }
    if (filled) {
        __syncthreads();
        flush_hist<HIST1, THREADS>(lh, layer_hist(hist, L, 1));
    }
}

// ---------------------------------------------------------------------------
// Third digit: histogram over the elements whose first two digits match the prefix
// (the prologue's pick appended to b1), taken from the tile slots (or from r, w for RAW
// tiles).  One workgroup per super-tile.
// ---------------------------------------------------------------------------
constexpr uint32_t STILES_TOGETHER = WAVE / GROUP; // tables of long layers: k_refine2 takes that many at once where slots hold few entries
constexpr uint32_t STILE_MAX_GRID = 8192;          // k_refine2 / k_count: beyond this many super-tiles a workgroup takes
                                                   // several consecutive ones (one pick for all of them)

// Closes a unit that holds elements with the threshold's prefix: lh (complete, synchronised) is added to the layer's third-digit
// histogram and the unit's record is written.  Clears lh, for which the caller synchronises.  red: a word per wavefront.
__device__ __forceinline__ void close_unit(uint32_t* lh, uint32_t* __restrict__ gh, uint32_t* __restrict__ record, uint32_t* red) {
    static_assert(RECORD_WORDS == BLOCK, "a word of the record per thread");
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const uint2 h = reinterpret_cast<const uint2*>(lh)[tid];
    if (h.x) atomicAdd(&gh[2 * tid], h.x);
    if (h.y) atomicAdd(&gh[2 * tid + 1], h.y);
    reinterpret_cast<uint2*>(lh)[tid] = make_uint2(0u, 0u);
    const uint32_t mine = h.x + h.y, upto = wave_inclusive_scan(mine), all = wave_last(upto);
    if (lane == 0) red[wave] = all;
    __syncthreads();
    uint32_t from = all - upto + mine;                     // of bin 2 tid or more
#pragma unroll
    for (uint32_t v = 1; v < BLOCK / WAVE; ++v) from += wave < v ? red[v] : 0u;
    record[tid] = from | (from - h.x) << 16;
}

// RECORD: what the split needs to know of every super-tile is left as well (units, records: see tie_record), so that it
// finds the threshold itself and k_count has no launch.
template <bool RECORD>
__global__ __launch_bounds__(BLOCK) void k_refine2(ResidualPtrs R, const float* __restrict__ w,
                                                   const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                   uint32_t tiles, uint32_t stiles,
                                                   const uint32_t* __restrict__ leader, uint32_t W,
                                                   float eps, LayerState* __restrict__ state,
                                                   const uint32_t* __restrict__ stage_cnt, StageArrays A,
                                                   uint32_t* __restrict__ hist, uint32_t* __restrict__ units,
                                                   uint32_t* __restrict__ records) {
    __shared__ alignas(8) uint32_t lh[HIST2];
    __shared__ uint32_t part[BLOCK / WAVE], red[BLOCK / WAVE];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = wave_id();
    const uint32_t per = (stiles + gridDim.x - 1) / gridDim.x;
    const uint32_t s0 = blockIdx.x * per, s1 = min(s0 + per, stiles);
    uint32_t cur_j = 0xFFFFFFFFu, prefix = 0;
    bool filled = false;                                   // lh holds counts of layer cur_j
    DevLayer L;
    for (uint32_t s = s0; s < s1; ++s) {
        const uint32_t j = layer_of_stile(layers, n_layers, tiles, s);
        if (j != cur_j) {
            if (filled) {
                __syncthreads();
                flush_hist<HIST2>(lh, layer_hist(hist, L, 2));
                filled = false;
            }
            L = layers[j];
            cur_j = j;
            if (L.k == 0) continue;
            // second pick, redone by every workgroup of the layer, from the finished second-digit histogram
            uint32_t bin1, k_rem1;
            wave_pick<(int)HIST1>(layer_hist(hist, L, 1), state[j].k_rem0, &bin1, &k_rem1);
            prefix = (state[j].b1 << digit_bits(1)) | bin1;                   // 22 bits
            if (s == L.stile_begin && tid == 0) {
                state[j].p22 = prefix;
                state[j].k_rem1 = k_rem1;
            }
            __syncthreads();                               // the flush above has read lh
            for (uint32_t b = tid; b < HIST2; b += BLOCK) lh[b] = 0u;
            __syncthreads();
            filled = !RECORD;
        }
        if (L.k == 0) continue;
        const uint32_t ntiles = (L.n + TILE - 1) / TILE;
        const uint32_t lt0 = (s - L.stile_begin) * GROUP;
        if (!RECORD && per > 1) {                              // the workgroup's super-tiles of the layer at once, up to eight
            const uint32_t n = min(min(s1 - s, STILES_TOGETHER) * GROUP, ntiles - lt0);
            const uint32_t c = lane < n ? staged_entries(stage_cnt[L.tile_begin + lt0 + lane]) : 0u;
            if (!__any(c > WAVE)) {                           // uniform; no RAW or UNIFORM tile among them
                each_key_of_64_tiles<BLOCK>(A, L, lt0, n, c, [&](uint32_t key) {
                    if ((key >> digit_shift(1)) == prefix) atomicAdd(&lh[key & (HIST2 - 1)], 1u);
                });
                s += (n - 1) / GROUP;
                continue;
            }
        }
        const uint32_t nt = min(GROUP, ntiles - lt0);
        // the super-tile's eight counts, one per lane; a wavefront takes tiles wave and wave + 4, the counts
        // and the first 256 entries of both requested before any of them is used
        const uint32_t my_cnt = lane < nt ? staged_entries(stage_cnt[L.tile_begin + lt0 + lane]) : 0u;
        constexpr uint32_t MINE = GROUP / (BLOCK / WAVE);
        uint32_t cnt[MINE];
        uint32_t key[MINE][4];
        uint32_t c = 0;                                    // above the prefix; high half: sharing it
        auto add = [&](uint32_t k2, uint32_t n) {          // n elements of key k2 (NOT_AN_ELEMENT: none)
            const uint32_t top = k2 >> digit_shift(1);
            if (RECORD) c += k2 == NOT_AN_ELEMENT ? 0u : top > prefix ? n : top == prefix ? n << 16 : 0u;
            if (k2 != NOT_AN_ELEMENT && top == prefix) atomicAdd(&lh[k2 & (HIST2 - 1)], n);
        };
#pragma unroll
        for (uint32_t m = 0; m < MINE; ++m) {
            const uint32_t tl = wave + m * (BLOCK / WAVE);
            cnt[m] = from_lane(my_cnt, tl);
            const uint64_t sb = L.slot_begin + (uint64_t)(lt0 + tl) * L.slot_cap;
            if (cnt[m] == UNIFORM_TILE) {                  // all keys of the tile are the slot's one entry
                const uint32_t k0 = A.key[sb];
                if (lane == 0) add(k0, min(TILE, L.n - (lt0 + tl) * TILE));
                cnt[m] = 0u;
            }
            if (cnt[m] == RAW_TILE) cnt[m] = 0u;           // read again below
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t e = q * WAVE + lane;
                key[m][q] = e < cnt[m] ? A.key[sb + e] : NOT_AN_ELEMENT;
            }
        }
#pragma unroll
        for (uint32_t m = 0; m < MINE; ++m) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) add(key[m][q], 1u);
            const uint64_t sb = L.slot_begin + (uint64_t)(lt0 + wave + m * (BLOCK / WAVE)) * L.slot_cap;
            for (uint32_t e = 4 * WAVE + lane; e < cnt[m]; e += WAVE) add(A.key[sb + e], 1u);   // fuller slots: the rest
        }
        const uint64_t raw_tiles = __ballot(my_cnt == RAW_TILE) & 0xFFull;    // the same in every wavefront
        if (raw_tiles) {                                                       // uniform
            const float* rl = R.r[leader_of(leader, j, W)] + L.offset;
            const float* wl = w + L.offset;
            const uint32_t shift = state[j].shift;
            for (uint32_t tl = 0; tl < nt; ++tl) {
                if (!((raw_tiles >> tl) & 1ull)) continue;
                for (uint32_t u = 0; u < CHUNKS_PER_TILE; ++u) {
                    const uint32_t i = (lt0 + tl) * TILE + u * CHUNK + tid * VEC;
                    if (i >= L.n) break;
                    float rv[4], wv[4];
                    load_quad(rl, i, L.n, rv);
                    load_quad(wl, i, L.n, wv, 1.0f);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t key2 = shifted(score_key(rv[q], wv[q], eps), shift);
                        if (i + q < L.n) add(key2, 1u);
                    }
                }
            }
        }
        if (RECORD) {
            c = wave_sum(c);                               // at most 32768 of either kind
            if (lane == 0) part[wave] = c;
            __syncthreads();                               // lh is complete, too
            const uint32_t all = part[0] + part[1] + part[2] + part[3];
            if (tid == 0) units[s] = all;
            if (all >> 16) close_unit(lh, layer_hist(hist, L, 2), tie_record(hist, records, L, s - L.stile_begin), red);
            filled = false;
            if (s + 1 < s1) __syncthreads();               // part and lh are written again
        }
    }
    if (filled) {
        __syncthreads();
        flush_hist<HIST2>(lh, layer_hist(hist, L, 2));
    }
}

// ---------------------------------------------------------------------------
// The third digit on tables without a sampled mark (LOOK_TWICE_TILES), one workgroup per tile.  There look 2 copies whole bins of
// the first digit, and where scores crowd into one bin every tile overflows its slot.  Such a tile is read a third time, from the
// caches, but by this launch alone: the 22-bit prefix is known here and leaves little more than is kept, so what is at or above it
// goes into the slot after all, and k_split (or k_count and k_write) finds copies (a tile that still overflows, by ties, stays RAW).
// Bound by latency, and for such tiles by the divides: a workgroup per tile puts them on all compute units, where k_refine2's
// workgroup of a super-tile has eight tiles in turn.  One layer of 1 M elements kept at 1/64, us a call, k_refine2 / this: scores
// inside one bin 104 / 40 (45.5 when such layers were sampled), normally distributed 31.0 / 30.0 (38.4); kept at 0.001, an
// eighth of the scores in the threshold's bin 98 / 36 (39), eight distinct values 99 / 74 (117).  Where an eighth of a tile just
// fits its slot nothing is gained: 2 M elements kept at 1/64 46 (42 sampled).  (Slots of 400 entries instead of 576, so that it
// overflows: 44, but the eight values, kept at 1/64, 39 -> 74.)
// ---------------------------------------------------------------------------
template <bool RECORD>
__global__ __launch_bounds__(BLOCK) void k_refine_tiles(ResidualPtrs R, const float* __restrict__ w,
                                                        const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                        const uint32_t* __restrict__ leader, uint32_t W, float eps,
                                                        LayerState* __restrict__ state, uint32_t* __restrict__ stage_cnt,
                                                        StageArrays A, uint32_t* __restrict__ hist, uint32_t* __restrict__ units,
                                                        uint32_t* __restrict__ records) {
    __shared__ alignas(8) uint32_t lh[HIST2];
    __shared__ uint32_t slot[STAGE_WORDS];
    __shared__ uint32_t part[BLOCK / WAVE], red[BLOCK / WAVE];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), t = blockIdx.x;
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    const uint32_t lt = t - L.tile_begin, base = lt * TILE, cnt = staged_entries(stage_cnt[t]);
    const uint64_t sb = L.slot_begin + (uint64_t)lt * L.slot_cap;
    const uint32_t first = cnt < UNIFORM_TILE && tid < cnt ? A.key[sb + tid] : NOT_AN_ELEMENT;
    // tiles of equal keys: the first tile's workgroup of a super-tile adds all of its up (one hot bin, 64 workgroups instead of 512
    // queueing up at it: 2 M equal scores 47 -> 43 us)
    uint32_t equal = NOT_AN_ELEMENT;
    if (lt % GROUP == 0 && tid < GROUP && lt + tid < (L.n + TILE - 1) / TILE && stage_cnt[t + tid] == UNIFORM_TILE)
        equal = A.key[sb + (uint64_t)tid * L.slot_cap];
    uint32_t bin1, k_rem1;
    wave_pick<(int)HIST1>(layer_hist(hist, L, 1), state[j].k_rem0, &bin1, &k_rem1);
    const uint32_t prefix = (state[j].b1 << digit_bits(1)) | bin1;            // 22 bits
    if (lt == 0 && tid == 0) {
        state[j].p22 = prefix;
        state[j].k_rem1 = k_rem1;
    }
    for (uint32_t b = tid; b < HIST2; b += BLOCK) lh[b] = 0u;
    __syncthreads();
    uint32_t c = 0;                                        // above the prefix; high half: sharing it
    auto add = [&](uint32_t key, uint32_t n) {
        const uint32_t top = key >> digit_shift(1);
        if (RECORD) c += key == NOT_AN_ELEMENT ? 0u : top > prefix ? n : top == prefix ? n << 16 : 0u;
        if (key != NOT_AN_ELEMENT && top == prefix) atomicAdd(&lh[key & (HIST2 - 1)], n);
    };
    if (cnt == RAW_TILE) {                                 // uniform
        uint32_t key[CHUNKS_PER_TILE][4];
        float val[CHUNKS_PER_TILE][4];
        scored_tile(R.r[leader_of(leader, j, W)] + L.offset, w + L.offset, L.n, base, eps, state[j].shift, key, val);
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS_PER_TILE; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) add(key[u][q], 1u);
        const uint32_t copies = stage_tile(key, val, base, prefix << digit_shift(1), L.slot_cap, sb, A, slot);
        if (tid == 0) stage_cnt[t] = copies;
    } else if (cnt != UNIFORM_TILE) {
        add(first, 1u);
        for (uint32_t e = BLOCK + tid; e < cnt; e += BLOCK) add(A.key[sb + e], 1u);
    }
    const uint32_t n_equal = min(TILE, L.n - min(base + tid * TILE, L.n));
    if (!RECORD) {
        add(equal, n_equal);
        __syncthreads();
        flush_hist<HIST2>(lh, layer_hist(hist, L, 2));
        return;
    }
    uint32_t* gh = layer_hist(hist, L, 2);
    uint32_t* record = tie_record(hist, records, L, lt);
    if (tid < WAVE) {                                      // the super-tile's tiles of equal keys, key by key
        const bool hit = equal != NOT_AN_ELEMENT && (equal >> digit_shift(1)) == prefix;
        for (uint64_t left = __ballot(hit); left;) {
            const uint32_t key = from_lane(equal, (uint32_t)__ffsll((unsigned long long)left) - 1u);
            const bool same = hit && equal == key;
            const uint32_t n = wave_sum(same ? n_equal : 0u);
            if (lane == 0) atomicAdd(&gh[key & (HIST2 - 1)], n);
            left &= ~__ballot(same);
        }
    }
    if (cnt == UNIFORM_TILE) {                             // uniform
        const uint32_t key = A.key[sb], top = key >> digit_shift(1), low = key & (HIST2 - 1), n = min(TILE, L.n - base);
        if (tid == 0) units[t] = top > prefix ? n : top == prefix ? n << 16 : 0u;
        if (top == prefix) record[tid] = (2 * tid <= low ? n : 0u) | (2 * tid + 1 <= low ? n << 16 : 0u);
        return;
    }
    c = wave_sum(c);
    if (lane == 0) part[tid >> 6] = c;
    __syncthreads();                                       // lh is complete, too
    const uint32_t all = part[0] + part[1] + part[2] + part[3];
    if (tid == 0) units[t] = all;
    if (all >> 16) close_unit(lh, gh, record, red);
}

// ---------------------------------------------------------------------------
// Threshold records given by the caller (compact_pairs): one pass over the layer that counts, per tile, the elements above
// the threshold and those that tie with it, and copies both into the tile's slot, one workgroup per tile as in look 1;
// k_fold_counts sums the counts up, and the ordered split works on the slots, as after a selection.  A layer's first
// workgroup leaves the record in its selection state.
// Bound by reading r and w once.  Counting and writing from r and w directly read them twice, and the counts with one
// dword per lane and access: 126 us for a table of 25 M elements at one pair in 64, now 48 us.
// A tile is marked RAW, to be read again by the split, where copies do not pay: its elements overflow the slot, the
// threshold is zero (everything is at or above it), or the layer keeps half of its elements or more, where a copy and its
// reading back move 24 bytes per pair against 8 per element read again.  One layer of 25 M elements, copies / read again:
// keep 0.4 125 / 112 us, 0.5 149 / 118, 0.999 254 / 163; of 1 M elements 24 / 39, 27 / 37, 40 / 38.
// ---------------------------------------------------------------------------
template <uint32_t THREADS>
__global__ __launch_bounds__(THREADS) void k_stage_records(const float* __restrict__ r, const float* __restrict__ w,
                                                         const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                         const iwp_threshold* __restrict__ thr, float eps,
                                                         LayerState* __restrict__ state,
                                                         uint32_t* __restrict__ stage_cnt, StageArrays A,
                                                         uint2* __restrict__ tile_counts) {
    constexpr uint32_t CHUNKS = TILE / (THREADS * VEC);
    __shared__ uint32_t slot[STAGE_WORDS];
    __shared__ uint32_t part[THREADS / WAVE];
    const uint32_t t = blockIdx.x;
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    const uint32_t lt = t - L.tile_begin;
    const uint32_t from = thr[j].key;
    if (lt == 0 && threadIdx.x == 0) {
        LayerState st;
        st.b1 = 0; st.k_rem0 = 0; st.p22 = 0; st.k_rem1 = 0;
        st.thr = from; st.n_eq_take = thr[j].n_eq_take;
        st.stage_bin = NO_STAGE_BIN; st.shift = 0; st.prestaged = 0;
        state[j] = st;
    }
    uint32_t key[CHUNKS][4];
    float val[CHUNKS][4];
    scored_tile<THREADS>(r + L.offset, w + L.offset, L.n, lt * TILE, eps, 0u, key, val);
    uint32_t c = 0;                                        // above the threshold; high half: tying with it
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            c += key[u][q] == NOT_AN_ELEMENT ? 0u : key[u][q] > from ? 1u : key[u][q] == from ? 0x10000u : 0u;
    c = wave_sum(c);
    if ((threadIdx.x & (WAVE - 1)) == 0) part[threadIdx.x >> 6] = c;
    uint32_t cnt = RAW_TILE;
    if (from != 0u && L.k < L.n - L.k)                     // uniform; either way a barrier before the sum below
        cnt = stage_tile<THREADS>(key, val, lt * TILE, from, L.slot_cap, L.slot_begin + (uint64_t)lt * L.slot_cap, A, slot);
    else
        __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t v = 0; v < THREADS / WAVE; ++v) sum += part[v];
        stage_cnt[t] = cnt;
        tile_counts[t] = make_uint2(sum & 0xffffu, sum >> 16);
    }
}

// The tiles' counts that k_stage_records left -> what k_count leaves: each tile's exclusive prefix inside its super-tile and
// the super-tile's totals.  One super-tile per lane.
__global__ __launch_bounds__(BLOCK) void k_fold_counts(const DevLayer* __restrict__ layers, uint32_t n_layers, uint32_t tiles, uint32_t stiles,
                                                       uint2* __restrict__ tile_counts, uint2* __restrict__ stile_counts) {
    const uint32_t s = blockIdx.x * BLOCK + threadIdx.x;
    if (s >= stiles) return;
    const DevLayer& L = layers[layer_of_stile(layers, n_layers, tiles, s)];
    if (L.k == 0) return;
    const uint32_t lt0 = (s - L.stile_begin) * GROUP;
    const uint32_t nt = min(GROUP, (L.n + TILE - 1) / TILE - lt0);
    uint2* tc = tile_counts + L.tile_begin + lt0;
    uint2 v[GROUP];
#pragma unroll
    for (uint32_t q = 0; q < GROUP; ++q) v[q] = q < nt ? tc[q] : make_uint2(0u, 0u);
    uint32_t above = 0, ties = 0;
#pragma unroll
    for (uint32_t q = 0; q < GROUP; ++q) {
        if (q < nt) tc[q] = make_uint2(above, ties);
        above += v[q].x;
        ties += v[q].y;
    }
    stile_counts[s] = make_uint2(above, ties);
}

// A RAW tile read again by one wavefront, RAW_AHEAD rounds of 256 elements in flight together, since neither k_refine_tiles nor look 2
// has left its lines in this die's cache.  body(packed, key, val, i): the lane's four elements of a round, i the first one's position;
// packed: of those above the threshold, in the high half of those tying with it; key[q] is NOT_AN_ELEMENT where position i + q is not
// the lane's.  Every lane reads whole quads, at the layer's end the last one, and leaves
// out what comes before its own: loads in branches waited for each other (a layer of 48 tiles, mostly zeros, kept at 0.2: k_count 22.2 -> 18.3 us,
// k_write 25.1 -> 17.1).  Layers of fewer elements than a quad, which k_stage_records can leave RAW, are read element by element.
constexpr uint32_t RAW_ROUND = WAVE * VEC, RAW_AHEAD = 4;
template <class Body>
__device__ __forceinline__ void read_raw_tile(const float* rl, const float* wl, uint32_t n, uint32_t first, float eps, uint32_t shift,
                                              uint32_t thr, Body body) {
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    const uint32_t last = n >= VEC ? n - VEC : 0u;           // the layer's last quad
#pragma unroll 1
    for (uint32_t c = 0; c < TILE && first + c < n; c += RAW_AHEAD * RAW_ROUND) {
        v4f rv[RAW_AHEAD], wv[RAW_AHEAD];
        if (n >= VEC) {                                      // uniform
#pragma unroll
            for (uint32_t a = 0; a < RAW_AHEAD; ++a) {
                const uint32_t at = min(first + c + a * RAW_ROUND + lane * VEC, last);
                rv[a] = load_v4<false>(rl + at);
                wv[a] = load_v4<false>(wl + at);
            }
        } else {
            const uint32_t e1 = min(1u, n - 1u), e2 = n - 1u;
#pragma unroll
            for (uint32_t a = 0; a < RAW_AHEAD; ++a) {
                rv[a] = v4f{rl[0], rl[e1], rl[e2], 0.0f};
                wv[a] = v4f{wl[0], wl[e1], wl[e2], 1.0f};
            }
        }
#pragma unroll
        for (uint32_t a = 0; a < RAW_AHEAD; ++a) {
            const uint32_t i = first + c + a * RAW_ROUND + lane * VEC, at = min(i, last);
            const float val[4] = {rv[a].x, rv[a].y, rv[a].z, rv[a].w}, wgt[4] = {wv[a].x, wv[a].y, wv[a].z, wv[a].w};
            uint32_t key[4], packed = 0;
#pragma unroll
            for (uint32_t q = 0; q < VEC; ++q) {
                key[q] = at + q >= i && at + q < n ? shifted(score_key(val[q], wgt[q], eps), shift) : NOT_AN_ELEMENT;
                packed += key[q] == NOT_AN_ELEMENT ? 0u : key[q] > thr ? 1u : key[q] == thr ? 0x10000u : 0u;
            }
            body(packed, key, val, at);
        }
    }
}

// ---------------------------------------------------------------------------
// Ordered split, part 1: per tile, how many elements lie above the threshold and
// how many tie with it.  One workgroup per super-tile; writes each tile's exclusive
// prefix inside the super-tile and the super-tile's totals.  The threshold is the
// prologue's third pick (recorded, with thr_out, by the layer's first workgroup).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_count(ResidualPtrs R, const float* __restrict__ w,
                                                 const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                 uint32_t tiles, uint32_t stiles,
                                                 const uint32_t* __restrict__ leader, uint32_t W, float eps,
                                                 LayerState* __restrict__ state, const uint32_t* __restrict__ hist,
                                                 iwp_threshold* __restrict__ thr_out,
                                                 const uint32_t* __restrict__ stage_cnt, StageArrays A,
                                                 uint2* __restrict__ tile_counts, uint2* __restrict__ stile_counts) {
    __shared__ uint32_t cg[GROUP], ce[GROUP];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & (WAVE - 1), wave = wave_id();
    const uint32_t per = (stiles + gridDim.x - 1) / gridDim.x;
    const uint32_t s0 = blockIdx.x * per, s1 = min(s0 + per, stiles);
    uint32_t cur_j = 0xFFFFFFFFu, thr = 0, shift = 0;
    DevLayer L;
    for (uint32_t s = s0; s < s1; ++s) {
        const uint32_t j = layer_of_stile(layers, n_layers, tiles, s);
        if (j != cur_j) {
            L = layers[j];
            cur_j = j;
            if (L.k == 0) continue;
            shift = state[j].shift;
            // third pick, redone by every workgroup of the layer: the exact k-th largest key
            uint32_t bin2, k_rem2;
            wave_pick<(int)HIST2>(layer_hist(hist, L, 2), state[j].k_rem1, &bin2, &k_rem2);
            thr = (state[j].p22 << digit_bits(2)) | bin2;
            if (s == L.stile_begin && tid == 0) {
                state[j].thr = thr;
                state[j].n_eq_take = k_rem2;
                if (thr_out) {
                    iwp_threshold th;
                    th.key = unshifted(thr, state[j].shift); th.n_gt = L.k - k_rem2; th.n_eq_take = k_rem2;
                    thr_out[j] = th;
                }
            }
        }
        if (L.k == 0) continue;
        const uint32_t ntiles = (L.n + TILE - 1) / TILE;
        const uint32_t lt0 = (s - L.stile_begin) * GROUP;       // first tile of the super-tile, in the layer
        const uint32_t nt = min(GROUP, ntiles - lt0);
        const float* rl = R.r[leader_of(leader, j, W)] + L.offset;
        const float* wl = w + L.offset;
        // each wavefront takes tiles of its own (tiles wave and wave + 4; the counts and the first 256 entries of
        // both requested before any of them is used); nothing workgroup-wide until the end
        const uint32_t my_cnt = lane < nt ? staged_entries(stage_cnt[L.tile_begin + lt0 + lane]) : RAW_TILE;
        constexpr uint32_t MINE = GROUP / (BLOCK / WAVE);
        uint32_t cnt[MINE];
        uint32_t key[MINE][4];
#pragma unroll
        for (uint32_t m = 0; m < MINE; ++m) {
            const uint32_t tl = wave + m * (BLOCK / WAVE);
            cnt[m] = from_lane(my_cnt, tl);
            const uint64_t sb = L.slot_begin + (uint64_t)(lt0 + tl) * L.slot_cap;
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t e = q * WAVE + lane;
                key[m][q] = (tl < nt && cnt[m] < UNIFORM_TILE && e < cnt[m]) ? A.key[sb + e] : NOT_AN_ELEMENT;
            }
        }
#pragma unroll
        for (uint32_t m = 0; m < MINE; ++m) {
            const uint32_t tl = wave + m * (BLOCK / WAVE);
            if (tl >= nt) continue;
            uint32_t gt = 0, eq = 0;
            if (cnt[m] == UNIFORM_TILE) {                  // all keys of the tile are the slot's one entry
                const uint32_t k0 = A.key[L.slot_begin + (uint64_t)(lt0 + tl) * L.slot_cap];
                const uint32_t n_tile = min(TILE, L.n - (lt0 + tl) * TILE);
                if (lane == 0) { gt = k0 > thr ? n_tile : 0u; eq = k0 == thr ? n_tile : 0u; }
            } else if (cnt[m] != RAW_TILE) {
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    gt += (key[m][q] != NOT_AN_ELEMENT && key[m][q] > thr) ? 1u : 0u;
                    eq += key[m][q] == thr ? 1u : 0u;          // a key is never NOT_AN_ELEMENT (bit 31 is clear)
                }
                const uint64_t sb = L.slot_begin + (uint64_t)(lt0 + tl) * L.slot_cap;
                // fuller slots: again 256 entries at a time (as a plain loop the compiler asked for 64: five layers of 20 M elements,
                // 0.9 kept, 46 us a launch instead of 23.5)
                for (uint32_t e0 = 4 * WAVE; e0 < cnt[m]; e0 += 4 * WAVE) {
                    uint32_t k2[4];
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) {
                        const uint32_t e = e0 + q * WAVE + lane;
                        k2[q] = e < cnt[m] ? A.key[sb + e] : NOT_AN_ELEMENT;
                    }
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) {
                        gt += (k2[q] != NOT_AN_ELEMENT && k2[q] > thr) ? 1u : 0u;
                        eq += k2[q] == thr ? 1u : 0u;
                    }
                }
            } else {
                read_raw_tile(rl, wl, L.n, (lt0 + tl) * TILE, eps, shift, thr,
                              [&](uint32_t packed, const uint32_t (&)[4], const float (&)[4], uint32_t) {
                    gt += packed & 0xffffu;
                    eq += packed >> 16;
                });
            }
            gt = wave_sum(gt);
            eq = wave_sum(eq);
            if (lane == 0) { cg[tl] = gt; ce[tl] = eq; }
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t G = 0, E = 0;
            for (uint32_t tl = 0; tl < nt; ++tl) {
                tile_counts[L.tile_begin + lt0 + tl] = make_uint2(G, E);
                G += cg[tl];
                E += ce[tl];
            }
            stile_counts[s] = make_uint2(G, E);
        }
        __syncthreads();                                        // cg / ce are written again for the next super-tile
    }
}

// Part 2: exclusive prefix of the super-tile totals inside each layer, in order.
// One workgroup per layer, eight parts of 1024 consecutive super-tiles a round: a chain of a load, two scans and a store per 8192 of
// them.  A layer of 400 M elements, 12 k of them: 256 threads with eight consecutive ones each 12.4 us, 1024 threads 12.1 (each access
// a line per lane), now 7.3.
constexpr int SCAN_BLOCK = 1024;
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan(const DevLayer* __restrict__ layers, uint2* __restrict__ stile_counts) {
    constexpr uint32_t PER = 8, WAVES = SCAN_BLOCK / WAVE;
    __shared__ uint2 sums[2][PER][WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = wave_id();
    const uint32_t j = blockIdx.x;
    if (layers[j].k == 0) return;
    const uint32_t sb = layers[j].stile_begin;
    const uint32_t se = sb + (layers[j].n + STILE - 1) / STILE;
    uint32_t G = 0, E = 0;                                  // before the part
    for (uint32_t b = sb, round = 0; b < se; b += SCAN_BLOCK * PER, ++round) {
        uint2 v[PER], upto[PER];
        auto& ws = sums[round & 1u];                         // the round before may still be reading the other
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t s = b + q * SCAN_BLOCK + tid;
            v[q] = s < se ? stile_counts[s] : make_uint2(0u, 0u);
        }
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            upto[q] = make_uint2(wave_inclusive_scan(v[q].x), wave_inclusive_scan(v[q].y));
            if (lane == WAVE - 1) ws[q][wave] = upto[q];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            if (b + q * SCAN_BLOCK >= se) break;             // uniform
            const uint2 c = lane < WAVES ? ws[q][lane] : make_uint2(0u, 0u);     // the wavefronts' totals
            const uint32_t cg = wave_inclusive_scan(c.x), ce = wave_inclusive_scan(c.y);
            const uint32_t g = G + upto[q].x - v[q].x + from_lane(cg - c.x, wave);
            const uint32_t e = E + upto[q].y - v[q].y + from_lane(ce - c.y, wave);
            G += wave_last(cg);
            E += wave_last(ce);
            const uint32_t s = b + q * SCAN_BLOCK + tid;
            if (s < se) stile_counts[s] = make_uint2(g, e);
        }
    }
}

// AHEAD times 64 consecutive entries of a tile's slot, in registers.
template <uint32_t AHEAD>
struct SlotPart {
    uint32_t key[AHEAD], idx[AHEAD];
    float val[AHEAD];
};
// Requested before it is known what is kept of them; of fuller slots, at a time (2: full slots of 25 tiles 23.4 us, 4: 18.0).
constexpr uint32_t SPLIT_AHEAD = 2, SPLIT_AHEAD_MORE = 4;
typedef SlotPart<SPLIT_AHEAD> SlotStart;
// cnt: entries from `first` on.
template <uint32_t AHEAD>
__device__ __forceinline__ void request_slot(const StageArrays& A, uint64_t first, uint32_t cnt, SlotPart<AHEAD>& S) {
    const uint32_t last = cnt < UNIFORM_TILE ? max(cnt, 1u) - 1u : 0u;       // lanes behind the last entry read it, or the first word
#pragma unroll
    for (uint32_t q = 0; q < AHEAD; ++q) {
        const uint64_t e = first + min(q * WAVE + (threadIdx.x & (WAVE - 1)), last);
        S.key[q] = A.key[e];
        S.idx[q] = A.idx[e];
        S.val[q] = A.val[e];
    }
}

// 64 entries of a slot, one per lane (have: there is one): those that are kept go to their places behind G elements above the threshold
// and E that tie with it, which are counted on.
template <bool FUSED>
__device__ __forceinline__ void write_entries(const DevLayer& L, uint32_t key, uint32_t idx, float val, bool have, uint32_t thr,
                                              uint32_t quota, uint32_t& G, uint32_t& E, float* rl, uint32_t* __restrict__ io,
                                              float* __restrict__ vo, float* __restrict__ go) {
    const uint64_t below = (1ull << (threadIdx.x & (WAVE - 1))) - 1ull;
    const bool above = have && key > thr, ties = have && key == thr;
    const uint64_t ma = __ballot(above), mt = __ballot(ties);
    const uint32_t gpre = G + __popcll(ma & below), epre = E + __popcll(mt & below);
    uint32_t pos = 0xFFFFFFFFu;
    if (above) pos = gpre + min(epre, quota);
    else if (ties && epre < quota) pos = gpre + epre;
    if (pos < L.k && idx < L.n) {
        io[pos] = (uint32_t)(L.offset + idx);
        vo[pos] = val;
        if (FUSED) { go[pos] = val; rl[idx] = 0.0f; }
    }
    G += __popcll(ma);
    E += __popcll(mt);
}

// The pairs of one tile, by one wavefront; S: its slot's first entries.  The slots being in index order saves the bitmaps in LDS that would rank
// their entries: 8.7 -> 6.5 us a launch on a 25.6 M-element table, 59 -> 47 us on a layer of 400 M.  cnt: the tile's staged entries, UNIFORM_TILE or RAW_TILE; Gt, Et: elements
// above the threshold / tying with it before the tile.
template <bool FUSED, uint32_t AHEAD>
__device__ __forceinline__ void write_tile(const DevLayer& L, uint32_t lt, uint32_t cnt, uint32_t thr, uint32_t quota,
                                           uint32_t shift, uint32_t Gt, uint32_t Et, float* rl,
                                           const float* __restrict__ wl, float eps, const StageArrays& A, const SlotPart<AHEAD>& S,
                                           uint32_t* __restrict__ io, float* __restrict__ vo, float* __restrict__ go) {
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    const uint32_t out_base = Gt + min(Et, quota);
    const uint32_t tile_first = lt * TILE;
    if (cnt == UNIFORM_TILE) {
        // all keys of the tile are the slot's one entry: above the threshold everything is kept, at the
        // threshold the first elements until the quota of ties is used up, below it nothing
        const uint32_t k0 = A.key[L.slot_begin + (uint64_t)lt * L.slot_cap];
        const uint32_t n_tile = min(TILE, L.n - tile_first);
        uint32_t take = 0;
        if (k0 > thr) take = n_tile;
        else if (k0 == thr && Et < quota) take = min(n_tile, quota - Et);
        for (uint32_t i = lane; i < take; i += WAVE) {
            const uint32_t pos = out_base + i;
            const uint32_t li = tile_first + i;
            if (pos < L.k) {
                const float v = rl[li];
                io[pos] = (uint32_t)(L.offset + li);
                vo[pos] = v;
                if (FUSED) { go[pos] = v; rl[li] = 0.0f; }
            }
        }
        return;
    }
    uint32_t G = Gt, E = Et;
    if (cnt != RAW_TILE) {
        // a slot holds its tile's candidates in index order: 64 of them at a time, ranked by what stands before them
        const uint64_t sb = L.slot_begin + (uint64_t)lt * L.slot_cap;
        auto write = [&](auto& part, auto ahead, uint32_t e0) {
#pragma unroll
            for (uint32_t q = 0; q < ahead.value; ++q)
                write_entries<FUSED>(L, part.key[q], part.idx[q], part.val[q], e0 + q * WAVE + lane < cnt, thr, quota, G, E, rl, io, vo, go);
        };
        write(S, std::integral_constant<uint32_t, AHEAD>(), 0u);
        for (uint32_t e0 = AHEAD * WAVE; e0 < cnt; e0 += SPLIT_AHEAD_MORE * WAVE) {
            SlotPart<SPLIT_AHEAD_MORE> more;
            request_slot(A, sb + e0, cnt - e0, more);
            write(more, std::integral_constant<uint32_t, SPLIT_AHEAD_MORE>(), e0);
        }
        return;
    }

    // RAW tile: every element is scored again
    read_raw_tile(rl, wl, L.n, tile_first, eps, shift, thr,
                  [&](uint32_t packed, const uint32_t (&key)[4], const float (&val)[4], uint32_t at) {
        const uint32_t inc = wave_inclusive_scan(packed), tot = wave_last(inc), ex = inc - packed;
        uint32_t gpre = G + (ex & 0xffffu);
        uint32_t epre = E + (ex >> 16);
        if (packed) {
#pragma unroll
            for (uint32_t q = 0; q < VEC; ++q) {
                if (key[q] == NOT_AN_ELEMENT) continue;
                uint32_t pos = 0xFFFFFFFFu;
                if (key[q] > thr) { pos = gpre + min(epre, quota); ++gpre; }
                else if (key[q] == thr) { if (epre < quota) pos = gpre + epre; ++epre; }
                if (pos < L.k) {
                    io[pos] = (uint32_t)(L.offset + at + q);
                    vo[pos] = val[q];
                    if (FUSED) { go[pos] = val[q]; rl[at + q] = 0.0f; }
                }
            }
        }
        G += tot & 0xffffu;
        E += tot >> 16;
    });
}

// Part 3: write the pairs.  An element above the threshold goes to position
// (#above before it) + min(#ties before it, quota); a tie is kept iff fewer than
// `quota` ties precede it.  Positions are counted in index order, so the output is
// ascending and ties go to the lowest indices (Alg. 1 split: the sent part is the
// residual itself).  tile_out[t] receives the position of the tile's first pair.
// FUSED (whole-step entry point): the value also goes into the leader's row of the
// gather matrix and the leader's residual is cleared at the sent position.
// One wavefront per tile, four tiles (half a super-tile) per workgroup.  What stands before a tile in its layer:
// FOLD_STILES: the super-tile totals are as k_count left them and the workgroup adds up the layer's earlier ones itself;
// FOLD_TILES: the tiles' own counts are (k_stage_records), and it adds up those, which saves k_fold_counts, 5 us, on layers of
// up to FOLD_MAX_TILES tiles (thresholds and pairs of 25.6 M elements 119.1 -> 116.3 us, one layer of 1 M, pairs alone, 15 -> 9);
// FOLDED: k_scan has turned the super-tile totals into prefixes.
constexpr int FOLDED = 0, FOLD_STILES = 1, FOLD_TILES = 2;
constexpr uint32_t FOLD_MAX_TILES = 4096;          // 16 loads per thread at most
template <bool FUSED, int FOLD>
__global__ __launch_bounds__(BLOCK) void k_write(ResidualPtrs R, const float* __restrict__ w,
                                                 const DevLayer* __restrict__ layers, uint32_t n_layers, uint32_t tiles,
                                                 const uint32_t* __restrict__ leader, uint32_t W, float eps,
                                                 const LayerState* __restrict__ state,
                                                 const uint32_t* __restrict__ stage_cnt, StageArrays A,
                                                 const uint2* __restrict__ tile_counts,
                                                 const uint2* __restrict__ stile_counts,
                                                 uint32_t* __restrict__ tile_out,
                                                 uint32_t* __restrict__ idx_out, float* __restrict__ val_out,
                                                 float* __restrict__ gathered, uint64_t K) {
    __shared__ uint32_t red[2][BLOCK / WAVE];
    const uint32_t lane = threadIdx.x & (WAVE - 1), wave = wave_id();
    const uint32_t s = blockIdx.x / (GROUP / (BLOCK / WAVE));            // the workgroup's super-tile
    const uint32_t part = blockIdx.x % (GROUP / (BLOCK / WAVE));
    const uint32_t j = layer_of_stile(layers, n_layers, tiles, s);
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    const uint32_t ntiles = (L.n + TILE - 1) / TILE;
    const uint32_t lt = (s - L.stile_begin) * GROUP + part * (BLOCK / WAVE) + wave;
    if (lt - wave >= ntiles) return;                                      // uniform: nothing of this part exists
    uint2 sc;
    if (FOLD != FOLDED) {
        // elements above / tying in the layer's earlier super-tiles, or tiles: summed here, by everybody
        const uint2* counts = FOLD == FOLD_TILES ? tile_counts : stile_counts;
        const uint32_t begin = FOLD == FOLD_TILES ? L.tile_begin : L.stile_begin;
        const uint32_t end = FOLD == FOLD_TILES ? L.tile_begin + lt - wave : s;
        uint32_t g = 0, e = 0;
        for (uint32_t q = begin + threadIdx.x; q < end; q += BLOCK) {
            const uint2 c = counts[q];
            g += c.x;
            e += c.y;
        }
        g = wave_sum(g);
        e = wave_sum(e);
        if (lane == 0) { red[0][wave] = g; red[1][wave] = e; }
        __syncthreads();
        sc.x = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        sc.y = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    } else {
        sc = stile_counts[s];                                             // already scanned (k_scan)
    }
    if (lt >= ntiles) return;
    const uint32_t t = L.tile_begin + lt;
    const LayerState st = state[j];
    const uint32_t thr = st.thr, quota = st.n_eq_take;
    const uint32_t lead = leader_of(leader, j, W);
    float* rl = R.r[lead] + L.offset;
    uint2 tc = make_uint2(0u, 0u);                                        // before the tile, from where sc ends
    if (FOLD == FOLD_TILES) {
        const uint2 c = lane < wave ? tile_counts[t - wave + lane] : tc;
        tc = make_uint2(wave_sum(c.x), wave_sum(c.y));
    } else {
        tc = tile_counts[t];
    }
    const uint32_t Gt = sc.x + tc.x, Et = sc.y + tc.y;         // elements above / tying, before this tile
    uint32_t* io = idx_out + L.out_offset;
    float* vo = val_out + L.out_offset;
    float* go = FUSED ? gathered + (size_t)lead * K + L.out_offset : nullptr;
    if (lane == 0) tile_out[t] = Gt + min(Et, quota);
    const uint32_t cnt = staged_entries(stage_cnt[t]);
    SlotStart S;
    request_slot(A, L.slot_begin + (uint64_t)lt * L.slot_cap, cnt, S);
    write_tile<FUSED>(L, lt, cnt, thr, quota, st.shift, Gt, Et, rl, w + L.offset, eps, A, S, io, vo, go);
}

// ---------------------------------------------------------------------------
// Counts and pairs of tables with a layer of more than FOLD_SCAN_MAX_STILES super-tiles whose slots hold few entries (SPARSE_MAX_CAP,
// iwp_api.hip), with k_scan between them: one wavefront per super-tile, the counts and the first 64 entries of all its tiles requested together.  Nothing is shared between wavefronts.
// Bound by the chain row -> state and counts -> entries, of which the chip has some ten thousand at once, not by what is read: of a
// layer of 400 M elements kept at 1/1000 a tile's slot holds six entries, and with a workgroup per super-tile or half of one the counts
// took 25 us and the pairs 45, now 8 and 27 (20 of which the clears of scattered residuals take); the whole step 1440 -> 1392 with look 2's and
// k_refine2's part (each_key_of_64_tiles), 300 M kept at 1/300 1079 -> 1050, at 1/180 1173 -> 1162.
// ---------------------------------------------------------------------------
template <class Body>
__device__ __forceinline__ void each_bit(uint32_t bits, Body body) {
#pragma unroll 1
    for (; bits; bits &= bits - 1u) body((uint32_t)__ffs((int)bits) - 1u);
}

__global__ __launch_bounds__(BLOCK) void k_count_stiles(ResidualPtrs R, const float* __restrict__ w,
                                                        const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                        uint32_t tiles, uint32_t stiles, const uint32_t* __restrict__ leader,
                                                        uint32_t W, float eps, LayerState* __restrict__ state,
                                                        const uint32_t* __restrict__ hist, iwp_threshold* __restrict__ thr_out,
                                                        const uint32_t* __restrict__ stage_cnt, StageArrays A,
                                                        uint2* __restrict__ tile_counts, uint2* __restrict__ stile_counts) {
    const uint32_t lane = threadIdx.x & (WAVE - 1), s = blockIdx.x * (BLOCK / WAVE) + wave_id();
    if (s >= stiles) return;
    const uint32_t j = layer_of_stile(layers, n_layers, tiles, s);
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    const uint32_t lt0 = (s - L.stile_begin) * GROUP, nt = min(GROUP, (L.n + TILE - 1) / TILE - lt0);
    const uint64_t sb0 = L.slot_begin + (uint64_t)lt0 * L.slot_cap;
    const uint32_t my_cnt = lane < nt ? staged_entries(stage_cnt[L.tile_begin + lt0 + lane]) : 0u;
    uint32_t key[GROUP];
#pragma unroll
    for (uint32_t q = 0; q < GROUP; ++q) {
        const uint32_t cnt = from_lane(my_cnt, q);
        key[q] = lane < cnt ? A.key[sb0 + (uint64_t)q * L.slot_cap + lane] : NOT_AN_ELEMENT;   // RAW, UNIFORM: not used
    }
    uint32_t bin2, quota;
    wave_pick<(int)HIST2>(layer_hist(hist, L, 2), state[j].k_rem1, &bin2, &quota);
    const uint32_t thr = (state[j].p22 << digit_bits(2)) | bin2, shift = state[j].shift;
    if (s == L.stile_begin && lane == 0) {
        state[j].thr = thr;
        state[j].n_eq_take = quota;
        if (thr_out) {
            iwp_threshold th;
            th.key = unshifted(thr, shift); th.n_gt = L.k - quota; th.n_eq_take = quota;
            thr_out[j] = th;
        }
    }
    uint32_t gt = 0, eq = 0;                                 // lane q: of tile q
#pragma unroll
    for (uint32_t q = 0; q < GROUP; ++q) {
        const uint32_t g = (uint32_t)__popcll(__ballot((int32_t)key[q] > (int32_t)thr));         // NOT_AN_ELEMENT: negative
        const uint32_t e = (uint32_t)__popcll(__ballot(key[q] == thr));
        gt = lane == q ? g : gt;
        eq = lane == q ? e : eq;
    }
    each_bit((uint32_t)__ballot(my_cnt > WAVE), [&](uint32_t q) {
        const uint32_t cnt = from_lane(my_cnt, q), first = (lt0 + q) * TILE;
        const uint64_t sb = sb0 + (uint64_t)q * L.slot_cap;
        uint32_t g = 0, e = 0;
        if (cnt == UNIFORM_TILE) {                           // all keys of the tile are the slot's one entry
            const uint32_t k0 = A.key[sb], n_tile = min(TILE, L.n - first);
            if (lane == 0) { g = k0 > thr ? n_tile : 0u; e = k0 == thr ? n_tile : 0u; }
        } else if (cnt == RAW_TILE) {
            read_raw_tile(R.r[leader_of(leader, j, W)] + L.offset, w + L.offset, L.n, first, eps, shift, thr,
                          [&](uint32_t packed, const uint32_t (&)[4], const float (&)[4], uint32_t) {
                g += packed & 0xffffu;
                e += packed >> 16;
            });
        } else {
            for (uint32_t e0 = 0; e0 < cnt; e0 += 4 * WAVE) {
                uint32_t k2[4];
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) k2[c] = e0 + c * WAVE + lane < cnt ? A.key[sb + e0 + c * WAVE + lane] : NOT_AN_ELEMENT;
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) {
                    g += (int32_t)k2[c] > (int32_t)thr ? 1u : 0u;
                    e += k2[c] == thr ? 1u : 0u;
                }
            }
        }
        g = wave_sum(g);
        e = wave_sum(e);
        gt = lane == q ? g : gt;
        eq = lane == q ? e : eq;
    });
    const uint32_t g = wave_inclusive_scan(gt), e = wave_inclusive_scan(eq);
    if (lane < nt) tile_counts[L.tile_begin + lt0 + lane] = make_uint2(g - gt, e - eq);
    if (lane == WAVE - 1) stile_counts[s] = make_uint2(g, e);
}

template <bool FUSED>
__global__ __launch_bounds__(BLOCK) void k_write_stiles(ResidualPtrs R, const float* __restrict__ w,
                                                        const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                        uint32_t tiles, uint32_t stiles, const uint32_t* __restrict__ leader,
                                                        uint32_t W, float eps, const LayerState* __restrict__ state,
                                                        const uint32_t* __restrict__ stage_cnt, StageArrays A,
                                                        const uint2* __restrict__ tile_counts,
                                                        const uint2* __restrict__ stile_counts,
                                                        uint32_t* __restrict__ tile_out,
                                                        uint32_t* __restrict__ idx_out, float* __restrict__ val_out,
                                                        float* __restrict__ gathered, uint64_t K) {
    const uint32_t lane = threadIdx.x & (WAVE - 1), s = blockIdx.x * (BLOCK / WAVE) + wave_id();
    if (s >= stiles) return;
    const uint32_t j = layer_of_stile(layers, n_layers, tiles, s);
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    const uint32_t lt0 = (s - L.stile_begin) * GROUP, nt = min(GROUP, (L.n + TILE - 1) / TILE - lt0), t0 = L.tile_begin + lt0;
    const uint64_t sb0 = L.slot_begin + (uint64_t)lt0 * L.slot_cap;
    const uint32_t my_cnt = lane < nt ? staged_entries(stage_cnt[t0 + lane]) : 0u;
    uint2 before = lane < nt ? tile_counts[t0 + lane] : make_uint2(0u, 0u);
    const uint2 sc = stile_counts[s];                        // before the super-tile (k_scan)
    before.x += sc.x;
    before.y += sc.y;
    SlotPart<1> S[GROUP];
#pragma unroll
    for (uint32_t q = 0; q < GROUP; ++q) request_slot(A, sb0 + (uint64_t)(q < nt ? q : 0u) * L.slot_cap, from_lane(my_cnt, q), S[q]);
    const uint32_t thr = state[j].thr, quota = state[j].n_eq_take, shift = state[j].shift;
    if (lane < nt) tile_out[t0 + lane] = before.x + min(before.y, quota);
    const uint32_t lead = leader_of(leader, j, W);
    float* rl = R.r[lead] + L.offset;
    uint32_t* io = idx_out + L.out_offset;
    float* vo = val_out + L.out_offset;
    float* go = FUSED ? gathered + (size_t)lead * K + L.out_offset : nullptr;
#pragma unroll
    for (uint32_t q = 0; q < GROUP; ++q) {
        const uint32_t cnt = from_lane(my_cnt, q);
        if (cnt > WAVE) continue;                            // uniform
        uint32_t G = from_lane(before.x, q), E = from_lane(before.y, q);
        write_entries<FUSED>(L, S[q].key[0], S[q].idx[0], S[q].val[0], lane < cnt, thr, quota, G, E, rl, io, vo, go);
    }
    each_bit((uint32_t)__ballot(my_cnt > WAVE), [&](uint32_t q) {
        const uint32_t cnt = from_lane(my_cnt, q);
        SlotStart more;
        request_slot(A, sb0 + (uint64_t)q * L.slot_cap, cnt, more);
        write_tile<FUSED>(L, lt0 + q, cnt, thr, quota, shift, from_lane(before.x, q), from_lane(before.y, q), rl, w + L.offset, eps, A,
                          more, io, vo, go);
    });
}

// ---------------------------------------------------------------------------
// The ordered split where the units' records are there (see tie_record; plans whose slots hold few entries).  The threshold's last
// digit is picked by every wavefront, so k_count has no launch.  One wavefront per tile, a super-tile per workgroup.  What
// stands above the threshold or ties with it before the workgroup's tiles: SPLIT_TILES: added up from the records of the layer's earlier
// tiles, SPLIT_STILES: of its earlier super-tiles, inside the workgroup's from the slots themselves.
// Bound by its chain of dependent loads (row, counts and state, entries and histogram, records) and, where residuals are cleared,
// by those scattered stores.  us a call, k_count and k_write / this: one layer of 1 M elements 30.1 / 26.7, six tensors of 235 k, four
// workers 35.6 / 32.5, one worker's share of 25.6 M 146.6 / 144.9, 16 tensors of 61 M, eight workers 1142 / 1133; with kept
// eighths instead of 64ths one layer of 1 M 59 / 54.  RECORD_MAX_CAP and RECORD_MAX_STILES (iwp_api.hip) are its lines.
// ---------------------------------------------------------------------------
constexpr int SPLIT_TILES = 0, SPLIT_STILES = 1;
constexpr int SPLIT_BLOCK = GROUP * WAVE;

// A unit's elements above the threshold (low half) and tying with it, from its word c.  low: the threshold's last digit.  No branch:
// a unit without a record reads some word instead, so that a thread's loads do not wait for each other.
typedef uint32_t u32_pair __attribute__((aligned(2)));
__device__ __forceinline__ uint32_t unit_counts(uint32_t c, uint32_t unit, const uint32_t* hist, const uint32_t* records,
                                                const DevLayer& L, uint32_t low) {
    const uint32_t* record = tie_record(const_cast<uint32_t*>(hist), const_cast<uint32_t*>(records), L, unit);
    // with the last digit of all, the upper half comes from the word behind the record (the workspace goes on there)
    const uint32_t two = *reinterpret_cast<const u32_pair*>(reinterpret_cast<const uint16_t*>(c >> 16 ? record : hist) + low);
    const uint32_t more = low + 1 < HIST2 ? two >> 16 : 0u;
    return (c & 0xffffu) + (c >> 16 ? more + (((two & 0xffffu) - more) << 16) : 0u);
}

template <bool FUSED, int BEFORE>
__global__ __launch_bounds__(SPLIT_BLOCK) void k_split(ResidualPtrs R, const float* __restrict__ w,
                                                       const DevLayer* __restrict__ layers, uint32_t n_layers, uint32_t tiles,
                                                       const uint32_t* __restrict__ leader, uint32_t W, float eps,
                                                       const LayerState* __restrict__ state, const uint32_t* __restrict__ hist,
                                                       const uint32_t* __restrict__ units, const uint32_t* __restrict__ records,
                                                       const uint32_t* __restrict__ stage_cnt, StageArrays A,
                                                       iwp_threshold* __restrict__ thr_out, uint32_t* __restrict__ tile_out,
                                                       uint32_t* __restrict__ idx_out, float* __restrict__ val_out,
                                                       float* __restrict__ gathered, uint64_t K) {
    constexpr uint32_t WAVES = SPLIT_BLOCK / WAVE;
    __shared__ uint2 red[WAVES], own[WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = wave_id();
    const uint32_t s = blockIdx.x;
    const uint32_t j = layer_of_stile(layers, n_layers, tiles, s);
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    const uint32_t ntiles = (L.n + TILE - 1) / TILE;
    const uint32_t lt0 = (s - L.stile_begin) * GROUP, lt = lt0 + wave;
    const bool have = lt < ntiles;
    const uint32_t t = L.tile_begin + lt;
    const uint32_t cnt = have ? staged_entries(stage_cnt[t]) : 0u;
    const uint32_t first = BEFORE == SPLIT_TILES ? L.tile_begin : L.stile_begin;
    const uint32_t before = BEFORE == SPLIT_TILES ? lt0 : lt0 / GROUP;       // units
    const uint32_t first_unit = tid < before ? units[first + tid] : 0u;
    const uint64_t sb = L.slot_begin + (uint64_t)(have ? lt : lt0) * L.slot_cap;
    SlotStart S;
    request_slot(A, sb, cnt, S);
    uint32_t low, quota;
    wave_pick<(int)HIST2>(layer_hist(hist, L, 2), state[j].k_rem1, &low, &quota);
    const uint32_t thr = (state[j].p22 << digit_bits(2)) | low, shift = state[j].shift;
    if (lt0 == 0 && tid == 0 && thr_out) {
        iwp_threshold th;
        th.key = unshifted(thr, shift); th.n_gt = L.k - quota; th.n_eq_take = quota;
        thr_out[j] = th;
    }
    const uint32_t lead = leader_of(leader, j, W);
    float* rl = R.r[lead] + L.offset;
    const float* wl = w + L.offset;
    uint32_t g = 0, e = 0;
    for (uint32_t u = tid; u < before; u += SPLIT_BLOCK) {
        const uint32_t c = unit_counts(u == tid ? first_unit : units[first + u], u, hist, records, L, low);
        g += c & 0xffffu;
        e += c >> 16;
    }
    g = wave_sum(g);
    e = wave_sum(e);
    if (lane == 0) red[wave] = make_uint2(g, e);
    uint32_t gt = 0, eq = 0;                                // of this tile; SPLIT_TILES: of the super-tile's earlier ones
    if (BEFORE == SPLIT_TILES) {
        const uint32_t c = lane < wave && lt0 + lane < ntiles
                               ? unit_counts(units[L.tile_begin + lt0 + lane], lt0 + lane, hist, records, L, low) : 0u;
        gt = c & 0xffffu;
        eq = c >> 16;
    } else if (cnt == UNIFORM_TILE) {
        const uint32_t k0 = A.key[sb], n_tile = min(TILE, L.n - lt * TILE);
        if (lane == 0) { gt = k0 > thr ? n_tile : 0u; eq = k0 == thr ? n_tile : 0u; }
    } else if (cnt == RAW_TILE) {
        read_raw_tile(rl, wl, L.n, lt * TILE, eps, shift, thr,
                      [&](uint32_t packed, const uint32_t (&)[4], const float (&)[4], uint32_t) {
            gt += packed & 0xffffu;
            eq += packed >> 16;
        });
    } else {
        for (uint32_t q = 0; q < SPLIT_AHEAD; ++q) {
            const bool there = q * WAVE + lane < cnt;
            gt += there && S.key[q] > thr ? 1u : 0u;
            eq += there && S.key[q] == thr ? 1u : 0u;
        }
        for (uint32_t e0 = SPLIT_AHEAD * WAVE; e0 < cnt; e0 += 4 * WAVE) {
            uint32_t k2[4];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) k2[q] = e0 + q * WAVE + lane < cnt ? A.key[sb + e0 + q * WAVE + lane] : NOT_AN_ELEMENT;
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                gt += k2[q] != NOT_AN_ELEMENT && k2[q] > thr ? 1u : 0u;
                eq += k2[q] == thr ? 1u : 0u;               // a key is never NOT_AN_ELEMENT (bit 31 is clear)
            }
        }
    }
    gt = wave_sum(gt);
    eq = wave_sum(eq);
    if (lane == 0) own[wave] = make_uint2(gt, eq);
    __syncthreads();
    uint32_t Gt = 0, Et = 0;                                // before this tile
#pragma unroll
    for (uint32_t v = 0; v < WAVES; ++v) { Gt += red[v].x; Et += red[v].y; }
    if (BEFORE == SPLIT_TILES) {
        Gt += gt; Et += eq;
    } else {
#pragma unroll
        for (uint32_t v = 0; v < WAVES; ++v) { Gt += v < wave ? own[v].x : 0u; Et += v < wave ? own[v].y : 0u; }
    }
    if (!have) return;
    if (lane == 0) tile_out[t] = Gt + min(Et, quota);
    write_tile<FUSED>(L, lt, cnt, thr, quota, shift, Gt, Et, rl, wl, eps, A, S, idx_out + L.out_offset, val_out + L.out_offset,
                      FUSED ? gathered + (size_t)lead * K + L.out_offset : nullptr);
}

// The importance keys themselves, for tests of the device arithmetic.
__global__ __launch_bounds__(BLOCK) void k_score_keys(const float* __restrict__ w, const float* __restrict__ r,
                                                      uint32_t n, float eps, uint32_t* __restrict__ key_out) {
    const uint64_t stride = (uint64_t)gridDim.x * BLOCK;
    for (uint64_t i = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += stride) key_out[i] = score_key(r[i], w[i], eps);
}

// Plain 128-bit copy, one quad per lane: the practical HBM ceiling every result is
// quoted against, and the known-size reference that scales the profiler's byte
// counters.
__global__ __launch_bounds__(BLOCK) void k_copy(float* __restrict__ dst, const float* __restrict__ src, uint64_t n) {
    const uint64_t quads = n / 4;
    const uint64_t q = (uint64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (q < quads) reinterpret_cast<v4f*>(dst)[q] = reinterpret_cast<const v4f*>(src)[q];
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) dst[quads * 4 + threadIdx.x] = src[quads * 4 + threadIdx.x];
}

}  // namespace iwp
