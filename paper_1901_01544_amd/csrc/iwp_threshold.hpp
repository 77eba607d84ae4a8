// Threshold mode: the front end exactly as Algorithm 1 prints it.  Each of the
// n_lead randomly chosen nodes of a layer marks the elements whose importance is
// strictly above the layer's threshold (mask line; fixed thresholds, Section 4.1),
// the masks are encoded one bit per element (encode_uint8: bit i%8 of byte i/8,
// i.e. bit i%32 of little-endian word i/32; a layer's mask is a whole number of
// words) and OR-ed, and every node splits its accumulated gradient by the common
// mask (G~ / G lines).  The number of sent elements is data dependent, so the
// layers' pairs are packed by a scan over device-resident counts.
//
// One look per chosen node (16 B/element), no selection at all; the other nodes
// stream once and hand over / clear their masked values on the way, with the
// 4096-bit tile mask taken straight from the encoded mask.
#pragma once

#include "iwp_common.hpp"
#include "iwp_exchange.hpp"
#include "iwp_stream.hpp"

namespace iwp {

constexpr uint32_t MAX_LEAD = 8;                 // chosen nodes per layer

// The node in slot q of layer j (out-of-range entries read as node 0).
__device__ __forceinline__ uint32_t chosen_at(const uint32_t* __restrict__ leaders, uint32_t n_lead, uint32_t j,
                                              uint32_t q, uint32_t W) {
    const uint32_t l = leaders[(size_t)j * n_lead + q];
    return l < W ? l : 0u;
}

// Is node p among the first `upto` chosen nodes of layer j?
__device__ __forceinline__ bool chosen_before(const uint32_t* __restrict__ leaders, uint32_t n_lead, uint32_t j,
                                              uint32_t upto, uint32_t W, uint32_t p) {
    for (uint32_t q = 0; q < upto; ++q)
        if (chosen_at(leaders, n_lead, j, q, W) == p) return true;
    return false;
}

// Where k_leader_mask leaves the sent values of the chosen nodes, in index order: the tile's slot of the node in slot q of
// its layer is val[(q * tiles + tile) * cap, + cap).  A tile that sends more than cap elements leaves none.
struct ChosenSlots {
    float* val;
    uint32_t cap, tiles;
};

// Status words at the end of count_out: [n_layers] = total pairs, [n_layers + 1] = 1 if
// the total exceeds the caller's capacity (then nothing is exchanged).
__device__ __forceinline__ bool overflowed(const uint32_t* __restrict__ count_out, uint32_t n_layers) {
    return count_out[n_layers + 1] != 0u;
}

// Random gradient selection (Section 3.3): an element not above the threshold is still
// sent with probability importance / threshold.  The draw comes from Philox-4x32 with 10
// rounds (Salmon et al., SC'11): key = the caller's 64-bit seed, counter = (i / 4, layer,
// step low, step high); element i of the layer takes output word i % 4, and
// u = (word >> 8) * 2^-24.  It depends on (seed, step, layer, position) only, so every
// node, and any other implementation of the same generator, sees the same draw.
struct RandomSel {
    uint32_t on, key0, key1, step0, step1;
};

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t (&out)[4]) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// The layer-wise rule (Section 3.4, Eq. 4) from a layer's mean and population variance.
struct LayerRule {
    double alpha, beta, C;
    double2* stats_out;                                      // per layer and slot: (mean, variance)
    float* thr_out;                                          // ... and the threshold, rounded to binary32
    __device__ __forceinline__ float threshold(double mean, double var) const {
        const double ratio = var / mean;
        return (float)(ratio > C ? alpha + beta * ratio : alpha - beta * ratio);
    }
    __device__ __forceinline__ void write(size_t slot, double mean, double var) const {
        stats_out[slot] = make_double2(mean, var);
        thr_out[slot] = threshold(mean, var);
    }
};

// What the masks' launch needs to merge the tiles' statistics by itself (RULE: layers of up to RULE_MAX_TILES tiles, tables of up to
// RULE_MAX_TABLE over all slots): every wavefront does, one tile per lane, in k_layer_thr's order of additions, while its tile's loads are on their way.  That saves a launch of a few
// workgroups: one chosen node, 20 k elements 19.0 -> 16.8 us a step, 400 k 23.6 -> 21.0, 3 M in 300 layers 60.5 -> 58.5; two, 400 k
// 26.2 -> 24.3; four, 100 k 25.5 -> 24.0.  Three nodes of 3 M (880 tiles) lose, 74.8 -> 76.1: the registers that it takes.
constexpr uint32_t RULE_MAX_TILES = WAVE, RULE_MAX_TABLE = 1024;
struct TileStats {
    const double2* of;                                       // slot by slot, the table's tiles
    uint32_t tiles;
    LayerRule rule;
};
__device__ __forceinline__ double wave_sum_f64(double v) {   // in all lanes
#pragma unroll
    for (int d = WAVE / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, WAVE);
    return v;
}
__device__ __forceinline__ double2 merged_by_wave(const DevLayer& L, const double2* ts) {
    const uint32_t lane = threadIdx.x & (WAVE - 1), ntiles = (L.n + TILE - 1) / TILE;
    const bool have = lane < ntiles;
    const double2 v = have ? ts[lane] : make_double2(0.0, 0.0);
    const double n = (double)L.n, mean = wave_sum_f64(v.x) / n;
    const double nt = (double)(have ? min(TILE, L.n - lane * TILE) : 1u), d = v.x / nt - mean;
    return make_double2(mean, wave_sum_f64(have ? v.y + nt * (d * d) : 0.0) / n);
}

// The lane's elements whose score is above a threshold -> bits of nib.  The score is |r| / d, d = |w| + eps, rounded.  No divide where the
// answer does not hang on the rounding: f = t * d - |r|, rounded once, has the sign of the exact value.  f > 0: |r| / d < t, and rounded it
// is at most t.  f + |r| / 2^21 < 0: |r| / d exceeds t by more than a unit in t's last place, and rounded it does, too; this takes a t
// well above the subnormal numbers (SHORT_MIN) and finite.  Where a lane has neither (a NaN, an infinity, a score within 2^-21 of t),
// its wavefront divides.  Two fused multiply-adds and two compares for a divide's dozen instructions, which count where a table is small:
// steps with thresholds, one chosen node 20 k elements 15.5 -> 15.0 us, 400 k 18.7 -> 18.1, two nodes 20 k 19.0 -> 17.9, 1 M 28.5 -> 27.2,
// three nodes 400 k 21.4 -> 20.0, 10 M 110.0 -> 108.4; one node of 10 M or more is bound by memory either way.  With random selection
// the score itself is needed.
constexpr float SHORT_MIN = 0x1p-100f, SHORT_MAX = 0x1p127f;
template <uint32_t CHUNKS>
__device__ __forceinline__ void add_above(const float (&rv)[CHUNKS][4], const float (&wv)[CHUNKS][4], float eps, float t,
                                          uint32_t (&nib)[CHUNKS]) {
    uint32_t mine[CHUNKS] = {};
    bool open = !(t >= SHORT_MIN && t <= SHORT_MAX);
    if (!open) {                                             // uniform
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
            for (uint32_t c = 0; c < VEC; ++c) {
                const float a = fabsf(rv[u][c]), d = fabsf(wv[u][c]) + eps;
                const float f = __builtin_fmaf(t, d, -a);
                const bool above = __builtin_fmaf(a, 0x1p-21f, f) < 0.0f;
                mine[u] |= above ? 1u << c : 0u;
                open = open || !(above || f > 0.0f);
            }
    }
    if (__any(open)) {
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) {
            mine[u] = 0u;
#pragma unroll
            for (uint32_t c = 0; c < VEC; ++c) mine[u] |= fabsf(rv[u][c]) / (fabsf(wv[u][c]) + eps) > t ? 1u << c : 0u;
        }
    }
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) nib[u] |= mine[u];
}

// The tile that starts at element `base` of its layer, CHUNKS chunks of it, for all chosen nodes of the layer: accumulate,
// score, compare, encode, and hand over what is sent.  Layers that end within a tile's first chunk take one chunk only, which
// spares them three quarters of the divides (and draws).  The nodes' values stay in registers until the common mask is known:
// NL nodes per group of THREADS threads (threadIdx.y), the groups' masks meet in LDS (meet, BLOCK words each; one group has none).
template <uint32_t CHUNKS, int NL, int GROUPS, bool RULE, uint32_t THREADS>
__device__ __forceinline__ void mask_tile(const WorkerPtrs& P, const float* __restrict__ wl, const DevLayer& L, uint32_t j,
                                          uint32_t t, uint32_t base, const uint32_t* __restrict__ leaders, uint32_t n_lead,
                                          uint32_t W, const float* __restrict__ thr, bool thr_per_slot, bool accumulate,
                                          const TileStats& stats, const RandomSel& rs, float eps, uint32_t* __restrict__ mw,
                                          uint32_t* __restrict__ tile_counts, const ChosenSlots& S, uint32_t* part,
                                          uint32_t (*meet)[BLOCK]) {
    constexpr uint32_t SPAN = THREADS * VEC;                 // elements of a chunk
    static_assert(GROUPS == 1 || THREADS == BLOCK, "groups are of BLOCK threads");
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1);
    const uint32_t group = GROUPS > 1 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.y) : 0u;   // the same in a wavefront
    const uint32_t q0 = group * NL;
    const uint32_t n = L.n, nwords = (n + 31) / 32;
    float wv[CHUNKS][4], rv[NL][CHUNKS][4], gv[NL][CHUNKS][4];
    Rest wv_rest, rv_rest[NL], gv_rest[NL];
    float* rl[NL];
    const float* gl[NL];
    float th[NL] = {};
    bool on[NL];
    uint32_t nib[CHUNKS] = {};
    request_tile<true, THREADS>(wl, n, base, wv, wv_rest);
    auto request = [&](int s, uint32_t q, bool there) {      // node in slot q of the layer -> registers s
        const uint32_t p = chosen_at(leaders, n_lead, j, q, W);
        on[s] = there && !chosen_before(leaders, n_lead, j, q, W, p);
        if (!RULE) th[s] = thr_per_slot ? thr[(size_t)j * n_lead + q] : thr[j];
        rl[s] = P.r[p] + L.offset;
        gl[s] = accumulate && P.g[p] ? P.g[p] + L.offset : nullptr;
        if (!on[s]) return;
        request_tile<true, THREADS>(rl[s], n, base, rv[s], rv_rest[s]);
        if (gl[s]) request_tile<true, THREADS>(gl[s], n, base, gv[s], gv_rest[s]);
    };
    auto settle = [&](int s) {
        if (!on[s]) return;
        settle_tile<THREADS>(n, base, rv[s], rv_rest[s]);
        if (!gl[s]) return;
        settle_tile<THREADS>(n, base, gv[s], gv_rest[s]);
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) rv[s][u][c] = accum(rv[s][u][c], gv[s][u][c], P.momentum);
    };
    // one group: exactly NL nodes, their slots constants
#pragma unroll
    for (int s = 0; s < NL; ++s) request(s, GROUPS > 1 ? min(q0 + s, n_lead - 1u) : (uint32_t)s, GROUPS == 1 || q0 + s < n_lead);
    if (RULE) {                                              // the loads are on their way
#pragma unroll 1
        for (uint32_t s = 0; s < NL && q0 + s < n_lead; ++s) {
            const uint32_t p = chosen_at(leaders, n_lead, j, q0 + s, W);
            uint32_t first = 0;                              // a slot that repeats an earlier node takes that node's tiles
            while (chosen_at(leaders, n_lead, j, first, W) != p) ++first;
            const double2 v = merged_by_wave(L, stats.of + (size_t)first * stats.tiles + L.tile_begin);
            const float t0 = stats.rule.threshold(v.x, v.y);
#pragma unroll
            for (uint32_t x = 0; x < NL; ++x) th[x] = x == s ? t0 : th[x];
            if (base == 0 && tid == 0) stats.rule.write((size_t)j * n_lead + q0 + s, v.x, v.y);
        }
    }
    settle_tile<THREADS>(n, base, wv, wv_rest);
#pragma unroll
    for (int s = 0; s < NL; ++s) settle(s);
    const bool ragged = base + CHUNKS * SPAN > n;           // uniform
    if (ragged) {                                            // behind the layer's end: a score that is far from a threshold
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
            for (uint32_t c = 0; c < VEC; ++c) {
                const bool behind = base + u * SPAN + tid * VEC + c >= n;
                wv[u][c] = behind ? 1.0f : wv[u][c];
#pragma unroll
                for (int s = 0; s < NL; ++s) rv[s][u][c] = behind ? 0.0f : rv[s][u][c];
            }
    }
    if (!RULE && rs.on) {
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) {
            const uint32_t i = base + u * SPAN + tid * VEC;
            uint32_t word4[4];
            philox4x32_10(i >> 2, j, rs.step0, rs.step1, rs.key0, rs.key1, word4);   // i is a multiple of 4
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                if (!on[s]) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float score = fabsf(rv[s][u][c]) / (fabsf(wv[u][c]) + eps);
                    const float draw = (float)(word4[c] >> 8) * 0x1p-24f;
                    const float prob = score / th[s];
                    if (score > th[s] || draw < prob) nib[u] |= 1u << c;
                }
            }
        }
    } else {                                                 // the elements that one of the nodes in registers sends
#pragma unroll
        for (int s = 0; s < NL; ++s)
            if (on[s]) add_above<CHUNKS>(rv[s], wv, eps, th[s], nib);
    }
    if (ragged) {
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) {
            const uint32_t i = base + u * SPAN + tid * VEC;
            nib[u] &= i < n ? 0xFu >> (VEC - min(n - i, (uint32_t)VEC)) : 0u;
        }
    }
    if (GROUPS > 1) {
        uint32_t bits = 0;
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) bits |= nib[u] << (4u * u);
        meet[group][tid] = bits;
        __syncthreads();
        bits = 0;
#pragma unroll
        for (int y = 0; y < GROUPS; ++y) bits |= meet[y][tid];
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) nib[u] = (bits >> (4u * u)) & 0xFu;
    }
    uint32_t count[CHUNKS], first[CHUNKS], word[CHUNKS];
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        // eight lanes (32 consecutive elements) make one word of the encoded mask
        word[u] = or_of_8_lanes(nib[u] << (4u * (lane & 7u)));
        const uint32_t widx = base / 32 + u * (SPAN / 32) + (tid >> 3);
        if (group == 0 && (lane & 7u) == 0u && widx < nwords) mw[widx] = word[u];
        count[u] = __popc(nib[u]);
    }
    const uint32_t total = tile_ranks<THREADS>(count, first, part + group * STAGE_WORDS);
    if (group == 0 && tid == 0) tile_counts[t] = total;
    const bool hand_over = total <= S.cap;                   // otherwise the next pass fetches and clears them
#pragma unroll
    for (int s = 0; s < NL; ++s) {
        if (!on[s]) continue;
        float* slot = S.val + ((size_t)(q0 + s) * S.tiles + t) * S.cap;
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) {
            if (!hand_over || !nib[u]) continue;
            uint32_t rank = first[u];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if ((nib[u] >> c) & 1u) { slot[rank++] = rv[s][u][c]; rv[s][u][c] = 0.0f; }
        }
        // a node that has not been accumulated here: only what holds a sent element, in whole lines of 32 elements
        // (single elements, partial lines, take 63 us instead of 49 where one of 59 of 25.6 M elements is sent)
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
            if (gl[s] || (hand_over && word[u])) store_quad<true>(rl[s], base + u * SPAN + tid * VEC, n, rv[s][u]);
    }
}

// ---------------------------------------------------------------------------
// Chosen nodes, one workgroup per tile for all of them: accumulate (if asked), score, compare, encode the OR of their masks
// (an output), count its bits, and split the nodes' residuals by it: the sent values go into a slot of the tile and +0 is
// left behind, as long as the slot holds them (S.cap; the packed position is only known once all tiles are counted).  If the
// total then exceeds the caller's capacity, k_follow_mask puts them back.
// thr: one value per layer, or per (layer, slot) with thr_per_slot.
// Bound by memory (two nodes, 61 M elements: 1.71 GB in 270 us, 6.3 TB/s).  A workgroup per node and tile read the weights
// once per node and left a mask for each, to be OR-ed and counted in a launch of its own (308 + 9 us), and the nodes' sent
// values were read and cleared pair by pair behind everything else (the update 177 us, now 66).  Whole steps: that table
// 1208 -> 1077 us, one node of 25.6 M elements with a line per layer 554 -> 522, three of 1.1 M 38 -> 29 (three launches less).
// Up to three nodes are one group's (59, 96 and 133 registers of 256 threads; 36, 56 and 78 of 512 on small tables, see WIDE_BLOCK in
// iwp_api.hip); more are taken two to a group, by workgroups of two to four
// groups, which read the weights once each.  One group that takes them one after the other, storing each and fetching
// its sent values again, had every node's loads wait for the one before: eight workers, four and eight nodes, us a step, against
// that (and against a workgroup per node and tile): 30 k elements 35 / 24 (31) and 47 / 27 (35), 1.2 M 69 / 43 (60) and 88 / 49
// (70), 61 M 1374 / 1064 (1327) and 1618 / 1268 (1571).
// ---------------------------------------------------------------------------
template <int NL, int GROUPS, bool RULE, uint32_t THREADS>
__global__ __launch_bounds__(THREADS * GROUPS) void k_leader_mask(WorkerPtrs P, const float* __restrict__ w,
                                                       const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                       const uint32_t* __restrict__ leaders, uint32_t n_lead, uint32_t W,
                                                       const float* __restrict__ thr, bool thr_per_slot, bool accumulate,
                                                       TileStats stats, RandomSel rs, float eps, uint32_t* __restrict__ mask_out,
                                                       uint32_t* __restrict__ tile_counts, ChosenSlots S) {
    __shared__ uint32_t part[GROUPS * STAGE_WORDS];
    __shared__ uint32_t meet[GROUPS > 1 ? GROUPS : 1][BLOCK];
    const uint32_t t = blockIdx.x;
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    const uint32_t base = (t - L.tile_begin) * TILE;
    const float* wl = w + L.offset;
    uint32_t* mw = mask_out + L.mask_begin;
    if (L.n - base <= THREADS * VEC)
        mask_tile<1, NL, GROUPS, RULE, THREADS>(P, wl, L, j, t, base, leaders, n_lead, W, thr, thr_per_slot, accumulate, stats, rs, eps, mw,
                                 tile_counts, S, part, meet);
    else
        mask_tile<TILE / (THREADS * VEC), NL, GROUPS, RULE, THREADS>(P, wl, L, j, t, base, leaders, n_lead, W, thr, thr_per_slot, accumulate, stats, rs, eps,
                                               mw, tile_counts, S, part, meet);
    if (RULE && threadIdx.y == 0)                            // layers without elements have no tile
        for (uint32_t l = t * THREADS + threadIdx.x; l < n_layers; l += gridDim.x * THREADS)
            if (layers[l].n == 0)
                for (uint32_t q = 0; q < n_lead; ++q) stats.rule.write((size_t)l * n_lead + q, 0.0, 0.0);
}

// One tile of a chosen node in registers: residual (after adding the gradient and storing
// it back when gp is set) and weights, 16 values per lane; positions past the layer's end hold
// values that are not meant for use.
__device__ __forceinline__ void chosen_tile(const float* gp, float* rl, const float* gl, const float* wl, float m,
                                            uint32_t n, uint32_t base, float (&rv)[CHUNKS_PER_TILE][4],
                                            float (&wv)[CHUNKS_PER_TILE][4]) {
    float gv[CHUNKS_PER_TILE][4];
    Rest rv_rest, gv_rest, wv_rest;
    request_tile<true>(rl, n, base, rv, rv_rest);
    if (gp) request_tile<true>(gl, n, base, gv, gv_rest);
    request_tile<true>(wl, n, base, wv, wv_rest);
    settle_tile(n, base, rv, rv_rest);
    settle_tile(n, base, wv, wv_rest);
    if (gp) {
        settle_tile(n, base, gv, gv_rest);
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS_PER_TILE; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) rv[u][c] = accum(rv[u][c], gv[u][c], m);
        store_tile<true>(rl, n, base, rv);
    }
}

// ---------------------------------------------------------------------------
// Layer-wise threshold, part 1 (Section 3.4, Eq. 4): the chosen nodes accumulate and
// score, and every tile leaves the sum of its importance values and the sum of their
// squared deviations from the tile's own mean, both binary64.  Grid: n_lead * tiles.
// tile_stats[q * tiles + t] = (sum, squared deviations).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double block_sum_f64(double v, double* slot) {
#pragma unroll
    for (int d = WAVE / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, WAVE);
    __syncthreads();                             // slot may still be read from an earlier call
    if ((threadIdx.x & (WAVE - 1)) == 0) slot[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((slot[0] + slot[1]) + slot[2]) + slot[3];
}

__global__ __launch_bounds__(BLOCK) void k_leader_stats(WorkerPtrs P, const float* __restrict__ w,
                                                        const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                        uint32_t tiles, const uint32_t* __restrict__ leaders,
                                                        uint32_t n_lead, uint32_t W, float eps,
                                                        double2* __restrict__ tile_stats) {
    __shared__ double slot[BLOCK / WAVE];
    const uint32_t tid = threadIdx.x;
    const uint32_t q = blockIdx.x / tiles;
    const uint32_t t = blockIdx.x - q * tiles;
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    const uint32_t p = chosen_at(leaders, n_lead, j, q, W);
    if (chosen_before(leaders, n_lead, j, q, W, p)) return;
    const uint32_t base = (t - L.tile_begin) * TILE;
    const float* gp = P.g[p];
    float rv[CHUNKS_PER_TILE][4], wv[CHUNKS_PER_TILE][4];
    chosen_tile(gp, P.r[p] + L.offset, gp ? gp + L.offset : nullptr, w + L.offset, P.momentum, L.n, base, rv, wv);
    float sc[CHUNKS_PER_TILE][4];
    double lane_sum = 0.0;
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS_PER_TILE; ++u) {
        const uint32_t i = base + u * CHUNK + tid * VEC;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            sc[u][c] = fabsf(rv[u][c]) / (fabsf(wv[u][c]) + eps);
            if (i + c < L.n) lane_sum += (double)sc[u][c];
        }
    }
    const double sum = block_sum_f64(lane_sum, slot);
    const double mean = sum / (double)min(TILE, L.n - base);
    double lane_m2 = 0.0;
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS_PER_TILE; ++u) {
        const uint32_t i = base + u * CHUNK + tid * VEC;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double d = (double)sc[u][c] - mean;
            if (i + c < L.n) lane_m2 += d * d;
        }
    }
    const double m2 = block_sum_f64(lane_m2, slot);
    if (tid == 0) tile_stats[(size_t)q * tiles + t] = make_double2(sum, m2);
}

// ---------------------------------------------------------------------------
// Layer-wise threshold, part 2: one workgroup per (layer, slot) merges the tiles
// (sum of squared deviations about the layer mean = sum over tiles of the tile's own
// plus n_t * (tile mean - layer mean)^2), then applies the rule:
// ratio = var / mean; thr = alpha + beta * ratio if ratio > C, else alpha - beta * ratio.
// stats_out[slot] = (mean, population variance), thr_out[slot] = thr rounded to binary32.
// A slot repeating an earlier node of the layer takes that node's tiles.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_layer_thr(const DevLayer* __restrict__ layers, uint32_t tiles,
                                                     const uint32_t* __restrict__ leaders, uint32_t n_lead, uint32_t W,
                                                     const double2* __restrict__ tile_stats, LayerRule rule) {
    __shared__ double slot[BLOCK / WAVE];
    const uint32_t j = blockIdx.x / n_lead;
    const uint32_t q = blockIdx.x - j * n_lead;
    const DevLayer L = layers[j];
    const uint32_t p = chosen_at(leaders, n_lead, j, q, W);
    uint32_t q0 = 0;
    while (chosen_at(leaders, n_lead, j, q0, W) != p) ++q0;      // ends at q at the latest
    const uint32_t ntiles = (L.n + TILE - 1) / TILE;
    const double2* ts = tile_stats + (size_t)q0 * tiles + L.tile_begin;
    double part = 0.0;
    for (uint32_t t = threadIdx.x; t < ntiles; t += BLOCK) part += ts[t].x;
    const double n = (double)L.n;
    const double mean = L.n ? block_sum_f64(part, slot) / n : 0.0;
    part = 0.0;
    for (uint32_t t = threadIdx.x; t < ntiles; t += BLOCK) {
        const double nt = (double)min(TILE, L.n - t * TILE);
        const double d = ts[t].x / nt - mean;
        part += ts[t].y + nt * (d * d);
    }
    const double var = L.n ? block_sum_f64(part, slot) / n : 0.0;
    if (threadIdx.x == 0) rule.write(blockIdx.x, mean, var);
}

// ---------------------------------------------------------------------------
// The tiles' counts -> where each tile's pairs start in the packed outputs (layers in table order), where each layer's do
// (lay_out[j], lay_out[n_layers] = total), the counts the caller sees, and the capacity check.  One workgroup, four quads of
// tiles per lane and round (tables of more than ADD_UP_TILES tiles; on others the workgroups of the next launch add up): a chain of one load, a scan and a store per 16384 tiles (5.3 us; sixteen dwords per lane, not
// coalesced, 15.5).  Both arrays hold whole 256-byte blocks.
// ---------------------------------------------------------------------------
constexpr int OFFSETS_BLOCK = 1024;
__global__ __launch_bounds__(OFFSETS_BLOCK) void k_tile_offsets(const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                                uint32_t tiles, const uint32_t* __restrict__ tile_counts,
                                                                uint32_t max_pairs, uint32_t* tile_pos,
                                                                uint32_t* __restrict__ lay_out,
                                                                uint32_t* __restrict__ count_out) {
    constexpr uint32_t PER = 4, STEP = OFFSETS_BLOCK * 4, WAVES = OFFSETS_BLOCK / WAVE;
    __shared__ uint32_t wave_sum[2][PER][WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    uint32_t total = 0;
    for (uint32_t b = 0, round = 0; b < tiles; b += STEP * PER, ++round) {
        uint4 v[PER];
        uint32_t sum[PER], inc[PER];
#pragma unroll
        for (uint32_t x = 0; x < PER; ++x) {
            const uint32_t t0 = b + x * STEP + tid * 4;
            v[x] = t0 < tiles ? *reinterpret_cast<const uint4*>(tile_counts + t0) : make_uint4(0u, 0u, 0u, 0u);
            if (t0 + 1 >= tiles) v[x].y = 0u;                // what lies behind the last tile's count
            if (t0 + 2 >= tiles) v[x].z = 0u;
            if (t0 + 3 >= tiles) v[x].w = 0u;
        }
        auto& ws = wave_sum[round & 1u];                     // the round before may still be reading the other
#pragma unroll
        for (uint32_t x = 0; x < PER; ++x) {
            sum[x] = v[x].x + v[x].y + v[x].z + v[x].w;
            inc[x] = wave_inclusive_scan(sum[x]);
            if (lane == WAVE - 1) ws[x][wave] = inc[x];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t x = 0; x < PER; ++x) {
            uint32_t pos = total + inc[x] - sum[x];
#pragma unroll
            for (uint32_t y = 0; y < WAVES; ++y) {
                pos += y < wave ? ws[x][y] : 0u;
                total += ws[x][y];
            }
            const uint32_t t0 = b + x * STEP + tid * 4;
            if (t0 < tiles)
                *reinterpret_cast<uint4*>(tile_pos + t0) =
                    make_uint4(pos, pos + v[x].x, pos + v[x].x + v[x].y, pos + v[x].x + v[x].y + v[x].z);
        }
    }
    __syncthreads();                                         // tile_pos is complete
    for (uint32_t j = tid; j < n_layers; j += OFFSETS_BLOCK) {
        const uint32_t f = layers[j].tile_begin, e = layers[j + 1].tile_begin;   // the sentinel row's is `tiles`
        const uint32_t first = f < tiles ? tile_pos[f] : total, end = e < tiles ? tile_pos[e] : total;
        lay_out[j] = first;
        count_out[j] = end - first;
    }
    if (tid == 0) {
        lay_out[n_layers] = total;
        count_out[n_layers] = total;
        count_out[n_layers + 1] = total > max_pairs ? 1u : 0u;
    }
}

// ---------------------------------------------------------------------------
// Every node that is not chosen for the layer and has a gradient: accumulate, and
// where the tile's mask has bits, copy the accumulated value into the node's gather
// row and leave +0 behind.  Grid: W * tiles; runs: see in_runs().  The workgroups of the chosen nodes, whose
// residuals k_leader_mask has been through, have nothing to accumulate: those of the first one write the
// tile's masked positions as ascending flat indices and move the sent values of all of them from the tile's
// slots to their gather rows.  A tile that sends more than a slot holds they stream, each its own: everything sent, eight workers,
// 6 M elements, one, two and four chosen nodes 247, 256 and 270 us a step (by the first one's workgroup, element by element for
// all of them, 344, 459 and 653); about half sent 181, 206 and 233 (215, 312, 506).
// ---------------------------------------------------------------------------
// The tile's mask in LDS (no bits unless wanted) and the number of bits before each word.
// map, pre, slot: LDS of TILE_WORDS, TILE_WORDS and 4 words.
__device__ __forceinline__ void tile_mask(const uint32_t* __restrict__ mask, const DevLayer& L, uint32_t base, bool wanted,
                                          uint32_t* map, uint32_t* pre, uint32_t* slot) {
    const uint32_t tid = threadIdx.x, nwords = (L.n + 31) / 32;
    if (tid < TILE_WORDS) {
        const uint32_t widx = base / 32 + tid;
        map[tid] = (wanted && widx < nwords) ? mask[L.mask_begin + widx] : 0u;
    }
    __syncthreads();
    bitmap_prefix(map, pre, slot);
}

// ADD_UP: on tables of up to ADD_UP_TILES tiles every workgroup adds the tiles' counts up itself, four per thread, and the first ones write
// what k_tile_offsets would have, which then has no launch: steps with thresholds, two workers, 1.5 M elements 22.3 -> 19.9 us, four, 4 M
// 49.4 -> 47.0, nine, 4 M 91.8 -> 89.2, with statistics 1.5 M 41.9 -> 39.2.
constexpr uint32_t ADD_UP_TILES = 4 * BLOCK;
template <bool ADD_UP>
__global__ __launch_bounds__(BLOCK) void k_follow_mask(WorkerPtrs P, const DevLayer* __restrict__ layers,
                                                       uint32_t n_layers, uint32_t tiles, uint32_t runs,
                                                       const uint32_t* __restrict__ leaders, uint32_t n_lead, uint32_t W,
                                                       const uint32_t* __restrict__ mask,
                                                       const uint32_t* __restrict__ tile_counts,
                                                       const uint32_t* __restrict__ tile_pos, uint32_t* lay_out, uint32_t* count_out,
                                                       uint32_t max_pairs, ChosenSlots S, uint32_t* __restrict__ idx_out,
                                                       float* __restrict__ gathered) {
    __shared__ uint32_t map[TILE_WORDS], pre[TILE_WORDS], slot[4];
    __shared__ alignas(16) uint32_t own_pos[ADD_UP ? ADD_UP_TILES : 1];
    const uint32_t tid = threadIdx.x;
    uint32_t total = 0;
    if (ADD_UP) {
        uint4 v = 4 * tid < tiles ? reinterpret_cast<const uint4*>(tile_counts)[tid] : make_uint4(0u, 0u, 0u, 0u);
        if (4 * tid + 1 >= tiles) v.y = 0u;                  // what lies behind the last tile's count
        if (4 * tid + 2 >= tiles) v.z = 0u;
        if (4 * tid + 3 >= tiles) v.w = 0u;
        const uint32_t pos = block_exclusive_scan(v.x + v.y + v.z + v.w, slot, &total);
        reinterpret_cast<uint4*>(own_pos)[tid] = make_uint4(pos, pos + v.x, pos + v.x + v.y, pos + v.x + v.y + v.z);
        __syncthreads();
        for (uint32_t l = blockIdx.x * BLOCK + tid; l < n_layers; l += gridDim.x * BLOCK) {
            const uint32_t f = layers[l].tile_begin, e = layers[l + 1].tile_begin;   // the sentinel row's is `tiles`
            const uint32_t first = f < tiles ? own_pos[f] : total;
            lay_out[l] = first;
            count_out[l] = (e < tiles ? own_pos[e] : total) - first;
        }
        if (blockIdx.x == 0 && tid == 0) {
            lay_out[n_layers] = total;
            count_out[n_layers] = total;
            count_out[n_layers + 1] = total > max_pairs ? 1u : 0u;
        }
    }
    const uint32_t b = runs ? in_runs(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t p = b / tiles;
    const uint32_t t = b - p * tiles;
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    const uint32_t base = (t - L.tile_begin) * TILE;
    const float* gp = P.g[p];
    uint32_t q = 0;
    while (q < n_lead && chosen_at(leaders, n_lead, j, q, W) != p) ++q;
    if (q == n_lead && !gp) return;                          // a node without a gradient: pair by pair later
    const uint32_t at = min(ADD_UP ? own_pos[t] : tile_pos[t], max_pairs), room = max_pairs - at;
    const bool exchange = ADD_UP ? total <= max_pairs : !overflowed(count_out, n_layers);
    float* row = gathered + (size_t)p * max_pairs + at;
    auto sent = [&]() {
        tile_mask(mask, L, base, exchange, map, pre, slot);
        return true;
    };
    if (q == n_lead) {
        float* rl = P.r[p] + L.offset;
        const float* gl = gp + L.offset;
        const uint32_t head = elements_to_line(rl);
        if (L.n - base <= CHUNK) follow_tile<1>(gl, rl, L.n, base, P.momentum, row, room, map, pre, sent);   // see mask_tile
        else if (head && base + TILE <= L.n) follow_tile_from(head, gl + base, rl + base, P.momentum, row, room, map, pre, sent);
        else follow_tile<CHUNKS_PER_TILE>(gl, rl, L.n, base, P.momentum, row, room, map, pre, sent);
        return;
    }
    // the chosen nodes' part of the tile
    const uint32_t cnt = tile_counts[t];
    const bool handed_over = cnt <= S.cap;
    uint32_t mine, first;                                    // the lane's 16 elements: which are sent, how many before them
    if (!handed_over) {
        if (!exchange) return;
        follow_tile<CHUNKS_PER_TILE, false>(nullptr, P.r[p] + L.offset, L.n, base, 1.0f, row, room, map, pre, sent);
        if (q > 0) return;
        mine = (map[tid >> 1] >> (16u * (tid & 1u))) & 0xffffu;
        first = bitmap_rank(map, pre, 16u * tid);
    } else {
        if (q > 0 || cnt == 0u) return;
        const uint32_t widx = base / 32 + (tid >> 1);
        mine = widx < (L.n + 31) / 32 ? (mask[L.mask_begin + widx] >> (16u * (tid & 1u))) & 0xffffu : 0u;
        uint32_t all;
        first = block_exclusive_scan(__popc(mine), slot, &all);
    }
    if (exchange) {
        uint32_t rank = first;
        for (uint32_t b = mine; b && rank < room; b &= b - 1u, ++rank)
            idx_out[at + rank] = (uint32_t)L.offset + base + 16u * tid + (uint32_t)__ffs(b) - 1u;
    }
    if (!handed_over) return;
    for (q = 0; q < n_lead; ++q) {
        const uint32_t c = chosen_at(leaders, n_lead, j, q, W);
        if (chosen_before(leaders, n_lead, j, q, W, c)) continue;
        const float* val = S.val + ((size_t)q * S.tiles + t) * S.cap;
        if (exchange) {
            for (uint32_t e = tid; e < min(cnt, room); e += BLOCK) gathered[(size_t)c * max_pairs + at + e] = val[e];
        } else {                                             // put back
            float* rl = P.r[c] + L.offset;
            uint32_t rank = first;
            for (uint32_t b = mine; b; b &= b - 1u, ++rank) rl[base + 16u * tid + (uint32_t)__ffs(b) - 1u] = val[rank];
        }
    }
}

// ---------------------------------------------------------------------------
// Ordered sum over the W nodes and the weight update, for a pair count that lives
// on the device.  Every node has left its value in its gather row (k_follow_mask), except those without a gradient (bits of
// static_mask) in layers that they are not chosen for: these are read and cleared here, pair by pair.  Fixed grid, strided
// over the pairs.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_reduce_update_counted(ResidualPtrs R, uint32_t static_mask, uint32_t n_layers,
                                                                 const uint32_t* __restrict__ leaders, uint32_t n_lead,
                                                                 uint32_t W, const uint32_t* __restrict__ lay_out,
                                                                 const uint32_t* __restrict__ count_out,
                                                                 uint32_t max_pairs, const float* __restrict__ gathered,
                                                                 const uint32_t* __restrict__ idx,
                                                                 float* __restrict__ w, float scale,
                                                                 float* __restrict__ sum_out, uint64_t flat_end) {
    if (overflowed(count_out, n_layers)) return;
    const uint32_t total = min(count_out[n_layers], max_pairs);
    for (uint64_t jj64 = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; jj64 < total; jj64 += (uint64_t)gridDim.x * BLOCK) {
        const uint32_t jj = (uint32_t)jj64;
        uint32_t direct = static_mask;
        if (static_mask) {
            uint32_t lo = 0, hi = n_layers;          // layer of pair jj: last layer with lay_out <= jj
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (lay_out[mid] <= jj) lo = mid; else hi = mid;
            }
            for (uint32_t q = 0; q < n_lead; ++q) direct &= ~(1u << chosen_at(leaders, n_lead, lo, q, W));
        }
        const uint32_t i = idx[jj];
        const bool ok = i < flat_end;
        float acc = 0.0f;
        if (!static_mask) acc = ordered_sum(W, [&](uint32_t p) { return gathered[(size_t)p * max_pairs + jj]; });
        for (uint32_t p = 0; static_mask && p < W; ++p) {
            float v;
            if ((direct >> p) & 1u) {
                v = ok ? R.r[p][i] : 0.0f;
                if (ok) R.r[p][i] = 0.0f;
            } else {
                v = gathered[(size_t)p * max_pairs + jj];
            }
            acc = p == 0 ? v : acc + v;
        }
        sum_out[jj] = acc;
        if (ok) {
            const float t = scale * acc;
            w[i] = w[i] + t;
        }
    }
}

}  // namespace iwp
