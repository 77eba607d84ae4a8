// Small tables: everything after the leaders' part of a step -- the other workers' accumulation, the exchange and the weight
// update -- in one launch, for the top-k and the threshold routes.
//
// Work unit: a chunk of 1024 elements, one quad per lane, for all workers: up to TOGETHER workers' loads are in flight at a
// time, the chunk's bits of sent elements are found once, and every lane keeps the running sums of its four elements, so that
// nothing is gathered into memory and read back by another launch.  The quads start at a multiple of 64 bytes of one worker's
// residual (see follow_tile_from); a layer's first and last chunk (PART) read a cut quad from the
// nearest whole one.
//
// Latency bound: launches count here, and a layer that takes a few workgroups.  Six tensors of 235 k elements, four workers
// 43.4 -> 40.7 us a step; 40 tensors of 300 k with two, four and eight workers 38.5, 40.8, 43.6 -> 36.4, 38.8, 43.4; with
// thresholds 21.8, 23.0, 24.8 -> 17.7, 18.7, 21.8.  From FOLLOW_SUM_MAX_TILES on (where the chip no longer holds all chunks at
// once) the workers' own launch, one worker at a time, streams faster: 300 tensors of 1 M elements 63 against 72 us, 61 M
// elements with eight workers 886 us (with the update) against 914.
// The workers are a serial chain here, TOGETHER at a time, where their own launch has workgroups of their own for each.  What the
// one launch gains over two, us a step, median over layouts, hints and keep ratios (steps of 20 to 110 us): up to 6 workers 1 to 4
// from 20 k to 1 M elements, -0.3 to 1.5 below.  7 and 8 lose 0.6 to 1.4 (thresholds; top-k 0.1 to 0.8) where layers average less than
// a chunk, gain up to 1 above that and 2.4 to 6 from 300 k elements on: they take it from a chunk a layer on.  More workers take it where
// its chunks give the chip enough to do, 14 a worker (140 for 9), not counting the two a layer that the layer may fill in part: 16
// workers -2.0 at 8 to 12 chunks a worker, -0.3 at 12, 0.6 at 16, 2.9 at 20; 24 -1.0, 1.2, 3.8, 5.1; 32 (thresholds) 1.7, 6.7, 8.4, 13.
// Cut quads were read and written element by element before, 32 loads in a row for four workers: packed layers then lost up to
// 14 us (60 layers of 270 k elements, 32 workers 60 us a step in two launches, 72 in one).
#pragma once

#include "iwp_common.hpp"
#include "iwp_stream.hpp"
#include "iwp_threshold.hpp"

namespace iwp {

constexpr uint32_t FOLLOW_SUM_MAX_TILES = 256;
constexpr uint32_t FOLLOW_SUM_ANY = 6, FOLLOW_SUM_FEW = 8;      // workers: always; from a chunk a layer on
constexpr uint32_t FOLLOW_SUM_CHUNKS = 140, FOLLOW_SUM_CHUNKS_EACH = 14;
constexpr uint32_t CHUNKS_A_TILE = TILE / CHUNK;
constexpr uint32_t TOGETHER = 4;                            // workers whose loads are in flight together
constexpr uint32_t NO_WORKER = 0xFFFFFFFFu;

// Elements by which a layer's chunks start before the layer, so that they start at a multiple of 64 bytes of `p`.
__device__ __forceinline__ uint32_t elements_past_line(const float* p) {
    return (uint32_t)(reinterpret_cast<uintptr_t>(p) / sizeof(float)) & (LINE - 1u);
}
// How a chunk's elements are reached.  WHOLE: all of them are the layer's.  PART: some are not (i counts modulo 2^32, elements
// outside the layer are left alone): a lane whose quad is cut reads the layer's nearest whole quad and shifts it (settle_quad)
// once all loads have been requested; ONES: layers of fewer elements than a quad.
enum ChunkForm { WHOLE, PART, ONES };
template <ChunkForm FORM>
__device__ __forceinline__ void chunk_load(const float* p, uint32_t i, uint32_t n, float (&v)[4]) {
    if (FORM == ONES) {
#pragma unroll
        for (uint32_t c = 0; c < VEC; ++c) {
            const uint32_t e = i + c;
            if (e < n) v[c] = p[e];
        }
        return;
    }
    const int at = FORM == WHOLE ? (int)i : min(max((int)i, 0), (int)(n - VEC));
    if (FORM == WHOLE || i < n || i + (VEC - 1u) < n) {
        const v4f t = load_v4<true>(p + at);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
}
template <ChunkForm FORM>
__device__ __forceinline__ void settle_quad(uint32_t i, uint32_t n, float (&v)[4]) {
    if (FORM != PART) return;
    const int by = (int)i - min(max((int)i, 0), (int)(n - VEC));    // v[c] is to be what v[c + by] is
    if (by == 0) return;
    const float t[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int c = 0; c < (int)VEC; ++c)
#pragma unroll
        for (int k = 0; k < (int)VEC; ++k) v[c] = c + by == k ? t[k] : v[c];
}
template <ChunkForm FORM>
__device__ __forceinline__ void chunk_store(float* p, uint32_t i, uint32_t n, const float (&v)[4]) {
    if (FORM == WHOLE || (FORM == PART && i < n && n - i >= VEC)) {
        v4f t; t.x = v[0]; t.y = v[1]; t.z = v[2]; t.w = v[3];
        store_v4<true>(p + i, t);
    } else {
#pragma unroll
        for (uint32_t c = 0; c < VEC; ++c) {
            const uint32_t e = i + c;
            if (e < n) p[e] = v[c];
        }
    }
}

// Runs body(chunk, first element, whole) for chunk c of a layer, and for what lies behind the layer's last chunk, less than a
// line, if c is that chunk.  first counts modulo 2^32 (a layer's first chunk starts before it); whole: all of the chunk's
// elements are the layer's.
template <class Body>
__device__ __forceinline__ void layer_chunk(const DevLayer& L, uint32_t c, uint32_t past, Body body) {
    const uint32_t chunks = (L.n + TILE - 1) / TILE * CHUNKS_A_TILE;
    uint32_t first = c * CHUNK - past;
    if (c > 0 && first >= L.n) return;
    for (;; ++c, first += CHUNK) {
        body(c, first, first < L.n && L.n - first >= CHUNK);
        if (c + 1 < chunks || L.n - first <= CHUNK) return;
        __syncthreads();                                     // what body keeps in LDS is written again
    }
}

// One chunk for all workers; i: the lane's first element.  sent(bits, pos), called once with the first loads in flight: the
// lane's bits of sent elements and the position of the first of them among the pairs.  special.is(p): a worker that does not
// stream the layer though it may have a gradient; special.take(p, bits, pos, i, r, v): its values there.  exchange: the sent
// positions are cleared, and done(bits, pos, acc) gets the ordered sums.
template <ChunkForm FORM, class Sent, class Special, class Done>
__device__ __forceinline__ void follow_chunk(const WorkerPtrs& P, uint64_t offset, uint32_t n, uint32_t W, uint32_t i,
                                             bool exchange, Sent sent, Special special, Done done) {
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t bits = 0, pos = 0;
    for (uint32_t p0 = 0; p0 < W; p0 += TOGETHER) {
        float rv[TOGETHER][4], gv[TOGETHER][4];
#pragma unroll
        for (uint32_t q = 0; q < TOGETHER; ++q) {
            const uint32_t p = p0 + q;
            if (p < W && P.g[p] && !special.is(p)) {
                chunk_load<FORM>(P.r[p] + offset, i, n, rv[q]);
                chunk_load<FORM>(P.g[p] + offset, i, n, gv[q]);
            }
        }
        if (p0 == 0) sent(bits, pos);
        const uint32_t cut = exchange ? bits : 0u;
#pragma unroll
        for (uint32_t q = 0; q < TOGETHER; ++q) {
            const uint32_t p = p0 + q;
            if (p >= W) break;
            float* r = P.r[p] + offset;
            float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (special.is(p)) {
                if (bits) special.take(p, bits, pos, i, r, v);
            } else if (P.g[p]) {
                settle_quad<FORM>(i, n, rv[q]);
                settle_quad<FORM>(i, n, gv[q]);
#pragma unroll
                for (uint32_t c = 0; c < VEC; ++c) {
                    v[c] = accum(rv[q][c], gv[q][c], P.momentum);
                    rv[q][c] = (cut >> c) & 1u ? 0.0f : v[c];
                }
                chunk_store<FORM>(r, i, n, rv[q]);
            } else if (cut) {                               // holds a residual and does not stream: only what is sent
#pragma unroll
                for (uint32_t c = 0; c < VEC; ++c)
                    if ((cut >> c) & 1u) { v[c] = r[i + c]; r[i + c] = 0.0f; }
            }
#pragma unroll
            for (uint32_t c = 0; c < VEC; ++c) acc[c] = p == 0 ? v[c] : acc[c] + v[c];   // the fold starts from worker 0's value
        }
    }
    if (exchange && bits) done(bits, pos, acc);
}

// The worker that leads the layer: its values at the sent positions are the pairs'.
struct LeaderValues {
    uint32_t lead;
    const float* val;                                        // of the layer's pairs
    __device__ __forceinline__ bool is(uint32_t p) const { return p == lead; }
    __device__ __forceinline__ void take(uint32_t, uint32_t bits, uint32_t pos, uint32_t, float*, float (&v)[4]) const {
#pragma unroll
        for (uint32_t c = 0; c < VEC; ++c)
            if ((bits >> c) & 1u) v[c] = val[pos++];
    }
};

// Top-k: after the leader's pairs are known.  tile_out[t] = position (inside the layer's pairs) of the first pair that falls into
// tile t; the pairs are ascending, so a chunk's are contiguous.  align: the worker whose residual the chunks
// are aligned to.  Grid: CHUNKS_A_TILE * tiles.
__global__ __launch_bounds__(BLOCK) void k_follow_sum(WorkerPtrs P, uint32_t align, const DevLayer* __restrict__ layers,
                                                      uint32_t n_layers, const uint32_t* __restrict__ leader, uint32_t W,
                                                      const uint32_t* __restrict__ idx, const float* __restrict__ val,
                                                      const uint32_t* __restrict__ tile_out, float* w, float scale,
                                                      float* __restrict__ sum_out) {
    __shared__ uint32_t map[CHUNK / 32], first_pair;
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1);
    const uint32_t t = blockIdx.x / CHUNKS_A_TILE;
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    const uint32_t ntiles = (L.n + TILE - 1) / TILE;
    const uint32_t* ix = idx + L.out_offset;
    const LeaderValues special{L.k > 0 ? leader_of(leader, j, W) : NO_WORKER, val + L.out_offset};
    float* wl = w + L.offset;
    float* so = sum_out + L.out_offset;
    layer_chunk(L, (t - L.tile_begin) * CHUNKS_A_TILE + blockIdx.x % CHUNKS_A_TILE, elements_past_line(P.r[align] + L.offset),
                [&](uint32_t, uint32_t first, bool whole) {
        const uint32_t i = first + tid * VEC;
        auto sent = [&](uint32_t& bits, uint32_t& pos) {
            if (L.k == 0) return;
            // the pairs of the one or two tiles that the chunk's elements lie in; positions are clamped to the layer's k
            // pairs: never index outside idx
            const uint32_t begin = first < L.n ? first : 0u, end = min(first + CHUNK, L.n);
            const uint32_t t0 = begin / TILE, t1 = (end - 1u) / TILE;
            const uint32_t lo = min(tile_out[L.tile_begin + t0], L.k);
            const uint32_t hi = t1 + 1 < ntiles ? min(tile_out[L.tile_begin + t1 + 1], L.k) : L.k;
            if (hi <= lo) return;                            // uniform
            if (tid < CHUNK / 32) map[tid] = 0u;
            __syncthreads();
            const uint32_t at = (uint32_t)L.offset + first;  // flat position of the chunk's first element
            for (uint32_t e = lo + tid; e < hi; e += BLOCK) {
                const uint32_t loc = ix[e] - at;
                if (loc < CHUNK) {
                    atomicOr(&map[loc >> 5], 1u << (loc & 31u));
                    if (e == lo || ix[e - 1] - at >= CHUNK) first_pair = e;      // ascending: the chunk's first
                }
            }
            __syncthreads();
            // every wavefront adds the words' bits up for itself
            const uint32_t word = lane < CHUNK / 32 ? map[lane] : 0u, ones = __popc(word);
            const uint32_t wd = tid * VEC / 32, b = tid * VEC % 32, mine = map[wd];
            bits = (mine >> b) & 0xFu;
            pos = first_pair + __shfl(wave_inclusive_scan(ones) - ones, (int)wd, WAVE) + __popc(mine & ((1u << b) - 1u));
        };
        auto done = [&](uint32_t bits, uint32_t pos, const float (&acc)[4]) {
#pragma unroll
            for (uint32_t c = 0; c < VEC; ++c)
                if ((bits >> c) & 1u) {
                    so[pos++] = acc[c];
                    const float u = scale * acc[c];          // rounded product ...
                    wl[i + c] = wl[i + c] + u;               // ... then rounded sum
                }
        };
        if (whole) follow_chunk<WHOLE>(P, L.offset, L.n, W, i, true, sent, special, done);
        else if (L.n >= VEC) follow_chunk<PART>(P, L.offset, L.n, W, i, true, sent, special, done);
        else follow_chunk<ONES>(P, L.offset, L.n, W, i, true, sent, special, done);
    });
}

// The same where thresholds decide: the bits and positions come from the mask.  The chosen nodes' values come from the tiles'
// slots (k_leader_mask has been through their residuals).  If the total exceeds the capacity, the others only accumulate, and
// what the chosen nodes have handed over is put back.
struct ChosenValues {
    const uint32_t* leaders;                     // of the layer
    uint32_t n_lead, W, chosen;                  // chosen: bit p: node p is chosen for the layer
    bool exchange;
    const uint32_t *tile_counts, *tile_pos;      // of the layer's tiles
    ChosenSlots S;                               // val: of the layer's first tile
    __device__ __forceinline__ bool is(uint32_t p) const { return (chosen >> p) & 1u; }
    __device__ __forceinline__ void take(uint32_t p, uint32_t bits, uint32_t pos, uint32_t i, float* r, float (&v)[4]) const {
        uint32_t q = 0;
        while (q + 1 < n_lead && chosen_at(leaders, n_lead, 0, q, W) != p) ++q;
#pragma unroll
        for (uint32_t c = 0; c < VEC; ++c) {
            if (!((bits >> c) & 1u)) continue;
            const uint32_t t = (i + c) / TILE;
            const bool handed_over = tile_counts[t] <= S.cap;
            const float* val = S.val + ((size_t)q * S.tiles + t) * S.cap + (pos - tile_pos[t]);
            ++pos;
            if (exchange) {
                v[c] = handed_over ? *val : r[i + c];
                if (!handed_over) r[i + c] = 0.0f;
            } else if (handed_over) {
                r[i + c] = *val;
            }
        }
    }
};

// The tables are so small that every workgroup finds where the tiles' pairs start for itself, one count per thread, which saves
// k_tile_offsets, a launch of one workgroup: steps with thresholds of 20 k elements 15.0 -> 11.8 us, 400 k 18.0 -> 15.0, 1 M, two
// chosen nodes 23.7 -> 20.7, with statistics 400 k 26.7 -> 23.7.  The counts that the caller sees are written on the way.
__global__ __launch_bounds__(BLOCK) void k_follow_mask_sum(WorkerPtrs P, uint32_t align, const DevLayer* __restrict__ layers,
                                                       uint32_t n_layers, uint32_t tiles, const uint32_t* __restrict__ leaders,
                                                       uint32_t n_lead, uint32_t W, const uint32_t* __restrict__ mask,
                                                       const uint32_t* __restrict__ tile_counts,
                                                       uint32_t* __restrict__ count_out, uint32_t max_pairs,
                                                       ChosenSlots S, uint32_t* __restrict__ idx_out, float* w, float scale,
                                                       float* __restrict__ sum_out) {
    static_assert(FOLLOW_SUM_MAX_TILES <= BLOCK, "a tile's count per thread");
    __shared__ uint32_t tile_pos[BLOCK], scan[4];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1);
    const uint32_t t = blockIdx.x / CHUNKS_A_TILE;
    uint32_t total;
    tile_pos[tid] = block_exclusive_scan(tid < tiles ? tile_counts[tid] : 0u, scan, &total);
    __syncthreads();
    for (uint32_t l = blockIdx.x * BLOCK + tid; l < n_layers; l += gridDim.x * BLOCK) {
        const uint32_t f = layers[l].tile_begin, e = layers[l + 1].tile_begin;   // the sentinel row's is `tiles`
        count_out[l] = (e < tiles ? tile_pos[e] : total) - (f < tiles ? tile_pos[f] : total);
    }
    if (blockIdx.x == 0 && tid == 0) {
        count_out[n_layers] = total;
        count_out[n_layers + 1] = total > max_pairs ? 1u : 0u;
    }
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    const uint32_t ntiles = (L.n + TILE - 1) / TILE, nwords = (L.n + 31) / 32;
    const uint32_t past = elements_past_line(P.r[align] + L.offset);
    const bool exchange = total <= max_pairs;
    ChosenValues special{leaders + (size_t)j * n_lead, n_lead, W, 0u, exchange, tile_counts + L.tile_begin,
                         tile_pos + L.tile_begin, S};
    special.S.val += (size_t)L.tile_begin * S.cap;
    for (uint32_t q = 0; q < n_lead; ++q) special.chosen |= 1u << chosen_at(leaders, n_lead, j, q, W);
    const uint32_t* mw = mask + L.mask_begin;
    float* wl = w + L.offset;
    layer_chunk(L, (t - L.tile_begin) * CHUNKS_A_TILE + blockIdx.x % CHUNKS_A_TILE, past,
                [&](uint32_t c, uint32_t first, bool whole) {
        const uint32_t i = first + tid * VEC;
        auto sent = [&](uint32_t& bits, uint32_t& pos) {
            // lane l holds mask word 32 c - 1 + l, of the first one only the bits from the chunk's first element on; every
            // wavefront does this for itself.  Pairs before the chunk: the tile's first, and the words of the tile before
            // word 32 c, less the bits just named.
            const uint32_t at = c * (CHUNK / 32), tc = min(c / CHUNKS_A_TILE, ntiles - 1u);
            const uint32_t wi = at + lane - 1u;              // the layer's word 0 has none before it: out of range
            uint32_t word = lane <= CHUNK / 32 && wi < nwords ? mw[wi] : 0u;
            if (lane == 0) word = past ? word >> (32u - past) << (32u - past) : 0u;
            const uint32_t tw = tc * TILE_WORDS;
            const uint32_t earlier = wave_sum((tw + lane < at ? __popc(mw[tw + lane]) : 0) +
                                              (tw + lane + WAVE < at ? __popc(mw[tw + lane + WAVE]) : 0));
            const uint32_t ones = __popc(word), upto = wave_inclusive_scan(ones);
            const uint32_t from = 32u - past + tid * VEC, wd = from / 32, b = from % 32;
            const uint32_t lo = __shfl(word, (int)wd, WAVE), hi = __shfl(word, (int)wd + 1, WAVE);
            bits = (uint32_t)(((uint64_t)hi << 32 | lo) >> b) & 0xFu;
            pos = tile_pos[L.tile_begin + tc] + earlier - from_lane(ones, 0) + __shfl(upto - ones, (int)wd, WAVE) +
                  __popc(lo & ((1u << b) - 1u));
        };
        auto done = [&](uint32_t bits, uint32_t pos, const float (&acc)[4]) {
#pragma unroll
            for (uint32_t q = 0; q < VEC; ++q)
                if ((bits >> q) & 1u) {
                    if (pos < max_pairs) {                   // always: nothing is exchanged otherwise
                        idx_out[pos] = (uint32_t)L.offset + i + q;
                        sum_out[pos] = acc[q];
                    }
                    ++pos;
                    const float u = scale * acc[q];          // rounded product, then rounded sum
                    wl[i + q] = wl[i + q] + u;
                }
        };
        if (whole) follow_chunk<WHOLE>(P, L.offset, L.n, W, i, exchange, sent, special, done);
        else if (L.n >= VEC) follow_chunk<PART>(P, L.offset, L.n, W, i, exchange, sent, special, done);
        else follow_chunk<ONES>(P, L.offset, L.n, W, i, exchange, sent, special, done);
    });
}

}  // namespace iwp
