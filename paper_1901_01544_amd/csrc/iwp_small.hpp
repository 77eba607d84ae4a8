// Tables of small layers: the leader's whole part of a step -- accumulate, score, select, split -- in one launch, one
// workgroup per layer with the layer in registers.
//
// Latency bound: a small layer's seven launches (k_init ... k_write) take about 4 us each, whatever the layer holds, and
// every one reads back what the one before has written.  Here the layer is read once and the three digits of the k-th
// largest key are found by three histograms in LDS.  One layer of 1000 elements: 30.6 -> 10.8 us a call.
// Layers of one tile take a workgroup of 4 wavefronts, eight of which a compute unit holds, longer ones 16 wavefronts,
// two or (beyond 16384 elements) one a unit; a large table of both takes a launch for each kind.  3000 layers of 300
// elements 119 us by 16 wavefronts, 30 by 4, 94 to 123 by the long route; 6000 ragged ones of 1 M elements, the longest
// 24 759, 394 us by 16 wavefronts, 87 in two launches, 171 to 225 by the long route.
// Beyond 32768 elements a lane would hold more than 32 keys and values (128 registers at 16 wavefronts), and one compute
// unit's share of the memory rate outweighs the launches.
#pragma once

#include "iwp_common.hpp"

namespace iwp {

constexpr int SMALL_BLOCK = 1024;
constexpr uint32_t SMALL_CHUNK = SMALL_BLOCK * VEC;        // elements that the workgroup takes at a time
constexpr uint32_t SMALL_CHUNKS_MAX = 8;                   // layers of up to 32768 elements
constexpr int TINY_BLOCK = 256;                            // tables whose layers all fit one tile
constexpr uint32_t TINY_CHUNKS = TILE / (TINY_BLOCK * VEC);

// FUSED: as in k_write -- the values also go into the leader's row of the gather matrix and the sent positions are
// cleared.  emit: write the pairs; otherwise (select_threshold) only the record, and the residual is only read.
// A single layer comes as `row` (layers == NULL).  Layers of less than min_n or more than max_n elements are another launch's.
template <bool FUSED, int THREADS, uint32_t CHUNKS>
__global__ __launch_bounds__(THREADS) void k_small(WorkerPtrs P, const float* __restrict__ w,
                                                       const DevLayer* __restrict__ layers, DevLayer row,
                                                       uint32_t min_n, uint32_t max_n,
                                                       const uint32_t* __restrict__ leader, uint32_t W, float eps,
                                                       iwp_threshold* __restrict__ thr_out, bool emit,
                                                       uint32_t* __restrict__ tile_out, uint32_t* __restrict__ idx_out,
                                                       float* __restrict__ val_out, float* __restrict__ gathered,
                                                       uint64_t K) {
    constexpr uint32_t WAVES = THREADS / WAVE, STEP = THREADS * VEC;         // STEP: elements of a chunk
    static_assert(TILE % STEP == 0, "tiles start where chunks start");
    __shared__ uint32_t lh[HIST0];
    __shared__ uint32_t sh[PICK_WORDS];
    __shared__ uint32_t tot[CHUNKS * WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = wave_id();
    const uint32_t j = blockIdx.x;
    const DevLayer L = layers ? layers[j] : row;
    if (L.k == 0 || L.n < min_n || L.n > max_n) return;
    const uint32_t p = leader_of(leader, j, W);
    const float* gp = P.g[p];
    float* rl = P.r[p] + L.offset;
    const float* gl = gp ? gp + L.offset : nullptr;
    const float* wl = w + L.offset;
    uint32_t key[CHUNKS][4];
    float val[CHUNKS][4];
#pragma unroll
    for (uint32_t u0 = 0; u0 < CHUNKS; u0 += 4) {          // four chunks' loads before their first use
        float gv[4][4], wv[4][4];
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
            const uint32_t i = (u0 + c) * STEP + tid * VEC;
            if (i < L.n) {
                load_quad(rl, i, L.n, val[u0 + c]);
                if (gp) load_quad(gl, i, L.n, gv[c]);
                load_quad(wl, i, L.n, wv[c], 1.0f);
            }
        }
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
            const uint32_t u = u0 + c, i = u * STEP + tid * VEC;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                key[u][q] = NOT_AN_ELEMENT;
                if (i + q < L.n) {
                    if (gp) val[u][q] = accum(val[u][q], gv[c][q], P.momentum);
                    key[u][q] = score_key(val[u][q], wv[c][q], eps);
                }
            }
            if (!FUSED && gp && i < L.n) store_quad(rl, i, L.n, val[u]);
        }
    }
    for (uint32_t b = tid; b < HIST0; b += THREADS) lh[b] = 0u;
    __syncthreads();
    uint32_t zeros = 0;                                    // counted in a register, as in look 1
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (key[u][q] == 0u) ++zeros;
            else if (key[u][q] != NOT_AN_ELEMENT) atomicAdd(&lh[key[u][q] >> digit_shift(0)], 1u);
        }
    if (__any(zeros != 0)) {
        zeros = wave_sum(zeros);
        if (lane == 0) atomicAdd(&lh[0], zeros);
    }
    __syncthreads();
    uint32_t prefix, rank;
    block_pick<(int)HIST0, THREADS>(lh, L.k, sh, &prefix, &rank);
#pragma unroll
    for (int level = 1; level < DIGITS; ++level) {
        static_assert(HIST2 <= HIST1, "the third digit leaves the upper half of the bins empty");
        for (uint32_t b = tid; b < HIST1; b += THREADS) lh[b] = 0u;
        __syncthreads();
        const uint32_t mask = (1u << digit_bits(level)) - 1u;
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (key[u][q] != NOT_AN_ELEMENT && (key[u][q] >> digit_shift(level - 1)) == prefix)
                    atomicAdd(&lh[(key[u][q] >> digit_shift(level)) & mask], 1u);
        __syncthreads();
        uint32_t bin, rest;
        block_pick<(int)HIST1, THREADS>(lh, rank, sh, &bin, &rest);
        prefix = (prefix << digit_bits(level)) | bin;
        rank = rest;
    }
    const uint32_t thr = prefix, quota = rank;             // the k-th largest key, ties to keep
    if (thr_out && tid == 0) {
        iwp_threshold th;
        th.key = thr; th.n_gt = L.k - quota; th.n_eq_take = quota;
        thr_out[j] = th;
    }
    if (!emit) return;
    // elements above the threshold (low half) and tying with it (high half): inside the lane's quad, before the lane in
    // its wavefront, before the wavefront in index order (chunk by chunk, wavefront by wavefront)
    uint32_t mine[CHUNKS], before[CHUNKS];
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        mine[u] = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            mine[u] += key[u][q] == NOT_AN_ELEMENT ? 0u : key[u][q] > thr ? 1u : key[u][q] == thr ? 0x10000u : 0u;
        const uint32_t inc = wave_inclusive_scan(mine[u]);
        before[u] = inc - mine[u];
        if (lane == WAVE - 1) tot[u * WAVES + wave] = inc;
    }
    __syncthreads();
    uint32_t carry = 0;                                    // at most 32768 of either kind in a layer: the halves hold them
    constexpr uint32_t PER_SCAN = CHUNKS < WAVE / WAVES ? CHUNKS : WAVE / WAVES;
#pragma unroll
    for (uint32_t u0 = 0; u0 < CHUNKS; u0 += PER_SCAN) {
        const uint32_t v = lane < PER_SCAN * WAVES ? tot[u0 * WAVES + lane] : 0u;
        const uint32_t inc = wave_inclusive_scan(v);
#pragma unroll
        for (uint32_t c = 0; c < PER_SCAN; ++c) {
            const uint32_t u = u0 + c;
            const uint32_t base = carry + from_lane(inc - v, c * WAVES + wave);
            if (FUSED && tid == 0 && u * STEP % TILE == 0 && u * STEP < L.n)
                tile_out[L.tile_begin + u * STEP / TILE] = (base & 0xffffu) + min(base >> 16, quota);
            before[u] += base;
        }
        carry += wave_last(inc);
    }
    uint32_t* io = idx_out + L.out_offset;
    float* vo = val_out + L.out_offset;
    float* go = FUSED ? gathered + (size_t)p * K + L.out_offset : nullptr;
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        const uint32_t i = u * STEP + tid * VEC;
        if (mine[u]) {
            uint32_t g = before[u] & 0xffffu, e = before[u] >> 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (key[u][q] == NOT_AN_ELEMENT) continue;
                uint32_t pos = 0xFFFFFFFFu;
                if (key[u][q] > thr) { pos = g + min(e, quota); ++g; }
                else if (key[u][q] == thr) { if (e < quota) pos = g + e; ++e; }
                if (pos < L.k) {
                    io[pos] = (uint32_t)(L.offset + i + q);
                    vo[pos] = val[u][q];
                    if (FUSED) {
                        go[pos] = val[u][q];
                        val[u][q] = 0.0f;
                        if (!gp) rl[i + q] = 0.0f;         // a worker that is not accumulated: only the sent positions
                    }
                }
            }
        }
        if (FUSED && gp && i < L.n) store_quad(rl, i, L.n, val[u]);
    }
}

}  // namespace iwp
