// Kernels of the index-driven half of the exchange: every worker's residual taken
// at the leader's index set and summed in a fixed order (arithmetic of the ring
// all-reduce line of Alg. 1), then the sparse SGD update and the clearing of the
// sent residuals (SGD line / Eq. 3, "not Mask" line).
#pragma once

#include "iwp_common.hpp"

namespace iwp {

// The ordered sum over a pair's values, value(p) for worker p, eight on their way at a time: one by one they are a chain of loads, which
// shows where pairs are few.  Steps of 1.4 k elements, 32 workers: whole 20.4 -> 16.1 us, three calls 30.4 -> 17.7, with thresholds 20.0
// -> 14.0; eight workers 16.1 -> 15.3, 17.1 -> 14.9 and 14.5 -> 12.8; tables of millions are alike.
template <uint32_t N, class Value>
__device__ __forceinline__ void add_workers(float& acc, uint32_t& p, uint32_t W, Value value) {
    for (; p + N <= W; p += N) {
        float v[N];
#pragma unroll
        for (uint32_t q = 0; q < N; ++q) v[q] = value(p + q);
#pragma unroll
        for (uint32_t q = 0; q < N; ++q) acc = p + q == 0 ? v[q] : acc + v[q];      // the fold starts from worker 0's value, not from 0
    }
}
template <class Value>
__device__ __forceinline__ float ordered_sum(uint32_t W, Value value) {
    float acc = 0.0f;
    uint32_t p = 0;
    add_workers<8>(acc, p, W, value);
    add_workers<4>(acc, p, W, value);
    add_workers<2>(acc, p, W, value);
    add_workers<1>(acc, p, W, value);
    return acc;
}

// Scattered 4-byte accesses, one 128-byte line each: bound by lines moved (955 k pairs of 61 M elements, eight workers:
// the sums at 5.9 TB/s counted in lines) and, for the clears, by partial writes to memory (about 22 G/s).  More loads in
// flight per lane, more pairs per lane or one worker per workgroup change neither.  Ordinary accesses: with a new index
// set and freshly written residuals in every pass the clears find the lines that the sum has just read, and
// non-temporal ones miss them.  Sum and update together, ordinary against non-temporal, eight workers, one pair in 64:
// 300 k pairs 147 / 181 us, 600 k 336 / 360, 955 k 532 / 557; after compress_segmented 410 / 461 us (61 M elements)
// and 168 / 203 us (25.6 M).  Non-temporal accesses win where pairs lie closer than about one in 28 and the lines exceed
// 1 GB (2 M pairs of one in 20: 832 / 732 us), a density that these calls cannot know from their arguments.
__global__ __launch_bounds__(BLOCK) void k_gather_sum(ResidualPtrs R, uint32_t W, const uint32_t* __restrict__ idx,
                                                      uint32_t k, float* __restrict__ sum_out) {
    const uint32_t j = blockIdx.x * BLOCK + threadIdx.x;
    if (j >= k) return;
    const uint32_t i = idx[j];
    sum_out[j] = ordered_sum(W, [&](uint32_t p) { return R.r[p][i]; });
}

// From the last pairs to the first, eight workgroups by eight, so that each stays on the die that has summed its pairs: the
// lines that the sum has read last are still in the caches.  Sum and update together, forwards / backwards: 955 k pairs of
// one in 64, eight workers 580 / 554 us, with freshly written residuals 525 / 498; 3 M of one in 20 1313 / 1291.  Workgroup
// by workgroup backwards the dies change, and 47 k pairs lose what their L2 held: 22 -> 24 us.  (Positions are distinct:
// the order changes no result.)
__global__ __launch_bounds__(BLOCK) void k_apply_update(float* __restrict__ w, const uint32_t* __restrict__ idx,
                                                        const float* __restrict__ sum, uint32_t k, float scale,
                                                        ResidualPtrs R, uint32_t W) {
    const uint32_t whole = gridDim.x & ~7u;
    const uint32_t b = blockIdx.x < whole ? whole - 8u - (blockIdx.x & ~7u) + (blockIdx.x & 7u) : blockIdx.x;
    const uint32_t j = b * BLOCK + threadIdx.x;
    if (j >= k) return;
    const uint32_t i = idx[j];
    const float t = scale * sum[j];              // rounded product ...
    w[i] = w[i] + t;                             // ... then rounded sum (contraction is off)
    for (uint32_t p = 0; p < W; ++p) R.r[p][i] = 0.0f;
}

// Whole-step route: the workers that streamed (and each layer's leader) left their
// values at the K pairs in `gathered` (row p = worker p) and cleared them on the way.
// A worker that does not accumulate (no gradient: bit p of static_mask) streams
// nothing, so unless it leads the pair's layer its value is fetched and cleared
// here, pair by pair.  Then the ordered sum over the workers and the weight update.
__global__ __launch_bounds__(BLOCK) void k_reduce_update(ResidualPtrs R, uint32_t static_mask,
                                                         const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                         const uint32_t* __restrict__ leader,
                                                         const float* __restrict__ gathered, uint32_t W, uint64_t K,
                                                         const uint32_t* __restrict__ idx, float* __restrict__ w,
                                                         float scale, float* __restrict__ sum_out, uint64_t flat_end) {
    const uint64_t j = (uint64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (j >= K) return;
    const uint32_t i = idx[j];
    const bool ok = i < flat_end;                // always true for pairs this library wrote
    uint32_t direct = 0;
    if (static_mask) {
        uint32_t lo = 0, hi = n_layers;          // layer of pair j: last row with out_offset <= j
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (layers[mid].out_offset <= j) lo = mid; else hi = mid;
        }
        direct = static_mask & ~(1u << leader_of(leader, lo, W));
    }
    float acc = 0.0f;
    if (!static_mask) acc = ordered_sum(W, [&](uint32_t p) { return gathered[(size_t)p * K + j]; });
    for (uint32_t p = 0; static_mask && p < W; ++p) {
        float v;
        if ((direct >> p) & 1u) {
            v = ok ? R.r[p][i] : 0.0f;
            if (ok) R.r[p][i] = 0.0f;
        } else {
            v = gathered[(size_t)p * K + j];
        }
        acc = p == 0 ? v : acc + v;
    }
    sum_out[j] = acc;
    if (!ok) return;
    const float t = scale * acc;
    w[i] = w[i] + t;
}

}  // namespace iwp
