// The streaming kernels: Alg. 1's accumulation line (r <- r + g for every worker
// and layer; r <- m * r + g with the momentum of Eq. 3) fused with what can ride along on the same pass over HBM --
//  * on the leader of a layer: the importance of every element and the histogram
//    of its most significant key digit (first look of the selection);
//  * on the other workers, once the leader's index set is known: the gather of
//    the residual at those indices and the clearing of the sent positions
//    (Alg. 1 split lines), so the exchange needs no scattered second pass.
//
// Work unit: one TILE (4096 elements = 4 quads per lane of 256, 2 of 512) per workgroup, all loads
// of a tile issued before the first use, non-temporal accesses for data that is
// not read again soon.  This shape measured fastest for a 2-read-1-write stream
// on MI355X (about 6.2 TB/s against 5.3 TB/s for 16K-element tiles and 4.6 TB/s
// for a grid-stride loop).
#pragma once

#include "iwp_common.hpp"

namespace iwp {

// What a leader's workgroup needs besides the data: its LDS histogram, and where the
// candidates go that look 1 copies out.
struct LeadCtx {
    uint32_t* lh;           // LDS, HIST0 bins
    uint32_t* slot;         // LDS, 2 x STAGE_WORDS words for the scans
    uint32_t stage_bin;     // NO_STAGE_BIN: no staging in look 1
    uint32_t shift;         // of the layer's keys
    uint32_t cap;           // slot entries per tile
    uint64_t slot_begin;    // the layer's first slot
    uint32_t* stage_cnt;    // the layer's first tile count
    StageArrays A;
};

// One tile of a worker that follows: accumulate, copy the values at sent positions into the worker's row of the gather
// matrix (row: the tile's first entry there, room: entries it may take), leave +0 behind.  sent(): builds the tile's bitmap
// in map / pre (LDS, TILE_WORDS words each) while the tile's loads are in flight; false: nothing of the tile is sent.
// ACC: false: nothing is accumulated (gl is not read).
template <uint32_t CHUNKS, bool ACC = true, class Sent>
__device__ __forceinline__ void follow_tile(const float* gl, float* rl, uint32_t n, uint32_t base, float m, float* row,
                                            uint32_t room, const uint32_t* map, const uint32_t* pre, Sent sent) {
    float rv[CHUNKS][4], gv[CHUNKS][4];
    Rest rv_rest, gv_rest;
    request_tile<true>(rl, n, base, rv, rv_rest);
    if (ACC) request_tile<true>(gl, n, base, gv, gv_rest);
    const bool any = sent();
    settle_tile(n, base, rv, rv_rest);
    if (ACC) settle_tile(n, base, gv, gv_rest);
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        const uint32_t loc = u * CHUNK + threadIdx.x * VEC;
#pragma unroll
        for (int q = 0; ACC && q < 4; ++q) rv[u][q] = accum(rv[u][q], gv[u][q], m);
        const uint32_t nib = any ? (map[loc >> 5] >> (loc & 31u)) & 0xFu : 0u;      // no bits past the layer's end
        if (nib) {
            uint32_t rank = bitmap_rank(map, pre, loc);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((nib >> q) & 1u) { if (rank < room) row[rank] = rv[u][q]; ++rank; rv[u][q] = 0.0f; }
        }
    }
    store_tile<true>(rl, n, base, rv);
}

// The same for a full tile whose residuals do not start at a multiple of 64 bytes but `head` elements before one: the lanes'
// quads start there, and the last four of them (four lanes) take the 16 elements before the first and behind the last 64
// bytes one by one.  A wavefront's 1024 bytes then are 16 whole lines of 64; with the quads at the tile's start it shares a
// line at either end with its neighbours, which streaming accesses fetch and write in parts: a thousand packed tensors of
// 115.5 M elements, eight workers, followers' pass 1898 -> 1792 us (1798 if every layer starts at a multiple of 64
// bytes; 1871 and 1843 at multiples of 16 and 32).  Ordinary loads or stores, which merge the parts in the caches, are slower
// than either (2150, 2124).  Only full tiles: a layer's last one takes the plain form.
constexpr uint32_t LINE = 16;                               // elements
__device__ __forceinline__ uint32_t elements_to_line(const float* p) {
    return (0u - (uint32_t)(reinterpret_cast<uintptr_t>(p) / sizeof(float))) & (LINE - 1u);
}
template <class Sent>
__device__ __forceinline__ void follow_tile_from(uint32_t head, const float* g0, float* r0, float m, float* row, uint32_t room,
                                                 const uint32_t* map, const uint32_t* pre, Sent sent) {
    constexpr uint32_t LAST = CHUNKS_PER_TILE - 1, ODD = BLOCK - LINE / VEC;    // lanes from ODD on: single elements
    const uint32_t tid = threadIdx.x;
    float rv[CHUNKS_PER_TILE][4], gv[CHUNKS_PER_TILE][4];
    auto single = [&](uint32_t c) {                         // position of such a lane's element c
        const uint32_t e = (tid - ODD) * VEC + c;
        return e < head ? e : TILE - LINE + e;
    };
    auto request = [&](const float* p, float (&v)[CHUNKS_PER_TILE][4]) {
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS_PER_TILE; ++u) {
            if (u < LAST || tid < ODD) {
                const v4f t = load_v4<true>(p + head + u * CHUNK + tid * VEC);
                v[u][0] = t.x; v[u][1] = t.y; v[u][2] = t.z; v[u][3] = t.w;
            } else {
#pragma unroll
                for (uint32_t c = 0; c < VEC; ++c) v[u][c] = p[single(c)];
            }
        }
    };
    request(r0, rv);
    request(g0, gv);
    const bool any = sent();
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS_PER_TILE; ++u) {
#pragma unroll
        for (int q = 0; q < 4; ++q) rv[u][q] = accum(rv[u][q], gv[u][q], m);
        if (u < LAST || tid < ODD) {
            const uint32_t loc = head + u * CHUNK + tid * VEC, wd = loc >> 5;
            uint32_t nib = 0u;
            if (any) {
                const uint64_t two = (uint64_t)map[min(wd + 1u, TILE_WORDS - 1u)] << 32 | map[wd];
                nib = (uint32_t)(two >> (loc & 31u)) & 0xFu;
            }
            if (nib) {
                uint32_t rank = bitmap_rank(map, pre, loc);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((nib >> q) & 1u) { if (rank < room) row[rank] = rv[u][q]; ++rank; rv[u][q] = 0.0f; }
            }
            v4f t; t.x = rv[u][0]; t.y = rv[u][1]; t.z = rv[u][2]; t.w = rv[u][3];
            store_v4<true>(r0 + loc, t);
        } else {
#pragma unroll
            for (uint32_t c = 0; c < VEC; ++c) {
                const uint32_t loc = single(c);
                if (any && ((map[loc >> 5] >> (loc & 31u)) & 1u)) {
                    const uint32_t rank = bitmap_rank(map, pre, loc);
                    if (rank < room) row[rank] = rv[u][c];
                    rv[u][c] = 0.0f;
                }
                r0[loc] = rv[u][c];
            }
        }
    }
}

// One tile of a layer's leader: accumulate (ACC), score every element, histogram
// the top key digit, and with a staging bin copy the candidates into the tile's
// slot.  On large tables everything streams with non-temporal accesses, the leader's
// residual included: the second look comes after the whole first look, far too late for
// any cache (the counters show it fetching every byte from HBM either way), and the
// non-temporal form measured about 10 % faster.  KEEP: on tables small enough for the
// chip's 256 MB memory-side cache the weights (KEEP_W) or the weights and the written
// residual (KEEP_W_AND_R) are accessed with ordinary loads and stores instead, so that
// what touches them again within the step (the ordered write clears the sent positions
// of the residual, the update adds to the weights at them) finds them there.  The host
// picks by the table's size (launch_leader_pass): a written residual that stays in the
// cache is written back during whatever comes next.
// clear: the histogram is cleared first, once the tile's loads are on their way; before them it kept every
// workgroup from its loads (look 1 of one layer of 1 M elements 13.6 -> 12.8 us, thresholds of 25.6 M 51.4 -> 50.3).
// With a gradient it is bound by the stream itself: 25.6 M elements 71 us, 69.5 without histogram and copies, 400 M in one layer 1069 and 1067,
// a thousand tensors of 115.5 M 316 and 320.  Without one, 25.6 M (weights kept, 3 us of it): 50 us, the stream 35, copies (1.6 per element that
// is kept, partial lines) 7 with the histogram and 11 without, histogram 3 to 5, most of it the flush; the divide is 1 of them: it hides
// behind the rest (an approximate one 48.5).  What a wavefront issues counts on small tables, where it is most of a workgroup's time, and
// without a gradient.  Hence no branch per element where a tile is whole and none of a wavefront's scores is zero.
// Look 1 of 25.6 M elements without / with a gradient 51.0 -> 48.5 / 75.0 -> 73.5 us;
// whole calls, with look 2 and the records' pass likewise: one layer of 1 M 26.6 -> 25.1, six tensors of 235 k, four workers 32.6 -> 31.4,
// thresholds and pairs of 25.6 M 116.7 -> 115.0, one worker's share of them 145.0 -> 142.8, a thousand tensors, eight workers 2334 -> 2323.
constexpr int KEEP_NOTHING = 0, KEEP_W = 1, KEEP_W_AND_R = 2;
template <bool ACC, int KEEP, uint32_t THREADS>
__device__ __forceinline__ void lead_tile(const float* __restrict__ gl, float* __restrict__ rl,
                                          const float* __restrict__ wl, uint32_t n, uint32_t lt,
                                          float eps, float m, const LeadCtx& C, bool clear) {
    constexpr uint32_t CHUNKS = TILE / (THREADS * VEC);
    const uint32_t tid = threadIdx.x;
    const uint32_t base = lt * TILE;
    uint32_t key[CHUNKS][4];
    float val[CHUNKS][4], gv[CHUNKS][4], wv[CHUNKS][4];
    Rest val_rest, gv_rest, wv_rest;
    request_tile<true, THREADS>(rl, n, base, val, val_rest);
    if (ACC) request_tile<true, THREADS>(gl, n, base, gv, gv_rest);
    request_tile<(KEEP < KEEP_W), THREADS>(wl, n, base, wv, wv_rest);
    if (clear) {                                            // uniform; the loads are on their way
        for (uint32_t b = tid; b < HIST0 / 4; b += THREADS) reinterpret_cast<uint4*>(C.lh)[b] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    }
    settle_tile<THREADS>(n, base, val, val_rest);
    if (ACC) settle_tile<THREADS>(n, base, gv, gv_rest);
    settle_tile<THREADS>(n, base, wv, wv_rest);
    if (ACC) {
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) val[u][q] = accum(val[u][q], gv[u][q], m);
        store_tile<(KEEP < KEEP_W_AND_R), THREADS>(rl, n, base, val);
    }
    const bool full = base + TILE <= n;
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) key[u][q] = shifted(score_key(val[u][q], wv[u][q], eps), C.shift);
    if (!full) leave_out_rest<THREADS>(n, base, key);                // uniform
    // zero scores (zero residuals: a layer's untouched part) are counted in a register and added once per
    // wavefront: a tile of zeros would otherwise be 4096 atomics on one LDS word
    uint32_t least = key[0][0];
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) least = min(least, key[u][q]);
    if (full && !__any(least == C.shift)) {                 // a key is never less
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) atomicAdd(&C.lh[key[u][q] >> digit_shift(0)], 1u);
    } else {
        uint32_t zeros = 0;
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (key[u][q] == C.shift) ++zeros;
                else if (key[u][q] != NOT_AN_ELEMENT) atomicAdd(&C.lh[key[u][q] >> digit_shift(0)], 1u);
            }
        zeros = wave_sum(zeros);
        if (zeros != 0 && (tid & (WAVE - 1)) == 0) atomicAdd(&C.lh[0], zeros);
    }
    if (C.stage_bin != NO_STAGE_BIN) {                      // uniform
        const uint32_t cnt = stage_tile<THREADS>(key, val, base, C.stage_bin << digit_shift(0), C.cap, C.slot_begin + (uint64_t)lt * C.cap, C.A,
                                        C.slot + (lt & 1u) * STAGE_WORDS);
        if (tid == 0) C.stage_cnt[lt] = cnt;
    }
}

// The leader's share of one group (up to LGROUP tiles of the same layer):
// one LDS histogram of the top digit for the whole group, flushed once.
template <int KEEP, uint32_t THREADS>
__device__ __forceinline__ void leader_group(const float* gp, float* rp, const float* __restrict__ w, const DevLayer& L,
                                             uint32_t first_tile /*in layer*/, uint32_t group_tiles, float eps, float m,
                                             LeadCtx& C, uint32_t* __restrict__ ghist) {
    float* rl = rp + L.offset;
    const float* gl = gp ? gp + L.offset : nullptr;
    const float* wl = w + L.offset;
    const uint32_t ntiles = (L.n + TILE - 1) / TILE;
    const uint32_t last = min(first_tile + group_tiles, ntiles);
    for (uint32_t t = first_tile; t < last; ++t) {
        if (gp) lead_tile<true, KEEP, THREADS>(gl, rl, wl, L.n, t, eps, m, C, t == first_tile);
        else lead_tile<false, KEEP, THREADS>(gl, rl, wl, L.n, t, eps, m, C, t == first_tile);
    }
    __syncthreads();
    // neighbouring lanes, neighbouring bins: with four to a lane, read at once, the atomics meet fewer lines each and look 1 of
    // 25.6 M elements takes 84 us instead of 49
    for (uint32_t b = threadIdx.x; b < HIST0; b += THREADS) {
        const uint32_t v = C.lh[b];
        if (v) atomicAdd(&ghist[b], v);
    }
}

__device__ __forceinline__ LeadCtx lead_ctx(uint32_t* lh, uint32_t* slot, const DevLayer& L, const LayerState* state,
                                            uint32_t j, uint32_t* stage_cnt, const StageArrays& A) {
    LeadCtx C;
    C.lh = lh;
    C.slot = slot;
    C.stage_bin = state[j].stage_bin;
    C.shift = state[j].shift;
    C.cap = L.slot_cap;
    C.slot_begin = L.slot_begin;
    C.stage_cnt = stage_cnt + L.tile_begin;
    C.A = A;
    return C;
}

// Every worker that is not the leader of the tile's layer (and every worker of a layer
// without selection): plain accumulation, W * tiles workgroups, worker-major.  A worker
// without a gradient pointer is not accumulated.  runs: see in_runs().  The leaders go through k_leader_pass.
// Tiles that end within their first chunk take one (see mask_tile): 32 workers on 1000 layers of 205 elements 39.1 -> 28.1 us a launch.
__global__ __launch_bounds__(BLOCK) void k_accumulate_rest(WorkerPtrs P, const DevLayer* __restrict__ layers,
                                                           uint32_t n_layers, uint32_t tiles, uint32_t runs,
                                                           const uint32_t* __restrict__ leader, uint32_t W) {
    const uint32_t b = runs ? in_runs(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t p = b / tiles;
    const uint32_t t = b - p * tiles;
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    const float* gp = P.g[p];
    if (!gp || (L.k > 0 && leader_of(leader, j, W) == p)) return;
    float* rl = P.r[p] + L.offset;
    const float* gl = gp + L.offset;
    const uint32_t base = (t - L.tile_begin) * TILE, head = elements_to_line(rl);
    auto nothing = []() { return false; };
    if (L.n - base <= CHUNK) follow_tile<1>(gl, rl, L.n, base, P.momentum, nullptr, 0u, nullptr, nullptr, nothing);
    else if (head && base + TILE <= L.n) follow_tile_from(head, gl + base, rl + base, P.momentum, nullptr, 0u, nullptr, nullptr, nothing);
    else follow_tile<CHUNKS_PER_TILE>(gl, rl, L.n, base, P.momentum, nullptr, 0u, nullptr, nullptr, nothing);
}

// Leaders only: one workgroup per group of LG tiles of every layer with k > 0.  The grid:
// with LG == 1 one workgroup per tile of the table, otherwise GROUP / LG per super-tile (some of them past the end
// of a short layer).
template <uint32_t LG, int KEEP, uint32_t THREADS>
__global__ __launch_bounds__(THREADS, 6) void k_leader_pass(WorkerPtrs P, const float* __restrict__ w,
                                                       const DevLayer* __restrict__ layers, uint32_t n_layers,
                                                       const uint32_t* __restrict__ leader, uint32_t W, float eps,
                                                       uint32_t* __restrict__ hist,
                                                       const LayerState* __restrict__ state,
                                                       uint32_t* __restrict__ stage_cnt, StageArrays A) {
    __shared__ alignas(16) uint32_t lh[HIST0];
    __shared__ uint32_t slot[2 * STAGE_WORDS];
    uint32_t j, first;
    if (LG == 1) {
        j = layer_of_tile(layers, n_layers, blockIdx.x);
    } else {
        j = layer_of_stile(layers, n_layers, layers[n_layers].tile_begin, blockIdx.x / (GROUP / LG));
    }
    const DevLayer L = layers[j];
    if (L.k == 0) return;
    if (LG == 1) {
        first = blockIdx.x - L.tile_begin;
    } else {
        constexpr uint32_t SUB = GROUP / LG;                 // workgroups per super-tile
        first = (blockIdx.x / SUB - L.stile_begin) * GROUP + (blockIdx.x % SUB) * LG;
        if (first * TILE >= L.n) return;
    }
    const uint32_t p = leader_of(leader, j, W);
    LeadCtx C = lead_ctx(lh, slot, L, state, j, stage_cnt, A);
    // consecutive workgroups of a layer flush into different copies of its first-digit histogram
    uint32_t* h0 = layer_hist(hist, L, 0) + (size_t)((first / LG) & (L.h0_copies - 1u)) * HIST0;
    leader_group<KEEP, THREADS>(P.g[p], P.r[p], w, L, first, LG, eps, P.momentum, C, h0);
}

// The other workers, after the leader's pairs are known: accumulate, and where the
// tile holds sent positions, copy the accumulated value into the worker's row of
// the gather matrix and leave +0 behind.  tile_out[t] = position (inside the
// layer's pairs) of the first pair that falls into tile t; the pairs are ascending,
// so a tile's pairs are contiguous.  `acc`: the workers that accumulate (have a
// gradient); the grid is acc.n * tiles.  runs: see in_runs().
__global__ __launch_bounds__(BLOCK) void k_follow_gather(WorkerPtrs P, WorkerList acc, const DevLayer* __restrict__ layers,
                                                         uint32_t n_layers, uint32_t tiles, uint32_t runs,
                                                         const uint32_t* __restrict__ leader, uint32_t W,
                                                         const uint32_t* __restrict__ idx,
                                                         const uint32_t* __restrict__ tile_out,
                                                         float* __restrict__ gathered, uint64_t K) {
    __shared__ uint32_t map[TILE_WORDS], pre[TILE_WORDS], slot[4];
    const uint32_t tid = threadIdx.x;
    const uint32_t b = runs ? in_runs(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t a = b / tiles;
    const uint32_t t = b - a * tiles;
    const uint32_t p = acc.id[a];
    const uint32_t j = layer_of_tile(layers, n_layers, t);
    const DevLayer L = layers[j];
    const bool has_sel = L.k > 0;
    if (has_sel && leader_of(leader, j, W) == p) return;       // done by the leader pass
    const uint32_t lt = t - L.tile_begin;
    const uint32_t base = lt * TILE;
    const float* gp = P.g[p];
    float* rl = P.r[p] + L.offset;
    uint32_t lo = 0, cnt = 0;
    if (has_sel) {
        const uint32_t ntiles = (L.n + TILE - 1) / TILE;
        // positions are clamped to the layer's k pairs: never index outside idx / the gather row
        lo = min(tile_out[t], L.k);
        const uint32_t hi = (lt + 1 < ntiles) ? min(tile_out[t + 1], L.k) : L.k;
        cnt = hi > lo ? min(hi - lo, TILE) : 0u;
    }
    const uint32_t* ix = idx + L.out_offset + lo;
    float* go = gathered + (size_t)p * K + L.out_offset + lo;
    const uint32_t first = (uint32_t)L.offset + base;           // flat position of the tile's first element
    const float* gl = gp + L.offset;
    auto sent = [&]() {
        if (!cnt) return false;                                  // uniform
        if (tid < TILE_WORDS) map[tid] = 0u;
        __syncthreads();
        for (uint32_t e = tid; e < cnt; e += BLOCK) {
            const uint32_t loc = ix[e] - first;
            if (loc < TILE) atomicOr(&map[loc >> 5], 1u << (loc & 31u));
        }
        __syncthreads();
        bitmap_prefix(map, pre, slot);
        return true;
    };
    const uint32_t head = elements_to_line(rl);
    if (head && base + TILE <= L.n) follow_tile_from(head, gl + base, rl + base, P.momentum, go, cnt, map, pre, sent);
    else follow_tile<CHUNKS_PER_TILE>(gl, rl, L.n, base, P.momentum, go, cnt, map, pre, sent);
}

}  // namespace iwp
