// Tables of small layers: the leader's whole part of a step -- accumulate, score, select, split -- in one launch, one
// workgroup per layer with the layer in registers.
//
// Latency bound: a small layer's five launches (k_init ... k_split; seven up to k_write when this was first measured) take about 4 us
// each, whatever the layer holds, and every one reads back what the one before has written.  Here the layer is read once and the three
// digits of the k-th largest key are found by three histograms in LDS.  One layer of 1000 elements: 30.6 -> 10.8 us a call, now 7.7; the
// times here are of events around every call, which add 2 to 3 us: of calls in a row 5.6 (the launch alone 5.3).
// A lone workgroup is bound by the instructions its wavefronts issue, one in four cycles, and by barriers: 2000 instructions in a row
// take 3.4 us.  So: everything that is the same for all lanes in scalar registers, chunks behind the layer's end skipped by a
// scalar branch, elements counted without branches, only the kept ones of a quad walked through, two barriers a digit (small_pick)
// where there were five.  us a call, before / now: 1000 elements 10.2 / 7.7, 4096 12.6 / 10.8, 16384 15.8 / 14.3, 20000 24.1 / 17.2,
// 32768 29.5 / 22.1 (all kept 38.0 / 33.9), of calls in a row 8.0 / 5.6, 10.4 / 8.7, 13.7 / 12.1, 21.3 / 14.5,
// 25.8 / 19.0 (34.5 / 30.5); whole steps, four workers, 300 layers of 300 18.5 / 14.6, 1000 of 16000 186 / 157.
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

// Digits of the key: 2048 bins for workgroups of 4 wavefronts, 4096 for those of 16, whose wavefronts crowd more into a bin.
template <int THREADS>
struct SmallDigits {
    static constexpr uint32_t BINS0 = THREADS > TINY_BLOCK ? 4096 : 2048, BINS1 = 1024, BINS2 = THREADS > TINY_BLOCK ? 512 : 1024;
    static constexpr int SHIFT0 = THREADS > TINY_BLOCK ? 19 : 20, SHIFT1 = SHIFT0 - 10;
    static_assert((uint64_t)BINS2 == 1ull << SHIFT1 && (uint64_t)BINS0 << SHIFT0 == 1ull << 31, "31 bits in all");
};

// Element i of a layer whose bytes 32 bits address: one register holds the offset, the base stays scalar.
__device__ __forceinline__ const float* at_byte(const float* base, uint32_t i) {
    return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + (uint32_t)(i * sizeof(float)));
}
__device__ __forceinline__ float* at_byte(float* base, uint32_t i) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + (uint32_t)(i * sizeof(float)));
}

// The bin of an LDS histogram that holds rank k_rem counted from the top, and the rank inside it, in every wavefront.  Each sums up its
// share of the bins; after the one barrier all of them look for the share, and in it for the bin, which saves the barriers that
// handing the result around would take.  tot: a word per wavefront.
template <uint32_t NB, int THREADS>
__device__ __forceinline__ void small_pick(const uint32_t* h, uint32_t k_rem, uint32_t* tot, uint32_t* bin_out, uint32_t* k_rem_out) {
    constexpr uint32_t WAVES = THREADS / WAVE;
    constexpr bool SHARED = NB >= WAVE * WAVES && NB > 8 * WAVE;       // short histograms: every wavefront takes all of it
    constexpr uint32_t SHARE = SHARED ? NB / WAVES : NB, PER = SHARE / WAVE;
    static_assert(WAVES <= WAVE, "a share per lane");
    const uint32_t lane = threadIdx.x & (WAVE - 1), wave = wave_id();
    uint32_t c[PER], sum = 0;
    auto share = [&](uint32_t v) {
        sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            c[q] = h[v * SHARE + lane * PER + q];
            sum += c[q];
        }
    };
    auto find = [&](uint32_t x, uint32_t rank, uint32_t& above) {      // lane that holds the rank, what the lanes above it hold
        const uint32_t upto = wave_inclusive_scan(x), incl = wave_last(upto) - upto + x;
        const uint64_t hit = __ballot(incl - x < rank && rank <= incl);
        const uint32_t src = hit ? (uint32_t)__ffsll((unsigned long long)hit) - 1u : 0u;
        above = from_lane(incl - x, src);
        return src;
    };
    uint32_t above, v = SHARED ? wave : 0u;
    share(v);
    if (SHARED) {
        const uint32_t all = wave_sum(sum);
        if (lane == 0) tot[wave] = all;
        __syncthreads();
        v = find(lane < WAVES ? tot[lane] : 0u, k_rem, above);
        k_rem -= above;
        if (v != wave) share(v);
    }
    const uint32_t src = find(sum, k_rem, above);
    k_rem -= above;
    uint32_t q_hit = 0, rest = k_rem, left = k_rem;
    bool found = false;
#pragma unroll
    for (uint32_t q = PER; q-- > 0;) {                      // lane src's bins, from the top
        const uint32_t x = from_lane(c[q], src);
        const bool here = !found && left <= x;
        q_hit = here ? q : q_hit;
        rest = here ? left : rest;
        found = found || here;
        left -= found ? 0u : x;
    }
    *bin_out = v * SHARE + src * PER + q_hit;
    *k_rem_out = rest;
}

// FUSED: as in k_write -- the values also go into the leader's row of the gather matrix and the sent positions are
// cleared.  emit: write the pairs; otherwise (select_threshold) only the record, and the residual is only read.
// ONE: a single layer, its row is `row`.  (Chosen at run time, the row was in vector registers, and with it every bound and base
// address.)  Layers of less than min_n or more than max_n elements are another launch's.
template <bool FUSED, bool ONE, int THREADS, uint32_t CHUNKS>
__global__ __launch_bounds__(THREADS) void k_small(WorkerPtrs P, const float* __restrict__ w,
                                                       const DevLayer* __restrict__ layers, DevLayer row,
                                                       uint32_t min_n, uint32_t max_n,
                                                       const uint32_t* __restrict__ leader, uint32_t W, float eps,
                                                       iwp_threshold* __restrict__ thr_out, bool emit,
                                                       uint32_t* __restrict__ tile_out, uint32_t* __restrict__ idx_out,
                                                       float* __restrict__ val_out, float* __restrict__ gathered,
                                                       uint64_t K) {
    typedef SmallDigits<THREADS> D;
    constexpr uint32_t WAVES = THREADS / WAVE, STEP = THREADS * VEC;         // STEP: elements of a chunk
    static_assert(TILE % STEP == 0, "tiles start where chunks start");
    // the three histograms, and a word per lane for what is not counted, so that counting takes no branch
    __shared__ alignas(16) uint32_t h0[D::BINS0 + D::BINS1 + D::BINS2 + WAVE];
    __shared__ uint32_t part[3][WAVES];
    __shared__ uint32_t tot[CHUNKS * WAVES];
    uint32_t *h1 = h0 + D::BINS0, *h2 = h1 + D::BINS1;
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = wave_id();
    const uint32_t j = blockIdx.x;
    const DevLayer L = ONE ? row : layers[j];
    if (L.k == 0 || L.n < min_n || L.n > max_n) return;
    const uint32_t p = leader_of(leader, j, W);
    const float* gp = P.g[p];
    float* rl = P.r[p] + L.offset;
    const float* gl = gp ? gp + L.offset : nullptr;
    const float* wl = w + L.offset;
    // A lane whose quad is cut by the layer's end takes the layer's last whole quad and leaves out what is not its own; chunks
    // behind the end are skipped by the whole workgroup.  first_of(u): the position of the lane's first element in registers;
    // skip(u): how many of the four are not its own.
    auto first_of = [&](uint32_t u) { return L.n >= VEC ? min(u * STEP + tid * VEC, L.n - VEC) : 0u; };
    auto skip = [&](uint32_t u) { return u * STEP + tid * VEC < L.n ? u * STEP + tid * VEC - first_of(u) : VEC; };
    auto load = [&](const float* base, uint32_t at) {
        v4f t;
        if (L.n >= VEC) {
            t = load_v4<false>(at_byte(base, at));
        } else {
            t.x = base[0]; t.y = base[min(1u, L.n - 1u)]; t.z = base[L.n - 1u]; t.w = 0.0f;
        }
        return t;
    };
    auto store = [&](uint32_t u, v4f v) {
        const uint32_t at = first_of(u), from = skip(u);
        if (from == 0u && L.n >= VEC) {
            store_v4<false>(at_byte(rl, at), v);
        } else {
            const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (uint32_t q = 0; q < VEC; ++q)
                if (q >= from && at + q < L.n) rl[at + q] = x[q];
        }
    };
    uint32_t key[CHUNKS][4];
    v4f val[CHUNKS];
    uint32_t zeros = 0;                                    // counted in a register, as in look 1
#pragma unroll
    for (uint32_t u0 = 0; u0 < CHUNKS; u0 += 4) {          // four chunks' loads before their first use
        if (u0 * STEP >= L.n) continue;
        v4f gv[4], wv[4];
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
            if ((u0 + c) * STEP >= L.n) continue;
            const uint32_t at = first_of(u0 + c);
            val[u0 + c] = load(rl, at);
            if (gp) gv[c] = load(gl, at);
            wv[c] = load(wl, at);
        }
        if (u0 == 0) {                                     // while they are on their way
            for (uint32_t b = tid; b < (D::BINS0 + D::BINS1 + D::BINS2) / 4; b += THREADS)
                reinterpret_cast<uint4*>(h0)[b] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
        }
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
            const uint32_t u = u0 + c;
            if (u * STEP >= L.n) continue;
            const uint32_t at = first_of(u), from = skip(u);
            if (gp) {
                val[u].x = accum(val[u].x, gv[c].x, P.momentum);
                val[u].y = accum(val[u].y, gv[c].y, P.momentum);
                val[u].z = accum(val[u].z, gv[c].z, P.momentum);
                val[u].w = accum(val[u].w, gv[c].w, P.momentum);
            }
            const float x[4] = {val[u].x, val[u].y, val[u].z, val[u].w}, y[4] = {wv[c].x, wv[c].y, wv[c].z, wv[c].w};
#pragma unroll
            for (uint32_t q = 0; q < VEC; ++q) {
                key[u][q] = q >= from && at + q < L.n ? score_key(x[q], y[q], eps) : NOT_AN_ELEMENT;
                zeros += key[u][q] == 0u ? 1u : 0u;
                // zero or NOT_AN_ELEMENT: not counted here
                atomicAdd(&h0[key[u][q] - 1u >= NOT_AN_ELEMENT - 1u ? D::BINS0 + D::BINS1 + D::BINS2 + lane : key[u][q] >> D::SHIFT0], 1u);
            }
            if (!FUSED && gp) store(u, val[u]);
        }
    }
    if (__any(zeros != 0)) {
        zeros = wave_sum(zeros);
        if (lane == 0) atomicAdd(&h0[0], zeros);
    }
    __syncthreads();
    uint32_t d0, d1, d2, rank;
    small_pick<D::BINS0, THREADS>(h0, L.k, part[0], &d0, &rank);
    auto count_in = [&](uint32_t* h, uint32_t prefix, int above, int shift, uint32_t bins) {    // elements with that prefix
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) {
            if (u * STEP >= L.n) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (key[u][q] >> above == prefix) atomicAdd(&h[(key[u][q] >> shift) & (bins - 1u)], 1u);
        }
        __syncthreads();
    };
    count_in(h1, d0, D::SHIFT0, D::SHIFT1, D::BINS1);      // NOT_AN_ELEMENT has bit 31 set: no prefix of a key
    small_pick<D::BINS1, THREADS>(h1, rank, part[1], &d1, &rank);
    d0 = d0 * D::BINS1 + d1;
    count_in(h2, d0, D::SHIFT1, 0, D::BINS2);
    small_pick<D::BINS2, THREADS>(h2, rank, part[2], &d2, &rank);
    const uint32_t thr = d0 * D::BINS2 + d2, quota = rank; // the k-th largest key, ties to keep
    if (thr_out && tid == 0) {
        iwp_threshold th;
        th.key = thr; th.n_gt = L.k - quota; th.n_eq_take = quota;
        thr_out[j] = th;
    }
    if (!emit) return;
    // elements above the threshold (low half) and tying with it (high half): inside the lane's quad, before the lane in
    // its wavefront, before the wavefront in index order (chunk by chunk, wavefront by wavefront)
    uint32_t before[CHUNKS], kept[CHUNKS];                 // kept: a bit per element above; in the next four bits: per tie
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        kept[u] = before[u] = 0u;
        if (u * STEP < L.n) {
            uint32_t mine = 0;
#pragma unroll
            for (uint32_t q = 0; q < VEC; ++q) {
                const bool above = key[u][q] > thr && key[u][q] != NOT_AN_ELEMENT, ties = key[u][q] == thr;
                mine += (above ? 1u : 0u) + (ties ? 0x10000u : 0u);
                kept[u] |= (above ? 1u << q : 0u) | (ties ? 16u << q : 0u);
            }
            const uint32_t inc = wave_inclusive_scan(mine);
            before[u] = inc - mine;
            if (lane == WAVE - 1) tot[u * WAVES + wave] = inc;
        } else if (lane == WAVE - 1) {
            tot[u * WAVES + wave] = 0u;
        }
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
        if (u * STEP >= L.n) continue;
        const uint32_t at = first_of(u);
        uint32_t g = before[u] & 0xffffu, e = before[u] >> 16, sent = 0;
        // element by element of those that are kept, not of all four
        for (uint32_t left = (kept[u] | kept[u] >> 4) & 0xFu; left; left &= left - 1u) {
            const uint32_t q = (uint32_t)__ffs((int)left) - 1u;
            const bool above = (kept[u] >> q) & 1u;
            const uint32_t pos = g + (above ? min(e, quota) : e);
            const bool keep = (above || e < quota) && pos < L.k;
            g += above ? 1u : 0u;
            e += above ? 0u : 1u;
            if (!keep) continue;
            const float low = q & 1u ? val[u].y : val[u].x, high = q & 1u ? val[u].w : val[u].z, x = q & 2u ? high : low;
            io[pos] = (uint32_t)(L.offset + at + q);
            vo[pos] = x;
            if (FUSED) {
                go[pos] = x;
                sent |= 1u << q;
                if (!gp) rl[at + q] = 0.0f;                // a worker that is not accumulated: only the sent positions
            }
        }
        if (FUSED && gp) {
            v4f t = val[u];
            t.x = sent & 1u ? 0.0f : t.x; t.y = sent & 2u ? 0.0f : t.y; t.z = sent & 4u ? 0.0f : t.z; t.w = sent & 8u ? 0.0f : t.w;
            store(u, t);
        }
    }
}

}  // namespace iwp
