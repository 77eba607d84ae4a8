// Shared device-side definitions of the gfx950 kernels: tile geometry, the
// importance key, quad (4 consecutive elements per lane) accesses, wavefront and
// workgroup scans, histogram pick and bitmap ranking.  Wavefronts are 64 lanes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/iwp.h"

// No fused multiply-add anywhere: the update is a rounded product followed by a
// rounded sum (Alg. 1 SGD line read as two fp32 operations).
#pragma clang fp contract(off)

namespace iwp {

typedef float v4f __attribute__((ext_vector_type(4)));   // one 128-bit access
// The same in memory at any multiple of 4 bytes: the hardware's 128-bit global accesses need no more than that, so
// a layer that starts anywhere in a flat buffer (a packed table, behind a tensor of odd length) moves at four
// elements per lane and access like any other.  Against one dword per lane and access on such layers, a thousand
// packed tensors of 115.5 M elements, eight workers: followers' pass 2401 -> 1881 us (4.1 -> 5.2 TB/s), leader pass 519
// -> 378 us, whole step 3285 -> 2704 us.  (Whole lines on top: see follow_tile_from.)
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

// Local accumulation with momentum (Eq. 3): the product is rounded, then the sum
// (contraction is off for the whole library).  m = 1 leaves the product exact, so the
// result is bit for bit the plain r + g.
__device__ __forceinline__ float accum(float r, float g, float m) {
    const float decayed = m * r;
    return decayed + g;
}

constexpr int BLOCK = 256;                         // 4 wavefronts
constexpr int WAVE = 64;
constexpr int VEC = 4;
constexpr uint32_t CHUNK = BLOCK * VEC;            // 1024 elements per workgroup iteration
constexpr uint32_t CHUNKS_PER_TILE = 4;
constexpr uint32_t TILE = CHUNK * CHUNKS_PER_TILE; // 4096 elements: the streaming unit (measured best on MI355X)
constexpr uint32_t GROUP = 8;                      // tiles per super-tile
#ifndef IWP_LGROUP
#define IWP_LGROUP 1                               // build-time tuning knob: -DIWP_LGROUP=1|2|4|8
#endif
constexpr uint32_t LGROUP = IWP_LGROUP;            // tiles that share one LDS histogram in look 1 (divides GROUP).
                                                   // With the first-digit histogram in several copies 1, 2 and 4 measure
                                                   // alike on the model-shaped sets; on a 10^9-element layer 1 streams
                                                   // about 6 % faster than 2
constexpr uint32_t STILE = TILE * GROUP;           // 32768 elements: unit of the leader-side passes
constexpr uint32_t TILE_WORDS = TILE / 32;         // words of a one-bit-per-element tile bitmap

// The 31-bit key (sign bit is always 0) is resolved most-significant digit first:
// 12 bits (exponent + 4 mantissa bits), then 10, then 9.
constexpr int DIGITS = 3;
__host__ __device__ constexpr int digit_shift(int level) { return level == 0 ? 19 : (level == 1 ? 9 : 0); }
__host__ __device__ constexpr int digit_bits(int level) { return level == 0 ? 12 : (level == 1 ? 10 : 9); }
constexpr uint32_t HIST0 = 1u << 12, HIST1 = 1u << 10, HIST2 = 1u << 9;
// A layer's histograms in the workspace: h0_copies copies of the first digit's (look 1 flushes one LDS
// histogram per workgroup with atomics, and atomics on one address serialise at about 20 ns each on this
// chip, so a layer with many workgroups spreads them over several copies), then one of the second
// digit's and one of the third's.
constexpr uint32_t MAX_H0_COPIES = 16;
// Look-1 workgroups that share one copy.  128 against 512: one layer of 1 M elements 39.2 -> 36.0 us a call, ten of 25 M 127
// -> 120, 161 of 25.6 M 130 -> 123 (thresholds and pairs); 256: 37.8, 120, 125; 64: 38.4, 120, 123.  The pick that adds the
// copies up pays for them.  512 (FEW) only in plans that would otherwise no longer fit the library's static scratch,
// or 32 bits.
constexpr uint32_t FLUSHES_PER_COPY = 128, FLUSHES_PER_COPY_FEW = 512;
__host__ __device__ constexpr uint32_t layer_hist_words(uint32_t copies) { return copies * HIST0 + HIST1 + HIST2; }

constexpr uint32_t RAW_TILE = 0xFFFFFFFFu;        // stage count of a tile whose candidates did not fit its slot
constexpr uint32_t UNIFORM_TILE = 0xFFFFFFFEu;    // stage count of such a tile whose keys are all the same (say, a tile of zero
                                                  // residuals): the key is the slot's only entry, and the later passes handle
                                                  // the tile from its element count instead of reading it again
constexpr uint32_t RESTAGED = 0x40000000u;        // flag on a stage count: look 2 filled this slot again (from b1) after look 1
                                                  // had overflowed it; look 2's reader of look-1 slots skips such tiles
// Entries in a tile's slot for the passes after look 2 (RAW_TILE and UNIFORM_TILE stay what they are).
__device__ __forceinline__ uint32_t staged_entries(uint32_t stage_count) {
    return stage_count >= UNIFORM_TILE ? stage_count : stage_count & ~RESTAGED;
}
constexpr uint32_t NO_STAGE_BIN = 0xFFFFFFFFu;    // LayerState.stage_bin: look 1 stages nothing for this layer
constexpr uint32_t NOT_AN_ELEMENT = 0xFFFFFFFFu;  // key slot of a lane position past the layer's end

struct alignas(64) DevLayer {      // a cache line's half: one scalar load
    uint64_t offset;       // first element in the flat buffers
    uint64_t slot_begin;   // first entry of the layer's first tile slot in the staging arrays
    uint32_t n;
    uint32_t k;
    uint32_t out_offset;   // first pair in idx_out / val_out
    uint32_t tile_begin;   // first TILE of the layer in the per-worker tile numbering
    uint32_t stile_begin;  // first STILE of the layer
    uint16_t slot_cap;     // staging entries per tile of this layer
    uint16_t h0_copies;    // copies of the first-digit histogram (a power of two)
    uint32_t mask_begin;   // first 32-bit word of the layer's encoded mask (threshold mode)
    uint32_t hist_begin;   // first word of the layer's histograms
    uint32_t sample;       // how k_init samples the layer: rank - 1 in the low half, runs in the high half
    uint32_t record_begin; // first of the layer's records outside its histograms (see tie_record)
};
static_assert(TILE <= 0xFFFF && MAX_H0_COPIES <= 0xFFFF, "16-bit fields of DevLayer");

// Where digit `level`'s histogram of a layer starts (level 0: the first copy).
__device__ __forceinline__ uint32_t* layer_hist(uint32_t* hist, const DevLayer& L, int level) {
    uint32_t* h = hist + L.hist_begin;
    return level == 0 ? h : (level == 1 ? h + L.h0_copies * HIST0 : h + L.h0_copies * HIST0 + HIST1);
}
__device__ __forceinline__ const uint32_t* layer_hist(const uint32_t* hist, const DevLayer& L, int level) {
    return layer_hist(const_cast<uint32_t*>(hist), L, level);
}

// What the ordered split needs to know of a unit (a tile, or a super-tile) before it can know the threshold's last digit: how many
// of its elements lie above the threshold's 22-bit prefix, how many share it (one word, the latter in the high half), and
// if any do, how many of those have a last digit of b or more, for every b: HIST2 counts of 16 bits (a unit holds at most
// 32768 elements), two to a word.  A layer's records lie in its first-digit histograms, which nobody reads any more by
// then; those that do not fit there lie apart.
constexpr uint32_t RECORD_WORDS = HIST2 / 2;
__host__ __device__ constexpr uint32_t records_inside(uint32_t copies) { return copies * (HIST0 / RECORD_WORDS); }
__device__ __forceinline__ uint32_t* tie_record(uint32_t* hist, uint32_t* apart, const DevLayer& L, uint32_t unit) {
    const uint32_t inside = records_inside(L.h0_copies);
    return unit < inside ? hist + L.hist_begin + unit * RECORD_WORDS
                         : apart + (size_t)(L.record_begin + unit - inside) * RECORD_WORDS;
}

struct LayerState {        // selection state of one layer, lives in the workspace.  Every field has one writer
                           // (one elected workgroup of one kernel) and is read only by later launches.
    uint32_t b1;           // top key digit of the threshold (first pick)
    uint32_t k_rem0;       // rank of the threshold inside that bin (1-based, counted from the largest key)
    uint32_t p22;          // top two digits (second pick)
    uint32_t k_rem1;       // rank inside that 22-bit group
    uint32_t thr;          // the threshold key (third pick, or given by the caller)
    uint32_t n_eq_take;    // ties to keep
    uint32_t stage_bin;    // look 1 copies out every element whose top digit is >= this bin (from the hint or a sample)
    uint32_t shift;        // what is added to every key of the layer before it is split into digits (see shifted())
    uint32_t prestaged;    // set with the first pick: stage_bin <= b1, so look 1's copies are complete
};

struct StageArrays {       // staged candidates, structure of arrays; tile t of a layer owns entries
    uint32_t* key;         // [slot_begin + t * slot_cap, + slot_cap), filled in index order
    uint32_t* idx;         // position inside the layer
    float* val;
};

struct WorkerPtrs {        // passed by value as a kernel argument
    const float* g[IWP_MAX_WORKERS];
    float* r[IWP_MAX_WORKERS];
    float momentum;        // local accumulation is r <- momentum * r + g (Eq. 3); 1 = plain accumulation
};

struct ResidualPtrs {
    float* r[IWP_MAX_WORKERS];
};

struct WorkerList {        // a subset of the workers, by index
    uint32_t n;
    uint8_t id[IWP_MAX_WORKERS];
};

// Importance of one element as an order-preserving integer (Alg. 1 mask line:
// |grad / w|, with eps added to |w| in fp32 before the correctly rounded divide).
__device__ __forceinline__ uint32_t score_key(float r, float w, float eps) {
    float denom = fabsf(w) + eps;
    float s = fabsf(r) / denom;
    return __float_as_uint(s) & 0x7fffffffu;
}

// The selection works on keys moved up by a layer's `shift` (less than one top-digit bin), which puts a bin's lower
// edge exactly at the key from which look 1 copies candidates out.  Keys of NaN (0 / 0 with eps = 0: quiet, from
// 0x7fc00000 up) stay where they are: a finite or infinite score ends below them shifted too, so the map keeps the
// order, loses nothing and ends inside 31 bits.
constexpr uint32_t QUIET_NAN_KEY = 0x7fc00000u;
__device__ __forceinline__ uint32_t shifted(uint32_t key, uint32_t shift) {
    return max(key, min(key + shift, QUIET_NAN_KEY - 1u));   // key + shift below the NaN keys, key itself among them
}
__device__ __forceinline__ uint32_t unshifted(uint32_t key, uint32_t shift) {
    return key - (key < QUIET_NAN_KEY ? shift : 0u);
}

// The worker that leads layer j.  The table lives in device memory, so it cannot
// be checked on the host: an entry that is out of range is read as worker 0, which
// keeps a bad entry from turning into a wild pointer.
__device__ __forceinline__ uint32_t leader_of(const uint32_t* __restrict__ leader, uint32_t j, uint32_t W) {
    const uint32_t l = leader ? leader[j] : 0u;
    return l < W ? l : 0u;
}

// Which layer does tile t belong to, or super-tile s.  Uniform across the workgroup.
// A table of more than one layer comes from a plan, which stores the answer behind the
// table's sentinel row: one word per tile, then one per super-tile (a binary search over a
// thousand layers is ten dependent loads before a workgroup can issue its first tile load).
__device__ __forceinline__ uint32_t layer_of_tile(const DevLayer* __restrict__ layers, uint32_t n_layers, uint32_t t) {
    return n_layers == 1 ? 0u : reinterpret_cast<const uint32_t*>(layers + n_layers + 1)[t];
}
__device__ __forceinline__ uint32_t layer_of_stile(const DevLayer* __restrict__ layers, uint32_t n_layers, uint32_t tiles,
                                                   uint32_t s) {
    return layer_of_tile(layers, n_layers, tiles + s);
}

// The chip's eight dies take consecutive workgroups in turn, so the workgroups of neighbouring tiles, which read the same table
// row, map words, pair positions and, where layers are packed, share a line, are on eight dies with an L2 each.  in_runs: the tile
// (numbered over all workers) of workgroup b of n such that each die gets runs of RUN consecutive ones; the last up to
// DIES * RUN - 1 workgroups stay as they are.  The followers' passes are run so where layers are short (RUN_TILES): their
// workgroups wait for that chain of loads less often.  us a step, one by one / in runs of 8: a thousand packed tensors of 115 M
// elements 2535 / 2430 (in runs of 4: 2503, 16: 2410, 32: 2450), 100 of 50 M 974 / 956 packed, 942 / 929 at multiples of
// 64, 60 packed of 100 M 1056 / 1046, 161 of 25.6 M 505 / 502 (16: 509, 32: 513), with statistics 527 / 523.  On few long layers
// there is nothing to share, and eight fronts through each buffer cost a little: one layer of 50 M 907 / 912 (4: 983, 16: 935),
// 16 of 61 M 1145 / 1148 (1222, 1165).
constexpr uint32_t DIES = 8, RUN = 8;
constexpr uint32_t RUN_TILES = 512;               // tiles per layer, on average, up to which runs are taken
__device__ __forceinline__ uint32_t in_runs(uint32_t b, uint32_t n) {
    const uint32_t first = b & ~(DIES * RUN - 1u), i = b - first;
    return n - first < DIES * RUN ? b : first + (i % DIES) * RUN + i / DIES;
}

template <bool NT>
__device__ __forceinline__ v4f load_v4(const float* p) {
    if (NT) return __builtin_nontemporal_load(reinterpret_cast<const v4f_any*>(p));
    return *reinterpret_cast<const v4f_any*>(p);
}
template <bool NT>
__device__ __forceinline__ void store_v4(float* p, v4f v) {
    if (NT) __builtin_nontemporal_store(v, reinterpret_cast<v4f_any*>(p));
    else *reinterpret_cast<v4f_any*>(p) = v;
}

// Four consecutive elements starting at element i of a layer of n elements: one 128-bit load, except at the layer's
// end.  Lanes past the end read nothing and get `fill`.
__device__ __forceinline__ void load_quad(const float* __restrict__ base, uint32_t i, uint32_t n, float (&v)[4],
                                          float fill = 0.0f) {
    if (i + 4 <= n) {
        const v4f t = load_v4<false>(base + i);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = (i + c < n) ? base[i + c] : fill;
    }
}

// NT: streaming (non-temporal) access for whole quads.
template <bool NT = false>
__device__ __forceinline__ void store_quad(float* __restrict__ base, uint32_t i, uint32_t n, const float (&v)[4]) {
    if (i + 4 <= n) {
        v4f t; t.x = v[0]; t.y = v[1]; t.z = v[2]; t.w = v[3];
        store_v4<NT>(base + i, t);
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) if (i + c < n) base[i + c] = v[c];
    }
}

// The 16 elements per lane of the tile that starts at element `base` of a layer of n elements, in one stretch of code
// for full and ragged tiles.  request_tile() only issues loads: the whole quads, and the up to three elements behind
// the layer's last whole quad, on the lane they belong to, into registers of their own; settle_tile() puts those into place
// once every array of the tile has been requested.  CHUNKS: fewer than CHUNKS_PER_TILE for tiles known to end there.  A second branch per quad for the elements behind the last whole one
// made the compiler wait for one quad before it asked for the next.  Values past the end are not meant for use.
// Against separate code for the two forms: look 1 364 -> 347 us, followers' pass 1898 -> 1877 us on a thousand packed
// tensors of 115.5 M elements; with thresholds, tables of 0.3 to 1.2 M elements 39.5 -> 35.5 and 61.3 -> 58.6 us a step.
struct Rest { float x[3]; };
template <uint32_t THREADS = BLOCK>
__device__ __forceinline__ bool holds_rest(uint32_t n, uint32_t base) {      // does this lane hold those elements?
    return base + TILE > n && (n & 3u) && (((n & ~3u) - base) & (THREADS * VEC - 1u)) == threadIdx.x * VEC;
}
template <bool NT, uint32_t THREADS = BLOCK, uint32_t CHUNKS>
__device__ __forceinline__ void request_tile(const float* __restrict__ p, uint32_t n, uint32_t base,
                                             float (&v)[CHUNKS][4], Rest& rest) {
    const float* pt = p + base;                              // uniform, with an offset of 32 bits per lane
    const uint32_t left = n - base;
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        const uint32_t i = (u * THREADS + threadIdx.x) * VEC;
        if (i + VEC <= left) {
            const v4f t = load_v4<NT>(pt + i);
            v[u][0] = t.x; v[u][1] = t.y; v[u][2] = t.z; v[u][3] = t.w;
        }
    }
    if (holds_rest<THREADS>(n, base)) {
        const uint32_t whole = n & ~3u;
#pragma unroll
        for (uint32_t c = 0; c < 3; ++c) rest.x[c] = p[min(whole + c, n - 1u)];
    }
}

template <uint32_t THREADS = BLOCK, uint32_t CHUNKS>
__device__ __forceinline__ void settle_tile(uint32_t n, uint32_t base, float (&v)[CHUNKS][4], const Rest& rest) {
    if (!holds_rest<THREADS>(n, base)) return;
    const uint32_t at = ((n & ~3u) - base) / (THREADS * VEC);          // which of the lane's quads
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
        for (int c = 0; c < 3; ++c) v[u][c] = u == at ? rest.x[c] : v[u][c];
}

// The keys behind the layer's end, which were computed from no element.
template <uint32_t THREADS = BLOCK, uint32_t CHUNKS>
__device__ __forceinline__ void leave_out_rest(uint32_t n, uint32_t base, uint32_t (&key)[CHUNKS][4]) {
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u)
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
            if (base + (u * THREADS + threadIdx.x) * VEC + q >= n) key[u][q] = NOT_AN_ELEMENT;
}

// Stores the tile's elements that lie inside the layer.
template <bool NT, uint32_t THREADS = BLOCK, uint32_t CHUNKS>
__device__ __forceinline__ void store_tile(float* __restrict__ p, uint32_t n, uint32_t base,
                                           const float (&v)[CHUNKS][4]) {
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) store_quad<NT>(p + base, (u * THREADS + threadIdx.x) * VEC, n - base, v[u]);
}

// Sums and scans across the 64 lanes of a wavefront, by data-parallel-primitive moves (row shifts by 1, 2, 4 and 8 lanes of
// 16, then the last lane of a row, and of two rows, broadcast to the rows behind): a handful of cycles a step, where a
// shuffle goes through the LDS unit and back.  All lanes of the wavefront take part.  The selection's kernels are chains of
// such scans and of the loads between them: with shuffles one layer of 1 M elements took 40.0 us a call, now 37.9, six
// tensors of 235 k elements and four workers 45.4 -> 43.0 us a step, one layer of 1000 elements 9.2 -> 8.5.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {        // 0 where the control names no lane
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
    x += dpp<0x111, 0xf>(x);                                 // row_shr 1, 2, 4, 8
    x += dpp<0x112, 0xf>(x);
    x += dpp<0x114, 0xf>(x);
    x += dpp<0x118, 0xf>(x);
    x += dpp<0x142, 0xa>(x);                                 // row_bcast 15 into rows 1 and 3
    x += dpp<0x143, 0xc>(x);                                 // row_bcast 31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t wave_last(uint32_t x) {  // lane 63's value, in all lanes
    return (uint32_t)__builtin_amdgcn_readlane((int)x, WAVE - 1);
}
__device__ __forceinline__ uint32_t from_lane(uint32_t x, uint32_t lane) {   // lane: the same in all lanes
    return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)lane);
}
// The wavefront's number in its workgroup, as a scalar: what is indexed by it then is, too.
__device__ __forceinline__ uint32_t wave_id() { return (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) { return wave_last(wave_inclusive_scan(x)); }
// The OR over each group of eight lanes, in all of them: quad_perm [1,0,3,2], [2,3,0,1], then the half row mirrored.
__device__ __forceinline__ uint32_t or_of_8_lanes(uint32_t x) {
    x |= dpp<0xB1, 0xf>(x);
    x |= dpp<0x4E, 0xf>(x);
    x |= dpp<0x141, 0xf>(x);
    return x;
}

// Exclusive scan over the 256 threads of a workgroup; *total receives the sum.
// `slot` (4 words of LDS) must not be reused before the next __syncthreads().
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* slot, uint32_t* total) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive_scan(x);
    if (lane == WAVE - 1) slot[wave] = inc;
    __syncthreads();
    const uint32_t w0 = slot[0], w1 = slot[1], w2 = slot[2], w3 = slot[3];
    const uint32_t before = (wave > 0 ? w0 : 0) + (wave > 1 ? w1 : 0) + (wave > 2 ? w2 : 0);
    *total = w0 + w1 + w2 + w3;
    return before + inc - x;
}

// Digit pick over a histogram of NB bins (LDS or global): the bin that holds rank
// k_rem counted from the top bin down, and the rank inside that bin.  All THREADS
// threads call it; the result is broadcast through `sh` (PICK_WORDS words of LDS).
// copies: histograms of NB bins one behind the other, added up.
// Requires sum(hist) >= k_rem >= 1.  Suffix sums inside each wavefront, then over the
// wavefronts' totals: three barriers, where a scan over all threads in LDS takes two per doubling.
constexpr uint32_t PICK_WORDS = 16 + 2;
template <int NB, int THREADS = BLOCK>
__device__ __forceinline__ void block_pick(const uint32_t* hist, uint32_t k_rem, uint32_t* sh,
                                           uint32_t* bin_out, uint32_t* k_rem_out, uint32_t copies = 1) {
    constexpr int PER = NB / THREADS, WAVES = THREADS / WAVE;
    static_assert(WAVES + 2 <= (int)PICK_WORDS, "one word per wavefront, two for the result");
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    uint32_t h[PER];
    uint32_t local = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) h[q] = hist[tid * PER + q];
#pragma unroll 4
    for (uint32_t c = 1; c < copies; ++c)
#pragma unroll
        for (int q = 0; q < PER; ++q) h[q] += hist[c * NB + tid * PER + q];
#pragma unroll
    for (int q = 0; q < PER; ++q) local += h[q];
    const uint32_t upto = wave_inclusive_scan(local), all = wave_last(upto);
    uint32_t incl = all - upto + local;    // this lane's bins and those of the lanes above it
    __syncthreads();                       // sh may still be in use by a previous call
    if (lane == 0) sh[wave] = incl;
    if (tid == 0) { sh[WAVES] = 0u; sh[WAVES + 1] = 1u; }
    __syncthreads();
#pragma unroll
    for (int v = 1; v < WAVES; ++v) incl += (int)wave < v ? sh[v] : 0u;
    const uint32_t above = incl - local;
    if (above < k_rem && k_rem <= incl) {  // true for exactly one thread
        uint32_t acc = above, bin = tid * PER;
#pragma unroll
        for (int q = PER - 1; q >= 0; --q) {
            if (acc + h[q] >= k_rem) { bin = tid * PER + q; break; }
            acc += h[q];
        }
        sh[WAVES] = bin;
        sh[WAVES + 1] = k_rem - acc;
    }
    __syncthreads();
    *bin_out = sh[WAVES];
    *k_rem_out = sh[WAVES + 1];
}

// The same pick by one wavefront, from a histogram in global memory that starts at a multiple of 16 bytes: no barriers, so a
// workgroup's wavefronts each do it for themselves.  For the later digits' histograms; the first digit's is too long for it.
template <int NB>
__device__ __forceinline__ void wave_pick(const uint32_t* __restrict__ hist, uint32_t k_rem, uint32_t* bin_out, uint32_t* k_rem_out) {
    constexpr int PER = NB / WAVE;
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    uint32_t h[PER], local = 0;
#pragma unroll
    for (int q = 0; q < PER; q += 4) {
        const uint4 x = reinterpret_cast<const uint4*>(hist)[(lane * PER + q) / 4];
        h[q] = x.x; h[q + 1] = x.y; h[q + 2] = x.z; h[q + 3] = x.w;
        local += x.x + x.y + x.z + x.w;
    }
    const uint32_t upto = wave_inclusive_scan(local);
    const uint32_t incl = wave_last(upto) - upto + local, above = incl - local;
    uint32_t acc = above, bin = 0, rest = 1;
    bool found = false;
#pragma unroll
    for (int q = PER - 1; q >= 0; --q) {
        const bool here = !found && acc + h[q] >= k_rem;
        bin = here ? lane * PER + q : bin;
        rest = here ? k_rem - acc : rest;
        found = found || here;
        acc += h[q];
    }
    const uint64_t hit = __ballot(above < k_rem && k_rem <= incl);         // one lane, if sum(hist) >= k_rem >= 1
    const uint32_t src = hit ? (uint32_t)__ffsll((unsigned long long)hit) - 1u : 0u;
    *bin_out = from_lane(bin, src);
    *k_rem_out = from_lane(rest, src);
}

// One bit per element of a tile.  prefix[w] = number of set bits in words < w.
// Called by all 256 threads after the bitmap is complete (and synchronised).
__device__ __forceinline__ void bitmap_prefix(const uint32_t* map, uint32_t* prefix, uint32_t* slot) {
    const uint32_t tid = threadIdx.x;
    const uint32_t c = tid < TILE_WORDS ? __popc(map[tid]) : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(c, slot, &tot);
    if (tid < TILE_WORDS) prefix[tid] = ex;
    __syncthreads();
}

// Number of set bits strictly below position `local` of the tile.
__device__ __forceinline__ uint32_t bitmap_rank(const uint32_t* map, const uint32_t* prefix, uint32_t local) {
    const uint32_t wd = local >> 5, b = local & 31u;
    return prefix[wd] + __popc(map[wd] & ((1u << b) - 1u));
}

// Of a tile's marked elements, how many stand before each lane's quads.  n[u]: marked elements (0 to 4) in the lane's quad of
// chunk u (the lane's elements are consecutive, chunks follow each other); first[u]: marked ones of the tile before that
// quad.  Returns the tile's total.  All threads call it; `slot`: STAGE_WORDS words of LDS, not to be used again before
// the next __syncthreads().
constexpr uint32_t STAGE_WORDS = 16;                        // a word per wavefront and pair of chunks
template <uint32_t THREADS = BLOCK, uint32_t CHUNKS>
__device__ __forceinline__ uint32_t tile_ranks(const uint32_t (&n)[CHUNKS], uint32_t (&first)[CHUNKS], uint32_t* slot) {
    static_assert(CHUNKS <= 4 && TILE < 65536, "two chunks' counts in one word");
    constexpr uint32_t PAIRS = (CHUNKS + 1) / 2;
    static_assert(PAIRS * (THREADS / WAVE) <= STAGE_WORDS, "a word per wavefront and pair of chunks");
    const uint32_t lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x >> 6;
    uint32_t c[PAIRS] = {}, inc[PAIRS], before[PAIRS], tot[PAIRS];
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) c[u / 2] += n[u] << (16 * (u % 2));
#pragma unroll
    for (uint32_t h = 0; h < PAIRS; ++h) {
        inc[h] = wave_inclusive_scan(c[h]);
        if (lane == WAVE - 1) slot[PAIRS * wave + h] = inc[h];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t h = 0; h < PAIRS; ++h) {
        before[h] = inc[h] - c[h];
        tot[h] = 0;
#pragma unroll
        for (uint32_t v = 0; v < THREADS / WAVE; ++v) {
            const uint32_t x = slot[PAIRS * v + h];
            before[h] += v < wave ? x : 0u;
            tot[h] += x;
        }
    }
    uint32_t done = 0;                                       // of the chunks so far
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        first[u] = done + (before[u / 2] >> (16 * (u % 2)) & 0xffffu);
        done += tot[u / 2] >> (16 * (u % 2)) & 0xffffu;
    }
    return done;
}

// Copy the elements of one tile whose key is >= from into the tile's slot,
// in index order, so that the ordered split can rank a slot's entries by their place in it.  key[u][q] / val[u][q]: the
// lane's element q of chunk u (the lane's elements are consecutive, chunks follow each other), NOT_AN_ELEMENT past
// the layer's end.  Returns the number of copies, or RAW_TILE if they exceed the
// slot (then nothing is written).  All threads call it; `slot`: STAGE_WORDS words of LDS, not to be used again
// before the next __syncthreads().
template <uint32_t THREADS = BLOCK, uint32_t CHUNKS>
__device__ __forceinline__ uint32_t stage_tile(const uint32_t (&key)[CHUNKS][4],
                                               const float (&val)[CHUNKS][4], uint32_t base, uint32_t from,
                                               uint32_t cap, uint64_t sb, const StageArrays& A, uint32_t* slot) {
    // as signed numbers NOT_AN_ELEMENT is less than any key (`from` beyond them all, from a caller's record: nothing of it is kept)
    const int32_t least = (int32_t)min(from, 0x7fffffffu);
    uint32_t n[CHUNKS], first[CHUNKS], any = 0u;
#pragma unroll
    for (uint32_t u = 0; u < CHUNKS; ++u) {
        n[u] = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) n[u] += (int32_t)key[u][q] >= least ? 1u : 0u;
        any |= n[u];
    }
    const uint32_t tot = tile_ranks<THREADS>(n, first, slot);
    if (tot > cap) return RAW_TILE;
    if (any) {
        // uniform pointers and a byte offset of 32 bits: one address register for the three stores
        char* const key_to = reinterpret_cast<char*>(A.key + sb);
        char* const idx_to = reinterpret_cast<char*>(A.idx + sb);
        char* const val_to = reinterpret_cast<char*>(A.val + sb);
#pragma unroll
        for (uint32_t u = 0; u < CHUNKS; ++u) {
            uint32_t at = first[u] * (uint32_t)sizeof(uint32_t);
            const uint32_t i = base + (u * THREADS + threadIdx.x) * VEC;
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                if ((int32_t)key[u][q] >= least) {
                    *reinterpret_cast<uint32_t*>(key_to + at) = key[u][q];
                    *reinterpret_cast<uint32_t*>(idx_to + at) = i + q;
                    *reinterpret_cast<float*>(val_to + at) = val[u][q];
                    at += (uint32_t)sizeof(uint32_t);
                }
        }
    }
    return tot;
}

}  // namespace iwp
