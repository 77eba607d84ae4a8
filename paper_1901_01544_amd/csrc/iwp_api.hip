// Host side of the C ABI declared in include/iwp.h: argument checks, workspace
// carving and the launch sequences.  Every compute step runs in the kernels of
// iwp_stream.hpp / iwp_select.hpp / iwp_exchange.hpp; nothing here touches element
// data and nothing falls back to the CPU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "iwp_common.hpp"
#include "iwp_exchange.hpp"
#include "iwp_select.hpp"
#include "iwp_small.hpp"
#include "iwp_stream.hpp"
#include "iwp_sum.hpp"
#include "iwp_threshold.hpp"

using namespace iwp;

namespace {

thread_local char g_hip_error[256] = "";

int hip_fail(hipError_t e, const char* what) {
    snprintf(g_hip_error, sizeof g_hip_error, "%s: %s", what, hipGetErrorString(e));
    return IWP_EHIP;
}

#define IWP_HIP(call)                                         \
    do {                                                      \
        hipError_t e_ = (call);                               \
        if (e_ != hipSuccess) return hip_fail(e_, #call);     \
    } while (0)

// Optional timing of one named kernel with HIP events on the stream it is launched
// on (iwp_timing_*): off by default, costs one string compare per launch when on.
struct Timing {
    static constexpr int MAX = 8192;
    bool enabled = false;
    char name[64] = "";
    std::vector<hipEvent_t> start, stop;
    int used = 0;
} g_timing;

struct TimedLaunch {       // records an event pair around the launch made while it is alive
    hipStream_t s;
    int slot = -1;
    TimedLaunch(const char* kernel, hipStream_t stream) : s(stream) {
        if (!g_timing.enabled || strcmp(kernel, g_timing.name) != 0) return;
        if (g_timing.used >= (int)g_timing.start.size()) return;
        slot = g_timing.used++;
        (void)hipEventRecord(g_timing.start[slot], s);
    }
    ~TimedLaunch() {
        if (slot >= 0) (void)hipEventRecord(g_timing.stop[slot], s);
    }
};

// Launch `kernel<<<grid, BLOCK, lds, s>>>(args...)`, timed if asked for, and turn a
// launch failure into IWP_EHIP.  lds: bytes of LDS that no one uses, see few_at_a_time().
#define IWP_LAUNCH(name, kernel, grid, s, ...) IWP_LAUNCH_AS(name, kernel, grid, BLOCK, 0u, s, __VA_ARGS__)
#define IWP_LAUNCH_BLOCK(name, kernel, grid, block, s, ...) IWP_LAUNCH_AS(name, kernel, grid, block, 0u, s, __VA_ARGS__)
#define IWP_LAUNCH_FEW(name, kernel, grid, lds, s, ...) IWP_LAUNCH_AS(name, kernel, grid, BLOCK, lds, s, __VA_ARGS__)
#define IWP_LAUNCH_AS(name, kernel, grid, block, lds, s, ...)         \
    do {                                                              \
        {                                                             \
            TimedLaunch tl_(name, s);                                 \
            kernel<<<(grid), (block), (lds), (s)>>>(__VA_ARGS__);     \
        }                                                             \
        hipError_t e_ = hipGetLastError();                            \
        if (e_ != hipSuccess) return hip_fail(e_, name);              \
    } while (0)

// Scratch of compress_segmented_static: device memory that belongs to the library, one copy per
// GPU, held until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; kernels and fills are given the address that call returns, looked up once
// per device with that device current.
static __device__ __align__(256) unsigned char scratch[IWP_STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[MAX_DEVICES] = {};

int static_scratch(void** out) {
    int dev = -1;
    IWP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return IWP_EINVAL;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        IWP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return IWP_EALIGN;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return IWP_OK;
}

inline bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }
inline size_t round256(size_t x) { return (x + 255) & ~size_t(255); }
inline uint32_t tiles_of(uint32_t n) { return (uint32_t)(((uint64_t)n + TILE - 1) / TILE); }
inline uint32_t stiles_of(uint32_t n) { return (uint32_t)(((uint64_t)n + STILE - 1) / STILE); }
// Staging entries per tile of a layer: three times the number of kept elements an
// average tile holds, twice what look 1 copies from its sampled mark (about 1.5 per
// kept element), plus 64 for tiles that hold more than the average.  A tile that
// overflows its slot is re-read by the later passes instead, which is exact as well.
inline uint32_t slot_cap_of(uint32_t n, uint32_t k) {
    if (k == 0) return 0u;
    const uint64_t per_tile = ((uint64_t)TILE * k + n - 1) / n;
    return (uint32_t)std::min<uint64_t>(TILE, 64 + 3 * per_tile);
}

// On small tables (looks_twice(), see LOOK_TWICE_TILES in iwp_select.hpp) the second look can have to copy out
// whole bins of the first digit: up to 1/16 of a tile where the scores lie evenly below the threshold, for which their slots
// have LOOK_TWICE_ROOM entries more.  Larger tables hold the same number of entries in reserve, so that a workspace that fits a table fits
// the smaller ones of its kind.
inline uint32_t roomy(uint32_t slot_cap) { return slot_cap ? std::min<uint32_t>(TILE, slot_cap + LOOK_TWICE_ROOM) : 0u; }
inline uint64_t roomy_reserve(uint64_t tiles) { return std::min<uint64_t>(tiles, LOOK_TWICE_TILES_MANY) * LOOK_TWICE_ROOM; }
// Likewise for the records of their tiles.
inline uint32_t record_reserve(uint64_t tiles) { return (uint32_t)std::min<uint64_t>(tiles, LOOK_TWICE_TILES_MANY); }
inline bool looks_twice(uint64_t tiles, uint32_t n_layers) {
    return tiles <= LOOK_TWICE_TILES || (tiles <= LOOK_TWICE_TILES_MANY && n_layers >= LOOK_TWICE_MANY);
}

// How k_init samples a layer: enough runs for the threshold's rank in the sample to be about SAMPLE_RANK, and the rank
// of the sample's element from whose key look 1 copies out (see iwp_select.hpp).
uint32_t sample_of(uint32_t n, uint32_t k) {
    if (n == 0 || k == 0) return 0u;
    const uint64_t runs_total = ((uint64_t)n + SAMPLE_RUN - 1) / SAMPLE_RUN;
    const uint64_t want = ((uint64_t)SAMPLE_RANK * n / k + SAMPLE_RUN - 1) / SAMPLE_RUN;
    const uint64_t runs = std::min({runs_total, (uint64_t)SAMPLE_RUNS, std::max<uint64_t>(SAMPLE_RUNS_MIN, want)});
    uint64_t rank = k;                                   // the whole layer
    if (runs < runs_total) {
        const uint64_t sampled = runs * SAMPLE_RUN;      // only a layer's last run can be short
        const uint64_t ks = std::max<uint64_t>(1, ((uint64_t)k * sampled + n - 1) / n);
        rank = std::min<uint64_t>(sampled, ks + ks / 4 + (uint64_t)(4.0 * std::sqrt((double)ks)) + 2);
    }
    return (uint32_t)(runs << 16 | (rank - 1));
}

// Copies of a layer's first-digit histogram: one per `flushes` look-1 workgroups, a power of two.
inline uint32_t h0_copies_of(uint32_t n, uint32_t k, uint32_t flushes = FLUSHES_PER_COPY) {
    if (k == 0) return 1u;
    const uint32_t groups = (tiles_of(n) + LGROUP - 1) / LGROUP;
    uint32_t c = 1;
    while (c < MAX_H0_COPIES && c * flushes < groups) c <<= 1;
    return c;
}

// Plans whose slots hold at most RECORD_MAX_CAP entries (an eighth of the elements kept) and whose layers at most RECORD_MAX_STILES
// super-tiles go by records.  Fuller slots are read twice by k_split: 25 M elements kept at 0.1 gain 0 to 1 %, small tables still 8.  Longer
// layers have every workgroup add up thousands of records; with a launch that does so once, 400 M elements kept at 1/1000
// took 107 us where k_count, k_scan and k_write take 75.
constexpr uint32_t RECORD_MAX_CAP = 64 + 3 * TILE / 8, RECORD_MAX_STILES = 4096;
inline bool goes_by_records(uint32_t max_cap, uint32_t max_stiles) {
    return max_cap <= RECORD_MAX_CAP && max_stiles <= RECORD_MAX_STILES;
}
// Units (see tie_record) of a layer, and how many of their records do not fit into its first-digit histograms.  Longer layers and
// fuller slots, which do not go by records, count as the longest layer that does, 4 MB at most, so that a workspace that fits
// them fits shorter and sparser ones.
inline uint32_t records_apart(uint32_t n, uint32_t k, uint32_t copies, bool per_tile) {
    const uint32_t units = k == 0 ? 0u : per_tile ? tiles_of(n) : std::min(stiles_of(n), RECORD_MAX_STILES);
    const uint32_t inside = records_inside(copies);
    return units > inside ? units - inside : 0u;
}

struct Sizes {                // everything the workspace layout depends on
    uint32_t n_layers, tiles, stiles;
    uint64_t pairs, slots;    // slots: staging entries over all tiles
    uint64_t mask_words;      // 32-bit words of all layers' encoded masks (threshold mode)
    uint64_t hist_words;      // words of all layers' histograms
    uint64_t records;         // units' records outside the histograms (see tie_record)
    uint32_t W_gather;        // rows of the gather matrix (whole-step entry point), else 0
};

// Carving of a caller-supplied workspace.
struct Workspace {
    DevLayer* single_table;   // 2 rows, used by the single-layer entry points
    uint64_t hist_words;      // what k_init clears
    uint32_t* hist;           // hist_words
    LayerState* state;        // n_layers
    uint32_t* stage;          // tiles: staged entries per tile, or RAW_TILE
    uint2* tile_counts;       // tiles
    uint2* stile_counts;      // stiles
    uint32_t* tile_out;       // tiles
    uint32_t* records;        // RECORD_WORDS each
    StageArrays A;            // `slots` entries each
    float* gathered;          // W_gather * pairs
    size_t bytes;
};

Workspace carve(void* base, const Sizes& z) {
    Workspace ws;
    const uintptr_t b = reinterpret_cast<uintptr_t>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) { uintptr_t p = b + off; off += round256(bytes); return p; };
    ws.single_table = reinterpret_cast<DevLayer*>(take(2 * sizeof(DevLayer)));
    const size_t hist_bytes = round256((size_t)z.hist_words * sizeof(uint32_t));
    const size_t state_bytes = round256((size_t)z.n_layers * sizeof(LayerState));
    ws.hist = reinterpret_cast<uint32_t*>(take(hist_bytes));
    ws.state = reinterpret_cast<LayerState*>(take(state_bytes));
    ws.hist_words = z.hist_words;
    ws.stage = reinterpret_cast<uint32_t*>(take((size_t)z.tiles * sizeof(uint32_t)));
    ws.tile_counts = reinterpret_cast<uint2*>(take((size_t)z.tiles * sizeof(uint2)));
    ws.stile_counts = reinterpret_cast<uint2*>(take((size_t)z.stiles * sizeof(uint2)));
    ws.tile_out = reinterpret_cast<uint32_t*>(take((size_t)z.tiles * sizeof(uint32_t)));
    ws.records = reinterpret_cast<uint32_t*>(take(z.records * RECORD_WORDS * sizeof(uint32_t)));
    ws.A.key = reinterpret_cast<uint32_t*>(take(z.slots * sizeof(uint32_t)));
    ws.A.idx = reinterpret_cast<uint32_t*>(take(z.slots * sizeof(uint32_t)));
    ws.A.val = reinterpret_cast<float*>(take(z.slots * sizeof(float)));
    ws.gathered = reinterpret_cast<float*>(take((size_t)z.W_gather * z.pairs * sizeof(float)));
    ws.bytes = off;
    return ws;
}

struct Table {                // what the launches need to know about a layer table
    const DevLayer* layers;   // device, n_layers rows + sentinel
    uint32_t n_layers, tiles, stiles;
    uint64_t pairs;
    bool any_k;
    uint32_t max_layer_stiles;   // super-tiles of the longest layer
    uint32_t max_copies;         // copies of its first-digit histogram
    bool look_twice;             // roomy slots, no sampled mark (LOOK_TWICE_TILES)
    bool by_records;             // the split goes by the units' records
    bool long_sparse;            // a layer of more than FOLD_SCAN_MAX_STILES super-tiles, and no slot of more than SPARSE_MAX_CAP entries
};

// Up to this many super-tiles per layer (128 Mi elements) k_write adds up the earlier super-tiles'
// counts itself (16 loads per thread at most); beyond, a scan launch is cheaper.
constexpr uint32_t FOLD_SCAN_MAX_STILES = 4096;
// Up to this many entries a slot (one of 170 elements kept), such tables' third digit, counts and pairs are found by wavefronts that take
// a super-tile or two at once (k_count_stiles).  Fuller slots have them go
// through most tiles one after the other: 300 M elements kept at 1/120 alike, at 1/64 1458 -> 1519 us a step.
constexpr uint32_t SPARSE_MAX_CAP = 64 + 3 * 24;
inline bool is_long_sparse(uint32_t max_cap, uint32_t max_stiles) {
    return max_stiles > FOLD_SCAN_MAX_STILES && max_cap <= SPARSE_MAX_CAP;
}

// Do the followers' passes take the tiles in runs (see in_runs)?
uint32_t takes_runs(uint32_t tiles, uint32_t n_layers) { return tiles <= (uint64_t)RUN_TILES * n_layers ? 1u : 0u; }

// LDS for a launch to ask for so that a compute unit holds no more than `resident` of its workgroups at a time.  The passes over
// whole buffers are bound by what the memory delivers, and it delivers more to fewer streams, as long as these keep it busy.
// own: what LDS the kernel itself has, or a little more; LDS is given out in pieces of 1280 bytes.
constexpr uint32_t LDS_BYTES = 160u << 10, LDS_PIECE = 1280;
constexpr uint32_t few_at_a_time(uint32_t resident, uint32_t own) {
    return LDS_BYTES / resident / LDS_PIECE * LDS_PIECE - own;
}

// Which tables that pays on.  Tiles that end early keep less on their way: ten thousand layers of 3000 elements take 101 us in look 1
// and 425 in the followers' pass, 111 and 484 four at a time; three thousand of 10000 elements 90 and 90, 430 and 413.
bool fills_tiles(uint32_t tiles, uint32_t n_layers) { return tiles >= 2 * n_layers; }

// Followers, n of them accumulating: 8 workers, a thousand tensors of 115.5 M elements, 1692 us with the eight workgroups a compute
// unit that the registers allow, 1632 with four, 20 % more with two; eight tensors of 62.4 M, 857 and 818.  Three workers, 120 M in
// one tensor, 468 and 457; two, 25 M in 16, 56.7 and 58.  Where many elements are sent, and written to the matrix as well, eight are better:
// 20 M of 4 workers 309 and 310 us a step at 1 / 10, 373 and 391 at 1 / 5; 12.5 M of 12, all of them, 1118 and 1252.
constexpr uint32_t FOLLOW_LDS = 2048;
uint32_t few_followers(const Table& T, uint32_t n) {
    return n >= 3 && fills_tiles(T.tiles, T.n_layers) && T.pairs * 16 <= (uint64_t)T.tiles * TILE ? few_at_a_time(4, FOLLOW_LDS) : 0u;
}

// Followers of a mask, n of them accumulating, in runs (others lose: 62.4 M in eight tensors 760 us, 775 five at a time): 8 workers, 25 M
// elements in 160 tensors 345 us, 332 five at a time, 335 four; 40 M in a thousand 458 and 440.  The last round costs more than that
// where there are few: 3 M in three tensors 44.8 and 46.3.
constexpr uint32_t MANY_ROUNDS = 16 * 5 * 256;        // workgroups: sixteen times what is resident
uint32_t few_mask_followers(uint32_t tiles, uint32_t n_layers, uint32_t n) {
    return n >= 4 && (uint64_t)n * tiles >= MANY_ROUNDS && fills_tiles(tiles, n_layers) ? few_at_a_time(5, FOLLOW_LDS) : 0u;
}

// Look 1, where it accumulates (a selection's, which stores nothing but candidates, is the faster the more are there: 25.6 M elements
// 46 us, 50 four at a time): 115.5 M in a thousand tensors 344.8 -> 333.3 us, 268 M in one 1105 -> 1087, 62.4 M in eight 169.5 -> 165.3;
// 1000 x 8000 elements 31.1 -> 32.2, 25.6 and 36 M alike, which is why smaller tables go without.  Statistics, 25.6 M: 73.2 -> 71.7.
constexpr uint64_t FEW_LEADERS_MIN_BYTES = 160ull << 20;
constexpr uint32_t LEAD_LDS = HIST0 * sizeof(uint32_t) + 512, FEW_READERS = few_at_a_time(4, 256);

// The reduction of `pairs` values with their update, where these are far apart: 62.4 M / 64 of 8 workers 51.6 -> 48.8 us, 268 M / 64 of one
// 185.6 -> 182.5; no difference at 1 / 20; all of 21 M elements of 7 workers are 20 % slower.  (The updates that follow a count on the
// device, or a caller's list, gain as much, 33.8 -> 31.0 and 21.5 -> 19.7 us, but the host cannot see how dense theirs are.)
uint32_t few_updates(uint32_t tiles, uint64_t pairs) { return pairs * 32 <= (uint64_t)tiles * TILE ? few_at_a_time(3, 0) : 0u; }

int check_eps(float eps) { return (eps >= 0.0f && std::isfinite(eps)) ? IWP_OK : IWP_EINVAL; }

// Sampling source of a call: the leaders' residuals and gradients (NULL entries allowed), or nothing (on: false, or no w).
SampleSource sample_from(const WorkerPtrs& P, const float* w, const uint32_t* leader, uint32_t W, float eps, bool on = true) {
    SampleSource S;
    S.P = P; S.w = w; S.leader = leader; S.W = W; S.eps = eps; S.on = w && on ? 1u : 0u; S.trust_hint = 0u;
    return S;
}

int launch_init(const Workspace& ws, uint32_t n_layers, uint32_t tiles, const iwp_threshold* hint, const DevLayer* layers,
                const DevLayer* row, const DevLayer* sentinel, SampleSource S, hipStream_t s) {
    if (hint && S.P.momentum == 1.0f && (tiles <= HINT_MAX_TILES || tiles / n_layers < STAGE_GROUP))
        S.trust_hint = n_layers <= HINT_FEW_LAYERS ? TRUST_ALWAYS : TRUST_DENSE;
    uint32_t zero_blocks = (uint32_t)std::min<uint64_t>((ws.hist_words + 4 * INIT_BLOCK - 1) / (4 * INIT_BLOCK), 1024);
    if (zero_blocks == 0) zero_blocks = 1;
    DevLayer zero;
    memset(&zero, 0, sizeof zero);
    IWP_LAUNCH_BLOCK("k_init", k_init, n_layers + zero_blocks, INIT_BLOCK, s, ws.hist, ws.hist_words, ws.state, zero_blocks, hint, layers,
               row ? ws.single_table : nullptr, row ? *row : zero, sentinel ? *sentinel : zero, S);
    return IWP_OK;
}

enum Stop { STOP_AT_THRESHOLD, FULL };

// Workgroups of look 1: one per tile, or GROUP / LGROUP per super-tile when a workgroup takes several tiles.
constexpr uint32_t leader_grid(uint32_t tiles, uint32_t stiles) {
    return LGROUP == 1 ? tiles : stiles * (GROUP / LGROUP);
}

// Up to these table sizes (bytes of one flat buffer's share of the table) look 1 leaves the weights, or the weights
// and the residual it writes, in the memory-side cache for the kernels that come back to them (see lead_tile).  Three
// states in turn / one state alone, us a call of one worker, r and w kept, w kept, nothing kept: 8 M elements 56.7 / 58.5, 57.6 /
// 59.4, 58.9 / 60.7; 15 M 97.0 / 83.9, 87.7 / 85.7, 88.1 / 87.8; 25.6 M 161 / 124.6, 142.7 / 124.4, 134.2 / 129.1; 36 M 208 / 166, 184 /
// 155.6, 176 / 163; whole steps of eight workers, w kept, nothing: 25.6 M 484 / 461, 477 / 466, 36 M 655 / 629, 650 / 632.  What one
// state alone gains beyond 64 MiB is what is left in the cache from call to call.  With 300 MB (1.2 GB) of other copies between the calls, as
// a training step has them, on one state, w kept, nothing: 17 M 104.9, 103.3 (106.9, 103.7), 25.6 M 144.2, 139.9 (143.5, 139.3), 36 M
// 181.2, 176.5 (179.6, 175.2), steps of eight workers 17 M 337, 334, 25.6 M 484.5, 478.5, 36 M 661, 651.
// Without a gradient (a selection) nothing is written, and the pairs' pass reads again what was read: 25.6 M 114.9 with w kept, 116.6.
constexpr uint64_t KEEP_W_AND_R_MAX_BYTES = 40ull << 20, KEEP_W_MAX_BYTES = 64ull << 20, KEEP_W_MAX_BYTES_READ_ONLY = 160ull << 20;

// Threads of a workgroup, which has one tile: 512 instead of 256 halve what each wavefront issues, and that is what counts where the chip
// holds all workgroups at once, or nearly, and where a gradient is streamed up to some rounds of them.  us a call, 256 / 512 in look
// 1, in look 2 (k_stage<true>), in the records' pass: one layer of 0.1 M elements 22.1 / 21.3, 21.1, - ; of 1 M 25.4 / 25.4, 24.3, -,
// in both 23.4 (1024: 24.5, 24.9); thresholds and pairs of 1 M 33.1 / 32.6, 32.3, 32.4.  Look 1: 8 M in one layer 55.6 / 54.3, one worker's
// share of 25.6 M 135.3 / 133.3, a whole step of eight on it 479.3 / 476.9, 36 M 177.3 / 174.6; without a gradient 25.6 M 114.7 / 115.9, 50 M
// 198 / 205; beyond 160 MiB a thousand tensors 2326 / 2345.  Look 2: 2.5 M 39.1 / 39.1, 4 M in 60 layers 40.3 / 40.8, 8 M in 40 62.8 /
// 64.1.  The records' pass: 8 M in 40 layers 62.8 / 62.2, 15 M in 100 81.0 / 81.4.  Masks of up to three nodes: 20 k elements 11.8 / 11.0,
// two nodes 14.7 / 13.5, 1 M, two nodes 24.7 / 23.6, with random selection 30.1 / 27.9, 10 M 109.3 / 108.0, three nodes 108.3 / 107.5.
constexpr uint32_t WIDE_BLOCK = 512;
constexpr uint32_t WIDE_STAGE_MAX_TILES = 512, WIDE_MASK_MAX_TILES = 2560;
constexpr uint64_t WIDE_LEADERS_MAX_BYTES = FEW_LEADERS_MIN_BYTES;

inline uint64_t buffer_bytes(const Table& T) { return (uint64_t)T.tiles * TILE * sizeof(float); }

int launch_leader_pass(const Table& T, const Workspace& ws, const WorkerPtrs& P, const float* w, const uint32_t* leader,
                       uint32_t W, float eps, hipStream_t s) {
    const uint32_t grid = leader_grid(T.tiles, T.stiles);
    const uint64_t bytes = buffer_bytes(T);
    bool accumulates = false;
    for (uint32_t p = 0; p < W; ++p) accumulates |= P.g[p] != nullptr;
#define IWP_LOOK1(KEEP, THREADS, LDS)                                                                                            \
    IWP_LAUNCH_AS("k_leader_pass", (k_leader_pass<LGROUP, KEEP, THREADS>), grid, THREADS, LDS, s, P, w, T.layers, T.n_layers,    \
                  leader, W, eps, ws.hist, ws.state, ws.stage, ws.A)
    if (bytes <= KEEP_W_AND_R_MAX_BYTES) IWP_LOOK1(KEEP_W_AND_R, WIDE_BLOCK, 0u);
    else if (bytes <= (accumulates ? KEEP_W_MAX_BYTES : KEEP_W_MAX_BYTES_READ_ONLY)) IWP_LOOK1(KEEP_W, BLOCK, 0u);
    else if (accumulates && bytes <= WIDE_LEADERS_MAX_BYTES) IWP_LOOK1(KEEP_NOTHING, WIDE_BLOCK, 0u);
    else IWP_LOOK1(KEEP_NOTHING, BLOCK, accumulates && fills_tiles(T.tiles, T.n_layers) ? few_at_a_time(4, LEAD_LDS) : 0u);
#undef IWP_LOOK1
    return IWP_OK;
}

template <bool FUSED>
int launch_write(const Table& T, const Workspace& ws, const ResidualPtrs& R, const float* w, const uint32_t* leader,
                 uint32_t W, float eps, uint32_t* idx_out, float* val_out, hipStream_t s) {
    const uint32_t grid = T.stiles * (GROUP / (BLOCK / WAVE));
    float* gathered = FUSED ? ws.gathered : nullptr;
    if (T.max_layer_stiles <= FOLD_SCAN_MAX_STILES) {
        IWP_LAUNCH("k_write", (k_write<FUSED, FOLD_STILES>), grid, s, R, w, T.layers, T.n_layers, T.tiles, leader, W, eps, ws.state,
                   ws.stage, ws.A, ws.tile_counts, ws.stile_counts, ws.tile_out, idx_out, val_out, gathered,
                   T.pairs);
    } else {
        IWP_LAUNCH_BLOCK("k_scan", k_scan, T.n_layers, SCAN_BLOCK, s, T.layers, ws.stile_counts);
        if (T.long_sparse)
            IWP_LAUNCH("k_write_stiles", k_write_stiles<FUSED>, (T.stiles + BLOCK / WAVE - 1) / (BLOCK / WAVE), s, R, w, T.layers,
                       T.n_layers, T.tiles, T.stiles, leader, W, eps, ws.state, ws.stage, ws.A, ws.tile_counts, ws.stile_counts,
                       ws.tile_out, idx_out, val_out, gathered, T.pairs);
        else
            IWP_LAUNCH("k_write", (k_write<FUSED, FOLDED>), grid, s, R, w, T.layers, T.n_layers, T.tiles, leader, W, eps, ws.state,
                       ws.stage, ws.A, ws.tile_counts, ws.stile_counts, ws.tile_out, idx_out, val_out, gathered, T.pairs);
    }
    return IWP_OK;
}

template <bool FUSED>
int launch_split(const Table& T, const Workspace& ws, const ResidualPtrs& R, const float* w, const uint32_t* leader,
                 uint32_t W, float eps, iwp_threshold* thr_out, uint32_t* idx_out, float* val_out, hipStream_t s) {
    const uint32_t* units = reinterpret_cast<const uint32_t*>(ws.tile_counts);
    float* gathered = FUSED ? ws.gathered : nullptr;
#define IWP_SPLIT(BEFORE)                                                                                                        \
    IWP_LAUNCH_BLOCK("k_split", (k_split<FUSED, BEFORE>), T.stiles, SPLIT_BLOCK, s, R, w, T.layers, T.n_layers, T.tiles, leader, W, \
                     eps, ws.state, ws.hist, units, ws.records, ws.stage, ws.A, thr_out, ws.tile_out, idx_out,    \
                     val_out, gathered, T.pairs)
    if (T.look_twice) {
        IWP_SPLIT(SPLIT_TILES);
    } else {
        IWP_SPLIT(SPLIT_STILES);
    }
#undef IWP_SPLIT
    return IWP_OK;
}

// Selection on the leaders' residuals after look 1 has filled the first-digit
// histograms, then (FULL) the ordered split.  fused: whole-step route (leader row
// of the gather matrix, leader residual cleared).
int run_select(const Table& T, const Workspace& ws, const ResidualPtrs& R, const float* w, const uint32_t* leader,
               uint32_t W, float eps, Stop stop, bool fused, uint32_t* idx_out, float* val_out,
               iwp_threshold* thr_out, hipStream_t s) {
    if (!T.any_k || T.tiles == 0) return IWP_OK;
    const bool own_pick = T.max_copies <= PICK_MAX_COPIES && T.tiles <= PICK_MAX_TILES;
    if (!own_pick) IWP_LAUNCH_BLOCK("k_first_pick", k_first_pick, T.n_layers, PICK_BLOCK, s, T.layers, ws.hist, ws.state);
    // Consecutive tiles per look-2 workgroup.  Where look 1's copies are complete only every STAGE_GROUP-th tile has work, and
    // few workgroups mean few flushes into a layer's one second-digit histogram; where they are not (a threshold among
    // zeros, a sample that misleads), tiles are read again, and few workgroups leave the chip idle.  Up to 32767 tiles at
    // least about a thousand workgroups, of three tiles at most; beyond, about as many as the chip holds at once (1280: five per
    // compute unit), of 64 tiles at most.  Threshold among zeros, selection alone, against 64 tiles from
    // 4096 tiles on and 4 below: one layer of 3 M elements 181 -> 92 us, 10 M 371 -> 158, 30 M 641 -> 319, 60 M 794 -> 580,
    // 150 M 1588 -> 1330; complete copies within 3 % from 1 M to 300 M (keep 0.2 of 10 M elements 192 -> 150).  Five tiles
    // instead of three: 326, 586; candidates crowded into blocks of nine tiles in 160 layers of 25 M 241 instead of 230;
    // one tile: keep 0.2 of 60 M elements 892 instead of 690.
    // Tables of short layers keep one tile each: a workgroup pays a chain of loads per layer.
    const uint32_t avg_tiles = T.tiles / std::max<uint32_t>(1u, T.n_layers);
    const uint32_t per_wg = avg_tiles < STAGE_GROUP ? 1u
        : T.tiles < STAGE_LARGE_TABLE ? std::min<uint32_t>(std::max<uint32_t>(T.tiles / 1024u, 1u), 3u)
        : std::min<uint32_t>((T.tiles + STAGE_RESIDENT - 1) / STAGE_RESIDENT, STAGE_TILES_MAX);
    const uint32_t stage_grid = std::max<uint32_t>(std::min<uint32_t>((T.tiles + per_wg - 1) / per_wg, STAGE_MAX_GRID),
                                                   (T.tiles + WAVE - 1) / WAVE);
#define IWP_LOOK2(PICK, THREADS)                                                                                                 \
    IWP_LAUNCH_BLOCK("k_stage", (k_stage<PICK, THREADS>), stage_grid, THREADS, s, R, w, T.layers, T.n_layers, T.tiles, leader, W, \
                     eps, ws.state, ws.hist, ws.stage, ws.A)
    if (!own_pick) IWP_LOOK2(false, BLOCK);
    else if (T.tiles <= WIDE_STAGE_MAX_TILES) IWP_LOOK2(true, WIDE_BLOCK);
    else IWP_LOOK2(true, BLOCK);
#undef IWP_LOOK2
    const uint32_t stile_grid = T.long_sparse ? (T.stiles + STILES_TOGETHER - 1) / STILES_TOGETHER : std::min<uint32_t>(T.stiles, STILE_MAX_GRID);
    const bool record = T.by_records && stop == FULL;
    uint32_t* units = reinterpret_cast<uint32_t*>(ws.tile_counts);       // a word per tile or super-tile
#define IWP_REFINE(RECORD)                                                                                                       \
    do {                                                                                                                         \
        if (T.look_twice)                                                                                                        \
            IWP_LAUNCH("k_refine_tiles", k_refine_tiles<RECORD>, T.tiles, s, R, w, T.layers, T.n_layers, leader, W, eps, ws.state, \
                       ws.stage, ws.A, ws.hist, units, ws.records);                                                              \
        else                                                                                                                     \
            IWP_LAUNCH("k_refine2", k_refine2<RECORD>, stile_grid, s, R, w, T.layers, T.n_layers, T.tiles, T.stiles, leader, W,  \
                       eps, ws.state, ws.stage, ws.A, ws.hist, units, ws.records);                                               \
    } while (0)
    if (record) IWP_REFINE(true);
    else IWP_REFINE(false);
#undef IWP_REFINE
    if (record) return fused ? launch_split<true>(T, ws, R, w, leader, W, eps, thr_out, idx_out, val_out, s)
                             : launch_split<false>(T, ws, R, w, leader, W, eps, thr_out, idx_out, val_out, s);
    if (stop == STOP_AT_THRESHOLD) {
        IWP_LAUNCH_BLOCK("k_final_pick", k_final_pick, T.n_layers, WAVE, s, T.layers, ws.hist, ws.state, thr_out);
        return IWP_OK;
    }
    if (T.long_sparse)
        IWP_LAUNCH("k_count_stiles", k_count_stiles, (T.stiles + BLOCK / WAVE - 1) / (BLOCK / WAVE), s, R, w, T.layers, T.n_layers,
                   T.tiles, T.stiles, leader, W, eps, ws.state, ws.hist, thr_out, ws.stage, ws.A, ws.tile_counts, ws.stile_counts);
    else
        IWP_LAUNCH("k_count", k_count, stile_grid, s, R, w, T.layers, T.n_layers, T.tiles, T.stiles, leader, W, eps, ws.state,
               ws.hist, thr_out, ws.stage, ws.A, ws.tile_counts, ws.stile_counts);
    if (fused) return launch_write<true>(T, ws, R, w, leader, W, eps, idx_out, val_out, s);
    return launch_write<false>(T, ws, R, w, leader, W, eps, idx_out, val_out, s);
}

constexpr uint32_t SMALL_MAX_N = SMALL_CHUNKS_MAX * SMALL_CHUNK;

// Up to this many layers a table of short and long ones takes one launch: two workgroups of 16 wavefronts per compute unit.
// Ragged tables, one launch / two: 300 layers 25.6 / 30.3 us, 512 28.1 / 31.6, 1000 45.5 / 31.9.
constexpr uint32_t SMALL_ONE_LAUNCH = 512;

// row: a single layer (layers == NULL); n_long: layers of more than a tile; fused: whole-step route.
int launch_small(const DevLayer* layers, const DevLayer* row, uint32_t n_layers, uint32_t n_long, uint32_t max_n, uint64_t pairs,
                 const Workspace& ws, const WorkerPtrs& P, const float* w, const uint32_t* leader, uint32_t W, float eps,
                 Stop stop, bool fused, uint32_t* idx_out, float* val_out, iwp_threshold* thr_out, hipStream_t s) {
    DevLayer none;
    memset(&none, 0, sizeof none);
    const DevLayer r = row ? *row : none;
    const bool emit = stop == FULL;
    float* gathered = fused ? ws.gathered : nullptr;
    const bool apart = max_n > TILE && n_layers > SMALL_ONE_LAUNCH && n_long < n_layers;
#define IWP_SMALL_AS(FUSED, ONE, THREADS, CHUNKS, FROM, TO)                                                                      \
    IWP_LAUNCH_BLOCK("k_small", (k_small<FUSED, ONE, THREADS, CHUNKS>), n_layers, THREADS, s, P, w, layers, r, FROM, TO, leader, W, \
                     eps, thr_out, emit, ws.tile_out, idx_out, val_out, gathered, pairs)
#define IWP_SMALL(THREADS, CHUNKS, FROM, TO)                                                                                     \
    do {                                                                                                                         \
        if (fused) IWP_SMALL_AS(true, false, THREADS, CHUNKS, FROM, TO);                                                         \
        else if (row) IWP_SMALL_AS(false, true, THREADS, CHUNKS, FROM, TO);                                                      \
        else IWP_SMALL_AS(false, false, THREADS, CHUNKS, FROM, TO);                                                              \
    } while (0)
    if (max_n <= TILE || apart) IWP_SMALL(TINY_BLOCK, TINY_CHUNKS, 0u, TILE);
    const uint32_t from = apart ? TILE + 1 : 0u;
    if (max_n > SMALL_MAX_N / 2) IWP_SMALL(SMALL_BLOCK, SMALL_CHUNKS_MAX, from, SMALL_MAX_N);
    else if (max_n > TILE) IWP_SMALL(SMALL_BLOCK, SMALL_CHUNKS_MAX / 2, from, SMALL_MAX_N / 2);
#undef IWP_SMALL_AS
#undef IWP_SMALL
    return IWP_OK;
}

// Ordered split from threshold records given by the caller.
int run_compact_from(const Table& T, const Workspace& ws, const ResidualPtrs& R, const float* w, float eps,
                     const iwp_threshold* thr, uint32_t* idx_out, float* val_out, hipStream_t s) {
    if (!T.any_k || T.tiles == 0) return IWP_OK;
#define IWP_RECORDS(THREADS)                                                                                                     \
    IWP_LAUNCH_BLOCK("k_stage_records", k_stage_records<THREADS>, T.tiles, THREADS, s, R.r[0], w, T.layers, T.n_layers, thr, eps, \
                     ws.state, ws.stage, ws.A, ws.tile_counts)
    if (buffer_bytes(T) <= KEEP_W_AND_R_MAX_BYTES) IWP_RECORDS(WIDE_BLOCK);
    else IWP_RECORDS(BLOCK);
#undef IWP_RECORDS
    if (T.max_layer_stiles <= FOLD_MAX_TILES / GROUP) {
        IWP_LAUNCH("k_write", (k_write<false, FOLD_TILES>), T.stiles * (GROUP / (BLOCK / WAVE)), s, R, w, T.layers, T.n_layers, T.tiles,
                   nullptr, 1u, eps, ws.state, ws.stage, ws.A, ws.tile_counts, ws.stile_counts, ws.tile_out, idx_out, val_out, nullptr,
                   T.pairs);
        return IWP_OK;
    }
    IWP_LAUNCH("k_fold_counts", k_fold_counts, (T.stiles + BLOCK - 1) / BLOCK, s, T.layers, T.n_layers, T.tiles, T.stiles,
               ws.tile_counts, ws.stile_counts);
    return launch_write<false>(T, ws, R, w, nullptr, 1u, eps, idx_out, val_out, s);
}

}  // namespace

struct iwp_plan {
    std::vector<iwp_layer> rows;
    DevLayer* dev = nullptr;      // n_layers + 1 rows
    Sizes z{};
    uint64_t flat_end = 0;        // one past the last element any layer covers
    uint64_t elements = 0;        // of all layers
    bool any_k = false;
    bool all_k = true;            // every non-empty layer selects something
    uint32_t max_layer_stiles = 0;
    uint32_t max_n = 0;           // elements of the longest layer
    uint32_t n_long = 0;          // layers of more than one tile
    bool all_dense = true;        // each of those keeps at least one element in HINT_KEEP
    bool look_twice = false;      // roomy slots; marks by samples only where samples() says so (LOOK_TWICE_TILES)
    bool by_records = false;      // the split goes by the units' records
    bool long_sparse = false;     // see is_long_sparse()
    uint32_t max_copies = 1;      // most copies of a layer's first-digit histogram
    float momentum = 1.0f;        // r <- momentum * r + g in every call that accumulates through this plan
};

// Does k_small replace k_init, look 1 and the selection?  Where all layers have at most 32768 elements; beyond 16384 a
// compute unit holds one layer at a time and nothing overlaps its loads with its barriers, so only up to 512 layers of more
// than a tile where the long route takes every mark from a hint (see HINT_BELOW), 1024 where it samples; the selection
// alone, which writes nothing, always.
// Layers of 16385 elements, k_small against the long route: 512 hinted 69 / 72 us, 768 107 / 97; unhinted 1024 137 / 145,
// 2048 253 / 243; of 32768: 114 / 119, 165 / 168, 213 / 212, 401 / 395; selection of 6000 layers of 16385 366 / 398.
// 700 layers of 17000 elements with a hint, kept at 0.004: k_small 86 / long route 105 us; at 1/64 92 / 84; at 1/64 and
// momentum 0.9 92 / 102.
bool takes_small(const iwp_plan& plan, bool hinted, bool select) {
    if (plan.max_n > SMALL_MAX_N) return false;
    const bool no_sample = hinted && plan.all_dense && plan.momentum == 1.0f;
    return select || plan.max_n <= SMALL_MAX_N / 2 || plan.n_long <= (no_sample ? 512u : 1024u);
}

// Do k_follow_sum / k_follow_mask_sum take the workers' pass, the exchange and the update?  streaming: workers with a gradient.
// The lines: see iwp_sum.hpp.
bool follows_together(const iwp_plan& plan, uint32_t streaming) {
    if (plan.z.tiles > FOLLOW_SUM_MAX_TILES) return false;
    if (streaming <= FOLLOW_SUM_ANY) return true;
    const uint64_t layers = plan.z.n_layers, chunks = std::max(FOLLOW_SUM_CHUNKS, FOLLOW_SUM_CHUNKS_EACH * streaming);
    return plan.elements >= (streaming <= FOLLOW_SUM_FEW ? layers : chunks + 2 * layers) * CHUNK;
}

// May a step's or a compression's marks be sampled?  The rule and its exception: see LOOK_TWICE_TILES.
bool samples(const iwp_plan& plan, bool hinted) {
    return !plan.look_twice || (!hinted && plan.momentum == 1.0f);
}

static Table table_of(const iwp_plan& p) {
    return Table{p.dev, p.z.n_layers, p.z.tiles, p.z.stiles, p.z.pairs, p.any_k, p.max_layer_stiles, p.max_copies, p.look_twice,
                 p.by_records, p.long_sparse};
}

extern "C" {

const char* iwp_strerror(int code) {
    switch (code) {
        case IWP_OK: return "ok";
        case IWP_EINVAL: return "invalid argument";
        case IWP_EALIGN: return "buffer not aligned as required";
        case IWP_EWORKSPACE: return "workspace missing or too small";
        case IWP_ERANGE: return "layer does not fit the 32-bit index range";
        case IWP_EHIP: return "HIP runtime error";
        case IWP_ESCRATCH: return "plan needs more scratch than the library's static buffer holds";
        default: return "unknown status";
    }
}

const char* iwp_last_hip_error(void) { return g_hip_error; }

// ----------------------------------------------------------------- single layer

static Sizes single_sizes(uint32_t n, uint32_t k) {
    Sizes z;
    z.n_layers = 1; z.tiles = tiles_of(n); z.stiles = stiles_of(n);
    z.pairs = k; z.slots = (uint64_t)z.tiles * slot_cap_of(n, k) + (k ? roomy_reserve(z.tiles) : 0u); z.mask_words = ((uint64_t)n + 31) / 32;
    z.hist_words = layer_hist_words(h0_copies_of(n, k));
    z.records = k ? std::max(records_apart(n, k, h0_copies_of(n, k), looks_twice(z.tiles, 1)), record_reserve(z.tiles)) : 0u;
    z.W_gather = 0;
    return z;
}

size_t iwp_workspace_bytes(uint32_t n, uint32_t k) { return carve(nullptr, single_sizes(n, std::min(n, k))).bytes; }

enum SingleOp { OP_COMPRESS, OP_SELECT, OP_COMPACT };

static int single_common(SingleOp op, const float* w, const float* g, float* r, uint32_t n, uint32_t k, float eps,
                         const iwp_threshold* from_thr, uint32_t* idx_out, float* val_out, iwp_threshold* thr_out,
                         void* workspace, size_t workspace_bytes, hipStream_t s) {
    if (k > n) return IWP_EINVAL;
    if (check_eps(eps)) return IWP_EINVAL;
    if (n > IWP_MAX_FLAT) return IWP_ERANGE;
    if (n == 0) return IWP_OK;
    const bool emits = op != OP_SELECT && k > 0;
    if (!r || (k > 0 && !w) || (emits && (!idx_out || !val_out))) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(g) || !aligned4(r) || !aligned4(idx_out) || !aligned4(val_out) ||
        !aligned4(thr_out) || !aligned4(from_thr))
        return IWP_EALIGN;
    const Sizes z = single_sizes(n, k);
    Workspace ws = carve(workspace, z);
    if (!workspace || workspace_bytes < ws.bytes) return IWP_EWORKSPACE;   // holds the one-row layer table too
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return IWP_EALIGN;

    WorkerPtrs P;
    memset(&P, 0, sizeof P);
    P.g[0] = g;
    P.r[0] = r;
    P.momentum = 1.0f;
    ResidualPtrs R;
    memset(&R, 0, sizeof R);
    R.r[0] = r;
    DevLayer row, sentinel;
    memset(&row, 0, sizeof row);
    memset(&sentinel, 0, sizeof sentinel);
    row.n = n; row.k = k; row.slot_cap = (uint16_t)(looks_twice(z.tiles, 1) ? roomy(slot_cap_of(n, k)) : slot_cap_of(n, k));
    row.sample = sample_of(n, k);
    row.hist_begin = 0; row.h0_copies = (uint16_t)h0_copies_of(n, k);
    sentinel.tile_begin = z.tiles; sentinel.stile_begin = z.stiles; sentinel.out_offset = k;
    if (op != OP_COMPACT && k > 0 && n <= SMALL_MAX_N)
        return launch_small(nullptr, &row, 1u, 1u, n, k, ws, P, w, nullptr, 1u, eps, op == OP_SELECT ? STOP_AT_THRESHOLD : FULL,
                            false, idx_out, val_out, thr_out, s);
    SampleSource S = sample_from(P, w, nullptr, 1u, eps);
    if (op == OP_COMPACT || k == 0 || looks_twice(z.tiles, 1)) S.on = 0;
    int rc = launch_init(ws, 1, z.tiles, nullptr, nullptr, &row, &sentinel, S, s);
    if (rc) return rc;
    const Table T{ws.single_table, 1, z.tiles, z.stiles, k, k > 0, z.stiles, row.h0_copies, looks_twice(z.tiles, 1),
                  goes_by_records(slot_cap_of(n, k), z.stiles), is_long_sparse(slot_cap_of(n, k), z.stiles)};
    if (op == OP_COMPACT) return run_compact_from(T, ws, R, w, eps, from_thr, idx_out, val_out, s);
    if (k > 0) {
        rc = launch_leader_pass(T, ws, P, w, nullptr, 1u, eps, s);
        if (rc) return rc;
    } else if (g)
        IWP_LAUNCH("k_accumulate_rest", k_accumulate_rest, z.tiles, s, P, T.layers, 1u, z.tiles, 0u, nullptr, 1u);
    return run_select(T, ws, R, w, nullptr, 1u, eps, op == OP_SELECT ? STOP_AT_THRESHOLD : FULL, false, idx_out,
                      val_out, thr_out, s);
}

int compress_layer(const float* w, const float* g, float* r, uint32_t n, uint32_t k, float eps,
                   uint32_t* idx_out, float* val_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (n > 0 && !g) return IWP_EINVAL;
    return single_common(OP_COMPRESS, w, g, r, n, k, eps, nullptr, idx_out, val_out, nullptr, workspace,
                         workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int select_threshold(const float* w, const float* r, uint32_t n, uint32_t k, float eps, iwp_threshold* thr_out,
                     void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (k == 0 || !thr_out) return IWP_EINVAL;
    // r is only read: no gradient pointer means no accumulation
    return single_common(OP_SELECT, w, nullptr, const_cast<float*>(r), n, k, eps, nullptr, nullptr, nullptr, thr_out,
                         workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int compact_pairs(const float* w, const float* r, uint32_t n, float eps, const iwp_threshold* thr, uint32_t k,
                  uint32_t* idx_out, float* val_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (k == 0 || !thr) return IWP_EINVAL;
    return single_common(OP_COMPACT, w, nullptr, const_cast<float*>(r), n, k, eps, thr, idx_out, val_out, nullptr,
                         workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

// ----------------------------------------------------------------- exchange

int gather_sum_at_indices(const float* const* residuals, uint32_t W, const uint32_t* idx, uint32_t k,
                          float* sum_out, void* hip_stream) {
    if (W == 0 || W > IWP_MAX_WORKERS || !residuals) return IWP_EINVAL;
    if (k == 0) return IWP_OK;
    if (!idx || !sum_out) return IWP_EINVAL;
    if (!aligned4(idx) || !aligned4(sum_out)) return IWP_EALIGN;
    ResidualPtrs R;
    memset(&R, 0, sizeof R);
    for (uint32_t p = 0; p < W; ++p) {
        if (!residuals[p]) return IWP_EINVAL;
        if (!aligned4(residuals[p])) return IWP_EALIGN;
        R.r[p] = const_cast<float*>(residuals[p]);
    }
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    IWP_LAUNCH("k_gather_sum", k_gather_sum, (k + BLOCK - 1) / BLOCK, s, R, W, idx, k, sum_out);
    return IWP_OK;
}

int apply_sparse_update(float* w, const uint32_t* idx, const float* sum, uint32_t k, float scale,
                        float* const* residuals_to_clear, uint32_t W, void* hip_stream) {
    if (W > IWP_MAX_WORKERS || (W > 0 && !residuals_to_clear)) return IWP_EINVAL;
    if (k == 0) return IWP_OK;
    if (!w || !idx || !sum) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(idx) || !aligned4(sum)) return IWP_EALIGN;
    ResidualPtrs R;
    memset(&R, 0, sizeof R);
    for (uint32_t p = 0; p < W; ++p) {
        if (!residuals_to_clear[p]) return IWP_EINVAL;
        if (!aligned4(residuals_to_clear[p])) return IWP_EALIGN;
        R.r[p] = residuals_to_clear[p];
    }
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    IWP_LAUNCH("k_apply_update", k_apply_update, (k + BLOCK - 1) / BLOCK, s, w, idx, sum, k, scale, R, W);
    return IWP_OK;
}

// ----------------------------------------------------------------- plans and segmented calls

int iwp_plan_create(const iwp_layer* layers, uint32_t n_layers, iwp_plan** plan_out) {
    if (!plan_out) return IWP_EINVAL;
    *plan_out = nullptr;
    if (!layers || n_layers == 0) return IWP_EINVAL;
    std::vector<DevLayer> dev(n_layers + 1);
    uint64_t pairs = 0, slots = 0, tiles = 0, stiles = 0, end = 0, mask_words = 0;
    bool any_k = false, all_k = true;
    uint32_t max_stiles = 0, max_n = 0, n_long = 0, max_cap = 0;
    bool all_dense = true;
    for (uint32_t j = 0; j < n_layers; ++j) {
        const iwp_layer& L = layers[j];
        if (L.offset < 0 || L.k > L.n) return IWP_EINVAL;
        if ((uint64_t)L.offset < end) return IWP_EINVAL;              // table order, no overlap
        if ((uint64_t)L.offset + L.n > IWP_MAX_FLAT) return IWP_ERANGE;
        if (L.out_offset != pairs) return IWP_EINVAL;                  // packed outputs
        DevLayer& D = dev[j];
        memset(&D, 0, sizeof D);
        D.offset = (uint64_t)L.offset;
        D.slot_begin = slots;
        D.n = L.n;
        D.k = L.k;
        D.out_offset = L.out_offset;
        D.tile_begin = (uint32_t)tiles;
        D.stile_begin = (uint32_t)stiles;
        D.slot_cap = (uint16_t)slot_cap_of(L.n, L.k);
        max_cap = std::max<uint32_t>(max_cap, D.slot_cap);
        D.mask_begin = (uint32_t)mask_words;
        D.sample = sample_of(L.n, L.k);
        end = (uint64_t)L.offset + L.n;
        pairs += L.k;
        slots += (uint64_t)tiles_of(L.n) * D.slot_cap;
        tiles += tiles_of(L.n);
        stiles += stiles_of(L.n);
        mask_words += ((uint64_t)L.n + 31) / 32;
        any_k = any_k || L.k > 0;
        max_stiles = std::max(max_stiles, stiles_of(L.n));
        max_n = std::max(max_n, L.n);
        n_long += L.n > TILE ? 1u : 0u;
        if (L.n > TILE && (uint64_t)L.k * HINT_KEEP < L.n) all_dense = false;
        if (L.n > 0 && L.k == 0) all_k = false;
        if (pairs > 0xFFFFFFFFull || tiles > 0x7FFFFFFFull / IWP_MAX_WORKERS) return IWP_ERANGE;
    }
    // one copy of the first-digit histogram per `flushes` look-1 workgroups of a layer -> words of all layers' histograms
    auto lay_out_histograms = [&](uint32_t flushes) {
        uint64_t words = 0;
        for (uint32_t j = 0; j < n_layers; ++j) {
            dev[j].hist_begin = (uint32_t)words;
            dev[j].h0_copies = (uint16_t)h0_copies_of(layers[j].n, layers[j].k, flushes);
            words += layer_hist_words(dev[j].h0_copies);
        }
        return words;
    };
    // the records that do not fit there, behind one another -> their number
    auto lay_out_records = [&](bool per_tile) {
        uint64_t records = 0;
        for (uint32_t j = 0; j < n_layers; ++j) {
            dev[j].record_begin = (uint32_t)records;
            records += records_apart(layers[j].n, layers[j].k, dev[j].h0_copies, per_tile);
        }
        return records;
    };
    uint64_t hist_words = lay_out_histograms(FLUSHES_PER_COPY);
    if (hist_words > 0xFFFFFFFFull) hist_words = lay_out_histograms(FLUSHES_PER_COPY_FEW);      // hist_begin holds 32 bits
    if (hist_words > 0xFFFFFFFFull) return IWP_ERANGE;
    DevLayer& S = dev[n_layers];
    memset(&S, 0, sizeof S);
    S.out_offset = (uint32_t)pairs;
    S.tile_begin = (uint32_t)tiles;
    S.stile_begin = (uint32_t)stiles;
    S.slot_begin = slots;
    iwp_plan* plan = new (std::nothrow) iwp_plan;
    if (!plan) return IWP_EINVAL;
    plan->rows.assign(layers, layers + n_layers);
    plan->z = Sizes{n_layers, (uint32_t)tiles, (uint32_t)stiles, pairs, slots, mask_words, hist_words, 0, 0};
    plan->any_k = any_k;
    plan->all_k = all_k;
    plan->max_layer_stiles = max_stiles;
    plan->max_n = max_n;
    plan->n_long = n_long;
    plan->all_dense = all_dense;
    plan->long_sparse = is_long_sparse(max_cap, max_stiles);
    // roomy slots and records, or what larger tables hold in reserve for them, unless the library's static scratch would no longer do
    Sizes roomier = plan->z;
    roomier.slots += any_k ? roomy_reserve(tiles) : 0u;
    roomier.records = any_k ? std::max<uint64_t>(lay_out_records(false), record_reserve(tiles)) : 0u;
    if (!goes_by_records(max_cap, max_stiles) && carve(nullptr, roomier).bytes > IWP_STATIC_SCRATCH_BYTES) roomier.records = 0;
    if (carve(nullptr, roomier).bytes <= IWP_STATIC_SCRATCH_BYTES) {
        plan->z = roomier;
        plan->look_twice = looks_twice(tiles, n_layers);
        plan->by_records = goes_by_records(max_cap, max_stiles);
    }
    if (plan->look_twice) {
        slots = 0;
        for (DevLayer& D : dev) {
            D.slot_begin = slots;
            D.slot_cap = (uint16_t)roomy(D.slot_cap);
            slots += (uint64_t)tiles_of(D.n) * D.slot_cap;
        }
        lay_out_records(true);                               // no more than the reserve: the table has no more tiles
    }
    if (carve(nullptr, plan->z).bytes > IWP_STATIC_SCRATCH_BYTES) {
        Sizes few = plan->z;
        few.hist_words = 0;
        for (uint32_t j = 0; j < n_layers; ++j)
            few.hist_words += layer_hist_words(h0_copies_of(layers[j].n, layers[j].k, FLUSHES_PER_COPY_FEW));
        if (carve(nullptr, few).bytes <= IWP_STATIC_SCRATCH_BYTES) {
            plan->z = few;
            lay_out_histograms(FLUSHES_PER_COPY_FEW);
        }
    }
    // the records, unless a plan that the static scratch holds without them would no longer fit
    if (!plan->by_records && goes_by_records(max_cap, max_stiles)) {
        Sizes with = plan->z;
        with.records = lay_out_records(false);
        plan->by_records = carve(nullptr, with).bytes <= IWP_STATIC_SCRATCH_BYTES || carve(nullptr, plan->z).bytes > IWP_STATIC_SCRATCH_BYTES;
        if (plan->by_records) plan->z = with;
    }
    for (const DevLayer& D : dev) plan->max_copies = std::max<uint32_t>(plan->max_copies, D.h0_copies);
    plan->flat_end = end;
    for (const iwp_layer& row : plan->rows) plan->elements += row.n;
    // the table, then the layer of every tile and of every super-tile (layer_of_tile and layer_of_stile read them)
    std::vector<uint32_t> map;
    map.reserve(tiles + stiles);
    for (uint32_t j = 0; j < n_layers; ++j) map.insert(map.end(), tiles_of(layers[j].n), j);
    for (uint32_t j = 0; j < n_layers; ++j) map.insert(map.end(), stiles_of(layers[j].n), j);
    const size_t table_bytes = dev.size() * sizeof(DevLayer), map_bytes = map.size() * sizeof(uint32_t);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&plan->dev), table_bytes + std::max<size_t>(map_bytes, 4));
    if (e == hipSuccess) e = hipMemcpy(plan->dev, dev.data(), table_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess && map_bytes)
        e = hipMemcpy(reinterpret_cast<char*>(plan->dev) + table_bytes, map.data(), map_bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (plan->dev) (void)hipFree(plan->dev);
        delete plan;
        return hip_fail(e, "iwp_plan_create");
    }
    *plan_out = plan;
    return IWP_OK;
}

void iwp_plan_destroy(iwp_plan* plan) {
    if (!plan) return;
    if (plan->dev) (void)hipFree(plan->dev);
    delete plan;
}

int iwp_plan_set_momentum(iwp_plan* plan, float momentum) {
    if (!plan || !std::isfinite(momentum)) return IWP_EINVAL;
    plan->momentum = momentum;
    return IWP_OK;
}

size_t iwp_plan_workspace_bytes(const iwp_plan* plan) { return plan ? carve(nullptr, plan->z).bytes : 0; }

size_t iwp_plan_step_workspace_bytes(const iwp_plan* plan, uint32_t W) {
    if (!plan) return 0;
    Sizes z = plan->z;
    z.W_gather = W;
    return carve(nullptr, z).bytes;
}

uint64_t iwp_plan_total_pairs(const iwp_plan* plan) { return plan ? plan->z.pairs : 0; }

static int check_ws(size_t need, void* workspace, size_t workspace_bytes) {
    if (!workspace || workspace_bytes < need) return IWP_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return IWP_EALIGN;
    return IWP_OK;
}

// The first worker with a gradient, or worker 0: the one whose residual k_follow_sum's chunks are aligned to.
static uint32_t first_streaming(const float* const* g, uint32_t W) {
    for (uint32_t p = 0; p < W; ++p)
        if (g[p]) return p;
    return 0u;
}

static int worker_tables(const float* const* g, float* const* r, uint32_t W, float momentum, WorkerPtrs* P,
                         ResidualPtrs* R) {
    if (!g || !r || W == 0 || W > IWP_MAX_WORKERS) return IWP_EINVAL;
    memset(P, 0, sizeof *P);
    memset(R, 0, sizeof *R);
    P->momentum = momentum;
    for (uint32_t p = 0; p < W; ++p) {
        if (!r[p]) return IWP_EINVAL;
        if (!aligned4(r[p]) || !aligned4(g[p])) return IWP_EALIGN;
        P->g[p] = g[p];
        P->r[p] = r[p];
        R->r[p] = r[p];
    }
    return IWP_OK;
}

// compress_segmented on a workspace that is either the caller's or the library's static scratch.
static int compress_segmented_on(const iwp_plan* plan, const float* w, const float* const* g, float* const* r,
                                 uint32_t W, const uint32_t* leader, const iwp_threshold* thr_hint, float eps,
                                 uint32_t* idx_out, float* val_out, iwp_threshold* thr_out, bool own_scratch,
                                 void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!plan) return IWP_EINVAL;
    if (check_eps(eps)) return IWP_EINVAL;
    if (plan->any_k && (!w || !idx_out || !val_out)) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(idx_out) || !aligned4(val_out) || !aligned4(thr_out) || !aligned4(leader) ||
        !aligned4(thr_hint))
        return IWP_EALIGN;
    if (thr_hint && thr_hint == thr_out) return IWP_EINVAL;   // the hint is read while the records are written
    WorkerPtrs P;
    ResidualPtrs R;
    int rc = worker_tables(g, r, W, plan->momentum, &P, &R);
    if (rc) return rc;
    if (own_scratch) {
        // the size check comes first: a plan that does not fit is turned away before anything is looked up
        if (carve(nullptr, plan->z).bytes > IWP_STATIC_SCRATCH_BYTES) return IWP_ESCRATCH;
        rc = static_scratch(&workspace);
        if (rc) return rc;
        workspace_bytes = IWP_STATIC_SCRATCH_BYTES;
    }
    Workspace ws = carve(workspace, plan->z);
    rc = check_ws(ws.bytes, workspace, workspace_bytes);
    if (rc) return rc;
    if (plan->z.tiles == 0) return IWP_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const Table T = table_of(*plan);
    const bool small = T.any_k && takes_small(*plan, thr_hint != nullptr, false);
    if (small) {
        rc = launch_small(T.layers, nullptr, T.n_layers, plan->n_long, plan->max_n, T.pairs, ws, P, w, leader, W, eps, FULL, false, idx_out,
                          val_out, thr_out, s);
        if (rc) return rc;
    } else {
        rc = launch_init(ws, T.n_layers, T.tiles, thr_hint, T.layers, nullptr, nullptr,
                         sample_from(P, w, leader, W, eps, samples(*plan, thr_hint != nullptr)), s);
        if (rc) return rc;
        if (T.any_k) {
            rc = launch_leader_pass(T, ws, P, w, leader, W, eps, s);
            if (rc) return rc;
        }
    }
    if (W > 1 || !plan->all_k)
        IWP_LAUNCH("k_accumulate_rest", k_accumulate_rest, W * T.tiles, s, P, T.layers, T.n_layers, T.tiles,
                   takes_runs(T.tiles, T.n_layers), leader, W);
    if (small) return IWP_OK;
    return run_select(T, ws, R, w, leader, W, eps, FULL, false, idx_out, val_out, thr_out, s);
}

int compress_segmented(const iwp_plan* plan, const float* w, const float* const* g, float* const* r, uint32_t W,
                       const uint32_t* leader, const iwp_threshold* thr_hint, float eps, uint32_t* idx_out,
                       float* val_out, iwp_threshold* thr_out, void* workspace, size_t workspace_bytes,
                       void* hip_stream) {
    return compress_segmented_on(plan, w, g, r, W, leader, thr_hint, eps, idx_out, val_out, thr_out, false, workspace,
                                 workspace_bytes, hip_stream);
}

int compress_segmented_static(const iwp_plan* plan, const float* w, const float* const* g, float* const* r,
                              uint32_t W, const uint32_t* leader, const iwp_threshold* thr_hint, float eps,
                              uint32_t* idx_out, float* val_out, iwp_threshold* thr_out, void* hip_stream) {
    return compress_segmented_on(plan, w, g, r, W, leader, thr_hint, eps, idx_out, val_out, thr_out, true, nullptr, 0,
                                 hip_stream);
}

int iwp_step_segmented(const iwp_plan* plan, float* w, const float* const* g, float* const* r, uint32_t W,
                       const uint32_t* leader, const iwp_threshold* thr_hint, float eps, float scale,
                       uint32_t* idx_out, float* val_out, float* sum_out, iwp_threshold* thr_out, void* workspace,
                       size_t workspace_bytes, void* hip_stream) {
    if (!plan) return IWP_EINVAL;
    if (check_eps(eps) || !std::isfinite(scale)) return IWP_EINVAL;
    if (!w) return IWP_EINVAL;
    if (plan->any_k && (!idx_out || !val_out || !sum_out)) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(idx_out) || !aligned4(val_out) || !aligned4(sum_out) || !aligned4(thr_out) ||
        !aligned4(leader) || !aligned4(thr_hint))
        return IWP_EALIGN;
    if (thr_hint && thr_hint == thr_out) return IWP_EINVAL;   // the hint is read while the records are written
    WorkerPtrs P;
    ResidualPtrs R;
    int rc = worker_tables(g, r, W, plan->momentum, &P, &R);
    if (rc) return rc;
    Sizes z = plan->z;
    z.W_gather = W;
    Workspace ws = carve(workspace, z);
    rc = check_ws(ws.bytes, workspace, workspace_bytes);
    if (rc) return rc;
    if (z.tiles == 0) return IWP_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const Table T = table_of(*plan);
    if (T.any_k && takes_small(*plan, thr_hint != nullptr, false)) {
        rc = launch_small(T.layers, nullptr, T.n_layers, plan->n_long, plan->max_n, T.pairs, ws, P, w, leader, W, eps, FULL, true, idx_out,
                          val_out, thr_out, s);
        if (rc) return rc;
    } else if (T.any_k) {
        rc = launch_init(ws, z.n_layers, z.tiles, thr_hint, plan->dev, nullptr, nullptr,
                         sample_from(P, w, leader, W, eps, samples(*plan, thr_hint != nullptr)), s);
        if (rc) return rc;
        rc = launch_leader_pass(T, ws, P, w, leader, W, eps, s);
        if (rc) return rc;
        rc = run_select(T, ws, R, w, leader, W, eps, FULL, true, idx_out, val_out, thr_out, s);
        if (rc) return rc;
    }
    WorkerList acc, stat;                       // workers with / without a gradient
    memset(&acc, 0, sizeof acc);
    memset(&stat, 0, sizeof stat);
    for (uint32_t p = 0; p < W; ++p) {
        if (g[p]) acc.id[acc.n++] = (uint8_t)p; else stat.id[stat.n++] = (uint8_t)p;
    }
    // a single accumulating worker that leads every layer (no leader table: worker 0) has been through look 1 on
    // every tile: nothing follows
    const bool leader_did_all = acc.n == 1 && acc.id[0] == 0 && !leader && plan->all_k;
    if (acc.n && !leader_did_all && follows_together(*plan, acc.n)) {
        IWP_LAUNCH("k_follow_sum", k_follow_sum, CHUNKS_A_TILE * T.tiles, s, P, first_streaming(g, W), T.layers, T.n_layers,
                   leader, W, idx_out, val_out, ws.tile_out, w, scale, sum_out);
        return IWP_OK;
    }
    if (acc.n && !leader_did_all)
        IWP_LAUNCH_FEW("k_follow_gather", k_follow_gather, acc.n * T.tiles, few_followers(T, acc.n), s, P, acc, T.layers, T.n_layers, T.tiles,
                   takes_runs(T.tiles, T.n_layers), leader, W, idx_out, ws.tile_out, ws.gathered, T.pairs);
    if (T.any_k) {
        uint32_t static_mask = 0;
        for (uint32_t q = 0; q < stat.n; ++q) static_mask |= 1u << stat.id[q];
        IWP_LAUNCH_FEW("k_reduce_update", k_reduce_update, (uint32_t)((T.pairs + BLOCK - 1) / BLOCK), few_updates(T.tiles, T.pairs), s, R, static_mask, T.layers,
                   T.n_layers, leader, ws.gathered, W, T.pairs, idx_out, w, scale, sum_out, plan->flat_end);
    }
    return IWP_OK;
}

int select_threshold_segmented(const iwp_plan* plan, const float* w, const float* r, float eps,
                               iwp_threshold* thr_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!plan || !w || !r || !thr_out) return IWP_EINVAL;
    if (check_eps(eps)) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(r) || !aligned4(thr_out)) return IWP_EALIGN;
    Workspace ws = carve(workspace, plan->z);
    int rc = check_ws(ws.bytes, workspace, workspace_bytes);
    if (rc) return rc;
    if (plan->z.tiles == 0 || !plan->any_k) return IWP_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    WorkerPtrs P;
    memset(&P, 0, sizeof P);
    P.r[0] = const_cast<float*>(r);       // no gradient pointer: the residual is only read
    P.momentum = 1.0f;
    if (takes_small(*plan, false, true))
        return launch_small(plan->dev, nullptr, plan->z.n_layers, plan->n_long, plan->max_n, plan->z.pairs, ws, P, w, nullptr, 1u, eps,
                            STOP_AT_THRESHOLD, false, nullptr, nullptr, thr_out, s);
    rc = launch_init(ws, plan->z.n_layers, plan->z.tiles, nullptr, plan->dev, nullptr, nullptr,
                     sample_from(P, w, nullptr, 1u, eps, !plan->look_twice), s);
    if (rc) return rc;
    ResidualPtrs R;
    memset(&R, 0, sizeof R);
    R.r[0] = const_cast<float*>(r);
    const Table T = table_of(*plan);
    rc = launch_leader_pass(T, ws, P, w, nullptr, 1u, eps, s);
    if (rc) return rc;
    return run_select(T, ws, R, w, nullptr, 1u, eps, STOP_AT_THRESHOLD, false, nullptr, nullptr, thr_out, s);
}

int compact_pairs_segmented(const iwp_plan* plan, const float* w, const float* r, float eps, const iwp_threshold* thr,
                            uint32_t* idx_out, float* val_out, void* workspace, size_t workspace_bytes,
                            void* hip_stream) {
    if (!plan || !w || !r || !thr) return IWP_EINVAL;
    if (check_eps(eps)) return IWP_EINVAL;
    if (plan->any_k && (!idx_out || !val_out)) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(r) || !aligned4(thr) || !aligned4(idx_out) || !aligned4(val_out)) return IWP_EALIGN;
    Workspace ws = carve(workspace, plan->z);
    int rc = check_ws(ws.bytes, workspace, workspace_bytes);
    if (rc) return rc;
    if (plan->z.tiles == 0 || !plan->any_k) return IWP_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    ResidualPtrs R;
    memset(&R, 0, sizeof R);
    R.r[0] = const_cast<float*>(r);
    const Table T = table_of(*plan);
    return run_compact_from(T, ws, R, w, eps, thr, idx_out, val_out, s);
}

// ----------------------------------------------------------------- threshold mode

namespace {

struct ThresholdWorkspace {
    uint32_t* tile_counts;    // tiles
    uint32_t* tile_pos;       // tiles
    uint32_t* lay_out;        // n_layers + 1
    double2* tile_stats;      // n_lead * tiles (layer-wise thresholds)
    ChosenSlots slots;        // n_lead * tiles * cap
    float* gathered;          // W * max_pairs
    size_t bytes;
};

// Values per tile and chosen node that k_leader_mask hands over: four times what an average tile can send within the
// caller's capacity, since layers differ, plus 64; at most 1024.  What a tile sends beyond that is fetched and cleared later.
static uint32_t chosen_cap(const Sizes& z, uint32_t max_pairs) {
    const uint64_t per_tile = z.tiles ? ((uint64_t)max_pairs + z.tiles - 1) / z.tiles : 0;
    return (uint32_t)std::min<uint64_t>(1024, 64 + 4 * per_tile);
}

static ThresholdWorkspace carve_threshold(void* base, const Sizes& z, uint32_t W, uint32_t n_lead, uint32_t max_pairs) {
    ThresholdWorkspace ws;
    const uintptr_t b = reinterpret_cast<uintptr_t>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) { uintptr_t p = b + off; off += round256(bytes); return p; };
    ws.tile_counts = reinterpret_cast<uint32_t*>(take((size_t)z.tiles * sizeof(uint32_t)));
    ws.tile_pos = reinterpret_cast<uint32_t*>(take((size_t)z.tiles * sizeof(uint32_t)));
    ws.lay_out = reinterpret_cast<uint32_t*>(take(((size_t)z.n_layers + 1) * sizeof(uint32_t)));
    ws.tile_stats = reinterpret_cast<double2*>(take((size_t)n_lead * z.tiles * sizeof(double2)));
    ws.slots.cap = chosen_cap(z, max_pairs);
    ws.slots.tiles = z.tiles;
    ws.slots.val = reinterpret_cast<float*>(take((size_t)n_lead * z.tiles * ws.slots.cap * sizeof(float)));
    ws.gathered = reinterpret_cast<float*>(take((size_t)W * max_pairs * sizeof(float)));
    ws.bytes = off;
    return ws;
}

// Rule of the layer-wise threshold; absent (NULL) for caller-supplied thresholds.
struct LayerwiseRule {
    double alpha, beta, C;
    double* stats_out;
    float* thr_out;
};

static int run_threshold_step(const iwp_plan* plan, float* w, const float* const* g, float* const* r, uint32_t W,
                       const uint32_t* leaders, uint32_t n_lead, const float* thr, const LayerwiseRule* rule,
                       RandomSel rs, float eps, float scale, uint8_t* mask_out, uint32_t* count_out, uint32_t* idx_out, float* sum_out,
                       uint32_t max_pairs, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!plan || !w || !leaders || !mask_out || !count_out || !idx_out || !sum_out) return IWP_EINVAL;
    if (n_lead == 0 || n_lead > MAX_LEAD || n_lead > W || max_pairs == 0) return IWP_EINVAL;
    if (check_eps(eps) || !std::isfinite(scale)) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(leaders) || !aligned4(thr) || !aligned4(mask_out) || !aligned4(count_out) ||
        !aligned4(idx_out) || !aligned4(sum_out))
        return IWP_EALIGN;
    WorkerPtrs P;
    ResidualPtrs R;
    int rc = worker_tables(g, r, W, plan->momentum, &P, &R);
    if (rc) return rc;
    const Sizes& z = plan->z;
    ThresholdWorkspace ws = carve_threshold(workspace, z, W, n_lead, max_pairs);
    rc = check_ws(ws.bytes, workspace, workspace_bytes);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    uint32_t* mask32 = reinterpret_cast<uint32_t*>(mask_out);
    const DevLayer* layers = plan->dev;
    TileStats stats;                                         // only where the masks' launch merges them
    memset(&stats, 0, sizeof stats);
    if (rule) {
        // the chosen nodes accumulate while their statistics are taken; the mask pass then only re-reads
        if (z.tiles)
            IWP_LAUNCH_FEW("k_leader_stats", k_leader_stats, n_lead * z.tiles, fills_tiles(z.tiles, z.n_layers) ? FEW_READERS : 0u, s, P, w, layers, z.n_layers, z.tiles, leaders,
                       n_lead, W, eps, ws.tile_stats);
        const LayerRule lr{rule->alpha, rule->beta, rule->C, reinterpret_cast<double2*>(rule->stats_out), rule->thr_out};
        if (z.tiles && (uint64_t)n_lead * z.tiles <= RULE_MAX_TABLE && plan->max_layer_stiles <= RULE_MAX_TILES / GROUP)
            stats = TileStats{ws.tile_stats, z.tiles, lr};
        else
            IWP_LAUNCH("k_layer_thr", k_layer_thr, z.n_layers * n_lead, s, layers, z.tiles, leaders, n_lead, W, ws.tile_stats, lr);
        thr = rule->thr_out;
    }
#define IWP_MASK_AS(NL, GROUPS, RULE, THREADS)                                                                               \
    IWP_LAUNCH_BLOCK("k_leader_mask", (k_leader_mask<NL, GROUPS, RULE, THREADS>), z.tiles, dim3(THREADS, GROUPS), s, P, w, layers, \
                     z.n_layers, leaders, n_lead, W, thr, rule != nullptr, rule == nullptr, stats, rs, eps, mask32, ws.tile_counts, \
                     ws.slots)
#define IWP_MASK(NL, GROUPS, THREADS)                       \
    do {                                                    \
        if (stats.of) IWP_MASK_AS(NL, GROUPS, true, THREADS); \
        else IWP_MASK_AS(NL, GROUPS, false, THREADS);       \
    } while (0)
    if (z.tiles) {
        static_assert(RULE_MAX_TABLE <= WIDE_MASK_MAX_TILES, "the rule is merged by workgroups of WIDE_BLOCK, or by groups");
        const bool wide = z.tiles <= WIDE_MASK_MAX_TILES;
        if (n_lead == 1 && wide) IWP_MASK(1, 1, WIDE_BLOCK);
        else if (n_lead == 1) IWP_MASK_AS(1, 1, false, BLOCK);
        else if (n_lead == 2 && wide) IWP_MASK(2, 1, WIDE_BLOCK);
        else if (n_lead == 2) IWP_MASK_AS(2, 1, false, BLOCK);
        else if (n_lead == 3 && wide) IWP_MASK(3, 1, WIDE_BLOCK);
        else if (n_lead == 3) IWP_MASK_AS(3, 1, false, BLOCK);
        else if (n_lead == 4) IWP_MASK(2, 2, BLOCK);
        else if (n_lead <= 6) IWP_MASK(2, 3, BLOCK);
        else IWP_MASK(2, 4, BLOCK);
    }
#undef IWP_MASK
#undef IWP_MASK_AS
    uint32_t static_mask = 0, streaming = 0;
    for (uint32_t p = 0; p < W; ++p) {
        if (g[p]) ++streaming; else static_mask |= 1u << p;
    }
    if (z.tiles && follows_together(*plan, streaming)) {
        IWP_LAUNCH("k_follow_mask_sum", k_follow_mask_sum, CHUNKS_A_TILE * z.tiles, s, P, first_streaming(g, W), layers, z.n_layers,
                   z.tiles, leaders, n_lead, W, mask32, ws.tile_counts, count_out, max_pairs, ws.slots, idx_out, w, scale, sum_out);
        return IWP_OK;
    }
    const bool add_up = z.tiles && z.tiles <= ADD_UP_TILES;
    if (!add_up)
        IWP_LAUNCH_BLOCK("k_tile_offsets", k_tile_offsets, 1u, OFFSETS_BLOCK, s, layers, z.n_layers, z.tiles, ws.tile_counts, max_pairs,
                         ws.tile_pos, ws.lay_out, count_out);
    if (z.tiles == 0) return IWP_OK;
    const uint32_t runs = takes_runs(z.tiles, z.n_layers);
    uint32_t few = runs ? few_mask_followers(z.tiles, z.n_layers, streaming) : 0u;
    if (few && add_up) few -= ADD_UP_TILES * (uint32_t)sizeof(uint32_t);         // what the kernel has more
#define IWP_FOLLOW_MASK(ADD_UP)                                                                                              \
    IWP_LAUNCH_FEW("k_follow_mask", k_follow_mask<ADD_UP>, W * z.tiles, few, s, P, layers, z.n_layers, z.tiles, runs, leaders, n_lead, \
                   W, mask32, ws.tile_counts, ws.tile_pos, ws.lay_out, count_out, max_pairs, ws.slots, idx_out, ws.gathered)
    if (add_up) IWP_FOLLOW_MASK(true);
    else IWP_FOLLOW_MASK(false);
#undef IWP_FOLLOW_MASK
    const uint32_t pair_blocks = std::min<uint32_t>((max_pairs + BLOCK - 1) / BLOCK, 8192u);
    IWP_LAUNCH("k_reduce_update_counted", k_reduce_update_counted, pair_blocks, s, R, static_mask, z.n_layers, leaders, n_lead, W,
               ws.lay_out, count_out, max_pairs, ws.gathered, idx_out, w, scale, sum_out, plan->flat_end);
    return IWP_OK;
}

}  // namespace

size_t iwp_plan_mask_bytes(const iwp_plan* plan) { return plan ? (size_t)plan->z.mask_words * 4 : 0; }

size_t iwp_plan_threshold_workspace_bytes(const iwp_plan* plan, uint32_t W, uint32_t n_lead, uint32_t max_pairs) {
    return plan ? carve_threshold(nullptr, plan->z, W, n_lead, max_pairs).bytes : 0;
}

int iwp_step_threshold_segmented(const iwp_plan* plan, float* w, const float* const* g, float* const* r, uint32_t W,
                                 const uint32_t* leaders, uint32_t n_lead, const float* thr, float eps, float scale,
                                 uint8_t* mask_out, uint32_t* count_out, uint32_t* idx_out, float* sum_out,
                                 uint32_t max_pairs, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!thr) return IWP_EINVAL;
    return run_threshold_step(plan, w, g, r, W, leaders, n_lead, thr, nullptr, RandomSel{0, 0, 0, 0, 0}, eps, scale, mask_out,
                              count_out, idx_out, sum_out, max_pairs, workspace, workspace_bytes, hip_stream);
}

int iwp_step_threshold_random_segmented(const iwp_plan* plan, float* w, const float* const* g, float* const* r,
                                        uint32_t W, const uint32_t* leaders, uint32_t n_lead, const float* thr,
                                        uint64_t seed, uint64_t step, float eps, float scale, uint8_t* mask_out,
                                        uint32_t* count_out, uint32_t* idx_out, float* sum_out, uint32_t max_pairs,
                                        void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!thr) return IWP_EINVAL;
    const RandomSel rs{1u, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32)};
    return run_threshold_step(plan, w, g, r, W, leaders, n_lead, thr, nullptr, rs, eps, scale, mask_out, count_out, idx_out,
                              sum_out, max_pairs, workspace, workspace_bytes, hip_stream);
}

int iwp_step_layerwise_segmented(const iwp_plan* plan, float* w, const float* const* g, float* const* r, uint32_t W,
                                 const uint32_t* leaders, uint32_t n_lead, double alpha, double beta, double C, float eps,
                                 float scale, double* stats_out, float* thr_out, uint8_t* mask_out, uint32_t* count_out,
                                 uint32_t* idx_out, float* sum_out, uint32_t max_pairs, void* workspace,
                                 size_t workspace_bytes, void* hip_stream) {
    if (!stats_out || !thr_out) return IWP_EINVAL;
    if (!std::isfinite(alpha) || !std::isfinite(beta) || !std::isfinite(C)) return IWP_EINVAL;
    if ((reinterpret_cast<uintptr_t>(stats_out) & 15u) || !aligned4(thr_out)) return IWP_EALIGN;
    LayerwiseRule rule{alpha, beta, C, stats_out, thr_out};
    return run_threshold_step(plan, w, g, r, W, leaders, n_lead, thr_out, &rule, RandomSel{0, 0, 0, 0, 0}, eps, scale, mask_out, count_out, idx_out,
                              sum_out, max_pairs, workspace, workspace_bytes, hip_stream);
}

// ----------------------------------------------------------------- helpers

int iwp_score_keys(const float* w, const float* r, uint32_t n, float eps, uint32_t* key_out, void* hip_stream) {
    if (check_eps(eps)) return IWP_EINVAL;
    if (n == 0) return IWP_OK;
    if (!w || !r || !key_out) return IWP_EINVAL;
    if (!aligned4(w) || !aligned4(r) || !aligned4(key_out)) return IWP_EALIGN;
    uint32_t grid = (uint32_t)std::min<uint64_t>(((uint64_t)n + BLOCK - 1) / BLOCK, 65536);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    IWP_LAUNCH("k_score_keys", k_score_keys, grid, s, w, r, n, eps, key_out);
    return IWP_OK;
}

int iwp_copy_f32(float* dst, const float* src, uint64_t n, void* hip_stream) {
    if (n == 0) return IWP_OK;
    if (!dst || !src) return IWP_EINVAL;
    if ((reinterpret_cast<uintptr_t>(dst) & 15u) || (reinterpret_cast<uintptr_t>(src) & 15u)) return IWP_EALIGN;
    const uint64_t blocks = (n / 4 + BLOCK - 1) / BLOCK;
    if (blocks > 0x7FFFFFFFull) return IWP_ERANGE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    IWP_LAUNCH("k_copy", k_copy, (uint32_t)std::max<uint64_t>(blocks, 1), s, dst, src, n);
    return IWP_OK;
}

int iwp_timing_enable(const char* kernel_name, uint32_t max_launches) {
    if (!kernel_name || strlen(kernel_name) >= sizeof g_timing.name) return IWP_EINVAL;
    if (max_launches == 0 || max_launches > (uint32_t)Timing::MAX) max_launches = Timing::MAX;
    while (g_timing.start.size() < max_launches) {
        hipEvent_t a, b;
        IWP_HIP(hipEventCreate(&a));
        IWP_HIP(hipEventCreate(&b));
        g_timing.start.push_back(a);
        g_timing.stop.push_back(b);
    }
    strcpy(g_timing.name, kernel_name);
    g_timing.used = 0;
    g_timing.enabled = true;
    return IWP_OK;
}

int iwp_timing_collect(double* total_ms, uint32_t* launches) {
    if (!total_ms || !launches) return IWP_EINVAL;
    g_timing.enabled = false;
    double sum = 0.0;
    for (int i = 0; i < g_timing.used; ++i) {
        IWP_HIP(hipEventSynchronize(g_timing.stop[i]));
        float ms = 0.f;
        IWP_HIP(hipEventElapsedTime(&ms, g_timing.start[i], g_timing.stop[i]));
        sum += ms;
    }
    *total_ms = sum;
    *launches = (uint32_t)g_timing.used;
    g_timing.used = 0;
    return IWP_OK;
}

}  // extern "C"
