// epic.hip -- dense flow from the tracked points by edge-preserving interpolation (DeGraF-Flow,
// Section 2 "Interpolation"; k from Section 3 "Parameters").  Every pixel takes an affine motion
// fitted to the k tracked points nearest to it in a geodesic distance that penalises crossing
// edges of an image-gradient map.  Geodesic neighbours are built as in the cited interpolator:
// a geodesic Voronoi partition of the pixels among the points, a graph on the points joining
// adjacent cells, and neighbour searches on that graph, so every pixel of a cell shares its
// point's model.
//
// GPU structure (one pass each unless noted):
//   k_epic_prep     edge map (uint16) and cleared tables, HBM bound
//   k_epic_seed     one 64-bit atomicMin per converged point: key = (0 << 32) | index
//   k_epic_relax    62x32 tiles relaxed in registers (Bellman-Ford sweeps), exchanging border
//                   pixels with their neighbours during the launch; a grid that fits the chip
//                   settles in one launch, a larger one is launched until nothing changes
//   k_epic_graph    adjacent-cell pairs, gathered per tile in LDS, inserted into fixed-size
//                   per-seed adjacency rows
//   k_epic_least    each seed's least edge
//   k_epic_knn_fit  one wavefront per seed: Dijkstra on the seed graph with the frontier and a
//                   hash index in LDS, stopped after k settles; FP64 weighted affine fit by
//                   modified Gram-Schmidt across the wavefront
//   k_epic_dense    every pixel evaluates its cell's model, HBM bound
// Keys pack (distance << 32 | seed index), so one unsigned 64-bit minimum orders by distance and
// breaks ties by the lower index; all distances are exact integers.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "dgf_internal.hpp"

namespace dgf {
namespace {

constexpr int kMaxDeg = 32;          // graph neighbours a seed can hold
constexpr int kCand = 384;           // candidates one neighbour search can hold (about 210 needed at k 128)
constexpr int kHash = 512;           // LDS hash slots of one search (power of two, > kCand + 64)
constexpr int kMaxK = 256;           // largest k
// Relaxation tile: a wavefront holds 64 columns, the outer two of them the neighbouring tiles', and
// kRRows rows of them, one column's run per lane; kRWaves wavefronts stack up.  The 1242x375 frame
// then has 252 tiles, one per CU.
constexpr int kRTX = 62;             // tile width
constexpr int kRRows = 8;            // rows per wavefront
constexpr int kRWaves = 4;
constexpr int kRTY = kRWaves * kRRows; // tile height
constexpr int kRelaxThreads = 64 * kRWaves;
constexpr int kInner = 4;            // relaxation iterations of a round, between two checks for changes
constexpr int kExchange = 8;         // rounds between two halo exchanges
constexpr int kMaxRounds = 2048;     // rounds per tile and launch
constexpr int kMaxPolls = 1 << 16;   // halo polls of a still tile per launch (some 40 ms)
constexpr int kPollSleep = 2;        // 64-cycle units between two polls
constexpr int kLinger = 32;          // halo polls of a still tile per launch of a grid that does not fit the chip
constexpr int kStartPolls = 256;     // polls a resident grid waits for tiles that have not started
constexpr int kChunk = 4;            // relaxation launches between two convergence checks, and sets of their counters
constexpr int kMaxRelaxLaunches = 1 << 14;
constexpr int kDefaultAsyncRelax = 32; // dgf_epic_async's relaxation launches when given 0
constexpr uint64_t kNoKey = ~0ull;
constexpr uint64_t kDistCap = 0xFFFFFFFEull;
constexpr int kMaxEdge = 510;        // largest edge-map value
constexpr uint32_t kLeastCap = 1u << 30; // a least edge at or above this bounds nothing (distances stay below)

enum : uint32_t { kErrDegree = 1u, kErrCand = 2u };

struct EpicWs {
    uint64_t *keys;  // [H*W]
    uint16_t *E;     // [H*W]
    uint64_t *adj;   // [n][kMaxDeg]: (edge length << 32) | neighbour, kNoKey = empty slot
    float *model;    // [n][8]: affine coefficients (6), least edge of the seed (uint32 bits), unused
    uint32_t *ctr;   // [kChunk] tiles changed by a relaxation launch, [1] error bits, [kChunk] open
                     // count and [kChunk] done flag of a relaxation launch (launch j uses set
                     // j mod kChunk of these, of mail and of state)
    uint32_t *mail;  // [kChunk][tiles]: a neighbour published keys into this tile's halo
    uint32_t *state; // [kChunk][tiles]: 0 before the tile starts, then 4 x times resumed + 2, + 1 while still
};

int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }

int64_t ws_layout(int W, int H, int64_t n, EpicWs *ws, char *base)
{
    const int64_t N = (int64_t)W * H;
    int64_t off = 0;
    auto take = [&](int64_t bytes) {
        const int64_t o = off;
        off += align256(bytes);
        return base ? base + o : nullptr;
    };
    char *keys = take(8 * N), *E = take(2 * N), *adj = take(8 * n * kMaxDeg);
    const int64_t tiles = (int64_t)((W + kRTX - 1) / kRTX) * ((H + kRTY - 1) / kRTY);
    char *model = take(32 * n), *ctr = take(4 * (3 * kChunk + 1)), *mail = take(8 * kChunk * tiles);
    if (ws) {
        ws->keys = (uint64_t *)keys;
        ws->E = (uint16_t *)E;
        ws->adj = (uint64_t *)adj;
        ws->model = (float *)model;
        ws->ctr = (uint32_t *)ctr;
        ws->mail = (uint32_t *)mail;
        ws->state = ws->mail + kChunk * tiles;
    }
    return off;
}

__device__ __forceinline__ uint64_t load_key(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t load_word(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_word(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_key(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The least edge length of a seed's row.
__device__ __forceinline__ uint32_t *least_edge_at(const EpicWs &ws, int64_t s) { return (uint32_t *)ws.model + 8 * s + 6; }
__device__ __forceinline__ uint32_t least_edge(const EpicWs &ws, int64_t s) { return *least_edge_at(ws, s); }

// Edge map and cleared key / adjacency tables / least edges / counters.
__global__ void k_epic_prep(const uint8_t *I, int64_t pitch, int W, int H, int64_t n, uint32_t tiles, EpicWs ws)
{
    const uint32_t N = (uint32_t)W * (uint32_t)H;
    const int64_t S = n * kMaxDeg, C = 2 * (int64_t)kChunk * tiles + 3 * kChunk + 1;
    const int64_t tot = max(max(S, (int64_t)N), C);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < tot; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < (int64_t)N) {
            const uint32_t q = (uint32_t)i, y = q / (uint32_t)W, x = q - y * (uint32_t)W;
            const int xl = x > 0 ? (int)x - 1 : 0, xr = (int)x + 1 < W ? (int)x + 1 : W - 1;
            const int yu = y > 0 ? (int)y - 1 : 0, yd = (int)y + 1 < H ? (int)y + 1 : H - 1;
            const uint8_t *row = I + (int64_t)y * pitch;
            const int gx = (int)row[xr] - (int)row[xl];
            const int gy = (int)I[(int64_t)yd * pitch + x] - (int)I[(int64_t)yu * pitch + x];
            ws.E[i] = (uint16_t)(abs(gx) + abs(gy));
            ws.keys[i] = kNoKey;
        }
        if (i < S) ws.adj[i] = kNoKey;
        if (i <= 3 * kChunk) ws.ctr[i] = 0u;
        if (i < 2 * (int64_t)kChunk * tiles) ws.mail[i] = 0u; // and state
    }
}

// Seed pixel of a point, (floor(x + 1/2), floor(y + 1/2)) clamped into the image; false for a
// point that takes no part (not converged, or a non-finite position or flow).
__device__ __forceinline__ bool seed_pixel(const float *pts, const float *flow, const uint8_t *status, int64_t i,
                                           int W, int H, uint32_t &q)
{
    if (status[i] != DGF_ST_CONVERGED) return false;
    const float x = pts[2 * i], y = pts[2 * i + 1];
    if (!isfinite(x) || !isfinite(y) || !isfinite(flow[2 * i]) || !isfinite(flow[2 * i + 1])) return false;
    const int px = (int)fminf(fmaxf(floorf(x + 0.5f), 0.f), (float)(W - 1));
    const int py = (int)fminf(fmaxf(floorf(y + 0.5f), 0.f), (float)(H - 1));
    q = (uint32_t)py * (uint32_t)W + (uint32_t)px;
    return true;
}

__global__ void k_epic_seed(const float *pts, const float *flow, const uint8_t *status, int64_t n, int W, int H,
                            uint64_t *keys)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t q;
    if (seed_pixel(pts, flow, status, i, W, H, q)) atomicMin((unsigned long long *)(keys + q), (unsigned long long)i);
}

// How the relaxation handles keys.  A key is the pair (distance, seed), the least first.
//   Fast: distances below kFar, whose keys as bit patterns are positive doubles, so that one
//         v_min_f64 takes the lesser of two (denormals are kept in double precision).  No key is
//         kFar in the distance half; kFar plus any step stays below the doubles' infinities.
//   else: any distance up to kDistCap, by 64-bit integer comparisons; a sum beyond that is no key.
constexpr uint32_t kFar = 0x3F000000u;

enum : uint32_t { kDone = 1u, kLeave = 2u };

// The counters of one relaxation launch.
struct RelaxCounters {
    uint32_t *changed; // tiles that changed anything
    uint32_t *open;    // tiles that left before the whole grid had settled
    uint32_t *done;    // kDone once it has, kLeave when the still tiles are to make room
    uint32_t *mail, *state; // [tiles]
};

RelaxCounters relax_counters(const EpicWs &ws, int launch, int64_t tiles)
{
    const int c = launch % kChunk;
    return {ws.ctr + c, ws.ctr + kChunk + 1 + c, ws.ctr + 2 * kChunk + 1 + c, ws.mail + c * tiles, ws.state + c * tiles};
}

template <bool FAST>
__device__ __forceinline__ uint64_t key_of(uint64_t k) // a stored key, as the relaxation holds it
{
    return FAST && k == kNoKey ? ((uint64_t)kFar << 32) | 0xFFFFFFFFu : k;
}

template <bool FAST>
constexpr uint32_t kWall = FAST ? kFar + 1u : 0xFFFFFFFFu; // a step nobody takes

// The lesser of `mine` and `from` (a neighbour's key) after a step of cost c.
template <bool FAST>
__device__ __forceinline__ uint64_t key_relax(uint64_t mine, uint64_t from, uint32_t c)
{
    const uint32_t lo = (uint32_t)from, hi = (uint32_t)(from >> 32);
    if constexpr (FAST) {
        double a = __builtin_bit_cast(double, mine);
        const double v = __builtin_bit_cast(double, ((uint64_t)(hi + c) << 32) | lo);
        // (written out: the library's minimum would first quiet signalling NaNs, which no key is)
        asm("v_min_f64 %0, %0, %1" : "+v"(a) : "v"(v));
        return __builtin_bit_cast(uint64_t, a);
    } else {
        // an overflowing sum is no key.  (Zero plus a wall does not overflow: the end lanes, into which the
        // shifts bring zeros, may take it, but nothing comes of it: no step leads out of all ones.)
        const uint32_t d = hi + c;
        const bool over = d < hi;
        const uint64_t v = ((uint64_t)(over ? 0xFFFFFFFFu : d) << 32) | (over ? 0xFFFFFFFFu : lo);
        return v < mine ? v : mine;
    }
}

// The key of the lane to the left / right (whole-wavefront shifts).
template <int CTRL>
__device__ __forceinline__ uint64_t key_shift(uint64_t k)
{
    auto half = [](unsigned v) { return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true); };
    return (uint64_t)half((unsigned)k) | ((uint64_t)half((unsigned)(k >> 32)) << 32);
}

// One relaxation launch: key(p) = min(key(p), min over 4-neighbours q of key(q) + step(q, p)) to the
// fixed point, over tiles of 62 x 32 pixels.  Pixels live in registers, a run of kRRows rows of one
// column per lane.  An iteration relaxes every pixel from its left and right neighbours (the lanes
// next to it), then down the run and up it again, so a path advances a column per iteration and any
// number of rows inside a run; the runs' end rows are exchanged through LDS, without a barrier,
// since keys only decrease and any interleaving converges to the same least keys.  Lanes 0 and 63
// hold the neighbouring tiles' columns and take no part themselves (their steps cost a wall).
// Every kInner iterations the tile looks for changes.  Every kExchange such rounds, and when it has
// stopped changing, it publishes its changed border pixels (a pixel is only ever written by its own
// tile) and posts mail to each neighbour tile whose halo they touch; a tile with mail re-reads its
// halo.  With `wait` (the whole grid fits the chip at once) a still tile polls its mailbox and resumes on
// mail; polls are bounded (kMaxPolls), so every tile exits, but the bound outlasts the longest paths of a
// resident grid: a tile that left before the front came would cost a launch (one seed in a 2048x1024 frame,
// whole call: 11.2 ms at 4,096 polls, 2.2 at 65,536).  Termination: a tile says in its state
// word that it is still, after its last mail was posted, and that it is working again before it takes
// the mail that woke it.  Tile 0, itself still, reads every state, then every mailbox and every state
// again: all still with unchanged words means that all were still between the two readings, and with
// every mailbox empty after that no tile can change anything any more, so it raises `done`, on
// which every still tile leaves; where other work on the chip has kept some tiles from starting for
// kStartPolls polls it sends the still tiles away instead, to make room.  (One count of working tiles and unread mail, kept with atomics,
// was the bottleneck: its address took an atomic from every exchange of every tile.)  Keys always
// belong to a real path, so a launch in which no tile changes anything is at the fixed point.
// What bounds it is the longest least path: its iterations (about 110 VALU instructions, 0.2 us with a
// wavefront per SIMD) and its tile crossings (an exchange, about 2 us).  1242x375: 228 -> 128 us for the
// launch that works and the one that confirms; 2048x1024 (1,088 tiles) 160 us in the working launch with
// 117,238 seeds all over the frame, 257 and 441 with as many and more that leave stretches empty.  The form before kept 32x64 tiles in LDS, four pixels a lane, at about 28
// instructions and 5 LDS accesses a pixel and iteration, one column or row per iteration.
// Without `wait` a still tile looks for mail kLinger times before it leaves, so that a front that comes
// down or up the rows of tiles on the chip together crosses more than one of them a launch: seeds along the
// lower edge of 8192x700 reach every pixel in 16 launches (33 without, 8 polls 29, 128 polls 9), and the
// whole call takes 1,627 us on 4096x2160, 137,459 seeds (1,940 without, 8 polls 1,760, 128 polls 1,893).
// The launch counts the tiles that changed anything and those that left before they saw the whole
// grid settled.  prev (nullable) is the counters of the launch before: when either of its counts is
// zero the distances are already at the fixed point and the launch returns at once, with nothing
// changed (so a fixed number of launches can be enqueued without reading anything back).  Each launch
// clears the counters of the launch after the next, `next`, which nobody reads or writes meanwhile.
template <bool FAST>
__global__ __launch_bounds__(kRelaxThreads, 5) void k_epic_relax(int W, int H, int kappa, uint64_t *keys,
                                                                 const uint16_t *E, RelaxCounters now, int wait,
                                                                 RelaxCounters prev, RelaxCounters next, int tiles_x)
{
    constexpr uint32_t wall = kWall<FAST>;
    constexpr int R = kRRows;
    uint32_t *const mail = now.mail, *const state = now.state;
    const int me = (int)blockIdx.x, tiles = (int)gridDim.x;
    if (threadIdx.x == 0) {
        next.mail[me] = next.state[me] = 0u;
        if (me == 0) *next.changed = *next.open = *next.done = 0u;
    }
    // (the same values in every block: an earlier kernel wrote them)
    if (prev.changed && (*prev.changed == 0u || *prev.open == 0u)) return;
    // row 0: the row above the tile; 1 + 2w, 2 + 2w: first and last row of wavefront w; then the row below
    __shared__ uint64_t rows[2 * kRWaves + 2][64];
    __shared__ uint32_t flags[2][kRWaves];
    __shared__ uint32_t sides, poll;
    const int tile_y = me / tiles_x, tile_x = me - tile_y * tiles_x;
    const int nbr_tile[4] = {tile_x > 0 ? me - 1 : -1, tile_x + 1 < tiles_x ? me + 1 : -1,
                             tile_y > 0 ? me - tiles_x : -1, me + tiles_x < tiles ? me + tiles_x : -1};
    if (wait && threadIdx.x == 0) store_word(state + me, 2u);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x = tile_x * kRTX - 1 + lane, y0 = tile_y * kRTY + wave * R;
    const bool halo = lane == 0 || lane == 63, in_x = x >= 0 && x < W;
    // the run's pixels that belong to the tile (bit j)
    const uint32_t mine = in_x && !halo ? (1u << clampi(H - y0, 0, R)) - 1u : 0u;
    auto at = [&](int y) { return (int64_t)y * W + x; };
    auto load = [&](int y) { return in_x && y >= 0 && y < H ? key_of<FAST>(load_key(keys + at(y))) : key_of<FAST>(kNoKey); };
    auto put_row = [&](int r, uint64_t k) {
        __hip_atomic_store(&rows[r][lane], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto get_row = [&](int r) {
        return __hip_atomic_load(&rows[r][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };

    uint64_t own[R], snap[R]; // the pixels' keys, now and at the last check
    uint32_t cl[R], cr[R];    // step costs from the left and the right neighbour
    uint32_t cv[R + 1];       // between rows j - 1 and j (both ways)
    {
        uint32_t e[R + 2]; // edge values of rows -1 .. R
#pragma unroll
        for (int j = -1; j <= R; ++j) {
            const int y = y0 + j;
            e[j + 1] = in_x && y >= 0 && y < H ? E[at(y)] : 0u;
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            own[j] = load(y0 + j);
            snap[j] = own[j];
            const uint32_t ke = (uint32_t)kappa + e[j + 1];
            const uint32_t l = ke + dppu<0x138>(e[j + 1]), r = ke + dppu<0x130>(e[j + 1]);
            const bool in = (mine >> j) & 1u; // (pixels outside the image stay without a key)
            cl[j] = in && x > 0 ? l : wall;
            cr[j] = in && x + 1 < W ? r : wall;
        }
#pragma unroll
        for (int j = 0; j <= R; ++j)
            cv[j] = in_x && !halo && y0 + j > 0 && y0 + j < H ? (uint32_t)kappa + e[j] + e[j + 1] : wall;
    }
    put_row(1 + 2 * wave, own[0]);
    put_row(2 + 2 * wave, own[R - 1]);
    if (wave == 0) put_row(0, load(y0 - 1));
    if (wave == kRWaves - 1) put_row(2 * kRWaves + 1, load(y0 + R));
    if (threadIdx.x == 0) sides = 0u;
    __syncthreads();

    // re-read the neighbouring tiles' pixels
    auto reload_halo = [&]() {
        if (halo)
#pragma unroll
            for (int j = 0; j < R; ++j) {
                own[j] = load(y0 + j);
                snap[j] = own[j];
            }
        if (wave == 0) put_row(0, load(y0 - 1));
        if (wave == kRWaves - 1) put_row(2 * kRWaves + 1, load(y0 + R));
        __syncthreads();
    };
    uint32_t pend = 0u, ever = 0u; // pixels changed since the last publication, and at all (bit j)
    // the sides of the tile that pixel j lies on (bit per neighbour tile)
    auto sides_of = [&](int j) {
        return (lane == 1 ? 1u : 0u) | (lane == kRTX ? 2u : 0u) | (wave == 0 && j == 0 ? 4u : 0u) |
               (wave == kRWaves - 1 && j == R - 1 ? 8u : 0u);
    };
    // publish changed border pixels and post mail to the tiles whose halos they touch
    auto publish = [&]() {
        uint32_t my_sides = 0u;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint32_t sd = sides_of(j);
            if (((pend >> j) & 1u) && sd) {
                store_key(keys + at(y0 + j), own[j]);
                my_sides |= sd;
            }
        }
        pend = 0u;
        if (my_sides) atomicOr(&sides, my_sides);
        if (__ballot(my_sides != 0u)) __builtin_amdgcn_s_waitcnt(0); // the keys are there before the mail
        __syncthreads();
        if (threadIdx.x < 4 && ((sides >> threadIdx.x) & 1u) && nbr_tile[threadIdx.x] >= 0)
            store_word(mail + nbr_tile[threadIdx.x], 1u);
        if (threadIdx.x == 0) sides = 0u;
    };
    // take this tile's mail and re-read the halo
    auto take_mail = [&]() {
        if (threadIdx.x == 0) {
            atomicExch(mail + me, 0u);
            __builtin_amdgcn_s_waitcnt(0); // taken before the halo is read: later mail is kept
        }
        __syncthreads();
        reload_halo();
    };
    // (tile 0, all threads) 0: some tile is working or may, 1: none can change anything any more, 2: some
    // have not started
    auto all_settled = [&]() {
        uint32_t first = 0u, second = 0u, letters = 0u, still = 1u, started = 2u;
        for (int i = (int)threadIdx.x; i < tiles; i += kRelaxThreads) {
            const uint32_t v = load_word(state + i);
            first += v; // (resume counts only grow, so sums will do)
            still &= v;
            started = v == 0u ? 0u : started;
        }
        if (!__syncthreads_and(still & 1u)) return __syncthreads_and(started) ? 0 : 2;
        for (int i = (int)threadIdx.x; i < tiles; i += kRelaxThreads) letters |= load_word(mail + i);
        __builtin_amdgcn_s_waitcnt(0); // the mailboxes before the states
        for (int i = (int)threadIdx.x; i < tiles; i += kRelaxThreads) {
            const uint32_t v = load_word(state + i);
            second += v;
            still &= v;
        }
        return __syncthreads_and((still & 1u) && letters == 0u && first == second) ? 1 : 0;
    };
    int polls = 0;
    uint32_t resumed = 0u;
    bool settled = false; // left because no tile can change anything
    for (int round = 0; round < kMaxRounds; ++round) {
        const bool exchange = (round + 1) % kExchange == 0;
        uint32_t mailed = 0u;
        if (exchange && threadIdx.x == 0) mailed = load_word(mail + me); // in flight during the round
        for (int it = 0; it < kInner; ++it) {
            const uint64_t above = get_row(2 * wave), below = get_row(2 * wave + 3);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const uint64_t l = key_shift<0x138>(own[j]), r = key_shift<0x130>(own[j]);
                own[j] = key_relax<FAST>(key_relax<FAST>(own[j], l, cl[j]), r, cr[j]);
            }
            own[0] = key_relax<FAST>(own[0], above, cv[0]);
#pragma unroll
            for (int j = 1; j < R; ++j) own[j] = key_relax<FAST>(own[j], own[j - 1], cv[j]);
            own[R - 1] = key_relax<FAST>(own[R - 1], below, cv[R]);
#pragma unroll
            for (int j = R - 2; j >= 0; --j) own[j] = key_relax<FAST>(own[j], own[j + 1], cv[j + 1]);
            put_row(1 + 2 * wave, own[0]);
            put_row(2 + 2 * wave, own[R - 1]);
        }
        uint32_t ch = 0u;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            ch |= (own[j] != snap[j] ? 1u : 0u) << j;
            snap[j] = own[j];
        }
        ch &= mine;
        pend |= ch;
        ever |= ch;
        // one barrier: each wavefront posts whether any of its lanes changed anything, the first also
        // the mail.  (No change anywhere in a whole round: the rows read were the final ones, so this
        // is the fixed point of the tile.)
        const bool changed_lanes = __ballot(ch != 0u) != 0ull;
        if (lane == 0) flags[round & 1][wave] = (changed_lanes ? 1u : 0u) | (mailed ? 2u : 0u);
        __syncthreads();
        uint32_t seen = 0u;
#pragma unroll
        for (int w = 0; w < kRWaves; ++w) seen |= flags[round & 1][w];
        const bool any = (seen & 1u) != 0u;
        if (any && !exchange) continue;
        publish();
        if (seen & 2u) {
            take_mail();
            continue;
        }
        if (any) continue;
        // still
        if (wait && threadIdx.x == 0) {
            __builtin_amdgcn_s_waitcnt(0); // the mail it posted is there
            store_word(state + me, 4u * resumed + 3u);
        }
        bool resume = false;
        while (polls < kMaxPolls) {
            if (threadIdx.x == 0)
                poll = (load_word(mail + me) ? 1u : 0u) | (wait && me != 0 ? load_word(now.done) << 1 : 0u);
            __syncthreads();
            const uint32_t p = poll;
            resume = (p & 1u) != 0u;
            settled = p == 2u * kDone;
            if (p || (!wait && polls >= kLinger)) break;
            ++polls;
            if (wait && me == 0) {
                const int all = all_settled();
                settled = all == 1;
                const bool leave = settled || (all == 2 && polls >= kStartPolls);
                if (leave && threadIdx.x == 0) store_word(now.done, settled ? kDone : kLeave);
                if (leave) break;
            }
            __builtin_amdgcn_s_sleep(kPollSleep);
            __syncthreads();
        }
        if (!resume) break;
        ++resumed;
        if (wait && threadIdx.x == 0) {
            store_word(state + me, 4u * resumed + 2u);
            __builtin_amdgcn_s_waitcnt(0); // working again before the mail is taken
        }
        take_mail();
    }
    // leave
#pragma unroll
    for (int j = 0; j < R; ++j)
        if ((ever >> j) & 1u) store_key(keys + at(y0 + j), own[j]);
    const bool wrote = __syncthreads_or(ever != 0u) != 0;
    if (threadIdx.x == 0) {
        if (!settled) {
            atomicAdd(now.open, 1u);
            if (wait) store_word(now.done, kLeave); // (out of rounds or polls: nobody waits for this tile)
        }
        if (wrote) atomicAdd(now.changed, 1u);
    }
}

// Insert (or lower) the edge s -> t of length w into s's adjacency row: a slot holds
// (length << 32) | t, so once t owns a slot a 64-bit atomicMin keeps the least length.  Four slots are
// read at a time: one round trip to memory instead of one a slot.
__device__ void adj_insert(const EpicWs &ws, uint32_t s, uint32_t t, uint32_t w, uint32_t *err)
{
    unsigned long long *row = (unsigned long long *)(ws.adj + (int64_t)s * kMaxDeg);
    const unsigned long long val = ((unsigned long long)w << 32) | t;
    for (int j0 = 0; j0 < kMaxDeg; j0 += 4) {
        unsigned long long c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = __hip_atomic_load(row + j0 + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned long long cur = c[i];
            if (cur == kNoKey) {
                cur = atomicCAS(row + j0 + i, (unsigned long long)kNoKey, val);
                if (cur == kNoKey) return;
            }
            if ((uint32_t)cur == t) {
                if (val < cur) atomicMin(row + j0 + i, val);
                return;
            }
        }
    }
    atomicOr(err, kErrDegree);
}

// Least value over the wavefront, returned to every lane (DPP and row swaps, as the sums).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    v = min(v, dppu<0xB1>(v));
    v = min(v, dppu<0x4E>(v));
    v = min(v, dppu<0x141>(v));
    v = min(v, dppu<0x140>(v));
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min((uint32_t)p[0], (uint32_t)p[1]);
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return min((uint32_t)r[0], (uint32_t)r[1]);
}

// Seed graph: every right / down pixel pair whose cells differ gives both cells an edge of
// length D(p) + step(p, q) + D(q); each row keeps the least length per neighbour.  A workgroup takes a
// tile of 64 columns and four wavefronts of ROWS rows and keeps the least length of each pair of cells it
// meets in a hash table in LDS; only the table's entries then go to the rows in device memory, whose
// atomics are what the launch waits for: a pair of cells meets along several pixels, and the rows took
// one insertion for each run of them.  An entry that finds no place in the table within kGraphProbes
// steps, or finds the table full but for an eighth, goes to the rows directly.
//
// A lane's pixels and insertions are a serial chain, so a frame that leaves CUs without a workgroup
// takes fewer rows: eight from 2^19 pixels on (2048x1024, a seed every 5 px: 53 us, 90 with two; the
// one insertion for each run 426), two below (640x480, every 2 px: 39 us, 107 with eight; 86), one below
// 2^16 (128x96, a seed on every pixel: 12 us, 23 with two, 133 with eight; 12).  A table of 1,024
// entries took 32 steps for each of the 1,500 pairs that meet in 64 x 32 pixels with a seed every 2 px
// (1242x375: 109 us, 51 now).
constexpr int kGraphW = 64, kGraphWaves = 4;
constexpr int kGraphHash = 2048;
constexpr int kGraphProbes = 8;
constexpr int kGraphFull = kGraphHash / 8 * 7;

int graph_rows(int64_t pixels) { return pixels >= 1 << 19 ? 8 : pixels >= 1 << 16 ? 2 : 1; }

template <int ROWS>
__global__ __launch_bounds__(64 * kGraphWaves) void k_epic_graph(int W, int H, int kappa, const uint64_t *keys,
                                                                 const uint16_t *E, EpicWs ws, uint32_t *err,
                                                                 const uint32_t *unsettled)
{
    if (unsettled && *unsettled) return; // the partition did not reach its fixed point
    __shared__ unsigned long long hkey[kGraphHash]; // lower seed << 32 | higher seed
    __shared__ uint32_t hlen[kGraphHash];
    __shared__ uint16_t list[kGraphHash]; // the used entries
    __shared__ int used;
    for (int i = threadIdx.x; i < kGraphHash; i += 64 * kGraphWaves) {
        hkey[i] = kNoKey;
        hlen[i] = 0xFFFFFFFFu;
    }
    if (threadIdx.x == 0) used = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int x = (int)blockIdx.x * kGraphW + lane, y0 = ((int)blockIdx.y * kGraphWaves + wave) * ROWS;
    auto length = [&](uint64_t kp, uint32_t ep, uint64_t kq, uint32_t eq) {
        const uint64_t w64 = (kp >> 32) + (uint64_t)kappa + ep + eq + (kq >> 32);
        return w64 < 0xFFFFFFFFull ? (uint32_t)w64 : 0xFFFFFFFFu;
    };
    // adjacent pixels p and q into the table; true when their cells' pair found no place
    auto meet = [&](uint64_t kp, uint32_t ep, uint64_t kq, uint32_t eq) {
        const uint32_t ls = (uint32_t)kp, lt = (uint32_t)kq;
        if (ls == lt) return false;
        const unsigned long long pair = ((unsigned long long)min(ls, lt) << 32) | max(ls, lt);
        uint32_t h = (ls ^ lt) * 2654435761u + (ls + lt) * 2246822519u;
        h = (h >> 16) & (kGraphHash - 1);
        if (__hip_atomic_load(&used, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= kGraphFull) return true;
        for (int probe = 0; probe < kGraphProbes; ++probe) {
            const unsigned long long cur = atomicCAS(&hkey[h], (unsigned long long)kNoKey, pair);
            if (cur == kNoKey) list[atomicAdd(&used, 1)] = (uint16_t)h;
            if (cur == kNoKey || cur == pair) {
                atomicMin(&hlen[h], length(kp, ep, kq, eq));
                return false;
            }
            h = (h + 1) & (kGraphHash - 1);
        }
        return true;
    };
    auto key_at = [&](int xx, int yy) { return keys[(int64_t)yy * W + xx]; };
    auto edge_at = [&](int xx, int yy) { return (uint32_t)E[(int64_t)yy * W + xx]; };
    if (x < W) {
        // all the keys first: the rows' and the column to the right of the tile
        uint64_t k[ROWS + 1], kr[ROWS];
        uint32_t e[ROWS + 1], er[ROWS], missed = 0u;
#pragma unroll
        for (int j = 0; j <= ROWS; ++j) {
            const int y = min(y0 + j, H - 1);
            k[j] = key_at(x, y);
            e[j] = edge_at(x, y);
            if (j < ROWS) {
                kr[j] = key_at(min(x + 1, W - 1), y);
                er[j] = edge_at(min(x + 1, W - 1), y);
            }
        }
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            if (y0 + j >= H) break;
            if (x + 1 < W && meet(k[j], e[j], kr[j], er[j])) missed |= 1u << (2 * j);
            if (y0 + j + 1 < H && meet(k[j], e[j], k[j + 1], e[j + 1])) missed |= 2u << (2 * j);
        }
        for (; missed; missed &= missed - 1u) {
            const int b = __builtin_ctz(missed), y = y0 + (b >> 1), qx = x + (b & 1 ? 0 : 1), qy = y + (b & 1);
            const uint64_t kp = key_at(x, y), kq = key_at(qx, qy);
            const uint32_t w = length(kp, edge_at(x, y), kq, edge_at(qx, qy));
            adj_insert(ws, (uint32_t)kp, (uint32_t)kq, w, err);
            adj_insert(ws, (uint32_t)kq, (uint32_t)kp, w, err);
        }
    }
    __syncthreads();
    // both directions of every entry
    for (int i = threadIdx.x; i < 2 * used; i += 64 * kGraphWaves) {
        const int h = list[i >> 1];
        const uint32_t a = (uint32_t)(hkey[h] >> 32), b = (uint32_t)hkey[h];
        adj_insert(ws, i & 1 ? b : a, i & 1 ? a : b, hlen[h], err);
    }
}

// The least edge of every seed's row, eight lanes to a row (rows fill from slot 0).
__global__ __launch_bounds__(256) void k_epic_least(int64_t n, EpicWs ws, const uint32_t *unsettled)
{
    if (unsettled && *unsettled) return;
    const int64_t s = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 3;
    const int slot = threadIdx.x & 7;
    if (s >= n) return; // (whole rows: blocks hold 32)
    const uint64_t *row = ws.adj + s * kMaxDeg + slot;
    uint32_t least = kLeastCap;
    for (int j = 0; j < kMaxDeg; j += 8) {
        const uint64_t e = row[j];
        least = min(least, (uint32_t)(e >> 32)); // an empty slot is all ones
        if ((__ballot(e != kNoKey) >> ((threadIdx.x & 56) + 7) & 1ull) == 0ull) break; // this row's eighth
    }
    least = min(least, dppu<0xB1>(least));
    least = min(least, dppu<0x4E>(least));
    least = min(least, dppu<0x141>(least));
    if (slot == 0) *least_edge_at(ws, s) = least;
}

struct EpicFit {
    const float *pts, *flow;
    const uint8_t *status;
    const uint64_t *keys;
    EpicWs ws;
    int64_t n;
    int W, H, k, h, kappa;
    uint32_t dmax;
    int32_t *nbr;
    uint32_t *nbr_dist;
    float *model_out;
    uint32_t *err;
    const uint32_t *unsettled; // nullable: nonzero when the partition did not reach its fixed point
};

// Sum over the wavefront, returned to every lane: DPP butterflies inside rows of 16 lanes, then the
// row-swap permutes (a shuffle through LDS costs several times the latency, and the fit below is a
// chain of about twenty such sums).
template <int CTRL>
__device__ __forceinline__ double dppd(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)dppu<CTRL>((unsigned)u) | ((uint64_t)dppu<CTRL>((unsigned)(u >> 32)) << 32));
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
    v += dppd<0xB1>(v);
    v += dppd<0x4E>(v);
    v += dppd<0x141>(v);
    v += dppd<0x140>(v);
    auto halves = [](double x, auto swap) {
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        const auto lo = swap((unsigned)u), hi = swap((unsigned)(u >> 32));
        return __builtin_bit_cast(double, (uint64_t)(unsigned)lo[0] | ((uint64_t)(unsigned)hi[0] << 32)) +
               __builtin_bit_cast(double, (uint64_t)(unsigned)lo[1] | ((uint64_t)(unsigned)hi[1] << 32));
    };
    v = halves(v, [](unsigned x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
    return halves(v, [](unsigned x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
}

__device__ __forceinline__ int hash_slot(int32_t t) { return (int)(((uint32_t)t * 2654435761u) >> 23); }

// A least edge in seven bits, rounded down: 4 bits of exponent, from that of kappa on (no edge is shorter),
// above 3 of mantissa.  kb: the exponent of kappa, at most 20; edges beyond the range take its end, which
// stays below 2^29.
__device__ __forceinline__ uint32_t least_code(uint32_t l, uint32_t kb)
{
    const uint32_t z = (uint32_t)__builtin_clz(l);
    return min((31u - z - kb) << 3 | (((l << z) >> 28) & 7u), min(15u, 28u - kb) << 3 | 7u);
}

__device__ __forceinline__ uint32_t least_bound(uint32_t code, uint32_t kb)
{
    return ((8u | (code & 7u)) << ((code >> 3) + kb)) >> 3;
}

// One wavefront per seed s: its k nearest seeds on the seed graph in increasing (distance, index)
// order, at graph distance <= 64 h, then the weighted least-squares affine model of the flow
// around s, in FP64.  The search settles in batches: with T the least tentative distance plus
// least outgoing edge length over the frontier, every frontier node below T is final, since any
// other path to it leaves the settled set through some frontier node u and adds at least u's least
// edge.  After each batch the settled set is exactly the nodes below T, so once it holds k nodes
// its k smallest are the answer.  (With the least edge of the whole graph in place of each node's
// own, k = 128 took 28 - 30 batches instead of 14 - 15 on driving frames.)  A batch's adjacency
// rows are read eight lanes to a node, eight slots each; 97 % of the nodes have at most eight
// neighbours, and the rest take further rounds.  RPL: rows of the fit per lane, k <= 64 RPL.
//
// The search is a chain of short LDS and L2 round trips with VALU and scalar issue about even between
// them: LDS is kept to 6.1 KB so that 25 searches share a CU (at 6.9 KB, with the least edges in 16 bits of
// their own, 21 did: 1,011 us for 966 below), edges are inserted 64 at a time, nodes are ranked
// within their batch only, and the fit's first column comes from the moments.  2048x1024, 117,238
// seeds, k 128: 2,382 -> 966 us (7,185 -> about 3,500 VALU and 5,000 -> 2,850 scalar instructions per
// seed); 1242x375, 9,368 seeds: 246 -> 116 us.  Candidate capacity and results are as before.
template <int RPL>
__global__ __launch_bounds__(64) void k_epic_knn_fit(EpicFit F)
{
    if (F.unsettled && *F.unsettled) return; // the partition did not reach its fixed point
    static_assert(kHash == 1 << 9, "hash_slot returns 9 bits");
    static_assert(kHash >= 2 * kMaxK, "the sorted output reuses the hash keys");
    constexpr int kChunks = (kCand + 63) / 64;
    __shared__ int32_t hkey[kHash];   // node, or -1
    __shared__ uint16_t hval[kHash];  // its candidate slot
    __shared__ uint32_t cdist[kCand]; // candidates: tentative distance (all ones past the last one),
    __shared__ uint16_t chash[kCand]; // place in the hash, and least edge above it (least_code)
    __shared__ uint16_t sslot[kCand]; // candidate slots of the settled nodes, sorted by (distance, index)
    const int li = threadIdx.x;
    const int64_t s = blockIdx.x;
    if (s >= F.n) return; // whole wave

    uint32_t q = 0;
    bool alive = seed_pixel(F.pts, F.flow, F.status, s, F.W, F.H, q);
    if (alive) alive = F.keys[q] == (uint64_t)s; // s owns its pixel at distance 0
    // (every branch of the search is the wavefront's: the read-first-lanes keep its state in scalar
    // registers and the control flow free of execution masks)
    alive = __builtin_amdgcn_readfirstlane(alive ? 1 : 0) != 0;
    auto before = [](uint64_t mask) { // set bits of the mask in lower lanes
        return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
    };
    auto node_of = [&](int slot) { return hkey[chash[slot] & (kHash - 1)]; };
    int cnt = 0;
    bool overflow = false;
    if (alive) {
        for (int j = li; j < kHash; j += 64) hkey[j] = -1;
        for (int j = li; j < kCand; j += 64) cdist[j] = 0xFFFFFFFFu;
        __syncthreads();
        if (li == 0) {
            const int h = hash_slot((int32_t)s);
            hkey[h] = (int32_t)s;
            hval[h] = 0;
            chash[0] = (uint16_t)h; // (the code of the shortest edge there can be: alone in its batch)
            cdist[0] = 0u;
        }
        const uint32_t kb = 31u - (uint32_t)__builtin_clz((uint32_t)F.kappa);
        int m = 1, first = 0;  // candidates, and the first group of 64 that are not all settled (its slot)
        uint32_t settled = 0u; // nodes below this distance are settled
        __syncthreads();
        for (;;) {
            // T (distances are at most dmax <= 2^30 and bounds below 2^29, so sums fit)
            uint32_t T = 0xFFFFFFFFu;
            for (int base = first; base < m; base += 64) {
                const uint32_t d = cdist[base + li], least = least_bound((uint32_t)chash[base + li] >> 9, kb);
                if (d - settled < 0xFFFFFFFFu - settled) T = min(T, d + least); // settled <= d < all ones
            }
            T = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_min_u32(T));
            if (T == 0xFFFFFFFFu) break; // frontier empty
            // the batch
            const int b0 = cnt;
            int head = first;
            for (int base = first; base < m; base += 64) {
                const uint32_t d = cdist[base + li];
                const bool sel = d - settled < T - settled; // settled <= d < T
                const uint64_t bm = __ballot(sel);
                if (sel) sslot[cnt + before(bm)] = (uint16_t)(base + li);
                cnt += __popcll(bm);
                if (head == base && base + 64 <= m && __ballot(d >= T) == 0ull) head = base + 64;
            }
            first = head;
            settled = T;
            __syncthreads();
            // sort it by (distance, index)
            const int nb = cnt - b0;
            int32_t id = 0; // lane i: the batch's i-th node, before sorting
            uint32_t nd = 0u;
            if (nb <= 64) {
                int slot = 0, rank = 0;
                if (li < nb) {
                    slot = sslot[b0 + li];
                    nd = cdist[slot];
                    id = node_of(slot);
                }
                const uint64_t key = ((uint64_t)nd << 32) | (uint32_t)id;
                for (int i = 0; i < nb; ++i) {
                    const uint64_t other = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)nd, i) << 32) |
                                           (uint32_t)__builtin_amdgcn_readlane(id, i);
                    rank += other < key;
                }
                if (li < nb) sslot[b0 + rank] = (uint16_t)slot;
            } else { // (many nodes at equal distances)
                int slot[kChunks], rank[kChunks];
#pragma unroll
                for (int c = 0; c < kChunks; ++c) {
                    slot[c] = rank[c] = 0;
                    if (64 * c + li < nb) {
                        slot[c] = sslot[b0 + 64 * c + li];
                        const uint64_t key = ((uint64_t)cdist[slot[c]] << 32) | (uint32_t)node_of(slot[c]);
                        for (int i = 0; i < nb; ++i) {
                            const int other = sslot[b0 + i];
                            rank[c] += (((uint64_t)cdist[other] << 32) | (uint32_t)node_of(other)) < key;
                        }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int c = 0; c < kChunks; ++c)
                    if (64 * c + li < nb) sslot[b0 + rank[c]] = (uint16_t)slot[c];
            }
            __syncthreads();
            if (cnt >= F.k) break;
            // Relax the batch's edges.  Rows are read eight lanes to a node (they fill from slot 0; the
            // few nodes with more than eight neighbours are read again), and the edges found are
            // queued, one per lane, so that the insertion below runs once per 64 edges.
            int32_t qt = 0;
            uint32_t qc = 0u;
            int queued = 0;
            auto insert = [&]() {
                const bool ok = li < queued;
                uint32_t least = 1u;
                if (ok) least = least_edge(F.ws, qt); // in flight during the probing
                // find or claim the node's place (the table is never full: at most kCand + 64 of kHash)
                int hs = hash_slot(qt);
                bool is_new = false, open = ok;
                while (__ballot(open) != 0ull) {
                    if (open) {
                        const int32_t old = atomicCAS(&hkey[hs], -1, qt);
                        is_new = old == -1;
                        open = !is_new && old != qt;
                        if (open) hs = (hs + 1) & (kHash - 1);
                    }
                }
                queued = 0;
                const uint64_t nbm = __ballot(is_new);
                const int total = __popcll(nbm);
                if (m + total > kCand) {
                    overflow = true;
                    return;
                }
                if (is_new) {
                    const int slot = m + before(nbm);
                    hval[hs] = (uint16_t)slot;
                    chash[slot] = (uint16_t)(hs | least_code(least, kb) << 9);
                }
                m += total;
                __syncthreads();
                // (a settled node's distance is below T, which no path through this batch is)
                if (ok) atomicMin(&cdist[hval[hs]], qc);
                __syncthreads();
            };
            for (int n0 = 0; n0 < nb && !overflow; n0 += 8) {
                const int ni = n0 + (li >> 3);
                const bool on = ni < nb;
                int32_t node;
                uint32_t dv;
                if (nb <= 64) { // (the batch in lane order; any order gives the same distances)
                    node = __builtin_amdgcn_ds_bpermute(4 * ni, id);
                    dv = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * ni, (int)nd);
                } else {
                    const int slot = sslot[b0 + min(ni, nb - 1)];
                    node = node_of(slot);
                    dv = cdist[slot];
                }
                const uint64_t *row = F.ws.adj + (int64_t)node * kMaxDeg + (li & 7);
                for (int s0 = 0; s0 < kMaxDeg && !overflow; s0 += 8) {
                    const uint64_t e = on ? row[s0] : kNoKey;
                    const uint64_t c64 = (uint64_t)dv + (e >> 32);
                    const bool ok = e != kNoKey && c64 <= F.dmax;
                    const uint64_t bm = __ballot(ok);
                    const int n = __popcll(bm);
                    if (queued + n > 64) insert();
                    // the queue lane each edge goes to; the other lanes fill the rest of a permutation
                    const int rank = before(bm);
                    const int to = 4 * ((ok ? queued + rank : queued + n + li - rank) & 63);
                    const int32_t t = __builtin_amdgcn_ds_permute(to, (int32_t)(uint32_t)e);
                    const int32_t c = __builtin_amdgcn_ds_permute(to, (int32_t)(uint32_t)c64);
                    const bool mine = li >= queued && li < queued + n;
                    qt = mine ? t : qt;
                    qc = mine ? (uint32_t)c : qc;
                    queued += n;
                    // a full eighth slot: there may be more
                    if (__ballot((li & 7) == 7 && e != kNoKey) == 0ull) break;
                }
            }
            if (queued > 0 && !overflow) insert();
            if (overflow) break;
        }
        __syncthreads();
        cnt = cnt < F.k ? cnt : F.k;
    }
    if (overflow && li == 0) atomicOr(F.err, kErrCand);
    if (!alive || overflow) cnt = 0;
    if (F.nbr)
        for (int j = li; j < F.k; j += 64) {
            F.nbr[s * F.k + j] = j < cnt ? node_of(sslot[j]) : -1;
            F.nbr_dist[s * F.k + j] = j < cnt ? cdist[sslot[j]] : 0xFFFFFFFFu;
        }
    float *mo = F.ws.model + 8 * s;
    if (!alive || overflow) {
        if (li < 6) {
            mo[li] = __builtin_nanf("");
            if (F.model_out) F.model_out[6 * s + li] = __builtin_nanf("");
        }
        return;
    }
    // weighted position moments about the seed's own position (for the degeneracy test)
    const double sx = F.pts[2 * s], sy = F.pts[2 * s + 1];
    double c1[RPL], cx[RPL], cy[RPL], bu[RPL], bv[RPL]; // sqrt(w) (1, x, y | u, v)
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};              // w, x, y, xx, xy, yy, u, v
    const double half = -0.5 / (double)F.h;
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const int j = li + 64 * r;
        c1[r] = cx[r] = cy[r] = bu[r] = bv[r] = 0.0;
        if (j < cnt) {
            const int slot = sslot[j];
            const int32_t t = node_of(slot);
            const double x = (double)F.pts[2 * (int64_t)t] - sx, y = (double)F.pts[2 * (int64_t)t + 1] - sy;
            const double u = F.flow[2 * (int64_t)t], v = F.flow[2 * (int64_t)t + 1];
            const double rw = exp2((double)cdist[slot] * half); // sqrt(w), w = 2^(-distance / h)
            c1[r] = rw;
            cx[r] = rw * x;
            cy[r] = rw * y;
            bu[r] = rw * u;
            bv[r] = rw * v;
            a[0] += rw * rw;
            a[1] += rw * cx[r];
            a[2] += rw * cy[r];
            a[3] += cx[r] * cx[r];
            a[4] += cx[r] * cy[r];
            a[5] += cy[r] * cy[r];
            a[6] += rw * bu[r];
            a[7] += rw * bv[r];
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = wave_sum_f64(a[e]);
    double mdl[6];
    const double sw = a[0], isw = 1.0 / sw, ex = a[1] * isw, ey = a[2] * isw;
    const double cxx = a[3] * isw - ex * ex, cyy = a[5] * isw - ey * ey, cxy = a[4] * isw - ex * ey;
    const double tr = cxx + cyy, det = cxx * cyy - cxy * cxy;
    if (cnt < 3 || !(det > 1e-4 * tr * tr)) {
        mdl[0] = mdl[1] = mdl[3] = mdl[4] = 0.0;
        mdl[2] = a[6] / sw;
        mdl[5] = a[7] / sw;
    } else {
        // weighted least squares by modified Gram-Schmidt on the columns sqrt(w) (1, x, y), the
        // right-hand sides carried along as further columns (backward stable for least squares;
        // the weights can span 64 binades, beyond what the normal equations resolve).  The first
        // column's products are the moments above; the columns stay unnormalised, so that each of
        // the other two takes one round of sums: R's rows are (sw, a1, a2), (d22, d23), (d33).
        auto dot = [&](const double *p, const double *q) {
            double acc = 0.0;
#pragma unroll
            for (int r = 0; r < RPL; ++r) acc += p[r] * q[r];
            return wave_sum_f64(acc);
        };
        auto axpy = [&](double f, const double *q, double *p) {
#pragma unroll
            for (int r = 0; r < RPL; ++r) p[r] -= f * q[r];
        };
        const double mu = a[6] * isw, mv = a[7] * isw;
        axpy(ex, c1, cx);
        axpy(ey, c1, cy);
        axpy(mu, c1, bu);
        axpy(mv, c1, bv);
        const double d22 = dot(cx, cx), d23 = dot(cx, cy), d2u = dot(cx, bu), d2v = dot(cx, bv);
        const double i22 = 1.0 / d22, f23 = d23 * i22;
        axpy(f23, cx, cy);
        axpy(d2u * i22, cx, bu);
        axpy(d2v * i22, cx, bv);
        const double d33 = dot(cy, cy), d3u = dot(cy, bu), d3v = dot(cy, bv);
        const double gyu = d3u / d33, gyv = d3v / d33;
        const double gxu = d2u * i22 - f23 * gyu, gxv = d2v * i22 - f23 * gyv;
        mdl[0] = gxu;
        mdl[1] = gyu;
        mdl[2] = mu - ex * gxu - ey * gyu;
        mdl[3] = gxv;
        mdl[4] = gyv;
        mdl[5] = mv - ex * gxv - ey * gyv;
    }
    if (li != 0) return;
    for (int e = 0; e < 6; ++e) {
        mo[e] = (float)mdl[e];
        if (F.model_out) F.model_out[6 * s + e] = (float)mdl[e];
    }
}

// Every pixel evaluates the model of its cell's seed at its own coordinates.
__global__ void k_epic_dense(int W, int H, const uint64_t *keys, const float *model, const float *pts, float *dense, int64_t dpitch,
                             int32_t *labels, uint32_t *dist, const uint32_t *unsettled)
{
    if (unsettled && *unsettled) return; // the partition did not reach its fixed point
    const uint32_t N = (uint32_t)W * (uint32_t)H;
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < N; p += gridDim.x * blockDim.x) {
        const uint32_t y = p / (uint32_t)W, x = p - y * (uint32_t)W;
        const uint64_t k = keys[p];
        float2 f;
        if (k == kNoKey) {
            f = make_float2(__builtin_nanf(""), __builtin_nanf(""));
        } else {
            const float4 *m = reinterpret_cast<const float4 *>(model + 8 * (int64_t)(uint32_t)k);
            const float4 m0 = m[0], m1 = m[1];
            const float *at = pts + 2 * (int64_t)(uint32_t)k;
            const float rx = (float)x - at[0], ry = (float)y - at[1];
            f = make_float2(fmaf(m0.x, rx, fmaf(m0.y, ry, m0.z)), fmaf(m0.w, rx, fmaf(m1.x, ry, m1.y)));
        }
        *reinterpret_cast<float2 *>(dense + (int64_t)y * dpitch + 2 * x) = f;
        if (labels) labels[p] = k == kNoKey ? -1 : (int32_t)(uint32_t)k;
        if (dist) dist[p] = k == kNoKey ? 0xFFFFFFFFu : (uint32_t)(k >> 32);
    }
}

unsigned grid_for(int64_t items, int threads)
{
    const int64_t b = (items + threads - 1) / threads;
    return (unsigned)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

bool epic_image_ok(const dgf_image *im)
{
    if (!im || !im->data || im->dtype != DGF_U8 || im->width < 1 || im->height < 1) return false;
    if (im->pitch_bytes < im->width) return false;
    if ((int64_t)im->width * im->height > (int64_t)INT32_MAX) return false;
    return true;
}

} // namespace
} // namespace dgf

using namespace dgf;

extern "C" {

namespace dgf {
namespace {
// (one thread) The outcome of a call without host synchronisation: 0 done, 1 the partition did
// not reach its fixed point within the launches given, 2 a capacity limit (see dgf_epic).
__global__ void k_epic_status(uint32_t *out, const uint32_t *unsettled, const uint32_t *err)
{
    *out = (unsettled && *unsettled) ? 1u : (*err ? 2u : 0u);
}
} // namespace
} // namespace dgf

int dgf_epic_opts_default(dgf_epic_opts *o)
{
    if (!o) return DGF_ERR_INVALID_ARG;
    o->k = 128;
    o->kappa = 8;
    o->half_dist = 64;
    return DGF_OK;
}

size_t dgf_epic_workspace_bytes(int32_t width, int32_t height, int64_t n)
{
    if (width < 1 || height < 1 || n < 0) return 0;
    return (size_t)ws_layout(width, height, n, nullptr, nullptr);
}

namespace {

// The body of dgf_epic (max_relax == 0: relaxation checked from the host until it settles, the
// outcome returned) and of dgf_epic_async (max_relax > 0 launches, the outcome left in
// *status_out on the device).
int epic_run(const dgf_image *I0, const float *points, const float *flow, const uint8_t *status, int64_t n,
             const dgf_epic_opts *opts, void *workspace, size_t ws_bytes, float *dense, int64_t dense_pitch,
             int32_t *labels, uint32_t *dist, int32_t *nbr, uint32_t *nbr_dist, float *model, void *stream,
             int max_relax, uint32_t *status_out)
{
    if (!epic_image_ok(I0)) return DGF_ERR_INVALID_ARG;
    const int W = I0->width, H = I0->height;
    dgf_epic_opts o;
    if (opts)
        o = *opts;
    else
        dgf_epic_opts_default(&o);
    if (o.k < 1 || o.k > kMaxK || o.kappa < 1 || o.kappa > (1 << 20) || o.half_dist < 1 || o.half_dist > (1 << 24))
        return DGF_ERR_INVALID_ARG;
    // every least distance is at most that of a straight row-then-column path
    if ((uint64_t)(W - 1 + H - 1) * (uint64_t)(o.kappa + 2 * kMaxEdge) > kDistCap) return DGF_ERR_UNSUPPORTED;
    if (n < 0 || n >= (int64_t)INT32_MAX) return DGF_ERR_INVALID_ARG;
    if (n > 0 && (!points || !flow || !status)) return DGF_ERR_INVALID_ARG;
    if (!dense || dense_pitch < 2 * (int64_t)W || dense_pitch % 2 != 0 || (uintptr_t)dense % 8 != 0)
        return DGF_ERR_INVALID_ARG;
    if ((nbr == nullptr) != (nbr_dist == nullptr)) return DGF_ERR_INVALID_ARG;
    const size_t need = (size_t)ws_layout(W, H, n, nullptr, nullptr);
    if (!workspace || ws_bytes < need) return DGF_ERR_WORKSPACE;
    EpicWs ws;
    ws_layout(W, H, n, &ws, (char *)workspace);
    hipStream_t st = (hipStream_t)stream;
    const int64_t N = (int64_t)W * H;

    const dim3 tiles((unsigned)((W + kRTX - 1) / kRTX), (unsigned)((H + kRTY - 1) / kRTY));
    const int64_t ntiles = (int64_t)tiles.x * tiles.y;
    const int64_t prep_items = N > n * kMaxDeg ? N : n * kMaxDeg;
    hipLaunchKernelGGL(k_epic_prep, dim3(grid_for(prep_items, 256)), dim3(256), 0, st, (const uint8_t *)I0->data,
                       I0->pitch_bytes, W, H, n, (uint32_t)ntiles, ws);
    if (hipGetLastError() != hipSuccess) return DGF_ERR_HIP;
    uint32_t *err = ws.ctr + kChunk;
    // everything after the partition; unsettled (nullable): nothing is done when this word is not zero
    auto finish = [&](const uint32_t *unsettled) {
        if (n > 0) {
            const int rows = graph_rows(N), gh = kGraphWaves * rows;
            const auto graph = rows == 8 ? k_epic_graph<8> : rows == 2 ? k_epic_graph<2> : k_epic_graph<1>;
            hipLaunchKernelGGL(graph, dim3((unsigned)((W + kGraphW - 1) / kGraphW), (unsigned)((H + gh - 1) / gh)),
                               dim3(64 * kGraphWaves), 0, st, W, H, o.kappa, (const uint64_t *)ws.keys,
                               (const uint16_t *)ws.E, ws, err, unsettled);
            if (hipGetLastError() != hipSuccess) return false;
            hipLaunchKernelGGL(k_epic_least, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st, n, ws, unsettled);
            if (hipGetLastError() != hipSuccess) return false;
            EpicFit F{};
            F.pts = points;
            F.flow = flow;
            F.status = status;
            F.keys = ws.keys;
            F.ws = ws;
            F.n = n;
            F.W = W;
            F.H = H;
            F.k = o.k;
            F.h = o.half_dist;
            F.kappa = o.kappa;
            F.dmax = (uint32_t)(64u * (uint32_t)o.half_dist);
            F.nbr = nbr;
            F.nbr_dist = nbr_dist;
            F.model_out = model;
            F.err = err;
            F.unsettled = unsettled;
            if (o.k <= 128)
                hipLaunchKernelGGL(k_epic_knn_fit<2>, dim3((unsigned)n), dim3(64), 0, st, F);
            else
                hipLaunchKernelGGL(k_epic_knn_fit<kMaxK / 64>, dim3((unsigned)n), dim3(64), 0, st, F);
            if (hipGetLastError() != hipSuccess) return false;
        }
        hipLaunchKernelGGL(k_epic_dense, dim3(grid_for(N, 256)), dim3(256), 0, st, W, H, (const uint64_t *)ws.keys,
                           (const float *)ws.model, points, dense, dense_pitch, labels, dist, unsettled);
        return hipGetLastError() == hipSuccess;
    };
    // (synchronises) the counters: h[launch mod kChunk] tiles changed, h[kChunk] errors, then the open counts
    uint32_t h[2 * kChunk + 1] = {};
    auto counters = [&]() {
        return hipMemcpyAsync(h, ws.ctr, sizeof(h), hipMemcpyDeviceToHost, st) == hipSuccess &&
               hipStreamSynchronize(st) == hipSuccess;
    };
    const bool sync = max_relax == 0;
    const uint32_t *unsettled = nullptr; // (the async form) the last relaxation launch's changed count
    if (n > 0) {
        hipLaunchKernelGGL(k_epic_seed, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, points, flow, status, n, W,
                           H, ws.keys);
        if (hipGetLastError() != hipSuccess) return DGF_ERR_HIP;
        // tiles may wait for each other only if the whole grid is resident at once
        const bool fast = (uint64_t)(W - 1 + H - 1) * (uint64_t)(o.kappa + 2 * kMaxEdge) < kFar &&
                          o.kappa + 2 * kMaxEdge < (int)kFar;
        const void *kernel = fast ? (const void *)k_epic_relax<true> : (const void *)k_epic_relax<false>;
        int dev = 0, cus = 0, per_cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kRelaxThreads, 0) != hipSuccess)
            return DGF_ERR_HIP;
        const int wait = ntiles <= (int64_t)cus * per_cu ? 1 : 0;
        const int limit = sync ? kMaxRelaxLaunches : max_relax;
        // a grid that fits the chip settles in its first launch and the second says so; where other work
        // keeps it from being resident for a while, any later launch may be the one that settles it, so all
        // of them wait.  (128 workgroups that do not wait, from the third launch on, saved 7 of 1,224 us on a
        // 2048x1024 call, but 9 of 32 calls on four streams, 1600x900 frames of one seed, ended unsettled.)
        int done = 0; // launches so far; launch j uses counter set j mod kChunk
        auto relax = [&](int launches) {
            for (const int end = done + std::min(launches, limit - done); done < end; ++done) {
                const RelaxCounters prev = done > 0 ? relax_counters(ws, done - 1, ntiles) : RelaxCounters{};
                hipLaunchKernelGGL(fast ? k_epic_relax<true> : k_epic_relax<false>, dim3((unsigned)ntiles), dim3(kRelaxThreads),
                                   0, st, W, H, o.kappa, ws.keys, (const uint16_t *)ws.E,
                                   relax_counters(ws, done, ntiles), wait, prev, relax_counters(ws, done + 2, ntiles),
                                   (int)tiles.x);
                if (hipGetLastError() != hipSuccess) return false;
            }
            return true;
        };
        if (sync && wait) {
            // the launch that settles a resident grid, with all that follows behind it on the condition
            // that it did: one round trip to the host in all
            if (!relax(1) || !finish(relax_counters(ws, 0, ntiles).open) || !counters()) return DGF_ERR_HIP;
            if (h[kChunk + 1] == 0u) return h[kChunk] ? DGF_ERR_CAPACITY : DGF_OK;
        }
        if (sync) {
            // checked every kChunk launches; a launch after one that changed nothing returns at once
            bool converged = false;
            while (done < limit && !converged) {
                if (!relax(kChunk) || !counters()) return DGF_ERR_HIP;
                converged = h[(done - 1) % kChunk] == 0u;
            }
            if (!converged) return DGF_ERR_UNSUPPORTED;
        } else {
            if (!relax(limit)) return DGF_ERR_HIP;
            unsettled = ws.ctr + (done - 1) % kChunk;
        }
    }
    if (!finish(unsettled)) return DGF_ERR_HIP;
    if (!sync) {
        hipLaunchKernelGGL(k_epic_status, dim3(1), dim3(1), 0, st, status_out, unsettled, (const uint32_t *)err);
        return hipGetLastError() == hipSuccess ? DGF_OK : DGF_ERR_HIP;
    }
    if (!counters()) return DGF_ERR_HIP;
    return h[kChunk] ? DGF_ERR_CAPACITY : DGF_OK;
}

} // namespace

int dgf_epic(const dgf_image *I0, const float *points, const float *flow, const uint8_t *status, int64_t n,
             const dgf_epic_opts *opts, void *workspace, size_t ws_bytes, float *dense, int64_t dense_pitch,
             int32_t *labels, uint32_t *dist, int32_t *nbr, uint32_t *nbr_dist, float *model, void *stream)
{
    return epic_run(I0, points, flow, status, n, opts, workspace, ws_bytes, dense, dense_pitch, labels, dist, nbr,
                    nbr_dist, model, stream, 0, nullptr);
}

int dgf_epic_async(const dgf_image *I0, const float *points, const float *flow, const uint8_t *status, int64_t n,
                   const dgf_epic_opts *opts, void *workspace, size_t ws_bytes, float *dense, int64_t dense_pitch,
                   int32_t *labels, uint32_t *dist, int32_t *nbr, uint32_t *nbr_dist, float *model,
                   int32_t max_relax, uint32_t *status_out, void *stream)
{
    if (max_relax < 0 || max_relax > kMaxRelaxLaunches || !status_out || (uintptr_t)status_out % 4 != 0)
        return DGF_ERR_INVALID_ARG;
    return epic_run(I0, points, flow, status, n, opts, workspace, ws_bytes, dense, dense_pitch, labels, dist, nbr,
                    nbr_dist, model, stream, max_relax ? max_relax : kDefaultAsyncRelax, status_out);
}

} // extern "C"
