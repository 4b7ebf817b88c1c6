// adjoint_tiled.hip -- the adjoint of a batch plan's points at a support fixed at compile time:
// tiles of neighbouring points, whose gradient cells are combined in LDS.
#include <algorithm>

#include "adjoint_point.hpp"

namespace dgf {

// The points of a batch plan in tiles of tx x ty grid neighbours, one workgroup of kAdjWaves
// wavefronts each.  Neighbouring points' patches overlap (64 points at stride 2 and support 21
// touch 36,864 dI0 cells, 2,116 of them distinct), so their cells are added up in two LDS tiles
// and go to the gradient maps once per workgroup.  The dI0 tile starts at the least patch origin
// of the workgroup's converged points; the dI1 tile is centred on the median patch origin (the
// points' flows differ); a patch that leaves its tile goes to device memory directly.  With one
// wavefront and about 1,060 device atomics per point the atomics bound the launch (four 2048x1024
// pairs, stride 2, support 21, 701,685 converged points: 4.97 ms against 1.55 here, of which 1.17 ms
// is VALU issue, 1,020 instructions per point); 16 x 8 points per workgroup leave about 110.
// Eight wavefronts and at most 78 KB keep two workgroups on a CU, so one's ends overlap the other.
// Where few of a tile's points converged, clearing and emptying its LDS tiles costs more than their
// atomics: up to kAdjFew go to the maps directly (four 1242x375 pairs, stride 5, support 21, 73,112
// points of which 2 % converged: 36 us, 48 through the tiles, 36 with a wavefront per point; 20 %:
// 85, 87 and 130).  A wavefront takes up to eight points one after the other, so a small block of
// converged points in a plan of others is the one pattern that a wavefront per point does faster (two
// 520x400 pairs, stride 2, support 9, one ninth of the points in a corner: 36 us against 45).
constexpr int kAdjWaves = 8;
constexpr int kAdjPoints = 128; // most points of a tile
constexpr int kAdjFew = 6;      // so few converged points of a tile go to device memory directly

template <typename PixT, int S, bool IM>
__global__ __launch_bounds__(64 * kAdjWaves, 4) void k_track_adjoint_tiled(AdjParams A)
{
    constexpr int W0 = S + 3, W1 = S + 1, r = S / 2;
    extern __shared__ __align__(16) float smem[];
    __shared__ int list[kAdjPoints], lx1[kAdjPoints], ly1[kAdjPoints];
    __shared__ int count, minx, miny, medx, medy, lock[2];
    const int t = threadIdx.x, li = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    int lo = 0, hi = A.npairs - 1; // last pair whose first tile is <= this one
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (A.pairs[mid].tile_first <= (int64_t)blockIdx.x)
            lo = mid;
        else
            hi = mid - 1;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const AdjPair Pr = A.pairs[lo];
    const int64_t p0 = A.pt_off[lo];
    const int np = (int)(A.pt_off[lo + 1] - p0);
    const int tile = (int)((int64_t)blockIdx.x - Pr.tile_first);
    const int tiles_x = (Pr.nx + Pr.tx - 1) / Pr.tx;
    // every row of tiles starts at a column of its own: the dispatcher deals workgroups out in a fixed turn
    // (8 dies, 4 engines each), and with 32 tiles a row those of a frame's left half would all go to the
    // same engines (two 520x400 pairs, stride 2, support 9, illumination model, left half converged: 196 us,
    // 148 now)
    const int by = tile / tiles_x, turn = (int)(((uint32_t)by * 2654435761u >> 8) % (uint32_t)tiles_x);
    const int at = tile - by * tiles_x + turn, bx = at < tiles_x ? at : at - tiles_x;
    if (t == 0) {
        count = lock[0] = lock[1] = 0;
        minx = 0x7fffffff;
        miny = 0x7fffffff;
    }
    __syncthreads();
    // the tile's converged points and their patch origins
    if (t < Pr.tx * Pr.ty) {
        const int ky = by * Pr.ty + t / Pr.tx, kx = bx * Pr.tx + t % Pr.tx;
        const int64_t k = (int64_t)ky * Pr.nx + kx;
        if (kx < Pr.nx && k < np && A.status[p0 + k] == DGF_ST_CONVERGED) {
            const AdjPlace pl = adj_place(reinterpret_cast<const float2 *>(A.pts)[p0 + k],
                                          reinterpret_cast<const float2 *>(A.flow)[p0 + k], r);
            const int e = atomicAdd(&count, 1);
            list[e] = (int)k;
            lx1[e] = pl.ox1;
            ly1[e] = pl.oy1;
            atomicMin(&minx, pl.ox0);
            atomicMin(&miny, pl.oy0);
        }
    }
    __syncthreads();
    const int n = count;
    if (n == 0) return;
    const bool tiled = n > kAdjFew;
    float *tile0 = smem + kAdjWaves * AdjSplit<S>::floats, *tile1 = tile0 + Pr.w0 * Pr.h0;
    if (tiled)
        for (int c = t; c < Pr.w0 * Pr.h0 + Pr.w1 * Pr.h1; c += 64 * kAdjWaves) tile0[c] = 0.f;
    if (t < n) { // median by rank
        const int x = lx1[t], y = ly1[t];
        int bxr = 0, byr = 0;
        for (int e = 0; e < n; ++e) {
            bxr += lx1[e] < x || (lx1[e] == x && e < t);
            byr += ly1[e] < y || (ly1[e] == y && e < t);
        }
        if (bxr == n / 2) medx = x;
        if (byr == n / 2) medy = y;
    }
    __syncthreads();
    AdjSink K;
    K.tile0 = tile0;
    K.tile1 = tile1;
    K.pair = A.pairs + lo;
    K.lock0 = lock;
    K.lock1 = lock + 1;
    K.tp0 = Pr.w0;
    K.tp1 = Pr.w1;
    K.tx0 = minx;
    K.ty0 = miny;
    K.tx1 = medx - (Pr.w1 - W1) / 2;
    K.ty1 = medy - (Pr.h1 - W1) / 2;
    float *own = smem + wave * AdjSplit<S>::floats;
    for (int e = wave; e < n; e += kAdjWaves) {
        const int64_t i = p0 + __builtin_amdgcn_readfirstlane(list[e]);
        const AdjPlace pl = adj_place(reinterpret_cast<const float2 *>(A.pts)[i],
                                      reinterpret_cast<const float2 *>(A.flow)[i], r);
        // (differences in 32-bit unsigned: an origin may lie anywhere)
        auto fits = [](int o, int t0, int w, int n0) {
            return n0 >= w && o >= t0 && (uint32_t)o - (uint32_t)t0 <= (uint32_t)(n0 - w);
        };
        K.fit0 = tiled && fits(pl.ox0, K.tx0, W0, Pr.w0) && fits(pl.oy0, K.ty0, W0, Pr.h0);
        K.fit1 = tiled && fits(pl.ox1, K.tx1, W1, Pr.w1) && fits(pl.oy1, K.ty1, W1, Pr.h1);
        adjoint_point<PixT, S, IM, false>(A, Pr, i, pl, own, li, K);
    }
    if (!tiled) return; // (the same for every wavefront)
    __syncthreads();
    // the tiles' cells at their clamped image positions, one row per wavefront and step
    const AdjPair M = *map_of(K.pair);
    auto flush = [&](const float *tl, int w, int h, int ox, int oy, float *map, int64_t pitch) {
        for (int y = wave; y < h; y += kAdjWaves) {
            float *row = map + (int64_t)clampi(oy + y, 0, M.H - 1) * pitch;
            for (int x = li; x < w; x += 64) {
                const float v = tl[y * w + x];
                if (v != 0.f) unsafeAtomicAdd(row + clampi(ox + x, 0, M.W - 1), v);
            }
        }
    };
    flush(tile0, M.w0, M.h0, K.tx0, K.ty0, A.grad0 + M.g0, M.gpitch0);
    flush(tile1, M.w1, M.h1, K.tx1, K.ty1, A.grad1 + M.g1, M.gpitch1);
}


namespace {

size_t wave_bytes(int s)
{
#define DGF_CASE(S_) if (s == S_) return sizeof(float) * AdjSplit<S_>::floats;
    DGF_ADJOINT_SUPPORTS(DGF_CASE)
#undef DGF_CASE
    return 0;
}

template <int S>
hipError_t launch_tiled(const AdjParams &A, unsigned tiles, size_t lds, hipStream_t st)
{
    const dim3 grid(tiles), block(64 * kAdjWaves);
    if (A.illum)
        hipLaunchKernelGGL((k_track_adjoint_tiled<uint8_t, S, true>), grid, block, lds, st, A);
    else
        hipLaunchKernelGGL((k_track_adjoint_tiled<uint8_t, S, false>), grid, block, lds, st, A);
    return hipGetLastError();
}

} // namespace

// Tile shape for a pair of nx x ny grid points of a plan of n points: the largest of a few shapes whose
// two LDS tiles let two workgroups share a CU and that leaves the chip at least kMinTiles workgroups
// (a wavefront takes its points one after the other, so a small plan needs more workgroups more than
// it needs fewer atomics; twice as many for the largest shape, whose wavefronts take sixteen: one 800x700
// pair, stride 2, support 15, illumination model, 137,016 points, 325 us for 347, and where one ninth of
// them converged in a corner 85 for 152).  The dI0 tile holds the patches of a full tile of windows wherever the
// centroids fall in them; the dI1 tile leaves room for a quarter more spread and 8 px of it.
void adjoint_tile_shape(AdjPair &P, int nx, int ny, int s, int win, int stride, int64_t n)
{
    constexpr int64_t kMinTiles = 1024;
    const size_t budget = 78 * 1024 - kAdjWaves * wave_bytes(s);
    const int W0 = s + 3, W1 = s + 1;
    static const int shapes[][2] = {{16, 8}, {8, 8}, {8, 4}, {4, 4}};
    for (const auto &sh : shapes) {
        if (n < (sh[0] == 16 ? 2 : 1) * kMinTiles * sh[0] * sh[1]) continue;
        const int64_t ex = (int64_t)(sh[0] - 1) * stride, ey = (int64_t)(sh[1] - 1) * stride;
        const int64_t w0 = W0 + ex + win - 1, h0 = W0 + ey + win - 1;
        const int64_t w1 = W1 + ex + ex / 4 + win + 7, h1 = W1 + ey + ey / 4 + win + 7;
        if ((size_t)(w0 * h0 + w1 * h1) * sizeof(float) > budget) continue;
        // worth it where the tiles hold at most a quarter of the cells their points would touch
        if (4 * (w0 * h0 + w1 * h1) > (int64_t)sh[0] * sh[1] * (W0 * W0 + W1 * W1)) break;
        P.nx = nx;
        P.ny = ny;
        P.tx = sh[0];
        P.ty = sh[1];
        P.w0 = (int)w0;
        P.h0 = (int)h0;
        P.w1 = (int)w1;
        P.h1 = (int)h1;
        return;
    }
    P.nx = nx * ny; // a point per wavefront, no tiles (in a plan that has tiles elsewhere)
    P.ny = 1;
    P.tx = kAdjWaves;
    P.ty = 1;
    P.w0 = P.h0 = P.w1 = P.h1 = 0;
}

size_t adjoint_tile_floats(const AdjPair &P) { return (size_t)P.w0 * P.h0 + (size_t)P.w1 * P.h1; }

int64_t adjoint_tiles(const AdjPair &P)
{
    return (int64_t)((P.nx + P.tx - 1) / P.tx) * ((P.ny + P.ty - 1) / P.ty);
}

hipError_t launch_adjoint_tiled(const AdjParams &A, int64_t tiles, size_t tile_floats, hipStream_t st)
{
    if (tiles <= 0) return hipSuccess;
    const size_t lds = kAdjWaves * wave_bytes(A.s) + sizeof(float) * tile_floats;
#define DGF_CASE(S_) if (A.s == S_) return launch_tiled<S_>(A, (unsigned)tiles, lds, st);
    DGF_ADJOINT_SUPPORTS(DGF_CASE)
#undef DGF_CASE
    return hipErrorInvalidValue;
}

} // namespace dgf
