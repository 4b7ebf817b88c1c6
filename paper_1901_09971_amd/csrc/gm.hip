// gm.hip -- the global-motion prior's robust affine fit (the "GM" of RLOF(IM-GM), Section 3
// "Parameters"): one affine motion v = A (x - cx, y - cy, 1)^T per frame pair, fitted in FP64 to
// the motions of the points that the coarsest-level pass reports converged, by weighted least
// squares and then ten Tukey-biweight reweightings.
//
// Pairs of up to 4096 points are fitted by one workgroup in one launch (k_gm_one).  The larger ones
// take one launch per weighting pass, each a grid of (nblk, npairs) workgroups.  Every workgroup first rebuilds the previous pass's model from the previous pass's partial sums (all workgroups of a pair
// reduce the same partials in the same order, so they agree bit for bit), then sums its slice of the
// pair's samples under the weights that model gives.  A last launch of one workgroup per pair turns
// the final partial sums into the model.
//
// A launch is bound by its own latency -- launch, fetch, sum, solve, sum -- not by bytes or FP64
// rate, so each part of that chain is kept short: a lane's samples are fetched before the model
// they are weighted with is rebuilt and a slice is two of them per lane; the sums halve the number
// of values a lane carries; every lane solves for the model (no broadcast, no second barrier) and
// pivots by selection.  12065 points: 119 us for the twelve launches with slices of 2048 points read one
// by one, full butterflies and one lane solving through indexed rows, 82 with the shorter chain,
// 68 with slices of 512, 63 with the narrow steps of the sums off the LDS pipe.
//
// Models and partials are double-buffered by pass parity, so
// a launch only reads what the launch before it wrote: no atomics and no counters to clear, and the
// sequence can be captured into a graph.
#include <cmath>

#include "dgf_internal.hpp"

namespace dgf {

namespace {

// Weighted sums of one pass: S, Sx, Sy, Sxx, Sxy, Syy, Su, Sxu, Syu, Sv, Sxv, Syv and the number
// of samples of positive weight (x, y about the centre; u, v the sample motion).
enum { kS, kSx, kSy, kSxx, kSxy, kSyy, kSu, kSxu, kSyu, kSv, kSxv, kSyv, kNz };
static_assert(kNz + 1 == kGmSums, "sum layout");

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
static_assert(kGmMaxBlocks <= kThreads, "one partial per lane");
constexpr int64_t kGmOne = 4096; // points of a pair that one workgroup fits in one launch
constexpr int kHold = 4; // samples a lane fetches at a time (slices above 131072 points in all are longer than two)

// v + the value of v in the lane that the DPP control pairs this one with.
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v)
{
    const uint2 u = __builtin_bit_cast(uint2, v);
    const uint2 o = {(unsigned)__builtin_amdgcn_mov_dpp((int)u.x, CTRL, 0xF, 0xF, true),
                     (unsigned)__builtin_amdgcn_mov_dpp((int)u.y, CTRL, 0xF, 0xF, true)};
    return v + __builtin_bit_cast(double, o);
}

// One halving step of the wavefront's sum over the lanes M apart: on return the lanes of the lower
// half hold a's sum and those of the upper half b's (a pair of swaps in place of two exchanges).
template <int M>
__device__ __forceinline__ double add_split(double a, double b)
{
    const uint2 ua = __builtin_bit_cast(uint2, a), ub = __builtin_bit_cast(uint2, b);
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    u32x2 lo, hi;
    if constexpr (M == 32) {
        lo = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
        hi = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap(ua.x, ub.x, false, false);
        hi = __builtin_amdgcn_permlane16_swap(ua.y, ub.y, false, false);
    }
    return __builtin_bit_cast(double, uint2{lo[0], hi[0]}) + __builtin_bit_cast(double, uint2{lo[1], hi[1]});
}

// Sums of v[k] over the wavefront, to one row of 16: the butterfly's two widest steps halve the number of
// values a lane carries instead of exchanging all of them, which leaves 4 of the 16 (13 and three
// zeros) for the four narrow steps, inside rows of lanes: 16 exchanges of a double against 78, none through LDS.
__device__ __forceinline__ void wave_sums(const double (&v)[kGmSums], double (&row)[16])
{
    double h[8], q[4];
#pragma unroll
    for (int k = 0; k < 8; ++k) h[k] = add_split<32>(v[k], k + 8 < kGmSums ? v[k + 8 < kGmSums ? k + 8 : 0] : 0.0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        q[k] = add_split<16>(h[k], h[k + 4]);
        q[k] = add_dpp<0xB1>(q[k]);  // lane ^ 1
        q[k] = add_dpp<0x4E>(q[k]);  // lane ^ 2
        q[k] = add_dpp<0x141>(q[k]); // the other four of eight
        q[k] = add_dpp<0x140>(q[k]); // the other eight of sixteen
    }
    const int lane = threadIdx.x & 63;
    if ((lane & 15) == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) row[(lane >> 5) * 8 + ((lane >> 4) & 1) * 4 + k] = q[k];
}

// Sum of v[k] over the workgroup in a fixed order (lane butterflies, then the four wavefronts in
// turn); after the call every lane's out[k] holds it.
__device__ void block_sum(const double (&v)[kGmSums], double (*red)[16], double (&out)[kGmSums])
{
    wave_sums(v, red[threadIdx.x >> 6]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kGmSums; ++k) {
        double x = red[0][k];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) x += red[w][k];
        out[k] = x;
    }
}

// Model from one pass's sums.  `A` holds the previous model on entry and keeps it when no sample
// carries weight or the normal matrix is singular; with fewer than three samples, or positions
// whose weighted covariance C has det C <= 1e-4 (tr C)^2 (collinear), the model is the weighted
// mean motion.  Otherwise the 3 x 3 normal equations of both motion components are solved by
// Gaussian elimination with partial pivoting.
__device__ __forceinline__ void gm_solve(const double (&S)[kGmSums], double (&A)[6])
{
    if (!(S[kNz] > 0.0)) return;
    const double is = 1.0 / S[kS];
    const double mx = S[kSx] * is, my = S[kSy] * is;
    const double cxx = S[kSxx] * is - mx * mx, cxy = S[kSxy] * is - mx * my, cyy = S[kSyy] * is - my * my;
    const double tr = cxx + cyy, det = cxx * cyy - cxy * cxy;
    if (S[kNz] < 3.0 || !(det > 1e-4 * tr * tr)) {
        A[0] = A[1] = A[3] = A[4] = 0.0;
        A[2] = S[kSu] / S[kS];
        A[5] = S[kSv] / S[kS];
        return;
    }
    // unknowns (slope in x, slope in y, offset), one right-hand side per motion component
    double N[3][5] = {{S[kSxx], S[kSxy], S[kSx], S[kSxu], S[kSxv]},
                      {S[kSxy], S[kSyy], S[kSy], S[kSyu], S[kSyv]},
                      {S[kSx], S[kSy], S[kS], S[kSu], S[kSv]}};
    // (rows are exchanged by selection: an index known only at run time would put N in memory)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        int piv = c;
        double best = fabs(N[c][c]);
#pragma unroll
        for (int r = c + 1; r < 3; ++r) {
            const double a = fabs(N[r][c]);
            if (a > best) {
                best = a;
                piv = r;
            }
        }
        if (!(best > 0.0)) return;
#pragma unroll
        for (int r = c + 1; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const double t = N[c][k], u = N[r][k];
                N[c][k] = piv == r ? u : t;
                N[r][k] = piv == r ? t : u;
            }
#pragma unroll
        for (int r = c + 1; r < 3; ++r) {
            const double f = N[r][c] / N[c][c];
#pragma unroll
            for (int k = c; k < 5; ++k) N[r][k] -= f * N[c][k];
        }
    }
    double x[2][3];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 2; r >= 0; --r) {
            double acc = N[r][3 + j];
#pragma unroll
            for (int k = r + 1; k < 3; ++k) acc -= N[r][k] * x[j][k];
            x[j][r] = acc / N[r][r];
        }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        A[k] = x[0][k];
        A[3 + k] = x[1][k];
    }
}

// A sample's part in the sums of pass `pass` under the model A (pass 0: weight 1).
__device__ __forceinline__ void add_sample(float2 p, float2 m, double cx, double cy, double c2, int pass,
                                           const double (&A)[6], double (&v)[kGmSums])
{
    if (!isfinite(m.x) || !isfinite(m.y)) return;
    const double x = (double)p.x - cx, y = (double)p.y - cy, mu = m.x, mv = m.y;
    double w = 1.0;
    if (pass > 0) {
        const double ex = mu - (A[0] * x + A[1] * y + A[2]);
        const double ey = mv - (A[3] * x + A[4] * y + A[5]);
        const double e2 = ex * ex + ey * ey;
        const double q = 1.0 - e2 / c2;
        w = e2 < c2 ? q * q : 0.0;
    }
    if (!(w > 0.0)) return;
    const double wx = w * x, wy = w * y;
    v[kS] += w;
    v[kSx] += wx;
    v[kSy] += wy;
    v[kSxx] += wx * x;
    v[kSxy] += wx * y;
    v[kSyy] += wy * y;
    v[kSu] += w * mu;
    v[kSxu] += wx * mu;
    v[kSyu] += wy * mu;
    v[kSv] += w * mv;
    v[kSxv] += wx * mv;
    v[kSyv] += wy * mv;
    v[kNz] += 1.0;
}

// The points of a pair and its frame size.
struct GmPair {
    int64_t p0, p1;
    int W, H;
};

__device__ __forceinline__ GmPair gm_pair(const GmFit &g, int pair)
{
    if (!g.pt_off) return {0, g.n, g.W, g.H};
    const LevelPair &l = g.blv[(size_t)pair * g.L];
    return {g.pt_off[pair], g.pt_off[pair + 1], l.W, l.H};
}

// The whole fit of a pair of up to kGmOne points by one workgroup, its samples in registers: a
// pass is then two barriers and the workgroup's FP64 issue instead of a launch.  Above, that issue
// costs more than a launch's latency.  The twelve launches against the one: 100 points 59 -> 27 us, 4,000 points
// 67 -> 43; 8,000 points would take 59 for 62.
constexpr int kOneThreads = 1024, kOneHold = kGmOne / kOneThreads;

__global__ __launch_bounds__(kOneThreads) void k_gm_one(GmFit g)
{
    __shared__ double red[kOneThreads / 64][16];
    __shared__ double model[6];
    const GmPair P = gm_pair(g, (int)blockIdx.x);
    if (P.p1 - P.p0 > kGmOne) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const double cx = 0.5 * (P.W - 1), cy = 0.5 * (P.H - 1), c2 = g.c * g.c;
    float2 hp[kOneHold], hm[kOneHold];
    uint8_t hs[kOneHold];
#pragma unroll
    for (int j = 0; j < kOneHold; ++j) {
        const int64_t i = P.p0 + t + kOneThreads * j;
        hs[j] = DGF_ST_CONVERGED + 1;
        if (i < P.p1) {
            hp[j] = g.pts[i];
            hm[j] = g.flow[i];
            hs[j] = g.status[i];
        }
    }
    double A[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int pass = 0; pass < kGmPasses; ++pass) {
        double v[kGmSums];
#pragma unroll
        for (int k = 0; k < kGmSums; ++k) v[k] = 0.0;
#pragma unroll
        for (int j = 0; j < kOneHold; ++j)
            if (hs[j] == DGF_ST_CONVERGED) add_sample(hp[j], hm[j], cx, cy, c2, pass, A, v);
        wave_sums(v, red[wave]);
        __syncthreads();
        if (wave == 0) {
            // lane k (mod 16) sums value k over four wavefronts, then the four rows of lanes
            double x = 0.0;
#pragma unroll
            for (int w = 0; w < kOneThreads / 256; ++w) x += red[(lane >> 4) * (kOneThreads / 256) + w][lane & 15];
            x += __shfl_xor(x, 16, 64);
            x += __shfl_xor(x, 32, 64);
            const uint2 u = __builtin_bit_cast(uint2, x);
            double S[kGmSums];
#pragma unroll
            for (int k = 0; k < kGmSums; ++k)
                S[k] = __builtin_bit_cast(double, uint2{(unsigned)__builtin_amdgcn_readlane((int)u.x, k),
                                                        (unsigned)__builtin_amdgcn_readlane((int)u.y, k)});
            gm_solve(S, A);
            if (lane == 0)
#pragma unroll
                for (int k = 0; k < 6; ++k) model[k] = A[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 6; ++k) A[k] = model[k];
    }
    if (t < 6) g.models[(size_t)blockIdx.x * 6 + t] = model[t];
}

// Pass `pass` (0 .. kGmPasses - 1) sums its slice under the weights of the model of pass - 1 (pass
// 0: weight 1 on every sample); pass kGmPasses only finishes the last model.
__global__ __launch_bounds__(kThreads) void k_gm_pass(GmFit g, int pass)
{
    __shared__ double red[2][kWaves][16];
    const int pair = blockIdx.y;
    const int t = threadIdx.x;
    const GmPair P = gm_pair(g, pair);
    const int64_t p0 = P.p0, p1 = P.p1;
    const int W = P.W, H = P.H;
    if (p1 - p0 <= kGmOne) return; // (k_gm_one's)
    const int nb = gm_blocks(p1 - p0); // this pair's workgroups (the grid covers the largest pair)
    if ((int)blockIdx.x >= nb) return;
    const int64_t chunk = (p1 - p0 + nb - 1) / nb;
    const int64_t b0 = p0 + chunk * blockIdx.x;
    const int64_t b1 = pass >= kGmPasses ? b0 : (b0 + chunk < p1 ? b0 + chunk : p1);
    // the slice's first samples are fetched before the model they are weighted with is rebuilt
    float2 hp[kHold], hm[kHold];
    uint8_t hs[kHold];
    auto fetch = [&](int64_t i0) {
#pragma unroll
        for (int j = 0; j < kHold; ++j) {
            const int64_t i = i0 + t + kThreads * j;
            hs[j] = DGF_ST_CONVERGED + 1;
            if (i < b1) {
                hp[j] = g.pts[i];
                hm[j] = g.flow[i];
                hs[j] = g.status[i];
            }
        }
    };
    fetch(b0);
    double v[kGmSums], A[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (pass > 0) {
        // the model of pass - 1 from its partial sums (kept from pass - 2 where it cannot be solved)
        const double *part = g.part + ((size_t)((pass - 1) & 1) * g.npairs + pair) * g.nblk * kGmSums;
        if (pass >= 2) {
            const double *prev = g.models + ((size_t)((pass - 2) & 1) * g.npairs + pair) * 6;
#pragma unroll
            for (int k = 0; k < 6; ++k) A[k] = prev[k];
        }
#pragma unroll
        for (int k = 0; k < kGmSums; ++k) v[k] = t < nb ? part[(size_t)t * kGmSums + k] : 0.0;
        double S[kGmSums];
        block_sum(v, red[0], S);
        gm_solve(S, A); // by every lane alike
        if (blockIdx.x == 0 && t == 0) {
            double *out = g.models + ((size_t)((pass - 1) & 1) * g.npairs + pair) * 6;
#pragma unroll
            for (int k = 0; k < 6; ++k) out[k] = A[k];
        }
    }
    if (pass >= kGmPasses) return;

    const double cx = 0.5 * (W - 1), cy = 0.5 * (H - 1);
    const double c2 = g.c * g.c;
#pragma unroll
    for (int k = 0; k < kGmSums; ++k) v[k] = 0.0;
    for (int64_t i0 = b0; i0 < b1; i0 += kThreads * kHold) {
        if (i0 != b0) fetch(i0);
#pragma unroll
        for (int j = 0; j < kHold; ++j) {
            if (hs[j] == DGF_ST_CONVERGED) add_sample(hp[j], hm[j], cx, cy, c2, pass, A, v);
        }
    }
    double S[kGmSums];
    block_sum(v, red[1], S);
    if (t == 0) {
        double *out = g.part + (((size_t)(pass & 1) * g.npairs + pair) * g.nblk + blockIdx.x) * kGmSums;
#pragma unroll
        for (int k = 0; k < kGmSums; ++k) out[k] = S[k];
    }
}

} // namespace

size_t gm_models_bytes(int npairs) { return (size_t)(2 * npairs * 6 * sizeof(double) + 255) / 256 * 256; }

size_t gm_state_bytes(int npairs, int nblk)
{
    return gm_models_bytes(npairs) + (size_t)2 * npairs * nblk * kGmSums * sizeof(double);
}

hipError_t launch_gm_fit(const GmFit &g, hipStream_t st)
{
    // a pair's form depends on its own point count; either launch leaves the other's pairs alone
    if (g.npairs > 1 || g.nblk <= gm_blocks(kGmOne)) {
        hipLaunchKernelGGL(k_gm_one, dim3(g.npairs), dim3(kOneThreads), 0, st, g);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (g.nblk <= gm_blocks(kGmOne)) return hipSuccess; // no larger pair
    for (int pass = 0; pass <= kGmPasses; ++pass) {
        const dim3 grid(pass < kGmPasses ? g.nblk : 1, g.npairs);
        hipLaunchKernelGGL(k_gm_pass, grid, dim3(kThreads), 0, st, g, pass);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace dgf

extern "C" {

size_t dgf_gm_workspace_bytes(void) { return dgf::gm_state_bytes(1, dgf::kGmMaxBlocks); }

int dgf_gm_fit(const float *points, const float *flow, const uint8_t *status, int64_t n, int32_t width, int32_t height,
               double scale, void *workspace, size_t ws_bytes, double *model, void *stream)
{
    using namespace dgf;
    if (n < 0 || width < 1 || height < 1 || !model || !(scale > 0.0) || !std::isfinite(scale)) return DGF_ERR_INVALID_ARG;
    if (n > 0 && (!points || !flow || !status)) return DGF_ERR_INVALID_ARG;
    if (!workspace || ws_bytes < dgf_gm_workspace_bytes()) return DGF_ERR_WORKSPACE;
    GmFit g{};
    g.pts = reinterpret_cast<const float2 *>(points);
    g.flow = reinterpret_cast<const float2 *>(flow);
    g.status = status;
    g.n = n;
    g.W = width;
    g.H = height;
    g.L = 1;
    g.npairs = 1;
    g.nblk = gm_blocks(n);
    g.c = kTukeyC * scale;
    g.models = reinterpret_cast<double *>(workspace);
    g.part = reinterpret_cast<double *>((uint8_t *)workspace + gm_models_bytes(1));
    hipStream_t st = (hipStream_t)stream;
    if (launch_gm_fit(g, st) != hipSuccess) return DGF_ERR_HIP;
    return hipMemcpyAsync(model, g.models, 6 * sizeof(double), hipMemcpyDeviceToDevice, st) == hipSuccess ? DGF_OK
                                                                                                       : DGF_ERR_HIP;
}

} // extern "C"
