// pyramid.hip -- pyramid reduction steps on gfx950, up to four levels per launch.
//
// Level l+1 = binomial [1 4 6 4 1] smoothing of level l along both axes with replicated borders,
// sampled at even pixels (size ceil(W/2) x ceil(H/2)).  uint8 levels keep the exact integer sum
// and round half up, (sum + 128) >> 8; float levels are scaled by 1/256.
//
// blockIdx.z selects the image, so both frames of a pair go in one launch.  (Batch plans use
// front_batch.hip.)
#include "dgf_internal.hpp"

namespace dgf {

// ---- several levels in one launch ----------------------------------------------------------
//
// Levels s+1 .. s+m (m <= 4) of one or two images from level s.  A block owns a
// PC_T x PC_T tile of the coarsest level s+m and the 2^(m-k) times larger tile of every finer
// level s+k, which tile each level exactly; it computes each level over its owned tile plus the
// halo the next coarser level's taps need (the needed range [lo, hi] at level k+1 needs
// [2 lo - 2, 2 hi + 2] at level k, clamped into the level), starting from a staged rectangle of
// level s, and writes the owned pixels, with the replicated border of every level.
constexpr int PC_T = 4, PC_MAXM = 4;
// Lanes per chain block: a block walks its levels one after another, each a few LDS passes with
// barriers between, and with one or two blocks per CU only its own waves hide the LDS latency;
// eight waves measured 15 % faster than four on the 1242x375 pair (sixteen: 11 %).
constexpr int kChainThreads = 512;
constexpr int pc_width(int m) { return m == 0 ? PC_T : 2 * pc_width(m - 1) + 3; } // region width m levels finer
constexpr int PC_N0 = pc_width(PC_MAXM);     // 109: staged source rectangle side
constexpr int PC_N1 = pc_width(PC_MAXM - 1); // 53: first produced level
constexpr int PC_N0P = (PC_N0 + 3) & ~3;     // 112: row pitch of the staged source rectangle

// The pixels [x0, x1] x [y0, y1] of every level that a chain block needs: coarsest first, each finer
// level's from the next coarser one's taps, clamped into the level.
__device__ __forceinline__ void chain_ranges(const PyrChain &A, int bx, int by, int (&x0)[PC_MAXM + 1],
                                             int (&x1)[PC_MAXM + 1], int (&y0)[PC_MAXM + 1], int (&y1)[PC_MAXM + 1])
{
    const int m = A.m;
    int lx = bx * PC_T, hx = lx + PC_T - 1, ly = by * PC_T, hy = ly + PC_T - 1;
#pragma unroll
    for (int k = PC_MAXM; k >= 0; --k) {
        if (k <= m) {
            if (k < m) {
                lx = 2 * lx - 2;
                hx = 2 * hx + 2;
                ly = 2 * ly - 2;
                hy = 2 * hy + 2;
            }
            x0[k] = lx > 0 ? lx : 0;
            x1[k] = hx < A.W[k] - 1 ? hx : A.W[k] - 1;
            y0[k] = ly > 0 ? ly : 0;
            y1[k] = hy < A.H[k] - 1 ? hy : A.H[k] - 1;
        }
    }
}

// One block of a chain launch: tile (bx, by) of the coarsest level of image f, with the LDS
// buffers the kernel provides.
__device__ __forceinline__ void pyr_chain_block(const PyrChain &A, int bx, int by, int f,
                                                uint8_t (*lvl)[PC_N0P * PC_N0], uint16_t *hs)
{
    const int m = A.m, tid = threadIdx.x;
    int x0[PC_MAXM + 1], x1[PC_MAXM + 1], y0[PC_MAXM + 1], y1[PC_MAXM + 1];
    chain_ranges(A, bx, by, x0, x1, y0, y1);
    // stage level s (row pitch 4 ceil(w / 4); the produced levels use their own width)
    const int w0 = x1[0] - x0[0] + 1, p0 = (w0 + 3) & ~3;
    stage_u8_block<4>(lvl[0], p0, A.src[f], A.src_pitch[f], A.W[0], x0[0], y0[0], w0, y1[0] - y0[0] + 1);
    __syncthreads();
    for (int k = 0; k < m; ++k) {
        const uint8_t *in = lvl[k & 1];
        uint8_t *out = lvl[(k + 1) & 1];
        const int wi = x1[k] - x0[k] + 1, hi = y1[k] - y0[k] + 1, pin = k == 0 ? p0 : wi;
        const int wo = x1[k + 1] - x0[k + 1] + 1, ho = y1[k + 1] - y0[k + 1] + 1;
        const float inv_wo = 1.0f / (float)wo;
        const int Wk = A.W[k], Hk = A.H[k];
        // horizontal pass: every staged row, at the output column rate
        for (int i = tid; i < hi * wo; i += kChainThreads) {
            const int r = div_small(i, inv_wo), xo = i - r * wo;
            const int c = 2 * (x0[k + 1] + xo);
            const uint8_t *row = in + r * pin;
            auto at = [&](int cc) { return (int)row[(cc < 0 ? 0 : (cc > Wk - 1 ? Wk - 1 : cc)) - x0[k]]; };
            hs[i] = (uint16_t)(at(c - 2) + at(c + 2) + 4 * (at(c - 1) + at(c + 1)) + 6 * at(c));
        }
        __syncthreads();
        // vertical pass, rounding, and the owned pixels to memory
        const int sh = m - (k + 1);
        const int ox0 = (bx * PC_T) << sh, oy0 = (by * PC_T) << sh;
        const int own = PC_T << sh;
        uint8_t *dst = A.dst[k][f];
        const int64_t dp = A.dst_pitch[k];
        for (int i = tid; i < ho * wo; i += kChainThreads) {
            const int yo = div_small(i, inv_wo), xo = i - yo * wo;
            const int gy = y0[k + 1] + yo, gx = x0[k + 1] + xo;
            const int rr = 2 * gy;
            auto at = [&](int r) { return (int)hs[((r < 0 ? 0 : (r > Hk - 1 ? Hk - 1 : r)) - y0[k]) * wo + xo]; };
            const int v = at(rr - 2) + at(rr + 2) + 4 * (at(rr - 1) + at(rr + 1)) + 6 * at(rr);
            const uint8_t q = (uint8_t)((v + 128) >> 8);
            out[i] = q;
            if (gx >= ox0 && gx < ox0 + own && gy >= oy0 && gy < oy0 + own) dst[(int64_t)gy * dp + gx] = q;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kChainThreads) void k_pyr_chain_u8(PyrChain A)
{
    __shared__ __align__(16) uint8_t lvl[2][PC_N0P * PC_N0];
    __shared__ uint16_t hs[PC_N0 * PC_N1];
    pyr_chain_block(A, (int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, lvl, hs);
}

// The chain launch with the detection tiles of one uint8 frame beside it: blocks 0 .. nchain - 1
// build pyramid tiles (x fastest, then y, then image), the rest are 16 x 16-window detection
// tiles staged in the chain's level buffer (lanes beyond the 256 windows only help staging).  The two kinds of work are independent, so one
// launch runs both in about the time of the longer.
__global__ __launch_bounds__(kChainThreads) void k_front_u8(PyrChain A, FrontDetect D, int chain_x, int chain_y, int nchain)
{
    __shared__ __align__(16) uint8_t lvl[2][PC_N0P * PC_N0];
    __shared__ uint16_t hs[PC_N0 * PC_N1];
    const int b = (int)blockIdx.x;
    if (b < nchain) {
        const int per = chain_x * chain_y, f = b / per, t = b - f * per, by = t / chain_x;
        pyr_chain_block(A, t - by * chain_x, by, f, lvl, hs);
        return;
    }
    const int t = b - nchain, ty = t / D.tiles_x;
    if (D.side == 8)
        detect_tile<8, 8>(&lvl[0][0], t - ty * D.tiles_x, ty, D.img, D.pitch, D.W, D.H, D.win, D.stride, D.nx, D.ny, 0,
                          D.o);
    else
        detect_tile<16, 16>(&lvl[0][0], t - ty * D.tiles_x, ty, D.img, D.pitch, D.W, D.H, D.win, D.stride, D.nx, D.ny, 0,
                            D.o);
}

// Largest detection tile the fused launch can stage (the chain's two level buffers).
constexpr size_t kFrontDetectLds = 2 * (size_t)PC_N0P * PC_N0;

// The float levels by the same tiles: sums of whole products, 4 (a + b) exact and 6 c fused into its
// sum, then the scale.  One launch for the three coarser levels of a 640x480 pair takes 10 us, where
// one launch per level took 24.  Dynamic LDS: the staged rectangle and the
// levels in turn in two buffers, then the horizontal sums.
__global__ __launch_bounds__(kChainThreads) void k_pyr_chain_f32(PyrChain A, int n0, int n1)
{
    extern __shared__ float chain_lds[];
    float *const buf[2] = {chain_lds, chain_lds + n0 * n0};
    float *const hs = buf[1] + n1 * n1;
    const int m = A.m, tid = threadIdx.x, bx = (int)blockIdx.x, by = (int)blockIdx.y, f = (int)blockIdx.z;
    int x0[PC_MAXM + 1], x1[PC_MAXM + 1], y0[PC_MAXM + 1], y1[PC_MAXM + 1];
    chain_ranges(A, bx, by, x0, x1, y0, y1);
    {
        const int w = x1[0] - x0[0] + 1, n = w * (y1[0] - y0[0] + 1);
        const float inv = 1.0f / (float)w;
        const uint8_t *src = A.src[f] + (int64_t)y0[0] * A.src_pitch[f] + 4 * (int64_t)x0[0];
        constexpr int kB = 6; // loads in flight
        for (int i0 = tid; i0 < n; i0 += kB * kChainThreads) {
            float v[kB];
#pragma unroll
            for (int k = 0; k < kB; ++k) {
                const int i = min(i0 + k * kChainThreads, n - 1), r = div_small(i, inv);
                v[k] = reinterpret_cast<const float *>(src + (int64_t)r * A.src_pitch[f])[i - r * w];
            }
#pragma unroll
            for (int k = 0; k < kB; ++k)
                if (i0 + k * kChainThreads < n) buf[0][i0 + k * kChainThreads] = v[k];
        }
    }
    __syncthreads();
    for (int k = 0; k < m; ++k) {
        const float *in = buf[k & 1];
        float *out = buf[(k + 1) & 1];
        const int wi = x1[k] - x0[k] + 1, hi = y1[k] - y0[k] + 1;
        const int wo = x1[k + 1] - x0[k + 1] + 1, ho = y1[k + 1] - y0[k + 1] + 1;
        const float inv_wo = 1.0f / (float)wo;
        const int Wk = A.W[k], Hk = A.H[k];
        auto five = [](float a, float b, float c, float d, float e) {
            return fmaf(6.0f, c, fmaf(4.0f, b + d, a + e));
        };
        for (int i = tid; i < hi * wo; i += kChainThreads) {
            const int r = div_small(i, inv_wo), c = 2 * (x0[k + 1] + i - r * wo);
            const float *row = in + r * wi - x0[k];
            auto at = [&](int cc) { return row[cc < 0 ? 0 : (cc > Wk - 1 ? Wk - 1 : cc)]; };
            hs[i] = five(at(c - 2), at(c - 1), at(c), at(c + 1), at(c + 2));
        }
        __syncthreads();
        const int sh = m - (k + 1), own = PC_T << sh, ox0 = (bx * PC_T) << sh, oy0 = (by * PC_T) << sh;
        for (int i = tid; i < ho * wo; i += kChainThreads) {
            const int yo = div_small(i, inv_wo), xo = i - yo * wo;
            const int gy = y0[k + 1] + yo, gx = x0[k + 1] + xo, rr = 2 * gy;
            auto at = [&](int r) { return hs[((r < 0 ? 0 : (r > Hk - 1 ? Hk - 1 : r)) - y0[k]) * wo + xo]; };
            const float v = five(at(rr - 2), at(rr - 1), at(rr), at(rr + 1), at(rr + 2)) * (1.0f / 256.0f);
            out[i] = v;
            if (gx >= ox0 && gx < ox0 + own && gy >= oy0 && gy < oy0 + own)
                reinterpret_cast<float *>(A.dst[k][f] + (int64_t)gy * A.dst_pitch[k])[gx] = v;
        }
        __syncthreads();
    }
}

static hipError_t launch_pyr_chain_f32(const PyrChain &A, int njobs, hipStream_t st)
{
    if (A.m < 1 || A.m > PC_MAXM || njobs < 1 || njobs > 2) return hipErrorInvalidValue;
    const int n0 = pc_width(A.m), n1 = pc_width(A.m - 1);
    const dim3 grid((A.W[A.m] + PC_T - 1) / PC_T, (A.H[A.m] + PC_T - 1) / PC_T, njobs);
    const size_t lds = sizeof(float) * (size_t)(n0 * n0 + n1 * n1 + n0 * n1);
    hipLaunchKernelGGL(k_pyr_chain_f32, grid, dim3(kChainThreads), lds, st, A, n0, n1);
    return hipGetLastError();
}

hipError_t launch_pyr_chain_u8(const PyrChain &A, int njobs, hipStream_t st, const FrontDetect *det)
{
    if (A.m < 1 || A.m > PC_MAXM || njobs < 1 || njobs > 2) return hipErrorInvalidValue;
    dim3 grid((A.W[A.m] + PC_T - 1) / PC_T, (A.H[A.m] + PC_T - 1) / PC_T, njobs);
    if (!det) {
        hipLaunchKernelGGL(k_pyr_chain_u8, grid, dim3(kChainThreads), 0, st, A);
        return hipGetLastError();
    }
    const int nchain = (int)(grid.x * grid.y * grid.z);
    const int blocks = nchain + det->tiles_x * det->tiles_y;
    hipLaunchKernelGGL(k_front_u8, dim3((unsigned)blocks), dim3(kChainThreads), 0, st, A, *det, (int)grid.x, (int)grid.y, nchain);
    return hipGetLastError();
}

bool front_detect_fits(int win, int stride) { return detect_tile_lds(win, stride) <= kFrontDetectLds; }

// Levels 1 .. levels-1 of one or two images (level 0 = srcs) as chains of up to four
// levels per launch; level l of image f goes to lvl[f][l], row pitch pitch[l].
hipError_t launch_pyr_chains(const uint8_t *const srcs[2], const int64_t src_pitch[2],
                             uint8_t *const lvl[2][DGF_MAX_LEVELS], const int64_t *pitch, int W, int H, int levels,
                             int njobs, int dtype, hipStream_t st, const FrontDetect *det)
{
    int Wl[DGF_MAX_LEVELS], Hl[DGF_MAX_LEVELS];
    Wl[0] = W;
    Hl[0] = H;
    for (int l = 1; l < levels; ++l) {
        Wl[l] = (Wl[l - 1] + 1) / 2;
        Hl[l] = (Hl[l - 1] + 1) / 2;
    }
    for (int s = 0; s + 1 < levels; s += PC_MAXM) {
        PyrChain A{};
        A.m = levels - 1 - s < PC_MAXM ? levels - 1 - s : PC_MAXM;
        for (int f = 0; f < njobs; ++f) {
            A.src[f] = s == 0 ? srcs[f] : lvl[f][s];
            A.src_pitch[f] = s == 0 ? src_pitch[f] : pitch[s];
            for (int k = 1; k <= A.m; ++k) A.dst[k - 1][f] = lvl[f][s + k];
        }
        for (int k = 0; k <= A.m; ++k) {
            A.W[k] = Wl[s + k];
            A.H[k] = Hl[s + k];
            if (k > 0) A.dst_pitch[k - 1] = pitch[s + k];
        }
        const hipError_t e = dtype == DGF_U8 ? launch_pyr_chain_u8(A, njobs, st, s == 0 ? det : nullptr)
                                             : launch_pyr_chain_f32(A, njobs, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace dgf
