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
// Levels s+1 .. s+m (m <= 4) of one or two images from level s.  A block owns a T x T tile of the
// coarsest level s+m (T = chain_tile(m)) and the 2^(m-k) times larger tile of every finer level
// s+k, which tile each level exactly; it computes each level over its owned tile plus the
// halo the next coarser level's taps need (the needed range [lo, hi] at level k+1 needs
// [2 lo - 2, 2 hi + 2] at level k), starting from a staged rectangle of level s, and writes the
// owned pixels, with the replicated border of every level.  Tiles of 32 level-s pixels for up to
// three levels and 64 for four: with tiles of 4 throughout, a block of one level made 16 pixels.
constexpr int PC_MAXM = 4;
inline __host__ __device__ constexpr int chain_tile(int m) { return m <= 1 ? 16 : m == 2 ? 8 : 4; }
// Lanes per chain block: a block walks its levels one after another, each a few LDS passes with
// barriers between, and with one or two blocks per CU only its own waves hide the LDS latency;
// eight waves measured 15 % faster than four on the 1242x375 pair (sixteen: 11 %).
constexpr int kChainThreads = 512;
// region width, j levels above the coarsest
constexpr int pc_width(int j, int T) { return j == 0 ? T : 2 * pc_width(j - 1, T) + 3; }
constexpr int pc_pitch(int j, int T) { return (pc_width(j, T) + 3) & ~3; } // bytes per LDS row of a uint8 chain
constexpr int PC_N0 = pc_width(PC_MAXM, chain_tile(PC_MAXM));  // 109: the largest staged rectangle's side
constexpr int PC_N0P = pc_pitch(PC_MAXM, chain_tile(PC_MAXM)); // 112

// ---- uint8 chains
//
// A block holds every level over its whole needed range, positions outside the image included, as
// replicas of the border pixel they clamp to; relative to the range's first column the taps of output q
// are then columns 2 q .. 2 q + 4 everywhere, four outputs take three dwords, and the sums are byte
// dot products (horizontal) and 16-bit pairs (vertical).  Sizes are those of pc_width, known when
// compiled.  A launch is a few hundred blocks, each bound by its own latency, or on large frames by LDS
// passes: against a byte per step with clamped columns, four levels of a 1242x375 pair take 8.0 us for 11.6,
// one level 3.5 for 36 (with the larger tiles); of a 4096x2160 pair 39 for 86 and 29 for 630.
struct ChainLds {
    uint8_t lvl[2][PC_N0P * PC_N0 + 16]; // levels in turn (+ the dword read past the last row)
    uint16_t hs[PC_N0 * pc_pitch(PC_MAXM - 1, chain_tile(PC_MAXM))];
};

// Positions of a level's range (columns from ux, rows from uy, HO of each at row pitch PO) that lie
// outside the W x H level take the border pixel they clamp to.
template <int HO, int PO, class Pix>
__device__ __forceinline__ void chain_replicate(Pix *out, int ux, int uy, int W, int H)
{
    if (ux >= 0 && uy >= 0 && ux + HO <= W && uy + HO <= H) return;
    for (int t = threadIdx.x; t < HO * HO; t += kChainThreads) {
        const int y = t / HO, x = t - y * HO;
        const int cy = clampi(uy + y, 0, H - 1) - uy, cx = clampi(ux + x, 0, W - 1) - ux;
        if ((cx != x || cy != y) && cx >= 0 && cx < HO && cy >= 0 && cy < HO) out[y * PO + x] = out[cy * PO + cx];
    }
    __syncthreads();
}

// The level J above the coarsest, from memory: four bytes from the aligned dwords that hold the first
// and the last of them, columns outside the row by a byte selection; all of a lane's loads are in
// flight together.
template <int J, int T>
__device__ __forceinline__ void chain_stage(const PyrChain &A, int f, int ux, int uy, uint8_t *lds)
{
    typedef const __attribute__((address_space(1))) uint32_t gword;
    typedef const __attribute__((address_space(1))) uint8_t gbyte;
    constexpr int P4 = pc_pitch(J, T) / 4, N = P4 * pc_width(J, T), NT = (N + kChainThreads - 1) / kChainThreads;
    const int W = A.W[0], H = A.H[0], tid = threadIdx.x;
    if (W < 4) { // (a dword of a row does not exist)
        for (int t = tid; t < N; t += kChainThreads) {
            const int r = t / P4, c = ux + 4 * (t - r * P4);
            gbyte *b = (gbyte *)(A.src[f] + (int64_t)clampi(uy + r, 0, H - 1) * A.src_pitch[f]);
            uint32_t v = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) v |= (uint32_t)b[clampi(c + e, 0, W - 1)] << (8 * e);
            reinterpret_cast<uint32_t *>(lds)[t] = v;
        }
        return;
    }
    uint32_t lo[NT], hi[NT];
    auto at = [&](int k, int &c) { // the row's bytes c .. c + 3, moved inside the row
        const int t = min(tid + kChainThreads * k, N - 1), r = t / P4;
        c = ux + 4 * (t - r * P4);
        return (uintptr_t)(A.src[f] + (int64_t)clampi(uy + r, 0, H - 1) * A.src_pitch[f] + clampi(c, 0, W - 4));
    };
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        int c;
        const uintptr_t p = at(k, c);
        gword *a = (gword *)(p & ~(uintptr_t)3);
        lo[k] = a[0];
        hi[k] = a[(p & 3) ? 1 : 0]; // (a second dword only where it holds a byte of these four)
    }
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        int c;
        const uintptr_t p = at(k, c);
        uint32_t v = __builtin_amdgcn_alignbyte(hi[k], lo[k], (uint32_t)p & 3u);
        const int b = clampi(c, 0, W - 4);
        if (b != c) { // part or all of the four lie outside: each takes the byte its column clamps to
            uint32_t sel = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) sel |= (uint32_t)(clampi(c + e, 0, W - 1) - b) << (8 * e);
            v = __builtin_amdgcn_perm(v, v, sel);
        }
        const int t = tid + kChainThreads * k;
        if (t < N) reinterpret_cast<uint32_t *>(lds)[t] = v;
    }
}

// One level: from level k = m - J in `in` to level k + 1 in `out` and, its owned part, to memory.
// bx, by: the block's tile.
template <int J, int T>
__device__ __forceinline__ void chain_level(const PyrChain &A, int f, int bx, int by, const uint8_t *in, uint8_t *out,
                                            uint16_t *hs)
{
    constexpr int PI = pc_pitch(J, T) / 4, HI = pc_width(J, T), PO = pc_pitch(J - 1, T), HO = pc_width(J - 1, T);
    constexpr int G = PO / 4; // groups of four outputs per row
    constexpr int kHalo = (2 << (J - 1)) - 2, kOwn = T << (J - 1); // owned columns kHalo .. kHalo + kOwn - 1
    const int tid = threadIdx.x, k1 = A.m - J + 1;
    const int W = A.W[k1], H = A.H[k1];
    const int ux = bx * kOwn - kHalo, uy = by * kOwn - kHalo;
    constexpr uint32_t kTaps = 0x04060401u; // 1 4 6 4 (the fifth tap, 1, is added)
    const uint32_t *in4 = reinterpret_cast<const uint32_t *>(in);
    for (int t = tid; t < HI * G; t += kChainThreads) {
        const int r = t / G, q = t - r * G;
        const uint32_t *p = in4 + r * PI + 2 * q;
        const uint32_t d0 = p[0], d1 = p[1], d2 = p[2];
        const uint32_t h0 = __builtin_amdgcn_udot4(d0, kTaps, d1 & 255u, false);
        const uint32_t h1 = __builtin_amdgcn_udot4(__builtin_amdgcn_alignbyte(d1, d0, 2), kTaps, (d1 >> 16) & 255u, false);
        const uint32_t h2 = __builtin_amdgcn_udot4(d1, kTaps, d2 & 255u, false);
        const uint32_t h3 = __builtin_amdgcn_udot4(__builtin_amdgcn_alignbyte(d2, d1, 2), kTaps, (d2 >> 16) & 255u, false);
        reinterpret_cast<uint2 *>(hs)[t] = make_uint2(h0 | (h1 << 16), h2 | (h3 << 16));
    }
    __syncthreads();
    uint8_t *dst = A.dst[k1 - 1][f];
    const int64_t dp = A.dst_pitch[k1 - 1];
    const bool even = (((uintptr_t)dst | (uintptr_t)dp) & 1) == 0; // (a caller's buffer may start anywhere)
    for (int t = tid; t < HO * G; t += kChainThreads) {
        const int y = t / G, q = t - y * G;
        const uint2 *p = reinterpret_cast<const uint2 *>(hs) + 2 * y * G + q;
        uint32_t o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u16x2 a[5];
#pragma unroll
            for (int e = 0; e < 5; ++e) a[e] = __builtin_bit_cast(u16x2, h ? p[e * G].y : p[e * G].x);
            // at most 16 x 4080 + 128 < 2^16: exact in 16 bits
            const u16x2 v = (u16x2)((a[0] + a[4]) + (u16x2)4 * (a[1] + a[3]) + (u16x2)6 * a[2] + (u16x2)128) >> (u16x2)8;
            o[h] = (uint32_t)v[0] | ((uint32_t)v[1] << 8);
        }
        if constexpr (J > 1) reinterpret_cast<uint32_t *>(out)[t] = o[0] | (o[1] << 16);
        // owned columns start and end on even ones, so a pair is owned or not as a whole
        const int gy = uy + y;
        if (y < kHalo || y >= kHalo + kOwn || gy >= H) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int x = 4 * q + 2 * h, gx = ux + x;
            if (x < kHalo || x >= kHalo + kOwn || gx >= W) continue;
            uint8_t *d = dst + (int64_t)gy * dp + gx;
            if (gx + 1 < W && even) {
                *reinterpret_cast<uint16_t *>(d) = (uint16_t)o[h];
            } else {
                d[0] = (uint8_t)o[h];
                if (gx + 1 < W) d[1] = (uint8_t)(o[h] >> 8);
            }
        }
    }
    __syncthreads();
    if constexpr (J > 1) chain_replicate<HO, PO>(out, ux, uy, W, H);
}

template <int M>
__device__ __forceinline__ void chain_levels(const PyrChain &A, int bx, int by, int f, ChainLds &L)
{
    constexpr int T = chain_tile(M), kHalo = (2 << M) - 2, kOwn = T << M;
    chain_stage<M, T>(A, f, bx * kOwn - kHalo, by * kOwn - kHalo, L.lvl[0]);
    __syncthreads();
    chain_level<M, T>(A, f, bx, by, L.lvl[0], L.lvl[1], L.hs);
    if constexpr (M > 1) chain_level<M - 1, T>(A, f, bx, by, L.lvl[1], L.lvl[0], L.hs);
    if constexpr (M > 2) chain_level<M - 2, T>(A, f, bx, by, L.lvl[0], L.lvl[1], L.hs);
    if constexpr (M > 3) chain_level<M - 3, T>(A, f, bx, by, L.lvl[1], L.lvl[0], L.hs);
}

// One block of a chain launch: tile (bx, by) of the coarsest level of image f.
__device__ __forceinline__ void pyr_chain_block(const PyrChain &A, int bx, int by, int f, ChainLds &L)
{
    static_assert(PC_MAXM == 4, "cases");
    switch (A.m) {
    case 1: chain_levels<1>(A, bx, by, f, L); break;
    case 2: chain_levels<2>(A, bx, by, f, L); break;
    case 3: chain_levels<3>(A, bx, by, f, L); break;
    default: chain_levels<4>(A, bx, by, f, L); break;
    }
}

__global__ __launch_bounds__(kChainThreads) void k_pyr_chain_u8(PyrChain A)
{
    __shared__ __align__(16) ChainLds L;
    pyr_chain_block(A, (int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, L);
}

// The chain launch with the detection tiles of one uint8 frame beside it: blocks 0 .. nchain - 1
// build pyramid tiles (x fastest, then y, then image), the rest are 16 x 16-window detection
// tiles staged in the chain's level buffer (lanes beyond the 256 windows only help staging).  The two kinds of work are independent, so one
// launch runs both in about the time of the longer.
__global__ __launch_bounds__(kChainThreads) void k_front_u8(PyrChain A, FrontDetect D, int chain_x, int chain_y, int nchain)
{
    __shared__ __align__(16) ChainLds L;
    const int b = (int)blockIdx.x;
    if (b < nchain) {
        const int per = chain_x * chain_y, f = b / per, t = b - f * per, by = t / chain_x;
        pyr_chain_block(A, t - by * chain_x, by, f, L);
        return;
    }
    const int t = b - nchain, ty = t / D.tiles_x;
    if (D.side == 8)
        detect_tile<8, 8>(&L.lvl[0][0], t - ty * D.tiles_x, ty, D.img, D.pitch, D.W, D.H, D.win, D.stride, D.nx, D.ny, 0,
                          D.o);
    else
        detect_tile<16, 16>(&L.lvl[0][0], t - ty * D.tiles_x, ty, D.img, D.pitch, D.W, D.H, D.win, D.stride, D.nx, D.ny, 0,
                            D.o);
}

// Largest detection tile the fused launch can stage (the chain's two level buffers).
constexpr size_t kFrontDetectLds = 2 * (size_t)PC_N0P * PC_N0;

// ---- float chains: the same tiles, a float per byte.  Sums of whole products, 4 (a + b) exact and
// 6 c fused into its sum, then the scale; four outputs per step from 16-byte LDS reads.  Four levels of a
// 640x480 pair take 8.9 us, a float per step 12.5, a launch per level 31 and the gaps between them.
template <int M, int T>
constexpr size_t chain_f32_floats(int part) // two level buffers in turn (+ the float4 read past the last row), horizontal sums
{
    const size_t n0 = (size_t)pc_width(M, T) * pc_pitch(M, T) + 4, n1 = (size_t)pc_width(M - 1, T) * pc_pitch(M - 1, T) + 4;
    const size_t h = (size_t)pc_width(M, T) * pc_pitch(M - 1, T);
    return part == 0 ? n0 : part == 1 ? n0 + n1 : n0 + n1 + h;
}

template <int J, int T>
__device__ __forceinline__ void chain_level_f32(const PyrChain &A, int f, int bx, int by, const float *in, float *out, float *hs)
{
    constexpr int PI = pc_pitch(J, T) / 4, HI = pc_width(J, T), PO = pc_pitch(J - 1, T), HO = pc_width(J - 1, T);
    constexpr int G = PO / 4;
    constexpr int kHalo = (2 << (J - 1)) - 2, kOwn = T << (J - 1);
    const int tid = threadIdx.x, k1 = A.m - J + 1;
    const int W = A.W[k1], H = A.H[k1];
    const int ux = bx * kOwn - kHalo, uy = by * kOwn - kHalo;
    auto five = [](float a, float b, float c, float d, float e) { return fmaf(6.0f, c, fmaf(4.0f, b + d, a + e)); };
    const float4 *in4 = reinterpret_cast<const float4 *>(in);
    for (int t = tid; t < HI * G; t += kChainThreads) {
        const int r = t / G, q = t - r * G;
        const float4 *p = in4 + r * PI + 2 * q;
        const float4 a = p[0], b = p[1], c = p[2];
        reinterpret_cast<float4 *>(hs)[t] = make_float4(five(a.x, a.y, a.z, a.w, b.x), five(a.z, a.w, b.x, b.y, b.z),
                                                        five(b.x, b.y, b.z, b.w, c.x), five(b.z, b.w, c.x, c.y, c.z));
    }
    __syncthreads();
    uint8_t *dst = A.dst[k1 - 1][f];
    const int64_t dp = A.dst_pitch[k1 - 1];
    const bool even = (((uintptr_t)dst | (uintptr_t)dp) & 7) == 0;
    for (int t = tid; t < HO * G; t += kChainThreads) {
        const int y = t / G, q = t - y * G;
        const float4 *p = reinterpret_cast<const float4 *>(hs) + 2 * y * G + q;
        const float4 a = p[0], b = p[G], c = p[2 * G], d = p[3 * G], e = p[4 * G];
        constexpr float k = 1.0f / 256.0f;
        const float4 v = make_float4(five(a.x, b.x, c.x, d.x, e.x) * k, five(a.y, b.y, c.y, d.y, e.y) * k,
                                     five(a.z, b.z, c.z, d.z, e.z) * k, five(a.w, b.w, c.w, d.w, e.w) * k);
        if constexpr (J > 1) reinterpret_cast<float4 *>(out)[t] = v;
        const int gy = uy + y;
        if (y < kHalo || y >= kHalo + kOwn || gy >= H) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int x = 4 * q + 2 * h, gx = ux + x;
            if (x < kHalo || x >= kHalo + kOwn || gx >= W) continue;
            float *o = reinterpret_cast<float *>(dst + (int64_t)gy * dp) + gx;
            const float2 w = h ? make_float2(v.z, v.w) : make_float2(v.x, v.y);
            if (gx + 1 < W && even) {
                *reinterpret_cast<float2 *>(o) = w;
            } else {
                o[0] = w.x;
                if (gx + 1 < W) o[1] = w.y;
            }
        }
    }
    __syncthreads();
    if constexpr (J > 1) chain_replicate<HO, PO>(out, ux, uy, W, H);
}

template <int M, int T>
__global__ __launch_bounds__(kChainThreads) void k_pyr_chain_f32(PyrChain A)
{
    extern __shared__ __align__(16) float chain_lds[];
    float *const b0 = chain_lds, *const b1 = chain_lds + chain_f32_floats<M, T>(0),
                *const hs = chain_lds + chain_f32_floats<M, T>(1);
    constexpr int kHalo = (2 << M) - 2, kOwn = T << M;
    const int bx = (int)blockIdx.x, by = (int)blockIdx.y, f = (int)blockIdx.z;
    {
        // (rows of any alignment: a float per lane, the columns past the range left out)
        constexpr int HI = pc_width(M, T), PI = pc_pitch(M, T), N = HI * HI;
        const int W = A.W[0], H = A.H[0], ux = bx * kOwn - kHalo, uy = by * kOwn - kHalo;
        constexpr int NT = (N + kChainThreads - 1) / kChainThreads, kB = NT < 12 ? NT : 12; // loads in flight
        for (int i0 = threadIdx.x; i0 < N; i0 += kB * kChainThreads) {
            float v[kB];
#pragma unroll
            for (int k = 0; k < kB; ++k) {
                const int i = min(i0 + k * kChainThreads, N - 1), r = i / HI;
                v[k] = reinterpret_cast<const float *>(A.src[f] + (int64_t)clampi(uy + r, 0, H - 1) * A.src_pitch[f])[clampi(
                    ux + i - r * HI, 0, W - 1)];
            }
#pragma unroll
            for (int k = 0; k < kB; ++k) {
                const int i = i0 + k * kChainThreads, r = i / HI;
                if (i < N) b0[r * PI + i - r * HI] = v[k];
            }
        }
    }
    __syncthreads();
    chain_level_f32<M, T>(A, f, bx, by, b0, b1, hs);
    if constexpr (M > 1) chain_level_f32<M - 1, T>(A, f, bx, by, b1, b0, hs);
    if constexpr (M > 2) chain_level_f32<M - 2, T>(A, f, bx, by, b0, b1, hs);
    if constexpr (M > 3) chain_level_f32<M - 3, T>(A, f, bx, by, b1, b0, hs);
}

// A large float frame's first level goes by itself: a block of more levels re-reads up to 2.9 times its
// pixels, which costs more than a launch from about a million pixels on (five levels of a 2048x1024
// pair: 15 us, 30 in one launch; of a 1242x375 pair 9 in one, 12 in two).  Its tiles are 32 pixels wide: with
// 16 a block stages 35 x 35 floats for 256 outputs and most of its lanes idle (2048x1024 pair, that
// level alone: 11.3 us, 6.4 now, 9.4 in tiles of 64 x 16 by 256 lanes; 4096x2160 35, 24, 35).
static bool chain_f32_alone(int W, int H) { return (int64_t)W * H > (1 << 20); }

static hipError_t launch_pyr_chain_f32(const PyrChain &A, int njobs, hipStream_t st)
{
    if (A.m < 1 || A.m > PC_MAXM || njobs < 1 || njobs > 2) return hipErrorInvalidValue;
    auto go = [&](auto m, auto tile) {
        constexpr int M = m.value, T = tile.value;
        const dim3 grid((A.W[M] + T - 1) / T, (A.H[M] + T - 1) / T, njobs);
        constexpr size_t lds = sizeof(float) * chain_f32_floats<M, T>(2);
        hipLaunchKernelGGL((k_pyr_chain_f32<M, T>), grid, dim3(kChainThreads), lds, st, A);
    };
    using std::integral_constant;
    static_assert(PC_MAXM == 4, "cases");
    switch (A.m) {
    case 1:
        if (chain_f32_alone(A.W[0], A.H[0]))
            go(integral_constant<int, 1>(), integral_constant<int, 32>());
        else
            go(integral_constant<int, 1>(), integral_constant<int, chain_tile(1)>());
        break;
    case 2: go(integral_constant<int, 2>(), integral_constant<int, chain_tile(2)>()); break;
    case 3: go(integral_constant<int, 3>(), integral_constant<int, chain_tile(3)>()); break;
    default: go(integral_constant<int, 4>(), integral_constant<int, chain_tile(4)>()); break;
    }
    return hipGetLastError();
}

hipError_t launch_pyr_chain_u8(const PyrChain &A, int njobs, hipStream_t st, const FrontDetect *det)
{
    if (A.m < 1 || A.m > PC_MAXM || njobs < 1 || njobs > 2) return hipErrorInvalidValue;
    const int T = chain_tile(A.m);
    dim3 grid((A.W[A.m] + T - 1) / T, (A.H[A.m] + T - 1) / T, njobs);
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
    for (int s = 0, m; s + 1 < levels; s += m) {
        PyrChain A{};
        const bool alone = dtype != DGF_U8 && chain_f32_alone(Wl[s], Hl[s]);
        m = alone ? 1 : levels - 1 - s < PC_MAXM ? levels - 1 - s : PC_MAXM;
        A.m = m;
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
