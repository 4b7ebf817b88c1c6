// detect.hip -- DeGraF key-point detection on gfx950.
//
// One key-point per window of a uniform grid (DeGraF-Flow, Section 2 "Point detection"):
// positive centroid from the intensity-weighted moments (Eq. 1), negative centroid from the
// inverted weights 1 + m - I with m the window maximum (Eq. 2), and the centroid with the larger
// weight sum is kept (strictly larger for the negative one).
//
// The image is read once from HBM: a workgroup owns a block of windows and stages the pixel
// rectangle they cover into LDS four bytes per lane (aligned dword pairs).  Where windows overlap
// much the sums over each window row are taken once and shared (detect_tile_rows), elsewhere each
// lane reduces its own window (detect_tile); both take four pixels per step with byte dot products.
// Only the positive moments are accumulated; the negative ones follow exactly from
// sum (1 + m - I) = (1 + m) w h - sum I (and likewise for the moments).
//
// A small grid is bound by latency (launch, one round of staging, the sums: about 5 us), a dense
// one by the instructions of staging and sums: window 9, stride 2 at 2048x1024, 520k windows, takes 7.4 us where
// a byte per step for every window took 12.9; stride 1 15 against 41; window 9, stride 8 at 1242x375 5.0 against
// 10.0 (smaller tiles).
#include "dgf_internal.hpp"

namespace dgf {

// LDS of one 16 x 16-window tile: rows of (15 stride + win) bytes at a pitch rounded up to 4
size_t detect_tile_lds(int win, int stride)
{
    return (size_t)((15 * stride + win + 3) & ~3) * (size_t)(15 * stride + win);
}

// Tiles of 16 x 16 windows that take more than two rounds of loads (8 KB: eight dwords per lane of
// 256) are cut into 8 x 8, one or two rounds each: 1242x375, window 9, stride 8, 8.8 -> 5.1 us.
int detect_tile_side(int win, int stride) { return detect_tile_lds(win, stride) > 8 * 1024 ? 8 : 16; }

template <int TX, int TY>
__global__ __launch_bounds__(256) void k_detect_tiled(const uint8_t *__restrict__ img, int64_t pitch, int W, int H,
                                                          int win, int stride, int nx, int ny, DetectOut o)
{
    extern __shared__ __align__(16) uint8_t tile[];
    detect_tile<TX, TY>(tile, (int)blockIdx.x, (int)blockIdx.y, img, pitch, W, H, win, stride, nx, ny, 0, o);
}

__global__ __launch_bounds__(256) void k_detect_rows(const uint8_t *__restrict__ img, int64_t pitch, int W, int H, int win,
                                                     int stride, int nx, int ny, DetectOut o)
{
    extern __shared__ __align__(16) uint8_t tile[];
    with_window(win, [&](auto nd, auto w) {
        detect_tile_rows<nd.value, w.value>(tile, (int)blockIdx.x, (int)blockIdx.y, img, pitch, W, H, win, stride, nx, ny, 0, o);
    });
}

// Direct form for windows too large to tile: one lane per window, reads through the cache.
__global__ __launch_bounds__(256) void k_detect_direct(const uint8_t *__restrict__ img, int64_t pitch, int win,
                                                        int stride, int nx, int64_t N, DetectOut o)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    const int kx = (int)(n % nx), ky = (int)(n / nx);
    const int x0 = kx * stride, y0 = ky * stride;
    int S = 0, Mi = 0, Mj = 0, m = 0;
    for (int i = 0; i < win; ++i) {
        const uint8_t *row = img + (int64_t)(y0 + i) * pitch + x0;
        int rs = 0, rj = 0;
        for (int j = 0; j < win; ++j) {
            const int v = row[j];
            rs += v;
            rj += j * v;
            m = max(m, v);
        }
        S += rs;
        Mi += i * rs;
        Mj += rj;
    }
    finish_window(S, Mi, Mj, m, win, x0, y0, n, o);
}

hipError_t launch_detect(const uint8_t *img, int64_t pitch, int W, int H, int win, int stride, float *pts,
                         uint8_t *sel, float *resp, hipStream_t st)
{
    const int nx = (W - win) / stride + 1, ny = (H - win) / stride + 1;
    DetectOut o{pts, sel, resp};
    const int64_t RW = (int64_t)15 * stride + win, RH = RW;
    const int64_t RP = (RW + 3) & ~(int64_t)3;
    const int high = detect_rows_high(stride);
    const bool many = (int64_t)((nx + 15) / 16) * ((ny + high - 1) / high) >= 256;
    if (detect_by_rows(win, stride, many) && detect_rows_lds(win, stride) <= kMaxLdsPerBlock) {
        dim3 grid((nx + 15) / 16, (ny + high - 1) / high);
        hipLaunchKernelGGL(k_detect_rows, grid, dim3(256), detect_rows_lds(win, stride), st, img, pitch, W, H, win, stride, nx, ny, o);
    } else if (RP * RH <= 48 * 1024) {
        const int side = detect_tile_side(win, stride), R = (side - 1) * stride + win;
        const auto k = side == 8 ? k_detect_tiled<8, 8> : k_detect_tiled<16, 16>;
        hipLaunchKernelGGL(k, dim3((nx + side - 1) / side, (ny + side - 1) / side), dim3(256),
                           (size_t)(((R + 3) & ~3) * R), st, img, pitch, W, H, win, stride, nx, ny, o);
    } else {
        const int64_t N = (int64_t)nx * ny;
        hipLaunchKernelGGL(k_detect_direct, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, img, pitch, win,
                           stride, nx, N, o);
    }
    return hipGetLastError();
}

} // namespace dgf
