// adjoint_point.hpp -- the implicit adjoint of one tracked point for a support size fixed at compile
// time (device code of adjoint_direct.hip and adjoint_tiled.hip; the equations are in adjoint.hip).
#pragma once

#include "dgf_internal.hpp"

namespace dgf {

// The pair of a batch plan that point i belongs to.
__device__ __forceinline__ int adj_pair_of(const AdjParams &A, int64_t i)
{
    int lo = 0, hi = A.npairs - 1; // last pair whose first point is <= i
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (A.pt_off[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// ---- the adjoint of one point for a support size fixed at compile time ------------------------
//
// The same quantities by the same formulas as k_track_adjoint and k_track_adjoint_illum, split so
// that a wavefront issues as little as possible (VALU issue bounds a launch once its gradient
// cells are combined in LDS): lanes are (column, run of rows) pairs, so vertical neighbours sit in
// one lane's registers and are computed once per row, every row offset is an immediate, and no
// index is divided.  At support 21 three runs of 7 rows make 63 of 64 lanes busy.
template <int S>
struct AdjSplit {
    static constexpr int W0 = S + 3, W1 = S + 1, G = S + 2; // raw I0 patch, raw I1 patch, resampled grid
    static constexpr int Q = (W0 + 3) / 4 * 4;              // LDS row pitch of all three
    // the fields c1 and -psi / 2, interleaved, with a zero border of 2 columns and 3 rows: support
    // (a, b) at column a + 2 of row b + 3
    static constexpr int PF = S + 4;
    static constexpr int runs(int n) { return 64 / n < n ? 64 / n : n; } // runs of rows of an n-column field
    static constexpr int rows(int n, int h) { return (h + runs(n) - 1) / runs(n); } // rows of one run
    static constexpr int up(int h, int r) { return (h + r - 1) / r * r; }
    static constexpr int RS = rows(S, S), RG = rows(G, G), R0 = rows(W0, W0), R1 = rows(W1, W1);
    // rows a full last run touches beyond the field are allocated (what is read there is discarded)
    static constexpr int field_rows = up(W0, R0) + 3 > up(W1, R1) + 3 ? up(W0, R0) + 3 : up(W1, R1) + 3;
    static constexpr int grid_rows = up(S, RS) + 2 > G ? up(S, RS) + 2 : G;
    static constexpr int raw1_rows = up(S, RS) + 1 > W1 ? up(S, RS) + 1 : W1;
    static constexpr int raw0_rows = up(G, RG) + 1 > W0 ? up(G, RG) + 1 : W0;
    static constexpr int patch_floats = (raw0_rows + (raw1_rows > grid_rows ? raw1_rows : grid_rows)) * Q;
    static constexpr int field_floats = (2 * PF * field_rows + 3) / 4 * 4;
    static constexpr int floats = patch_floats > field_floats ? patch_floats : field_floats; // per wavefront
};

// The lane's left / right neighbour's value (whole-wavefront shift by one lane; 0 comes in).
__device__ __forceinline__ float lane_left(float v) { return dpp<0x138>(v); }
__device__ __forceinline__ float lane_right(float v) { return dpp<0x130>(v); }

// Cells of one gradient map that a lane holds: column X, rows Y0 .. Y0 + R - 1 of a patch with
// top-left cell (ox, oy) and `rows` rows (WHOLE: a multiple of R), added to the map in device memory
// at their clamped positions.
template <int R, bool WHOLE>
__device__ __forceinline__ void add_cells_device(float *map, int64_t pitch, int W, int H, int ox, int oy, int X, int Y0,
                                                 int rows, const float (&v)[R], bool on)
{
    if (!on) return;
    float *col = map + clampi(ox + X, 0, W - 1);
#pragma unroll
    for (int k = 0; k < R; ++k)
        if ((WHOLE || Y0 + k < rows) && v[k] != 0.f) unsafeAtomicAdd(col + (int64_t)clampi(oy + Y0 + k, 0, H - 1) * pitch, v[k]);
}

// The same into a tile in LDS (row pitch `pitch`) that holds the whole patch from cell (ox, oy) and
// is shared by the wavefronts of a workgroup: reads, adds and writes under the tile's lock.  (LDS
// float atomics take about 3 cycles a lane on this chip: 145 cycles for a 48-lane ds_add_f32, where
// a 12-row read and write of the same lanes takes 7 a row.)  The wait for the lock ends: its holder
// only reads and writes LDS before it lets go, and every wavefront takes it a bounded number of times.
template <int R, bool WHOLE>
__device__ __forceinline__ void add_cells_tile(float *tile, int *lock, int pitch, int ox, int oy, int X, int Y0, int rows,
                                               const float (&v)[R], bool on, int li)
{
    float *at = tile + (oy + Y0) * pitch + ox + X;
    // one lane tries for the whole wavefront; the read-first-lane keeps the others from running ahead
    // (the lock is the wavefront's, which a lane's own control flow does not show the compiler)
    for (;;) {
        int held = 1;
        if (li == 0) held = atomicCAS(lock, 0, 1);
        if (__builtin_amdgcn_readfirstlane(held) == 0) break;
        __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if (on) {
        float t[R];
#pragma unroll
        for (int k = 0; k < R; ++k) t[k] = WHOLE || Y0 + k < rows ? at[k * pitch] : 0.f;
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (WHOLE || Y0 + k < rows) at[k * pitch] = t[k] + v[k];
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (li == 0) __hip_atomic_store(lock, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Where a point's patches lie: integer bases and shared fractions of the template samples (p + k)
// and of the I1 samples (p + k + u).
struct AdjPlace {
    float fx0, fy0, fx1, fy1;
    int ox0, oy0, ox1, oy1; // dI0 patch origin ((s + 3)^2 cells), dI1 patch origin ((s + 1)^2)
};

__device__ __forceinline__ AdjPlace adj_place(float2 p, float2 u, int r)
{
    AdjPlace a;
    const float pbx = floorf(p.x), pby = floorf(p.y);
    a.fx0 = p.x - pbx;
    a.fy0 = p.y - pby;
    const float tx = a.fx0 + u.x, ty = a.fy0 + u.y;
    const float qbx = floorf(tx), qby = floorf(ty);
    a.fx1 = tx - qbx;
    a.fy1 = ty - qby;
    a.ox0 = (int)pbx - r - 1;
    a.oy0 = (int)pby - r - 1;
    a.ox1 = (int)pbx + (int)fminf(fmaxf(qbx, -1048576.f), 1048576.f) - r;
    a.oy1 = (int)pby + (int)fminf(fmaxf(qby, -1048576.f), 1048576.f) - r;
    return a;
}

// 4x4 system M^T x = v by Gaussian elimination with partial pivoting, fully unrolled (M row-major,
// both copied); x is not finite when a pivot is zero.
__device__ __forceinline__ void solve4_transposed(const float *M, const float *v, float *x)
{
    float a[4][5];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int c = 0; c < 4; ++c) a[r][c] = M[c * 4 + r];
        a[r][4] = v[r];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        // pivot: largest |a[r][c]| for r >= c, brought to row c by selects (no dynamic indexing)
#pragma unroll
        for (int r = c + 1; r < 4; ++r) {
            const bool sw = fabsf(a[r][c]) > fabsf(a[c][c]);
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const float t = a[c][k];
                a[c][k] = sw ? a[r][k] : t;
                a[r][k] = sw ? t : a[r][k];
            }
        }
        const float inv = 1.f / a[c][c];
#pragma unroll
        for (int r = c + 1; r < 4; ++r) {
            const float f = a[r][c] * inv;
#pragma unroll
            for (int k = c; k < 5; ++k) a[r][k] = fmaf(-f, a[c][k], a[r][k]);
        }
    }
#pragma unroll
    for (int r = 3; r >= 0; --r) {
        float acc = a[r][4];
#pragma unroll
        for (int k = r + 1; k < 4; ++k) acc = fmaf(-a[r][k], x[k], acc);
        x[r] = acc / a[r][r];
    }
}

// One wavefront computes the adjoint of the converged point i (wave-uniform).  `lds` is the
// wavefront's own AdjSplit<S>::floats floats, 16-byte aligned.  Where fit0 / fit1 is set the
// point's dI0 / dI1 cells go to the LDS tile tile0 / tile1 (pitch tp0 / tp1) whose cell (0, 0) is
// image cell (tx0, ty0) / (tx1, ty1), otherwise to the gradient map in device memory.
struct AdjSink {
    float *tile0, *tile1;
    int *lock0, *lock1;
    const AdjPair *pair; // the point's pair in device memory, for the maps' addresses (null: as given)
    int tp0, tp1, tx0, ty0, tx1, ty1;
    bool fit0, fit1;
};

// The pair descriptor, read where the maps in device memory are written and not before (the compiler
// would otherwise hold their addresses in scalar registers through the whole point, and spill).
__device__ __forceinline__ const AdjPair *map_of(const AdjPair *p)
{
    asm volatile("" : "+s"(p));
    return p;
}

template <typename PixT, int S, bool IM, bool DP>
__device__ __forceinline__ void adjoint_point(const AdjParams &A, const AdjPair &Pr, int64_t i, const AdjPlace &pl,
                                              float *lds, int li, const AdjSink &K)
{
    typedef AdjSplit<S> D;
    constexpr int W0 = D::W0, W1 = D::W1, G = D::G, Q = D::Q, PF = D::PF, R = D::RS;
    constexpr float kInvN = 1.f / (float)(S * S);
    const float2 lam = reinterpret_cast<const float2 *>(A.dflow)[i];
    const int W = Pr.W, H = Pr.H;
    const float fx0 = pl.fx0, fy0 = pl.fy0, fx1 = pl.fx1, fy1 = pl.fy1;
    float g1m = 1.f, moff = 0.f;
    if constexpr (IM) {
        const float2 mc = reinterpret_cast<const float2 *>(A.illum)[i];
        g1m = 1.f + mc.x;
        moff = mc.y;
    }

    float *raw0 = lds, *raw1 = lds + D::raw0_rows * Q, *grid = raw1; // (the grid replaces the raw I1 patch)
    wave_sync(); // the wavefront's reads of its last point are done
    stage_tile<64, PixT, (W0 + 7) / 8, (W0 + 7) / 8, W0>(raw0, Q, Pr.I0, Pr.pitch0, W, H, pl.ox0, pl.oy0, W0, W0, li);
    stage_tile<64, PixT, (W1 + 7) / 8, (W1 + 7) / 8, W1>(raw1, Q, Pr.I1, Pr.pitch1, W, H, pl.ox1, pl.oy1, W1, W1, li);
    wave_sync();

    // support pixels of the lane: column cs, rows ys .. ys + R - 1
    const int rs = li / S, cs0 = li - rs * S;
    const bool lane_on = rs * R < S;
    const int cs = lane_on ? cs0 : 0, ys = lane_on ? rs * R : 0;
    // (where the runs tile the column, an idle lane holds pixels of run 0 and is told apart by its
    // zero gradients alone)
    constexpr bool tiles = S % R == 0;
    auto in_support = [&](int k) { return tiles ? lane_on : lane_on && ys + k < S; };
    auto usable = [&](int k) { return tiles || in_support(k); }; // holds pixel values, not overrun

    // I1 sample and its gradient: horizontal lerps once per row, then the vertical ones
    float g0[R], g1[R], djx[R], djy[R], res[R], ps[R], dps[R], T[R];
    {
        const float *q = raw1 + ys * Q + cs;
        float a[R + 1], b[R + 1], h[R + 1];
#pragma unroll
        for (int k = 0; k <= R; ++k) {
            a[k] = q[k * Q];
            b[k] = q[k * Q + 1];
            h[k] = fmaf(fx1, b[k] - a[k], a[k]);
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            res[k] = fmaf(fy1, h[k + 1] - h[k], h[k]);
            djx[k] = (1.f - fy1) * (b[k] - a[k]) + fy1 * (b[k + 1] - a[k + 1]);
            djy[k] = (1.f - fx1) * (a[k + 1] - a[k]) + fx1 * (b[k + 1] - b[k]);
        }
    }
    wave_sync();
    // the resampled I0 patch on the (S + 2)^2 grid of support offsets -r - 1 .. r + 1
    {
        const int rg = li / G, cg = li - rg * G, yg = rg * D::RG;
        if (yg < G) {
            const float *q = raw0 + yg * Q + cg;
            float *o = grid + yg * Q + cg;
            float h0 = fmaf(fx0, q[1] - q[0], q[0]);
#pragma unroll
            for (int k = 0; k < D::RG; ++k) {
                const float h1 = fmaf(fx0, q[(k + 1) * Q + 1] - q[(k + 1) * Q], q[(k + 1) * Q]);
                if (yg + k < G) o[k * Q] = fmaf(fy0, h1 - h0, h0);
                h0 = h1;
            }
        }
    }
    wave_sync();
    {
        const float *gc = grid + (ys + 1) * Q + cs + 1;
        float c[R + 2];
#pragma unroll
        for (int k = 0; k < R + 2; ++k) c[k] = gc[(k - 1) * Q];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const float half = in_support(k) ? 0.5f : 0.f;
            T[k] = c[k + 1];
            g0[k] = usable(k) ? half * (gc[k * Q + 1] - gc[k * Q - 1]) : 0.f;
            g1[k] = usable(k) ? half * (c[k + 2] - c[k]) : 0.f;
            res[k] = IM ? res[k] - g1m * T[k] - moff : res[k] - T[k];
        }
    }
    float Tm = 0.f, iTs = 1.f; // illumination model: the centred, scaled template T' = (T - Tm) iTs
    if constexpr (IM) {
        float sT = 0.f, sTT = 0.f, z0 = 0.f, z1 = 0.f, z2 = 0.f;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const float t = in_support(k) ? T[k] : 0.f;
            sT += t;
            sTT = fmaf(t, t, sTT);
        }
        wave_sum5(sT, sTT, z0, z1, z2);
        Tm = sT * kInvN;
        float Ts = sqrtf(fmaxf(sTT * kInvN - Tm * Tm, 0.f));
        if (!(Ts > 1e-6f)) Ts = 1.f;
        iTs = 1.f / Ts;
#pragma unroll
        for (int k = 0; k < R; ++k) T[k] = in_support(k) ? (T[k] - Tm) * iTs : 0.f;
    }

    // psi and psi' of every pixel
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const float a = fabsf(res[k]);
        const bool inner = A.mode == ROBUST_L2 || a <= A.s1, outer = A.mode == ROBUST_HARD || a >= A.s2;
        const float mid = copysignf(-A.dpsi_mid * (A.s2 - a), res[k]);
        ps[k] = inner ? res[k] : outer ? 0.f : mid;
        dps[k] = inner ? 1.f : outer ? 0.f : A.dpsi_mid;
        if (IM || DP || !tiles) {
            ps[k] = in_support(k) ? ps[k] : 0.f;
            dps[k] = in_support(k) ? dps[k] : 0.f;
        }
    }
    // psi(r) / r for the test below.  An idle lane's pixels are run 0's (see above): a residual of zero
    // among them would give 0 / 0 where ps and dps are cleared outside the support, so they weigh 1.
    auto weight = [&](int k) {
        return dps[k] == 1.f || !in_support(k) ? 1.f : ps[k] / res[k];
    };
    // the least-squares equations' psi
    auto least_squares = [&]() {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            ps[k] = in_support(k) ? res[k] : 0.f;
            dps[k] = in_support(k) ? 1.f : 0.f;
        }
    };

    // gradient of the bilinear interpolant of I0 inside the cell at local (lx, ly)
    auto I0g = [&](int lx, int ly, float &gx, float &gy) {
        const float *q = raw0 + ly * Q + lx;
        gx = (1.f - fy0) * (q[1] - q[0]) + fy0 * (q[Q + 1] - q[Q]);
        gy = (1.f - fx0) * (q[Q] - q[0]) + fx0 * (q[Q + 1] - q[1]);
    };

    // pass 1: the system matrix, the point dependence K with DP, and the solve (see k_track_adjoint
    // and k_track_adjoint_illum); then the fields' coefficients: dI0 gathers
    // ka c1 + kb h + mx (h(x - 1) - h(x + 1)) + my (h(y - 1) - h(y + 1)) with h = -psi / 2
    float ka = 1.f, kb = 0.f, mx, my;
    float c1[R];
    if constexpr (IM) {
        if (A.mode != ROBUST_L2) {
            // the norm of the equation the forward pass stopped on: where its weighted system falls
            // back at the converged parameters (its determinant at most 1e-6 of the unweighted one's,
            // or not a number) the fixed point solves the least-squares equations
            float M[10], M0[10];
#pragma unroll
            for (int e = 0; e < 10; ++e) M[e] = M0[e] = 0.f;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const float w = in_support(k) ? weight(k) : 0.f;
                const float ph[4] = {g1m * g0[k], g1m * g1[k], -T[k], in_support(k) ? -1.f : 0.f};
                int e = 0;
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int b = a; b < 4; ++b, ++e) {
                        M[e] = fmaf(w * ph[a], ph[b], M[e]);
                        M0[e] = fmaf(ph[a], ph[b], M0[e]);
                    }
            }
            wave_sum5(M[0], M[1], M[2], M[3], M[4]);
            wave_sum5(M[5], M[6], M[7], M[8], M[9]);
            wave_sum5(M0[0], M0[1], M0[2], M0[3], M0[4]);
            wave_sum5(M0[5], M0[6], M0[7], M0[8], M0[9]);
            if (!(ldl4(M, nullptr, nullptr) > 1e-6f * ldl4(M0, nullptr, nullptr))) least_squares();
        }
        float Kp[8], Am[16];
#pragma unroll
        for (int e = 0; e < 8; ++e) Kp[e] = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) Am[e] = 0.f;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const float ph[4] = {g1m * g0[k], g1m * g1[k], -T[k], -1.f};
            const float dr[4] = {djx[k], djy[k], -T[k], -1.f};
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    Am[a * 4 + b] = fmaf(dps[k] * ph[a], usable(k) ? dr[b] : 0.f, Am[a * 4 + b]);
            if constexpr (DP) {
                if (in_support(k)) {
                    const int lx = cs + 1, ly = ys + k + 1;
                    float tgx, tgy, pxx, pxy, mxx, mxy, pyx, pyy, myx, myy;
                    I0g(lx, ly, tgx, tgy);
                    I0g(lx + 1, ly, pxx, pxy);
                    I0g(lx - 1, ly, mxx, mxy);
                    I0g(lx, ly + 1, pyx, pyy);
                    I0g(lx, ly - 1, myx, myy);
                    const float cg = -g1m * dps[k], hp = 0.5f * g1m * ps[k];
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        Kp[2 * a] = fmaf(cg * ph[a], tgx, Kp[2 * a]);
                        Kp[2 * a + 1] = fmaf(cg * ph[a], tgy, Kp[2 * a + 1]);
                    }
                    Kp[0] = fmaf(hp, pxx - mxx, Kp[0]);
                    Kp[1] = fmaf(hp, pxy - mxy, Kp[1]);
                    Kp[2] = fmaf(hp, pyx - myx, Kp[2]);
                    Kp[3] = fmaf(hp, pyy - myy, Kp[3]);
                    Kp[4] = fmaf(-ps[k] * iTs, tgx, Kp[4]);
                    Kp[5] = fmaf(-ps[k] * iTs, tgy, Kp[5]);
                }
            }
        }
        float z0 = 0.f, z1 = 0.f;
        wave_sum5(Am[0], Am[1], Am[2], Am[3], Am[4]);
        wave_sum5(Am[5], Am[6], Am[7], Am[8], Am[9]);
        wave_sum5(Am[10], Am[11], Am[12], Am[13], Am[14]);
        Am[15] = group_sum<64>(Am[15]);
        if constexpr (DP) {
            wave_sum5(Kp[0], Kp[1], Kp[2], Kp[3], Kp[4]);
            wave_sum5(Kp[5], Kp[6], Kp[7], z0, z1);
        }
        const float v[4] = {lam.x, lam.y, 0.f, 0.f};
        float mu[4];
        solve4_transposed(Am, v, mu);
        if (!(isfinite(mu[0]) && isfinite(mu[1]) && isfinite(mu[2]) && isfinite(mu[3]))) return; // uniform
        if constexpr (DP)
            if (li == 0)
                reinterpret_cast<float2 *>(A.dpoints)[i] =
                    make_float2(-lam.x - (Kp[0] * mu[0] + Kp[2] * mu[1] + Kp[4] * mu[2] + Kp[6] * mu[3]),
                                -lam.y - (Kp[1] * mu[0] + Kp[3] * mu[1] + Kp[5] * mu[2] + Kp[7] * mu[3]));
#pragma unroll
        for (int k = 0; k < R; ++k)
            c1[k] = dps[k] * (g1m * (mu[0] * g0[k] + mu[1] * g1[k]) - mu[2] * T[k] - mu[3]);
        ka = g1m;
        kb = -2.f * mu[2] * iTs;
        mx = g1m * mu[0];
        my = g1m * mu[1];
    } else {
        float J00, J01, J10, J11, z = 0.f;
        auto matrix = [&]() { // J = sum psi' g (grad J)^T, the lane's part
            J00 = J01 = J10 = J11 = 0.f;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const float e0 = dps[k] * g0[k], e1 = dps[k] * g1[k];
                const float jx = usable(k) ? djx[k] : 0.f, jy = usable(k) ? djy[k] : 0.f;
                J00 = fmaf(e0, jx, J00);
                J01 = fmaf(e0, jy, J01);
                J10 = fmaf(e1, jx, J10);
                J11 = fmaf(e1, jy, J11);
            }
        };
        matrix();
        if (A.mode != ROBUST_L2) {
            // the norm of the equation the forward pass stopped on (as above, on the 2 x 2 system)
            float a = 0.f, b = 0.f, c = 0.f, a0 = 0.f, b0 = 0.f, c0 = 0.f;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const float w = weight(k);
                const float wx = w * g0[k], wy = w * g1[k];
                a = fmaf(wx, g0[k], a);
                b = fmaf(wx, g1[k], b);
                c = fmaf(wy, g1[k], c);
                a0 = fmaf(g0[k], g0[k], a0);
                b0 = fmaf(g0[k], g1[k], b0);
                c0 = fmaf(g1[k], g1[k], c0);
            }
            wave_sum5(a, b, c, a0, b0);
            wave_sum5(J00, J01, c0, J10, J11);
            if (!(fmaf(a, c, -b * b) > 1e-6f * fmaf(a0, c0, -b0 * b0))) {
                least_squares();
                matrix();
                wave_sum5(J00, J01, z, J10, J11);
            }
        } else {
            wave_sum5(J00, J01, z, J10, J11);
        }
        float K00 = 0.f, K01 = 0.f, K10 = 0.f, K11 = 0.f;
        if constexpr (DP) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                if (in_support(k)) {
                    const float e0 = dps[k] * g0[k], e1 = dps[k] * g1[k];
                    const int lx = cs + 1, ly = ys + k + 1;
                    float tgx, tgy, pxx, pxy, mxx, mxy, pyx, pyy, myx, myy;
                    I0g(lx, ly, tgx, tgy);
                    I0g(lx + 1, ly, pxx, pxy);
                    I0g(lx - 1, ly, mxx, mxy);
                    I0g(lx, ly + 1, pyx, pyy);
                    I0g(lx, ly - 1, myx, myy);
                    K00 += -e0 * tgx + 0.5f * ps[k] * (pxx - mxx);
                    K01 += -e0 * tgy + 0.5f * ps[k] * (pxy - mxy);
                    K10 += -e1 * tgx + 0.5f * ps[k] * (pyx - myx);
                    K11 += -e1 * tgy + 0.5f * ps[k] * (pyy - myy);
                }
            }
            wave_sum5(K00, K01, z, K10, K11);
        }
        const float det = J00 * J11 - J01 * J10;
        if (!(det != 0.f) || !isfinite(det)) return; // uniform across the wave
        const float mux = (J11 * lam.x - J10 * lam.y) / det;
        const float muy = (J00 * lam.y - J01 * lam.x) / det;
        if constexpr (DP)
            if (li == 0)
                reinterpret_cast<float2 *>(A.dpoints)[i] =
                    make_float2(-lam.x - (K00 * mux + K10 * muy), -lam.y - (K01 * mux + K11 * muy));
#pragma unroll
        for (int k = 0; k < R; ++k) c1[k] = dps[k] * (mux * g0[k] + muy * g1[k]);
        mx = mux;
        my = muy;
    }

    // the fields, over the patches (no longer read)
    wave_sync();
    float4 *z4 = reinterpret_cast<float4 *>(lds);
    for (int c = li; c < D::field_floats / 4; c += 64) z4[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    wave_sync();
    float2 *field = reinterpret_cast<float2 *>(lds);
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (in_support(k)) field[(ys + k + 3) * PF + cs + 2] = make_float2(c1[k], -0.5f * ps[k]);
    wave_sync();

    // dI1 cells: minus the 4 bilinear taps of c1, the horizontal pair once per row.  The left tap
    // of column 0 is the previous run's last column, a border column, so zero.
    {
        constexpr int R1 = D::R1;
        const int rr = li / W1, x0 = li - rr * W1;
        const bool on = rr * R1 < W1;
        const int X = on ? x0 : 0, Y0 = on ? rr * R1 : 0;
        const float2 *e = field + (Y0 + 2) * PF + X + 2;
        float v[R1], up = 0.f;
#pragma unroll
        for (int k = 0; k <= R1; ++k) {
            const float c = e[k * PF].x;
            const float h = (1.f - fx1) * c + fx1 * lane_left(c);
            if (k > 0) v[k - 1] = -((1.f - fy1) * h + fy1 * up);
            up = h;
        }
        if (K.fit1)
            add_cells_tile<R1, W1 % R1 == 0>(K.tile1, K.lock1, K.tp1, pl.ox1 - K.tx1, pl.oy1 - K.ty1, X, Y0, W1, v, on, li);
        else {
            const AdjPair M = K.pair ? *map_of(K.pair) : Pr;
            add_cells_device<R1, W1 % R1 == 0>(A.grad1 + M.g1, M.gpitch1, W, H, pl.ox1, pl.oy1, X, Y0, W1, v, on);
        }
    }
    // dI0 cells: the 4 bilinear taps of F; with C and P the horizontal pairs of c1 and h at a cell's
    // columns, F's pair is ka C + kb P + mx (P(X - 1) - P(X + 1)) + my (P(y - 1) - P(y + 1)).
    // P of columns 0 and W0 - 1 is zero, so the lane shifts bring zeros in across runs.
    {
        constexpr int R0 = D::R0;
        const int rr = li / W0, x0 = li - rr * W0;
        const bool on = rr * R0 < W0;
        const int X = on ? x0 : 0, Y0 = on ? rr * R0 : 0;
        const float2 *e = field + Y0 * PF + X + 1; // field row Y0 is support row Y0 - 3
        float v[R0], Cm = 0.f, Pm = 0.f, Pp = 0.f, Dm = 0.f, up = 0.f;
#pragma unroll
        for (int k = 0; k < R0 + 3; ++k) {
            const float2 f = e[k * PF];
            const float C = (1.f - fx0) * f.x + fx0 * lane_left(f.x);
            const float P = (1.f - fx0) * f.y + fx0 * lane_left(f.y);
            const float Dx = lane_left(P) - lane_right(P);
            if (k >= 2) { // F's pair of row k - 1, from rows k - 2, k - 1 and k
                float F = fmaf(mx, Dm, fmaf(my, Pm - P, IM ? fmaf(ka, Cm, kb * Pp) : Cm));
                if (k >= 3) v[k - 3] = (1.f - fy0) * F + fy0 * up;
                up = F;
            }
            Cm = C;
            Pm = Pp;
            Pp = P;
            Dm = Dx;
        }
        if (K.fit0)
            add_cells_tile<R0, W0 % R0 == 0>(K.tile0, K.lock0, K.tp0, pl.ox0 - K.tx0, pl.oy0 - K.ty0, X, Y0, W0, v, on, li);
        else {
            const AdjPair M = K.pair ? *map_of(K.pair) : Pr;
            add_cells_device<R0, W0 % R0 == 0>(A.grad0 + M.g0, M.gpitch0, W, H, pl.ox0, pl.oy0, X, Y0, W0, v, on);
        }
    }
}

// Support sizes compiled (those of the row-run tracker).
#define DGF_ADJOINT_SUPPORTS(X) X(5) X(7) X(9) X(11) X(15) X(21)

} // namespace dgf
