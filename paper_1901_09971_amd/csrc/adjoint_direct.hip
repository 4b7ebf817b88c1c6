// adjoint_direct.hip -- the adjoint at a support fixed at compile time, one wavefront per point, its
// gradient cells added to the maps in device memory: the points of a float32 pair, which come in any
// order, and those of a uint8 batch plan too sparse for tiles (adjoint_tiled.hip).
#include "adjoint_point.hpp"

namespace dgf {

// One wavefront per point, its gradient cells added to the maps one by one.
template <typename PixT, int S, bool IM, bool DP>
__global__ __launch_bounds__(64) void k_track_adjoint_fixed(AdjParams A)
{
    extern __shared__ __align__(16) float smem[];
    const int li = threadIdx.x;
    const int64_t i = (int64_t)(((uint64_t)blockIdx.x * (uint64_t)A.perm_mul) % (uint64_t)A.n);
    if (DP && li == 0) reinterpret_cast<float2 *>(A.dpoints)[i] = make_float2(0.f, 0.f);
    if (A.status[i] != DGF_ST_CONVERGED) return;
    const AdjPlace pl = adj_place(reinterpret_cast<const float2 *>(A.pts)[i], reinterpret_cast<const float2 *>(A.flow)[i],
                                  S / 2);
    if constexpr (sizeof(PixT) == 1)
        adjoint_point<PixT, S, IM, DP>(A, A.pairs[__builtin_amdgcn_readfirstlane(adj_pair_of(A, i))], i, pl, smem, li,
                                       AdjSink{});
    else
        adjoint_point<PixT, S, IM, DP>(A, A.one, i, pl, smem, li, AdjSink{});
}


template <int S>
static hipError_t launch_direct(const AdjParams &A, hipStream_t st)
{
    const dim3 grid((unsigned)A.n), block(64);
    const size_t lds = sizeof(float) * AdjSplit<S>::floats;
    if (A.npairs) { // (batch plans hold uint8 frames and take no point gradients)
        if (A.illum)
            hipLaunchKernelGGL((k_track_adjoint_fixed<uint8_t, S, true, false>), grid, block, lds, st, A);
        else
            hipLaunchKernelGGL((k_track_adjoint_fixed<uint8_t, S, false, false>), grid, block, lds, st, A);
    } else if (A.illum) {
        if (A.dpoints)
            hipLaunchKernelGGL((k_track_adjoint_fixed<float, S, true, true>), grid, block, lds, st, A);
        else
            hipLaunchKernelGGL((k_track_adjoint_fixed<float, S, true, false>), grid, block, lds, st, A);
    } else if (A.dpoints)
        hipLaunchKernelGGL((k_track_adjoint_fixed<float, S, false, true>), grid, block, lds, st, A);
    else
        hipLaunchKernelGGL((k_track_adjoint_fixed<float, S, false, false>), grid, block, lds, st, A);
    return hipGetLastError();
}

bool adjoint_support_compiled(int s)
{
#define DGF_CASE(S_) if (s == S_) return true;
    DGF_ADJOINT_SUPPORTS(DGF_CASE)
#undef DGF_CASE
    return false;
}

hipError_t launch_adjoint_direct(const AdjParams &A, hipStream_t st)
{
#define DGF_CASE(S_) if (A.s == S_) return launch_direct<S_>(A, st);
    DGF_ADJOINT_SUPPORTS(DGF_CASE)
#undef DGF_CASE
    return hipErrorInvalidValue;
}

} // namespace dgf
