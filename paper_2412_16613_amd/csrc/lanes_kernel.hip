// The lanes engine's launches: one replica per thread, Frank-family networks.

#include "lanes_device.h"

namespace bwg {

// 8 words per 256-thread block, NQ quads of threshold planes; the launch's
// piece starts at word w0.
template <int NQ, bool FULL>
__global__ __launch_bounds__(256) void wm_lanes_kernel(WmArgs a, uint64_t w0)
{
    __shared__ __align__(16) uint32_t sq[8][LanesRow<NQ>::HALF];
    const int half = threadIdx.x >> 5;
    wm_lanes<NQ, FrankReplica<FULL>>(a, w0 + 8 * (uint64_t)blockIdx.x + half, sq[half]);
}

__global__ __launch_bounds__(256) void wm_lanes_shared_kernel(WmArgs a, uint64_t w0)
{
    wm_lanes_shared<FrankReplica<false>>(a, w0 + 8 * (uint64_t)blockIdx.x + (threadIdx.x >> 5));
}

template <int NQ>
static void lanes_piece(const WmArgs &a, uint64_t i0, dim3 g, hipStream_t s)
{
    if (a.fa >= 0 && a.fi >= 0 && a.cu < 65536u)
        hipLaunchKernelGGL((wm_lanes_kernel<NQ, true>), g, dim3(256), 0, s, a, i0 / 32);
    else
        hipLaunchKernelGGL((wm_lanes_kernel<NQ, false>), g, dim3(256), 0, s, a, i0 / 32);
}

hipError_t launch_wm_lanes(const WmArgs &a, hipStream_t s)
{
    using Piece = void (*)(const WmArgs &, uint64_t, dim3, hipStream_t);
    static const Piece kPieces[8] = {lanes_piece<1>, lanes_piece<2>, lanes_piece<3>,
                                     lanes_piece<4>, lanes_piece<5>, lanes_piece<6>,
                                     lanes_piece<7>, lanes_piece<8>};
    if (a.B < 1 || a.B > 32) return hipErrorInvalidValue;
    // one work-item per replica slot: pieces of kLaunchSpan / 32 words
    return launch_pieces(32 * a.n_words, 256, [&](uint64_t i0, dim3 g) {
        if (a.zs)
            hipLaunchKernelGGL(wm_lanes_shared_kernel, g, dim3(256), 0, s, a, i0 / 32);
        else
            kPieces[(a.B - 1) / 4](a, i0, g, s);
    });
}

}  // namespace bwg
