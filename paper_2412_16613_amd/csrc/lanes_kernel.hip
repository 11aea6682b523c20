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

// Two words per 128-thread block: one wave keeps their replicas, the other
// draws the next window.  Where most SIMDs are without a wave, the draws (about
// a third of a window's instructions) then cost the replicas' wave a barrier
// only: 6144 events of 512 words, N_tot = 1024, 679 -> 561 us; 21210 events,
// N_tot = 3535, 2227 -> 1819 us.
template <int NQ, bool FULL>
__global__ __launch_bounds__(128) void wm_lanes_pair_kernel(WmArgs a)
{
    __shared__ __align__(16) uint32_t sq[4][LanesRow<NQ>::HALF];
    __shared__ uint32_t ended[2];
    const uint32_t half = (threadIdx.x >> 5) & 1;
    const bool draws = __builtin_amdgcn_readfirstlane(threadIdx.x >= 64);
    wm_lanes<NQ, FrankReplica<FULL>, true>(a, 2 * (uint64_t)blockIdx.x + half, sq[half], draws,
                                           ended);
}

__global__ __launch_bounds__(256) void wm_lanes_shared_kernel(WmArgs a, uint64_t w0)
{
    wm_lanes_shared<FrankReplica<false>>(a, w0 + 8 * (uint64_t)blockIdx.x + (threadIdx.x >> 5));
}

// Ensembles up to which a block of two waves takes two words: a workgroup per
// CU.  Beyond it the second workgroup of a CU shares its SIMDs; with six quads
// of draws and more that still gains a little up to one wave that keeps
// replicas per SIMD (1024 to 2048 words, N_tot = 1024: 684 -> 659 us; 3535:
// 2244 -> 2169), with fewer it loses (N_tot = 200: 165 -> 173), and past that
// the draws' waves only take issue slots (4096 words, N_tot = 1024: 986 -> 1000).
static bool lanes_in_pairs(const WmArgs &a, int nq)
{
    return a.n_words <= (nq >= 6 ? 2048u : 512u);
}

template <int NQ>
static void lanes_piece(const WmArgs &a, uint64_t i0, dim3 g, hipStream_t s)
{
    const bool full = a.fa >= 0 && a.fi >= 0 && a.cu < 65536u;
    if (lanes_in_pairs(a, NQ)) {
        // one piece holds them all
        const dim3 gp((unsigned)((a.n_words + 1) / 2));
        if (full)
            hipLaunchKernelGGL((wm_lanes_pair_kernel<NQ, true>), gp, dim3(128), 0, s, a);
        else
            hipLaunchKernelGGL((wm_lanes_pair_kernel<NQ, false>), gp, dim3(128), 0, s, a);
    } else if (full) {
        hipLaunchKernelGGL((wm_lanes_kernel<NQ, true>), g, dim3(256), 0, s, a, i0 / 32);
    } else {
        hipLaunchKernelGGL((wm_lanes_kernel<NQ, false>), g, dim3(256), 0, s, a, i0 / 32);
    }
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
