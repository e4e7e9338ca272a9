// parametric_narrow.hip -- the transform's kernel for segments of 1 to 8 lanes:
// large calls of strategies of few stages.  (A code object of its own: beside
// these kernels the others ran 2 us longer a call.)
#include "parametric.h"

namespace dsim {
namespace {

// Bound by the wavefronts in flight (19 to 39 KB of LDS each for the lanes'
// programs, up to 256 registers: four to eight on a CU) and their recording.
// Few blocks that take the wavefronts in turn, each class from its last one
// on (a strategy grid lists microbatch counts ascending), so that a call
// without any pays little for the launch.  A call against 16 lanes a
// candidate, us: 100,000 MLP strategies of one stage and up to 4, 64, 256
// microbatches 389 -> 42, 582 -> 84, 669 -> 126, of up to four stages 388 ->
// 92, 625 -> 234, 777 -> 343; transformer ones 479 -> 55, 687 -> 130, 721 ->
// 201 and 495 -> 148, 749 -> 421, 831 -> 686.
template <bool TF, bool RC, bool ZR, bool OV>
__global__ __launch_bounds__(kLanes) __attribute__((amdgpu_waves_per_eu(ZR ? 1 : 2))) void k_parametric_narrow(const ParArgs g)
{
    const uint32_t n = g.meta[24 + kNarrow];
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) parametric_body<TF, true, RC, ZR, OV>(g, n - 1 - i);
}

template <bool RC, bool ZR, bool OV>
void launch_variant(bool tf, unsigned blocks, hipStream_t s, const ParArgs &g)
{
    if (tf) hipLaunchKernelGGL((k_parametric_narrow<true, RC, ZR, OV>), dim3(blocks), dim3(kLanes), 0, s, g);
    else hipLaunchKernelGGL((k_parametric_narrow<false, RC, ZR, OV>), dim3(blocks), dim3(kLanes), 0, s, g);
}

}  // namespace

// (ZeRO and overlap exclude one another)
void launch_narrow(bool rc, bool zr, bool ov, bool tf, unsigned blocks, hipStream_t s, const ParArgs &g)
{
    if (rc) {
        if (zr) launch_variant<true, true, false>(tf, blocks, s, g);
        else if (ov) launch_variant<true, false, true>(tf, blocks, s, g);
        else launch_variant<true, false, false>(tf, blocks, s, g);
    } else {
        if (zr) launch_variant<false, true, false>(tf, blocks, s, g);
        else if (ov) launch_variant<false, false, true>(tf, blocks, s, g);
        else launch_variant<false, false, false>(tf, blocks, s, g);
    }
}

}  // namespace dsim
