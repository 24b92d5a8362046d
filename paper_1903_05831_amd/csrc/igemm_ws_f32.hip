// Split-role implicit GEMM on binary32 tensors (igemm_ws_body.h with F32): forward and data gradient of the
// single-precision path; tiles and their choice: conv_f32.hip.
#include "igemm_ws_body.h"

namespace sdconv {

// Bound by the matrix pipe (64 cycles for 4096 FLOP), so a tile needs few loads a step and one or two waves send
// them; the rest is barriers and the last round of tiles.  128x128 has eight
// multiplying waves, because with the second set of sums (kFoldSteps) four would need more registers than two a SIMD
// leave; and a ring of three stages, because a compute unit holds one such workgroup.  The second set costs 2-5 %
// of a layer and halves its error against 64-bit sums (data gradient of a res4 block 3.1e-7 -> 1.5e-7).
// P counts channels of the contraction in halves (two to a float), those of the destination in floats.
template <int MODE, int BM, int BN, int WGM, int WGN, int KS, int S, int NP>
__global__ __launch_bounds__(64 * (WGM * WGN * KS + NP)) void igemm_ws_f32_kernel(IgemmParams P)
{
    ask_for_parameters(P);
    const int tile = xcd_run_tile(blockIdx.x);
    if (tile >= P.total_tiles) return;
    igemm_ws_body<MODE, BM, BN, WGM, WGN, S, 64, NP, 32, false, true, KS>(P, tile, P.tiles_n, 0);
}

template <int MODE, int BM, int BN, int WGM, int WGN, int KS, int S, int NP>
static hipError_t launch_one(const IgemmParams& P, hipStream_t st)
{
    constexpr size_t lds = ws_ring_bytes<BM, BN, WGM * WGN * KS, S, NP>() + (size_t)BM * 16;
    static_assert(lds <= 160 * 1024, "LDS budget");
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&igemm_ws_f32_kernel<MODE, BM, BN, WGM, WGN, KS, S, NP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    const int grid = ((P.total_tiles + 63) / 64) * 64;   // whole runs of tiles on each of 8 XCDs
    hipLaunchKernelGGL((igemm_ws_f32_kernel<MODE, BM, BN, WGM, WGN, KS, S, NP>), dim3(grid),
                       dim3(64 * (WGM * WGN * KS + NP)), lds, st, P);
    return hipGetLastError();
}

#define SDCONV_F32_CASE(idx, ...)                                                       \
    case idx: return P.mode ? launch_one<1, __VA_ARGS__>(P, st) : launch_one<0, __VA_ARGS__>(P, st);

hipError_t launch_igemm_ws_f32(int variant, const IgemmParams& P0, hipStream_t st)
{
    IgemmParams P = P0;
    set_tap_bias(&P);
    switch (variant) {
        SDCONV_F32_CASE(0, 128, 128, 2, 4, 1, 3, 2)
        SDCONV_F32_CASE(1, 128, 64, 2, 2, 1, 2, 2)
        SDCONV_F32_CASE(2, 64, 64, 2, 2, 1, 3, 2)
        SDCONV_F32_CASE(3, 64, 32, 2, 1, 2, 3, 1)
        SDCONV_F32_CASE(4, 32, 32, 1, 1, 4, 3, 1)
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sdconv
