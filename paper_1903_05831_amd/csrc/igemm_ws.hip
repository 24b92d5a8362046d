// Split-role implicit GEMM: kernels and launches (the work of a workgroup: igemm_ws_body.h).
#include <algorithm>
#include "igemm_ws_body.h"

namespace sdconv {

template <int MODE, int BM, int BN, int WGM, int WGN, int S, int BK, int NP, int MF = 32, bool TAIL = false>
__global__ __launch_bounds__(64 * (WGM * WGN + NP)) void igemm_ws_kernel(IgemmParams P)
{
    ask_for_parameters(P);
    const int tile = xcd_run_tile(blockIdx.x);
    if (tile >= P.total_tiles) return;
    igemm_ws_body<MODE, BM, BN, WGM, WGN, S, BK, NP, MF, TAIL>(P, tile, P.tiles_n, 0);
}

// Two tile widths in one launch.  A layer whose tiles make a few whole rounds of the chip's
// compute units plus half a round (896 tiles of 224 x 256 on 256 CUs: the 1x1 layers of the RoI
// head) leaves half the units idle for the last round.  Here the first mix_big_tiles tiles are
// BN wide and the row tiles after them are cut into tiles of half the width, twice as many and
// ~0.64 of the time each, so the last round fills the chip.  Undivided images only (one parity
// class); both bodies have the same waves.
template <int MODE, int BM, int BN, int BNS, int WGM, int WGN, int S, int SS, int BK, int MF, bool TAIL>
__global__ __launch_bounds__(64 * WGM * WGN) void igemm_ws_mixed_kernel(IgemmParams P)
{
    ask_for_parameters(P);
    int b = blockIdx.x;
    if (b < P.mix_big_blocks) {
        const int tile = xcd_run_tile(b);
        if (tile >= P.mix_big_tiles) return;
        igemm_ws_body<MODE, BM, BN, WGM, WGN, S, BK, 0, MF, TAIL>(P, tile, P.tiles_n, 0);
    } else {
        const int tile = xcd_run_tile(b - P.mix_big_blocks);
        if (tile >= P.mix_small_tiles) return;
        igemm_ws_body<MODE, BM, BNS, WGM, WGN, SS, BK, 0, MF, TAIL>(P, tile, P.mix_small_tiles_n, P.mix_small_tm0);
    }
}

template <int MODE, int BM, int BN, int BNS, int WGM, int WGN, int S, int SS, int BK, int MF, bool TAIL>
static hipError_t launch_ws_mixed_impl(const IgemmParams& P0, hipStream_t st)
{
    constexpr size_t lds_big = ws_ring_bytes<BM, BN, WGM * WGN, S, 0>(), lds_small = ws_ring_bytes<BM, BNS, WGM * WGN, SS, 0>();
    constexpr size_t lds = (lds_big > lds_small ? lds_big : lds_small) + (size_t)BM * 16;
    static_assert(lds <= 160 * 1024, "LDS budget");
    if (P0.nclasses != 1) return hipErrorInvalidValue;
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void*>(&igemm_ws_mixed_kernel<MODE, BM, BN, BNS, WGM, WGN, S, SS, BK, MF, TAIL>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    // P0.tiles_n / P0.total_tiles describe the launch in BN-wide tiles.
    IgemmParams P = P0;
    const int row_tiles = P0.total_tiles / P0.tiles_n;
    const int big_rows = (int)mixed_wide_rows(row_tiles, P0.tiles_n);
    P.mix_big_tiles = big_rows * P0.tiles_n;
    P.mix_big_blocks = (P.mix_big_tiles + 63) / 64 * 64;
    P.mix_small_tm0 = big_rows;
    P.mix_small_tiles_n = (P0.Cd + BNS - 1) / BNS;
    P.mix_small_tiles = (row_tiles - big_rows) * P.mix_small_tiles_n;
    const int grid = P.mix_big_blocks + (P.mix_small_tiles + 63) / 64 * 64;
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL((igemm_ws_mixed_kernel<MODE, BM, BN, BNS, WGM, WGN, S, SS, BK, MF, TAIL>), dim3(grid),
                       dim3(64 * WGM * WGN), lds, st, P);
    return hipGetLastError();
}

template <int MODE, int BM, int BN, int BNS, int WGM, int WGN, int S, int SS, int BK, int MF>
static hipError_t launch_ws_mixed(const IgemmParams& P, hipStream_t st)
{
    return P.ep.any() ? launch_ws_mixed_impl<MODE, BM, BN, BNS, WGM, WGN, S, SS, BK, MF, true>(P, st)
                      : launch_ws_mixed_impl<MODE, BM, BN, BNS, WGM, WGN, S, SS, BK, MF, false>(P, st);
}

template <int MODE, int BM, int BN, int WGM, int WGN, int S, int BK, int NP, int MF = 32, bool TAIL>
static hipError_t launch_ws_variant_impl(const IgemmParams& P, hipStream_t st)
{
    constexpr size_t lds = ws_ring_bytes<BM, BN, WGM * WGN, S, NP>() + (size_t)BM * 16;
    static_assert(lds <= 160 * 1024, "LDS budget");
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void*>(&igemm_ws_kernel<MODE, BM, BN, WGM, WGN, S, BK, NP, MF, TAIL>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    const int grid = ((P.total_tiles + 63) / 64) * 64;   // whole runs of tiles on each of 8 XCDs
    hipLaunchKernelGGL((igemm_ws_kernel<MODE, BM, BN, WGM, WGN, S, BK, NP, MF, TAIL>), dim3(grid),
                       dim3(64 * (WGM * WGN + NP)), lds, st, P);
    return hipGetLastError();
}

template <int MODE, int BM, int BN, int WGM, int WGN, int S, int BK, int NP, int MF = 32>
static hipError_t launch_ws_variant(const IgemmParams& P, hipStream_t st)
{
    // the tail has kernels of its own: see store_rows_via_lds
    return P.ep.any() ? launch_ws_variant_impl<MODE, BM, BN, WGM, WGN, S, BK, NP, MF, true>(P, st) : launch_ws_variant_impl<MODE, BM, BN, WGM, WGN, S, BK, NP, MF, false>(P, st);
}

// number - 300, tile, multiplying waves, ring stages, fetching waves, matrix block, name.  64- and 80-row tiles give every
// compute unit a workgroup in layers with few pixels; 144 and 160 rows divide the pixels of the backbone's maps
// into whole rounds of 256 where 128 and 256 do not, 224 those of the RoI head.
#define SDCONV_WS_VARIANTS(X) \
    X(10, 224, 256, 2, 4, 2, 0, 16, "224x256x64_8w0f_s2_m16") \
    X(11, 256, 256, 2, 4, 2, 0, 16, "256x256x64_8w0f_s2_m16") \
    X(16, 224, 128, 2, 4, 3, 0, 16, "224x128x64_8w0f_s3_m16") \
    X(25, 144, 64, 3, 1, 4, 4, 16, "144x64x64_3w4f_s4_m16") \
    X(26, 144, 256, 1, 4, 2, 4, 16, "144x256x64_4w4f_s2_m16") \
    X(27, 64, 64, 2, 2, 4, 4, 32, "64x64x64_4w4f_s4") \
    X(28, 64, 64, 2, 2, 4, 4, 16, "64x64x64_4w4f_s4_m16") \
    X(29, 64, 128, 2, 2, 4, 4, 32, "64x128x64_4w4f_s4") \
    X(30, 128, 128, 2, 2, 3, 4, 32, "128x128x64_4w4f_s3") \
    X(31, 256, 128, 4, 2, 3, 4, 16, "256x128x64_8w4f_s3_m16") \
    X(32, 224, 128, 2, 2, 3, 4, 16, "224x128x64_4w4f_s3_m16") \
    X(33, 96, 128, 2, 2, 4, 4, 16, "96x128x64_4w4f_s4_m16") \
    X(34, 80, 128, 1, 4, 4, 4, 16, "80x128x64_4w4f_s4_m16") \
    X(35, 160, 128, 2, 2, 3, 4, 16, "160x128x64_4w4f_s3_m16") \
    X(36, 192, 128, 2, 2, 3, 4, 16, "192x128x64_4w4f_s3_m16") \
    X(37, 96, 64, 2, 2, 4, 4, 16, "96x64x64_4w4f_s4_m16") \
    X(38, 160, 256, 2, 4, 2, 0, 16, "160x256x64_8w0f_s2_m16") \
    X(39, 128, 128, 2, 2, 2, 4, 16, "128x128x64_4w4f_s2_m16") \
    X(40, 128, 64, 2, 2, 2, 4, 32, "128x64x64_4w4f_s2")

constexpr int kMixed = 24;      // 224x256 tiles for the whole rounds of 256 workgroups, 224x128 for the rest
const std::array<IgemmVariant, kNumIgemmWsVariants> kIgemmWsVariants = [] {
    std::array<IgemmVariant, kNumIgemmWsVariants> v{};
#define SDCONV_WS_NAME(idx, BM, BN, WGM, WGN, S, NP, MF, name) v[idx] = {BM, BN, "igemm_fwd_ws_" name, "igemm_dgrad_ws_" name};
    SDCONV_WS_VARIANTS(SDCONV_WS_NAME)
    v[kMixed] = {224, 256, "igemm_fwd_ws_224x256x64_8w0f_s2_m16_tail128", "igemm_dgrad_ws_224x256x64_8w0f_s2_m16_tail128"};
    return v;
}();

template <int MODE> static hipError_t launch_mode(int variant, const IgemmParams& P, hipStream_t st)
{
    switch (variant) {
#define SDCONV_WS_CASE(idx, BM, BN, WGM, WGN, S, NP, MF, name) \
        case idx: return launch_ws_variant<MODE, BM, BN, WGM, WGN, S, 64, NP, MF>(P, st);
        SDCONV_WS_VARIANTS(SDCONV_WS_CASE)
        case kMixed: return launch_ws_mixed<MODE, 224, 256, 128, 2, 4, 2, 3, 64, 16>(P, st);
        default: return hipErrorInvalidValue;
    }
}

void set_tap_bias(IgemmParams* P)
{
    long low = 0, high = 0;     // least and greatest displacement of any class, in bytes
    bool served = true;
    for (int a = 0; a * P->sw_cls < P->nclasses; ++a)
        for (int b = 0; b < P->sw_cls; ++b) {
            const AxisTaps h = P->taps_h[a], w = P->taps_w[b];
            if (h.count * w.count == 0) continue;
            if (h.count * w.count > 32) served = false;
            const long h1 = h.disp + (h.count - 1) * (long)P->tap_dh, w1 = w.disp + (w.count - 1) * (long)P->tap_dw;
            low = std::min(low, (std::min<long>(h.disp, h1) * P->Ws + std::min<long>(w.disp, w1)) * P->Cs * 2);
            high = std::max(high, (std::max<long>(h.disp, h1) * P->Ws + std::max<long>(w.disp, w1)) * P->Cs * 2);
        }
    // out-of-range offsets start at 2^31, past whatever a descriptor covers
    const long source = (long)P->NB * P->Hs * P->Ws * P->Cs * 2;
    const long filter = (long)std::max(P->Cs, P->Cd) * P->b_row_pitch * 2, most = (1L << 31) - kRunSlack;
    // and a scalar offset stays within its descriptor, also that of a tap that lies outside every image (the range
    // check takes it from the descriptor's size)
    served = served && high + 2L * P->Cs <= source + kRunSlack;
    P->tap_bias = served && source - low <= most && filter <= most ? (int)-low : -1;
}

hipError_t launch_igemm_ws(int variant, const IgemmParams& P0, hipStream_t st)
{
    IgemmParams P = P0;
    set_tap_bias(&P);
    return P.mode ? launch_mode<1>(variant, P, st) : launch_mode<0>(variant, P, st);
}

}  // namespace sdconv
