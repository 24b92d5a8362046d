// Parameters of the implicit-GEMM forward / data-gradient kernel.
#pragma once
#include <array>
#include "common.h"

namespace sdconv {

constexpr int kMaxTaps = 64;      // R*S the MFMA route accepts
constexpr int kMaxClasses = 16;   // stride_h*stride_w parity classes of a strided dgrad

// The filter taps of one image axis that meet a stride-parity class of destination pixels (all of
// them in a forward pass): numbers first, first + step, ...  The source pixel of the t-th one lies
// disp + t * spacing from the class pixel's own (step, spacing: IgemmParams, the same for all classes).
struct AxisTaps { int first, count, disp; };

struct IgemmParams {
    const __half* A;   // gathered activations: x (forward) or dy (data gradient)
    const __half* B;   // filter matrix, one row per destination channel: [Cd][R][S][Cs]
    __half* D;         // destination activations
    int NB;            // batch
    int Hs, Ws, Cs;    // source image extents and channels (contraction channels per tap)
    int Hd, Wd, Cd;    // destination image extents and channels
    int R, S;
    int sh, sw, ph, pw, dh, dw;
    int mode;          // 0 forward, 1 data gradient
    int nclasses;      // 1, or stride_h*stride_w for a data gradient
    int sw_cls;        // classes along w (stride_w for a data gradient, else 1)
    int tiles_n;       // column tiles
    int total_tiles;   // row tiles (all classes) x column tiles
    int b_row_pitch;   // R*S*Cs
    int class_tile_start[kMaxClasses + 1];   // first row-tile of each class, then the total
    AxisTaps taps_h[kMaxClasses], taps_w[kMaxClasses];      // by class along h and along w
    int tap_sh, tap_sw;     // tap numbers between two consecutive ones
    int tap_dh, tap_dw;     // source pixels between two consecutive ones
    int pointwise;          // one tap, and GEMM row m reads source pixel m
    int tap_bias;           // what the fetching waves of igemm_ws_body.h add to a tap's displacement to have no
                            // negative one, or -1: the layer takes their general loop (set_tap_bias)
    int tiles_h, tiles_w;   // spatial tiles per image (patch kernels only)
    // launches with two tile widths (igemm_ws_mixed_kernel; set by its launcher)
    int mix_big_tiles, mix_big_blocks;                        // wide tiles, and the workgroups that cover them
    int mix_small_tiles, mix_small_tiles_n, mix_small_tm0;    // narrow tiles: count, per row tile, first row tile
    Epilogue ep;            // elementwise tail before the rounding to binary16 (all null: none)
};

void set_taps(const Geom& g, bool dgrad, IgemmParams* P);      // the tap fields (dispatch.hip)

void set_tap_bias(IgemmParams* P);      // once the other fields are set

// GEMM rows (destination pixels) and filter taps that meet them, by parity class of a strided data gradient;
// other passes have one class.
struct RowClasses { int n; unsigned pixels[kMaxClasses]; int taps[kMaxClasses]; };
RowClasses row_classes(const Geom& g, bool dgrad);

// Tile variants.  Their numbers are those of the committed timings and of the models fitted to them (fit_models.py);
// numbers without a name are tiles that were measured and are not in the library.
struct IgemmVariant { int bm, bn; const char* fwd_name; const char* dgrad_name; };
constexpr int kNumIgemmVariants = 4;            // register-staged, 0 and up
extern const std::array<IgemmVariant, kNumIgemmVariants> kIgemmVariants;

constexpr int kNumIgemmDmaVariants = 13;        // every wave fetches its share, 100 and up: forward passes only
extern const std::array<IgemmVariant, kNumIgemmDmaVariants> kIgemmDmaVariants;
hipError_t launch_igemm_dma(int variant, const IgemmParams& P, hipStream_t st);
constexpr int kNumIgemmWsVariants = 41;         // split roles, 300 and up
extern const std::array<IgemmVariant, kNumIgemmWsVariants> kIgemmWsVariants;
// Row tiles that a launch with two tile widths takes at full width: whole rounds of 256 workgroups
// (rounded down to whole row tiles), or all of them where the rest would make two rounds of half tiles.
inline long mixed_wide_rows(long row_tiles, int tiles_n)
{
    const long total = row_tiles * tiles_n;
    return 2 * (total % 256) > 256 + tiles_n ? row_tiles : total / 256 * 256 / tiles_n;
}
hipError_t launch_igemm_ws(int variant, const IgemmParams& P, hipStream_t st);
hipError_t launch_igemm_ws_f32(int variant, const IgemmParams& P, hipStream_t st);     // binary32 tensors
struct PatchVariant { int th, tw, bn, stages; const char* fwd_name; const char* dgrad_name; bool one_slab; };
// stages: of the filter ring; a step is a filter row (three taps), so R*S must be a multiple of 3 and R*S/3 at least stages-1.
// one_slab: the variant has a single patch buffer and takes layers with 64 source channels only
constexpr int kNumPatchVariants = 38;           // 400 and up
extern const std::array<PatchVariant, kNumPatchVariants> kPatchVariants;
hipError_t launch_conv_patch(int variant, const IgemmParams& P, hipStream_t st);
hipError_t launch_igemm(int variant, const IgemmParams& P, int total_tiles, hipStream_t st);
hipError_t launch_filter_transpose(const __half* w, __half* wT, int K, int RS, int C, hipStream_t st);

}  // namespace sdconv
