// Pointwise layers with few filters (narrow.hip).
#pragma once
#include "common.h"

namespace sdconv {

bool narrow_supported(const Geom& g, int pass);
int narrow_wgrad_ranges(const Geom& g);
size_t narrow_wgrad_partial_bytes(const Geom& g);
hipError_t launch_narrow_fwd(const Geom& g, const __half* x, const __half* w, __half* y, hipStream_t st, const Epilogue& ep);
hipError_t launch_narrow_dgrad(const Geom& g, const __half* dy, const __half* w, __half* dx, hipStream_t st, const Epilogue& ep);
// dw, or the partial sums [ranges][K][C] that launch_splitk_reduce adds up
hipError_t launch_narrow_wgrad(const Geom& g, const __half* x, const __half* dy, float* out, hipStream_t st);

}  // namespace sdconv
