// Pointwise layers (1x1, stride 1, no padding) with at most 64 filters, their number not a multiple
// of 8: the objectness and box heads of a region proposal network (3, 12, 15, 60 filters).
//
// All three passes are bound by the C-channel tensor, which each of them reads or writes once
// (2 * C bytes a pixel; the K-channel one is a fraction of it).  On the general kernels such a layer
// runs with K rounded up to 8, on padded copies of the filter and of the K-channel tensor: two to
// four launches, whose small ones take 2-6 us each while the large one takes 5-20 us.  Here the K axis
// is a fragment of v_mfma_f32_16x16x* that is filled with zeros as it is loaded, so a pass is one
// kernel (the weight gradient: two) and needs no copies.
#include "narrow.h"
#include "wgrad.h"

namespace sdconv {

typedef _Float16 half4v __attribute__((ext_vector_type(4)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kNarrowThreads = 256, kNarrowWaves = 4;
constexpr int kNarrowMaxFilters = 64;
constexpr int kNarrowBlocks = 1024;             // persistent: four workgroups a compute unit, at 33 KB of LDS each
constexpr int kNarrowChunk = 128;               // weight gradient: channels of a wave

static int filter_tiles(const Geom& g) { return (g.K + 15) / 16; }
static long narrow_pixels(const Geom& g) { return (long)g.N * g.Ho * g.Wo; }

// Where these kernels are the faster ones, from timings of both routes with 3 to 63 filters, 32 to 1024 channels
// and 64 to 134 400 pixels.  Forward and data gradient: each workgroup lays the filter out in LDS, 32
// bytes a channel and tile of 16 filters.  Up to 1024 channels x tiles they take 0.61 and 0.50 of the
// time on padded copies (380 sizes, 0.21-1.03 of it); above, 1.17 and 1.09 (60 filters, 512 channels, 4200
// pixels: forward 13.5 us against 10.6, data gradient 11.8 against 9.7).  Weight gradient: dy is read in
// 2-byte loads, for each 128 channels again.  One tile 0.79 (0.59-0.96), two tiles 0.93 up to 128 channels and
// 1.01 above, more tiles 1.22 (60 filters, 512 channels: 15.5 us against 12.1); with two tiles a few
// hundred pixels make two ranges and a reduction where the padded route has one (1.11-1.17).
bool narrow_supported(const Geom& g, int pass)
{
    const int tiles = filter_tiles(g);
    if (g.R != 1 || g.S != 1 || g.sh != 1 || g.sw != 1 || g.ph != 0 || g.pw != 0 || g.C % 8 != 0 ||
        g.K > kNarrowMaxFilters)
        return false;
    if (pass != SDCONV_WGRAD) return tiles * g.C <= 1024;
    const long pixels = narrow_pixels(g);
    return tiles == 1 || (tiles == 2 && g.C <= 128 && (pixels <= 256 || pixels >= 1024));
}

// Four values of one row of a [rows][K] tensor from column k on, zeros past its end.  Rows start at
// any multiple of 2 bytes; where K is a multiple of 4 the four lie at a multiple of 8.
__device__ __forceinline__ half4v load_row4(const _Float16* row, int k, int K)
{
    if (K % 4 == 0) {
        if (k < K) return *reinterpret_cast<const half4v*>(row + k);
        return half4v{0, 0, 0, 0};
    }
    half4v v = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (k + j < K) v[j] = row[k + j];
    return v;
}

// y[p][k] = sum over c of x[p][c] * w[k][c].  A wave takes 16 pixels: the filters are the rows of
// the product, the pixels its columns, so a lane ends with 4 consecutive filters of one pixel.
// The tail sees the sum rounded to binary16, as conv2d_fwd_fused defines it for such filter counts.
// 200x336x2 pixels, 256 channels, 12 filters: 17.6 us, 4.1 TB/s (30.0 us on padded copies).
template <int KT>
__global__ __launch_bounds__(kNarrowThreads) void narrow_fwd_kernel(
    const _Float16* __restrict__ x, const _Float16* __restrict__ w, _Float16* __restrict__ y,
    long P, int C, int K, Epilogue E)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    _Float16* wl = reinterpret_cast<_Float16*>(smem);       // [KT*16][C + 8]: rows 16 bytes apart in the banks
    const int pitch = C + 8;
    for (int i = threadIdx.x; i < KT * 16 * (C / 8); i += kNarrowThreads) {
        const int k = i / (C / 8), c = (i - k * (C / 8)) * 8;
        half8v v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (k < K) v = *reinterpret_cast<const half8v*>(w + (long)k * C + c);
        *reinterpret_cast<half8v*>(wl + k * pitch + c) = v;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const long tiles = (P + 15) / 16;
    for (long t = (long)blockIdx.x * kNarrowWaves + (threadIdx.x >> 6); t < tiles; t += (long)gridDim.x * kNarrowWaves) {
        const long p = t * 16 + r;
        const bool live = p < P;
        const _Float16* xp = x + (live ? p : P - 1) * C;    // a lane past the end writes nothing: any pixel will do
        float4v acc[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) acc[kt] = float4v{0.f, 0.f, 0.f, 0.f};
        for (int cb = 0; cb < C; cb += 256) {
            half8v v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = cb + j * 32 + q * 8;
                v[j] = half8v{0, 0, 0, 0, 0, 0, 0, 0};
                if (c < C) v[j] = *reinterpret_cast<const half8v*>(xp + c);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = cb + j * 32 + q * 8;
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    half8v f = {0, 0, 0, 0, 0, 0, 0, 0};
                    if (c < C) f = *reinterpret_cast<const half8v*>(wl + (kt * 16 + r) * pitch + c);
                    acc[kt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f, v[j], acc[kt], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const int k = kt * 16 + 4 * q;
            if (!live || k >= K) continue;
            half4v o = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k + j < K) o[j] = (_Float16)epilogue_apply(E, (float)(_Float16)acc[kt][j], k + j, p * K + k + j);
            if (K % 4 == 0) {
                *reinterpret_cast<half4v*>(y + p * K + k) = o;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k + j < K) y[p * K + k + j] = o[j];
            }
        }
    }
}

// The 16 bytes of the lane eight places on in its row of 16 lanes.
__device__ __forceinline__ half8v from_half_row(half8v v)
{
    typedef int int4v __attribute__((ext_vector_type(4)));
    int4v i = __builtin_bit_cast(int4v, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) i[e] = __builtin_amdgcn_mov_dpp(i[e], 0x128, 0xf, 0xf, true);     // row_ror:8
    return __builtin_bit_cast(half8v, i);
}

// dx[p][c] = sum over k of dy[p][k] * w[k][c].  The channels are the rows of the product, the
// pixels its columns.  Two tiles make 32 channels, dealt to their rows so that a lane's four rows of
// the first and four of the second are 8 consecutive channels.  Of two such pairs the lanes of pixels
// 0-7 and 8-15 exchange one chunk, after which a store writes 8 pixels x 128 bytes, whole lines.  The filter
// lies in LDS as the fragments that the lanes read.
// 200x336x2 pixels, 256 channels, 12 filters: 17.0 us, 4.3 TB/s (35.6 us on
// padded copies; 25 us with 64-byte store segments and the filter read by halves).
template <int KT, bool TAIL>
__global__ __launch_bounds__(kNarrowThreads) void narrow_dgrad_kernel(
    const _Float16* __restrict__ dy, const _Float16* __restrict__ w, _Float16* __restrict__ dx,
    long P, int C, int K, Epilogue E)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    _Float16* fill = reinterpret_cast<_Float16*>(smem);
    const half4v* frag = reinterpret_cast<const half4v*>(smem);     // [64 channels][2 pairs][2 tiles][KT][lane]
    const int couples = (C + 63) / 64;
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const long tiles = (P + 15) / 16, stride = (long)gridDim.x * kNarrowWaves;
    long t = (long)blockIdx.x * kNarrowWaves + (threadIdx.x >> 6);
    half4v g[KT];
    auto load = [&](long tile) {
        const long p = tile * 16 + r;       // a pixel past the end: nothing is stored for it, any will do
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) g[kt] = load_row4(dy + (p < P ? p : P - 1) * K, kt * 16 + 4 * q, K);
    };
    load(t < tiles ? t : tiles - 1);        // in flight while the filter is laid out
    for (int i = threadIdx.x; i < KT * 16 * couples * 8; i += kNarrowThreads) {
        const int k = i / (couples * 8), chunk = i - k * (couples * 8), c = chunk * 8;
        half8v v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (k < K && c < C) v = *reinterpret_cast<const half8v*>(w + (long)k * C + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int tile = (chunk >> 2) * 2 + (e >> 2), row = (chunk & 3) * 4 + (e & 3);
            fill[((tile * KT + (k >> 4)) * 64 + ((k & 15) >> 2) * 16 + row) * 4 + (k & 3)] = v[e];
        }
    }
    __syncthreads();
    const bool upper = r >= 8;
    for (; t < tiles; t += stride) {
        half4v cur[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) cur[kt] = g[kt];
        if (t + stride < tiles) load(t + stride);
        const long p_lo = t * 16 + (r & 7), p_hi = p_lo + 8;    // pixels of this lane's two stores
#pragma unroll 2
        for (int cc = 0; cc < couples; ++cc) {
            half8v o[2];
#pragma unroll
            for (int pair = 0; pair < 2; ++pair) {
                const half4v* f = frag + (long)(cc * 2 + pair) * 2 * KT * 64 + lane;
                float4v lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    lo = __builtin_amdgcn_mfma_f32_16x16x16f16(f[kt * 64], cur[kt], lo, 0, 0, 0);
                    hi = __builtin_amdgcn_mfma_f32_16x16x16f16(f[(KT + kt) * 64], cur[kt], hi, 0, 0, 0);
                }
                const int c = cc * 64 + pair * 32 + q * 8;
                if (TAIL && E.scale && c < C) {
                    lo *= *reinterpret_cast<const float4v*>(E.scale + c);
                    hi *= *reinterpret_cast<const float4v*>(E.scale + c + 4);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) { o[pair][j] = (_Float16)lo[j]; o[pair][4 + j] = (_Float16)hi[j]; }
            }
            const half8v got = from_half_row(upper ? o[0] : o[1]);
            half8v first = upper ? got : o[0];          // pixel p_lo: pair 0 from its own lane, pair 1 from the lane above
            half8v second = upper ? o[1] : got;         // pixel p_hi
            const int c = cc * 64 + (upper ? 32 : 0) + q * 8;
            if (c < C) {
                if (p_lo < P) {
                    if (TAIL && E.mask) {
                        const half8v m = *reinterpret_cast<const half8v*>(reinterpret_cast<const _Float16*>(E.mask) + p_lo * C + c);
#pragma unroll
                        for (int j = 0; j < 8; ++j) first[j] = (float)m[j] > 0.f ? first[j] : (_Float16)0.f;
                    }
                    __builtin_nontemporal_store(first, reinterpret_cast<half8v*>(dx + p_lo * C + c));
                }
                if (p_hi < P) {
                    if (TAIL && E.mask) {
                        const half8v m = *reinterpret_cast<const half8v*>(reinterpret_cast<const _Float16*>(E.mask) + p_hi * C + c);
#pragma unroll
                        for (int j = 0; j < 8; ++j) second[j] = (float)m[j] > 0.f ? second[j] : (_Float16)0.f;
                    }
                    __builtin_nontemporal_store(second, reinterpret_cast<half8v*>(dx + p_hi * C + c));
                }
            }
        }
    }
}

// dw[k][c] = sum over p of dy[p][k] * x[p][c].  The contraction runs over pixels, along which neither
// tensor is contiguous.  A lane loads 8 channels of each of 8 pixels (16 lanes: 256 consecutive
// bytes of a pixel) and holds with them one column of eight tiles, once the 8x8 values are
// transposed in its registers: no LDS, no exchange between lanes.  The waves of a workgroup take
// different pixels; their sums are added in LDS in a fixed order.
// 200x336x2 pixels, 256 channels, 12 filters: 16.0 us and 6.6 us for the sum of
// the ranges (31.6 us on padded copies; 31 us with a branch round each load).
template <int KT>
__global__ __launch_bounds__(kNarrowThreads) void narrow_wgrad_kernel(
    const _Float16* __restrict__ x, const _Float16* __restrict__ dy, float* __restrict__ out,
    long P, int C, int K, int chunks, int steps_per_wave)
{
    __shared__ __attribute__((aligned(16))) float sums[KT * 16 * kNarrowChunk];
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4, wave = threadIdx.x >> 6;
    const int chunk = blockIdx.x % chunks, range = blockIdx.x / chunks;
    const int c = chunk * kNarrowChunk + r * 8;
    const long first = ((long)range * kNarrowWaves + wave) * steps_per_wave * 32;
    const half8v zero = {0, 0, 0, 0, 0, 0, 0, 0};
    float4v acc[KT][8];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[kt][e] = float4v{0.f, 0.f, 0.f, 0.f};
    half8v xv[8], gv[KT];
    // Columns past the channels and rows past the filters are computed from whatever the last of them
    // holds, and not stored; pixels past the end count as zeros in both factors.
    const int cl = c < C ? c : C - 8;
    int kl[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) kl[kt] = kt * 16 + r < K ? kt * 16 + r : K - 1;
    auto load = [&](long p0) {
        const long p = p0 + q * 8;
        if (p0 + 32 <= P) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                xv[j] = *reinterpret_cast<const half8v*>(x + (p + j) * C + cl);
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) gv[kt][j] = dy[(p + j) * K + kl[kt]];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                xv[j] = zero;
                if (p + j < P) xv[j] = *reinterpret_cast<const half8v*>(x + (p + j) * C + cl);
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) gv[kt][j] = p + j < P ? dy[(p + j) * K + kl[kt]] : (_Float16)0.f;
            }
        }
    };
    load(first);
    for (int s = 0; s < steps_per_wave; ++s) {
        half8v col[8], g[KT];
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int j = 0; j < 8; ++j) col[e][j] = xv[j][e];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) g[kt] = gv[kt];
        if (s + 1 < steps_per_wave) load(first + (long)(s + 1) * 32);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
                acc[kt][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(g[kt], col[e], acc[kt][e], 0, 0, 0);
    }
    for (int turn = 0; turn < kNarrowWaves; ++turn) {
        if (wave == turn) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float4v* s = reinterpret_cast<float4v*>(sums + (kt * 16 + 4 * q + i) * kNarrowChunk + r * 8);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        float4v v = {acc[kt][4 * h][i], acc[kt][4 * h + 1][i], acc[kt][4 * h + 2][i], acc[kt][4 * h + 3][i]};
                        s[h] = turn ? s[h] + v : v;
                    }
                }
        }
        __syncthreads();
    }
    float* o = out + (long)range * K * C;
    for (int i = threadIdx.x; i < K * (kNarrowChunk / 4); i += kNarrowThreads) {
        const int k = i / (kNarrowChunk / 4), cc = (i % (kNarrowChunk / 4)) * 4;
        if (chunk * kNarrowChunk + cc < C)
            *reinterpret_cast<float4v*>(o + (long)k * C + chunk * kNarrowChunk + cc) =
                *reinterpret_cast<const float4v*>(sums + k * kNarrowChunk + cc);
    }
}

static int narrow_chunks(const Geom& g) { return (g.C + kNarrowChunk - 1) / kNarrowChunk; }

// Steps of 32 pixels that each wave takes: as few as make at most 512 workgroups (two a compute unit,
// which hold 64 KB of loads in flight there; more would only add partial sums), and at least two,
// behind which the next loads are in flight.
static int narrow_wgrad_steps(const Geom& g)
{
    const long steps = (narrow_pixels(g) + 31) / 32;
    long ranges = 512 / narrow_chunks(g);
    if (ranges < 1) ranges = 1;
    const long per_wave = (steps + ranges * kNarrowWaves - 1) / (ranges * kNarrowWaves);
    return (int)(per_wave < 2 ? 2 : per_wave);
}

int narrow_wgrad_ranges(const Geom& g)
{
    const long per_block = (long)narrow_wgrad_steps(g) * kNarrowWaves * 32;
    return (int)((narrow_pixels(g) + per_block - 1) / per_block);
}

size_t narrow_wgrad_partial_bytes(const Geom& g)
{
    const int ranges = narrow_wgrad_ranges(g);
    return ranges > 1 ? (size_t)ranges * g.K * g.C * sizeof(float) : 0;
}

static unsigned narrow_grid(const Geom& g)
{
    const long blocks = (narrow_pixels(g) + 16 * kNarrowWaves - 1) / (16 * kNarrowWaves);
    return (unsigned)(blocks < kNarrowBlocks ? blocks : kNarrowBlocks);
}

template <int KT>
static hipError_t fwd_tiles(const Geom& g, const _Float16* x, const _Float16* w, _Float16* y, hipStream_t st, const Epilogue& ep)
{
    hipLaunchKernelGGL(narrow_fwd_kernel<KT>, dim3(narrow_grid(g)), dim3(kNarrowThreads), (size_t)KT * 32 * (g.C + 8), st,
                       x, w, y, narrow_pixels(g), g.C, g.K, ep);
    return hipGetLastError();
}

template <int KT>
static hipError_t dgrad_tiles(const Geom& g, const _Float16* dy, const _Float16* w, _Float16* dx, hipStream_t st, const Epilogue& ep)
{
    const size_t lds = (size_t)((g.C + 63) / 64) * 4 * KT * 64 * sizeof(half4v);
    auto* kernel = ep.any() ? narrow_dgrad_kernel<KT, true> : narrow_dgrad_kernel<KT, false>;
    hipLaunchKernelGGL(kernel, dim3(narrow_grid(g)), dim3(kNarrowThreads), lds, st, dy, w, dx, narrow_pixels(g), g.C, g.K, ep);
    return hipGetLastError();
}

hipError_t launch_narrow_fwd(const Geom& g, const __half* x, const __half* w, __half* y, hipStream_t st, const Epilogue& ep)
{
    const _Float16 *xf = reinterpret_cast<const _Float16*>(x), *wf = reinterpret_cast<const _Float16*>(w);
    _Float16* yf = reinterpret_cast<_Float16*>(y);
    switch (filter_tiles(g)) {
        case 1: return fwd_tiles<1>(g, xf, wf, yf, st, ep);
        case 2: return fwd_tiles<2>(g, xf, wf, yf, st, ep);
        case 3: return fwd_tiles<3>(g, xf, wf, yf, st, ep);
        case 4: return fwd_tiles<4>(g, xf, wf, yf, st, ep);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_narrow_dgrad(const Geom& g, const __half* dy, const __half* w, __half* dx, hipStream_t st, const Epilogue& ep)
{
    const _Float16 *gf = reinterpret_cast<const _Float16*>(dy), *wf = reinterpret_cast<const _Float16*>(w);
    _Float16* xf = reinterpret_cast<_Float16*>(dx);
    switch (filter_tiles(g)) {
        case 1: return dgrad_tiles<1>(g, gf, wf, xf, st, ep);
        case 2: return dgrad_tiles<2>(g, gf, wf, xf, st, ep);
        case 3: return dgrad_tiles<3>(g, gf, wf, xf, st, ep);
        case 4: return dgrad_tiles<4>(g, gf, wf, xf, st, ep);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_narrow_wgrad(const Geom& g, const __half* x, const __half* dy, float* out, hipStream_t st)
{
    const _Float16 *xf = reinterpret_cast<const _Float16*>(x), *gf = reinterpret_cast<const _Float16*>(dy);
    const long P = narrow_pixels(g);
    const int chunks = narrow_chunks(g), steps = narrow_wgrad_steps(g);
    const dim3 grid((unsigned)(chunks * narrow_wgrad_ranges(g))), block(kNarrowThreads);
    switch (filter_tiles(g)) {
        case 1: hipLaunchKernelGGL(narrow_wgrad_kernel<1>, grid, block, 0, st, xf, gf, out, P, g.C, g.K, chunks, steps); break;
        case 2: hipLaunchKernelGGL(narrow_wgrad_kernel<2>, grid, block, 0, st, xf, gf, out, P, g.C, g.K, chunks, steps); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sdconv
