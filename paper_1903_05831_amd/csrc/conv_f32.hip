// Single-precision companion of the convolution path: the same three passes on binary32
// tensors with v_mfma_f32_32x32x2_f32 (binary32 products, binary32 accumulation).  It exists so
// that the FP32 -> FP16 speedup of section 2.2 / Figure 1(b) of the paper can be measured on this
// hardware with both sides on the matrix cores.
//
// The fp32 matrix rate is 1/16 of the fp16 one (157.3 against 2516.6 TFLOP/s), so the
// kernels are bound by the matrix pipe: a 128x128 tile needs 32 KB of operands per 4096 cycles of
// MFMA.  What costs time on the small layers is that few tiles divide badly by 256 compute units, hence
// tiles down to 32x32, and that a workgroup waits for its loads, hence waves that only fetch
// (igemm_ws_f32.hip, wgrad_ws_f32.hip).  The kernels of this file, global -> registers -> LDS double buffer,
// serve tensors of 2^29 elements and more and the layers on which they are the faster ones.  One res4 block of
// one image (1x1, 3x3 stride 2, 1x1, projection; 16 800 pixels in), three passes: register-staged 695 us,
// now 604; blocks of res2 - res4 on other maps 1.15 to 1.9 times as fast.
//
// Forward / data gradient: implicit GEMM, rows = pixels, 32 floats of contraction per step (a
// 128-byte row, 16-byte chunks XOR-swizzled with the row number).  An MFMA takes one float per
// lane and operand: lane l supplies row l%32 at contraction slot l/32.  A lane reads the 16-byte
// chunk 2j + l/32 of its row and uses its four floats in four consecutive MFMAs; the filter
// operand does the same, so both sides agree on which contraction index sits in which slot.
// The data gradient contracts over a transposed copy wT[c][r][s][k] of the filter (workspace).
//
// Weight gradient: rows = filters, columns = channels of one tap, contraction = pixels, 32 per
// step, tiles kept [pixel][channel] as they sit in memory: lane l reads channel l%32 of pixel
// 2t + l/32 with a 4-byte LDS read (odd pixel rows are stored with their columns XOR 32, which
// puts the two pixel rows of one read on different banks).  Split along the pixels, partial
// sums added in a fixed order by the reduction kernel of wgrad.hip.
#include "common.h"
#include "igemm.h"
#include "wgrad.h"

namespace sdconv {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct F32Params {
    const float* A;
    const float* B;
    float* D;
    int NB, Hs, Ws, Cs, Hd, Wd, Cd, R, S;
    int sh, sw, ph, pw, dh, dw;
    int nclasses, sw_cls, tiles_n, total_tiles, b_row_pitch;
    int class_tile_start[kMaxClasses + 1];
};

constexpr int kF32BK = 32;              // contraction floats per step
constexpr int kF32RowBytes = kF32BK * 4;

template <int BM, int BN, int WGK>
constexpr size_t f32_lds_bytes()
{
    const size_t loop = 2 * (BM + BN) * kF32RowBytes + (3 * kMaxTaps + 4) * sizeof(int);
    const size_t sums = (size_t)(WGK - 1) * BM * BN * sizeof(float);    // over the same memory after the loop
    return loop > sums ? loop : sums;
}

// WGK > 1: the waves divide the 32 contraction floats of a step among WGK groups, and the groups' sums
// meet in LDS after the loop.  That is what makes tiles possible whose sides four waves cannot
// divide into 32x32 blocks.
template <int MODE, int BM, int BN, int WGM, int WGN, int WGK>
__global__ __launch_bounds__(256) void igemm_f32_kernel(F32Params P)
{
    static_assert(WGM * WGN * WGK == 4, "four waves per workgroup");
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int FM = WM / 32, FN = WN / 32;
    constexpr int PA = BM / 32, PB = BN / 32;       // staging passes (32 rows per pass)
    static_assert(WM % 32 == 0 && WN % 32 == 0 && WM * WGM == BM && WN * WGN == BN, "wave tile is a multiple of the MFMA block");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* ldsA = smem;                                 // [2][BM rows][128 B]
    unsigned char* ldsB = smem + 2 * BM * kF32RowBytes;         // [2][BN rows][128 B]
    int* tap_oh = reinterpret_cast<int*>(smem + 2 * (BM + BN) * kF32RowBytes);
    int* tap_ow = tap_oh + kMaxTaps;
    int* tap_bo = tap_ow + kMaxTaps;
    int* tap_cnt = tap_bo + kMaxTaps;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wk = wave / (WGM * WGN), wmn = wave % (WGM * WGN);
    const int wm = wmn / WGN, wn = wmn % WGN;

    const int tile = blockIdx.x;
    const int tn = tile % P.tiles_n;
    int tm = tile / P.tiles_n;
    int cls = 0;
    while (cls + 1 < P.nclasses && tm >= P.class_tile_start[cls + 1]) ++cls;
    tm -= P.class_tile_start[cls];
    const int ca = cls / P.sw_cls, cb = cls % P.sw_cls;   // stride parity class (data gradient) or (0,0)

    int Hi, Wj, mh, mw, eh, ew;
    if (MODE == 0) { Hi = P.Hd; Wj = P.Wd; mh = P.sh; mw = P.sw; eh = 1; ew = 1; }
    else {
        Hi = (P.Hd - ca + P.sh - 1) / P.sh; Wj = (P.Wd - cb + P.sw - 1) / P.sw;
        mh = 1; mw = 1; eh = P.sh; ew = P.sw;
    }
    const int Mcls = P.NB * Hi * Wj;
    const int m0 = tm * BM, n0 = tn * BN;

    if (wave == 0) {
        const int ntap_all = P.R * P.S;
        bool ok = false;
        int oh = 0, ow = 0;
        const int r = lane / P.S, s = lane % P.S;
        if (lane < ntap_all) {
            if (MODE == 0) { ok = true; oh = r * P.dh - P.ph; ow = s * P.dw - P.pw; }
            else {
                int th = ca + P.ph - r * P.dh, tw = cb + P.pw - s * P.dw;
                ok = (th % P.sh == 0) && (tw % P.sw == 0);
                oh = th / P.sh; ow = tw / P.sw;
            }
        }
        unsigned long long mask = __ballot(ok);
        int pos = __popcll(mask & ((1ull << lane) - 1ull));
        if (ok) { tap_oh[pos] = oh; tap_ow[pos] = ow; tap_bo[pos] = (r * P.S + s) * P.Cs; }
        if (lane == 0) tap_cnt[0] = __popcll(mask);
    }
    __syncthreads();
    const int ntaps = __builtin_amdgcn_readfirstlane(tap_cnt[0]);
    const int kchunks = (P.Cs + kF32BK - 1) / kF32BK;
    const int nk = ntaps * kchunks;

    const int lrow = tid >> 3;        // 0..31
    const int kc = tid & 7;           // 16-byte chunk (4 floats) within the 128-byte row
    int a_base[PA], a_ih[PA], a_jw[PA];
#pragma unroll
    for (int p = 0; p < PA; ++p) {
        int m = m0 + lrow + 32 * p;
        if (m < Mcls) {
            int n = m / (Hi * Wj);
            int rem = m - n * (Hi * Wj);
            int i = rem / Wj, j = rem - i * Wj;
            a_base[p] = n * P.Hs * P.Ws * P.Cs;
            a_ih[p] = i * mh;
            a_jw[p] = j * mw;
        } else {
            a_base[p] = 0; a_ih[p] = -(1 << 28); a_jw[p] = -(1 << 28);
        }
    }
    int b_base[PB];
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        int n = n0 + lrow + 32 * p;
        b_base[p] = (n < P.Cd) ? n * P.b_row_pitch : -1;
    }

    f32x4 ra[PA], rb[PB];
    auto prefetch = [&](int it) {
        const int t = it / kchunks;
        const int c = (it - t * kchunks) * kF32BK + kc * 4;
        const int oh = tap_oh[t], ow = tap_ow[t], bo = tap_bo[t];
        const bool cok = c < P.Cs;                 // Cs is a multiple of 4: all four floats or none
#pragma unroll
        for (int p = 0; p < PA; ++p) {
            int hs = a_ih[p] + oh, ws = a_jw[p] + ow;
            bool ok = cok && (unsigned)hs < (unsigned)P.Hs && (unsigned)ws < (unsigned)P.Ws;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (ok) v = *reinterpret_cast<const f32x4*>(P.A + (a_base[p] + (hs * P.Ws + ws) * P.Cs + c));
            ra[p] = v;
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            bool ok = cok && b_base[p] >= 0;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (ok) v = *reinterpret_cast<const f32x4*>(P.B + (b_base[p] + bo + c));
            rb[p] = v;
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int p = 0; p < PA; ++p) {
            int row = lrow + 32 * p;
            *reinterpret_cast<f32x4*>(ldsA + buf * BM * kF32RowBytes + row * kF32RowBytes + ((kc ^ (row & 7)) << 4)) = ra[p];
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            int row = lrow + 32 * p;
            *reinterpret_cast<f32x4*>(ldsB + buf * BN * kF32RowBytes + row * kF32RowBytes + ((kc ^ (row & 7)) << 4)) = rb[p];
        }
    };

    f32x16 acc[FN][FM];
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
        for (int b = 0; b < FM; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;

    const int l32 = lane & 31, lhi = lane >> 5;
    auto compute = [&](int buf) {
        const unsigned char* sa = ldsA + buf * BM * kF32RowBytes;
        const unsigned char* sb = ldsB + buf * BN * kF32RowBytes;
#pragma unroll
        for (int j = 0; j < 4 / WGK; ++j) {
            const int chunk = 2 * (j + wk * (4 / WGK)) + lhi;   // contraction floats 4*chunk .. 4*chunk+3 of the step
            f32x4 fa[FM], fb[FN];
#pragma unroll
            for (int b = 0; b < FM; ++b) {
                int row = wm * WM + b * 32 + l32;
                fa[b] = *reinterpret_cast<const f32x4*>(sa + row * kF32RowBytes + ((chunk ^ (row & 7)) << 4));
            }
#pragma unroll
            for (int a = 0; a < FN; ++a) {
                int row = wn * WN + a * 32 + l32;
                fb[a] = *reinterpret_cast<const f32x4*>(sb + row * kF32RowBytes + ((chunk ^ (row & 7)) << 4));
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int a = 0; a < FN; ++a)
#pragma unroll
                    for (int b = 0; b < FM; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[a][t], fa[b][t], acc[a][b], 0, 0, 0);
        }
    };

    if (nk > 0) {
        prefetch(0);
        stage(0);
        __syncthreads();
        for (int it = 0; it < nk; ++it) {
            const bool more = it + 1 < nk;
            if (more) prefetch(it + 1);
            compute(it & 1);
            if (more) stage((it + 1) & 1);
            __syncthreads();
        }
    }

    if constexpr (WGK > 1) {        // add the groups' sums, in the order of the groups
        float* sums = reinterpret_cast<float*>(smem);
        auto slot = [&](int group, int a, int b, int e) {
            return ((((group - 1) * WGM * WGN + wmn) * FN + a) * FM + b) * 1024 + e * 64 + lane;
        };
        __syncthreads();            // the last step's reads, and those of the tap count where there was no step
        if (wk > 0) {
#pragma unroll
            for (int a = 0; a < FN; ++a)
#pragma unroll
                for (int b = 0; b < FM; ++b)
#pragma unroll
                    for (int e = 0; e < 16; ++e) sums[slot(wk, a, b, e)] = acc[a][b][e];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int group = 1; group < WGK; ++group)
#pragma unroll
            for (int a = 0; a < FN; ++a)
#pragma unroll
                for (int b = 0; b < FM; ++b)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[a][b][e] += sums[slot(group, a, b, e)];
    }

    // ---- epilogue: a lane holds 4 consecutive destination channels of one pixel per group ----
#pragma unroll
    for (int b = 0; b < FM; ++b) {
        int m = m0 + wm * WM + b * 32 + l32;
        if (m >= Mcls) continue;
        int n = m / (Hi * Wj);
        int rem = m - n * (Hi * Wj);
        int i = rem / Wj, j = rem - i * Wj;
        int hd = i * eh + ca, wd = j * ew + cb;
        float* drow = P.D + ((long)(n * P.Hd + hd) * P.Wd + wd) * P.Cd;
#pragma unroll
        for (int a = 0; a < FN; ++a) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int col = n0 + wn * WN + a * 32 + 8 * q + 4 * lhi;
                if (col < P.Cd) {                   // Cd is a multiple of 4
                    f32x4 v = {acc[a][b][4 * q + 0], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
                    *reinterpret_cast<f32x4*>(drow + col) = v;
                }
            }
        }
    }
}

// wT[c][r][s][k] = w[k][r][s][c]
__global__ __launch_bounds__(256) void filter_transpose_f32_kernel(const float* __restrict__ w, float* __restrict__ wT,
                                                                   int K, int RS, int C)
{
    __shared__ float tile[32][33];
    const int tap = blockIdx.z;
    const int k0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    for (int i = ty; i < 32; i += 8) {
        int k = k0 + i, c = c0 + tx;
        tile[i][tx] = (k < K && c < C) ? w[((long)k * RS + tap) * C + c] : 0.f;
    }
    __syncthreads();
    for (int i = ty; i < 32; i += 8) {
        int c = c0 + i, k = k0 + tx;
        if (c < C && k < K) wT[((long)c * RS + tap) * K + k] = tile[tx][i];
    }
}

// ---- weight gradient ---------------------------------------------------------------------------
template <int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void wgrad_f32_kernel(F32WgradParams P)
{
    static_assert(WGM * WGN == 4, "four waves");
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int FM = WM / 32, FN = WN / 32;
    constexpr int TA = BM / 4, TB = BN / 4;                 // threads per tile row (16 B each)
    constexpr int PA = kF32BP * TA / 256, PB = kF32BP * TB / 256;
    constexpr int RA = 256 / TA, RB = 256 / TB;             // rows per pass
    static_assert(PA >= 1 && PB >= 1 && WM % 32 == 0 && WN % 32 == 0, "tile shape");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float* ldsG = reinterpret_cast<float*>(smem);                            // [2][32][BM]
    float* ldsX = reinterpret_cast<float*>(smem) + 2 * kF32BP * BM;          // [2][32][BN]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WGN, wn = wave % WGN;

    int b = blockIdx.x;
    const int tc = b % P.tiles_c; b /= P.tiles_c;
    const int tk = b % P.tiles_k; b /= P.tiles_k;
    const int tap = b % (P.R * P.S);
    const int split = b / (P.R * P.S);
    const int r = tap / P.S, s = tap % P.S;
    const int k0 = tk * BM, c0 = tc * BN;
    const int oh = r * P.dh - P.ph, ow = s * P.dw - P.pw;

    const int step0 = split * P.steps_per_split;
    int nsteps = (P.P + kF32BP - 1) / kF32BP - step0;
    if (nsteps > P.steps_per_split) nsteps = P.steps_per_split;

    const int ga_row = tid / TA, ga_col = (tid % TA) * 4;
    const int xb_row = tid / TB, xb_col = (tid % TB) * 4;
    const bool ga_ok = k0 + ga_col < P.K;                   // K and C are multiples of 4
    const bool xb_ok = c0 + xb_col < P.C;

    f32x4 rg[PA], rx[PB];
    auto prefetch = [&](int step) {
        const int p0 = (step0 + step) * kF32BP;
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            int p = p0 + ga_row + i * RA;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (ga_ok && p < P.P) v = *reinterpret_cast<const f32x4*>(P.G + ((long)p * P.K + k0 + ga_col));
            rg[i] = v;
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            int p = p0 + xb_row + i * RB;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (xb_ok && p < P.P) {
                int n = p / (P.Ho * P.Wo);
                int rem = p - n * (P.Ho * P.Wo);
                int ho = rem / P.Wo, wo = rem - ho * P.Wo;
                int h = ho * P.sh + oh, w = wo * P.sw + ow;
                if ((unsigned)h < (unsigned)P.H && (unsigned)w < (unsigned)P.W)
                    v = *reinterpret_cast<const f32x4*>(P.X + ((((long)n * P.H + h) * P.W + w) * P.C + c0 + xb_col));
            }
            rx[i] = v;
        }
    };
    // odd pixel rows keep their columns XOR 32: the two rows one fragment read touches then lie
    // on different banks
    auto stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            int row = ga_row + i * RA;
            *reinterpret_cast<f32x4*>(ldsG + (buf * kF32BP + row) * BM + (ga_col ^ ((row & 1) << 5))) = rg[i];
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            int row = xb_row + i * RB;
            *reinterpret_cast<f32x4*>(ldsX + (buf * kF32BP + row) * BN + (xb_col ^ ((row & 1) << 5))) = rx[i];
        }
    };

    f32x16 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][c][e] = 0.f;

    const int l32 = lane & 31, lhi = lane >> 5;
    auto compute = [&](int buf) {
#pragma unroll
        for (int t = 0; t < kF32BP / 2; ++t) {
            const int row = 2 * t + lhi;            // pixel of the step: parity == lhi
            const float* sg = ldsG + (buf * kF32BP + row) * BM;
            const float* sx = ldsX + (buf * kF32BP + row) * BN;
            float fa[FM], fb[FN];
#pragma unroll
            for (int a = 0; a < FM; ++a) fa[a] = sg[(wm * WM + a * 32 + l32) ^ (lhi << 5)];
#pragma unroll
            for (int c = 0; c < FN; ++c) fb[c] = sx[(wn * WN + c * 32 + l32) ^ (lhi << 5)];
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int c = 0; c < FN; ++c)
                    acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[a], fb[c], acc[a][c], 0, 0, 0);
        }
    };

    if (nsteps > 0) {
        prefetch(0);
        stage(0);
        __syncthreads();
        for (int it = 0; it < nsteps; ++it) {
            const bool more = it + 1 < nsteps;
            if (more) prefetch(it + 1);
            compute(it & 1);
            if (more) stage((it + 1) & 1);
            __syncthreads();
        }
    }

    const long numel = (long)P.K * P.R * P.S * P.C;
    float* out = P.out + (long)split * numel;
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int c = 0; c < FN; ++c) {
            int col = c0 + wn * WN + c * 32 + l32;
            if (col >= P.C) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                int k = k0 + wm * WM + a * 32 + 8 * (e >> 2) + 4 * lhi + (e & 3);
                if (k < P.K) out[((long)k * P.R * P.S + tap) * P.C + col] = acc[a][c][e];
            }
        }
}

// ---- host side -----------------------------------------------------------------------------------
static size_t f32_align256(size_t b) { return (b + 255) & ~(size_t)255; }

bool f32_supported(const Geom& g)
{
    return g.C % 4 == 0 && g.K % 4 == 0 && g.R * g.S <= kMaxTaps && g.sh * g.sw <= kMaxClasses;
}

// The split-role kernels address with 32-bit byte offsets, of which those from 2^31 on mean "outside".
static bool f32_byte_offsets_fit_31_bits(const Geom& g)
{
    const long lim = 1L << 29;
    return (long)g.N * g.H * g.W * g.C < lim && (long)g.N * g.Ho * g.Wo * g.K < lim && (long)g.K * g.R * g.S * g.C < lim;
}

static void f32_staged_wgrad_shape(const Geom& g, int* bm, int* bn, int* splits, int* sps)
{
    *bm = g.K <= 64 ? 64 : 128;
    *bn = g.C <= 64 ? 64 : 128;
    const long tiles = (long)((g.K + *bm - 1) / *bm) * ((g.C + *bn - 1) / *bn) * g.R * g.S;
    const long total_steps = ((long)g.N * g.Ho * g.Wo + kF32BP - 1) / kF32BP;
    // enough pixel ranges for two workgroups per compute unit, in whole multiples of the unit count
    long cap = total_steps / 8;
    if (cap < 1) cap = 1;
    long want = 1;
    double best = -1.0;
    for (long sp = 1; sp <= cap && sp * tiles <= 2048; ++sp) {
        const long wgs = sp * tiles;
        const double fill = (double)wgs / (double)(((wgs + 255) / 256) * 256);
        const double enough = wgs >= 512 ? 1.0 : (double)wgs / 512.0;
        const double score = fill * enough - 1e-5 * sp;         // ties: fewer partial sums
        if (score > best) { best = score; want = sp; }
    }
    const long per = (total_steps + want - 1) / want;
    *sps = (int)per;
    *splits = (int)((total_steps + per - 1) / per);
}

// Tiles of the split-role weight gradient and their times, as for the tiles below; partial sums and dw are
// stored at `store` MB/us and added at kF32ReduceRate, after kF32ReduceFixed for the second kernel.  Fitted to 162
// layers: on layers left out 1.7 % slower than the fastest pair of tile and ranges (5.8 % at the 90th
// percentile).  Layers of 20 GFLOP and more run at 103 to 135 TFLOP/s where they are pointwise (a 128x128x32 step
// takes 1.9-2.1 us) and at 79 to 109 where pixels are gathered (2.5-2.8 us; one `step` serves both, so the
// choice leans a little away from that tile in pointwise layers); the register-staged kernel ran at 70 to 95.
struct F32WgradTile { int bm, bn, per_cu; float step, shared, tile, fixed, store; };
static const F32WgradTile kF32WgradTiles[] = {
    {128, 128, 2, 2.209f, 2.224f, 0.056f, 4.515f, 2.655f},
    {128, 64, 2, 1.356f, 1.199f, 0.863f, 3.357f, 2.591f},
    {64, 128, 2, 1.372f, 1.233f, 1.405f, 2.979f, 2.647f},
    {64, 64, 3, 0.630f, 0.587f, 0.824f, 2.690f, 2.480f},
};
constexpr float kF32ReduceFixed = 2.5f, kF32ReduceRate = 6.0f;

static F32WgradShape f32_wgrad_shape(const Geom& g)
{
    F32WgradShape out;
    f32_staged_wgrad_shape(g, &out.bm, &out.bn, &out.splits, &out.sps);
    out.ws = f32_byte_offsets_fit_31_bits(g) && g.K < 1 << 24 && g.C < 1 << 24;     // 32 pixels' rows within the offsets
    if (!out.ws) return out;
    // no more ranges, hence no more workspace, than the register-staged kernel takes
    const int forced = forced_f32_tile() - 100, forced_splits = forced_wgrad_splits();
    const int total = (int)(((long)g.N * g.Ho * g.Wo + kF32BP - 1) / kF32BP);
    const int least = forced_splits > 0 && forced_splits <= total ? forced_splits : 1, most = forced_splits > 0 ? least : out.splits;
    const float mb = 4e-6f * g.K * g.R * g.S * g.C;
    float best = 0.f;
    bool any = false;
    for (int i = 0; i < 4; ++i) {
        const F32WgradTile& t = kF32WgradTiles[i];
        if (forced >= 0 && forced < 4 && i != forced) continue;
        const int tiles = ((g.K + t.bm - 1) / t.bm) * ((g.C + t.bn - 1) / t.bn) * g.R * g.S;
        // no compute unit takes less than an even share of all steps, at its best rate
        const float rate = t.shared > t.step / t.per_cu ? t.shared : t.step / t.per_cu;
        const float even = (t.fixed + (float)tiles * total * rate / 256) * 0.9999f;
        int last = 0;
        for (const int workgroups : {0, 32, 64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048}) {
            int n = workgroups / tiles;
            n = n < least ? least : n > most ? most : n;
            if (n == last) continue;
            last = n;
            const int sps = (total + n - 1) / n, splits = (total + sps - 1) / sps;
            if (any && even + splits * mb / t.store * 0.9999f >= best) break;       // and so do more ranges
            const int fullest = (splits * tiles + 255) / 256, rest = fullest % t.per_cu;
            auto round = [&](int c) { return sps * (c * t.shared > t.step ? c * t.shared : t.step) + t.tile; };
            float us = t.fixed + fullest / t.per_cu * round(t.per_cu) + (rest ? round(rest) : 0.f) + splits * mb / t.store;
            if (splits > 1) us += kF32ReduceFixed + splits * mb / kF32ReduceRate;
            if (!any || us < best) {
                any = true;
                best = us;
                out.bm = t.bm; out.bn = t.bn; out.splits = (int)splits; out.sps = (int)sps;
            }
        }
    }
    return out;
}

F32Plan plan_f32(const Geom& g, int pass)
{
    F32Plan p{};
    if (!f32_supported(g)) return p;
    const size_t w = (size_t)g.K * g.R * g.S * g.C * sizeof(float);
    if (pass == SDCONV_DGRAD) p.workspace_bytes = f32_align256(w);
    if (pass == SDCONV_WGRAD) {
        p.wgrad = f32_wgrad_shape(g);
        if (p.wgrad.splits > 1) p.workspace_bytes = f32_align256(p.wgrad.splits * w);
    }
    return p;
}

template <int MODE, int BM, int BN, int WGM, int WGN, int WGK>
static hipError_t launch_f32_variant(const F32Params& P, hipStream_t st)
{
    constexpr size_t lds = f32_lds_bytes<BM, BN, WGK>();
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&igemm_f32_kernel<MODE, BM, BN, WGM, WGN, WGK>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((igemm_f32_kernel<MODE, BM, BN, WGM, WGN, WGK>), dim3(P.total_tiles), dim3(256), lds, st, P);
    return hipGetLastError();
}

// Tiles, and the time each takes: us per step and tile where a tile has a compute unit to itself (`step`) or
// several share one (`shared` each, at most `per_cu` at a time), us per tile besides, launch
// and first loads.  Fits to the fp32 timings in profiles/layer_timings_before_runs.jsonl.gz (fit_models.py: 710 passes of
// 354 layers of random size, 200 to 150 000 pixels, 8 to 2048 channels): on layers left out of the fit the
// choice is 1.2 % slower than the fastest tile (5.4 % at the 90th percentile).  On 1190 passes of the present kernels
// (layer_timings.jsonl.gz) it is 2.32 % slower, and a fit to those 2.30 % on layers left out.  Against the fastest register-staged
// tile it takes 16 % less time on average.  Those are the faster ones at times, with few channels on one
// side or four steps of contraction, and serve tensors that the split-role kernels do not address: they stay in
// the choice, which without them is 0.2 % slower.  A split-role 32x32 tile takes 0.19 us a step beside
// others where a staged one takes 0.22 (alone 0.36 and 0.64), 64x64 0.55 and 0.67: nothing is left between the
// loads and the matrix pipe but the barrier.  160x64, 96x128, 96x64, 96x32, 128x32 and 32x64 split-role tiles were
// measured too and gain 0.3 % together.
struct F32Tile {
    int bm, bn, per_cu;
    float step, shared, tile, fixed;
    hipError_t (*launch[2])(const F32Params&, hipStream_t);     // forward, data gradient
};
#define F32_TILE(BM, BN, WGM, WGN, WGK) {launch_f32_variant<0, BM, BN, WGM, WGN, WGK>, launch_f32_variant<1, BM, BN, WGM, WGN, WGK>}
static const F32Tile kF32Tiles[] = {
    // launch_igemm_ws_f32
    {128, 128, 1, 2.243f, 2.243f, 3.814f, 2.247f, {}},
    {128, 64, 2, 1.370f, 1.173f, 4.633f, 0.500f, {}},
    {64, 64, 3, 0.717f, 0.545f, 3.935f, 0.984f, {}},
    {64, 32, 4, 0.530f, 0.331f, 3.465f, 1.755f, {}},
    {32, 32, 6, 0.361f, 0.191f, 4.505f, 0.522f, {}},
    // register-staged
    {128, 128, 2, 2.525f, 2.341f, 5.690f, 0.500f, F32_TILE(128, 128, 2, 2, 1)},
    {128, 64, 3, 1.554f, 1.242f, 5.307f, 0.500f, F32_TILE(128, 64, 2, 2, 1)},
    {96, 64, 3, 1.247f, 0.952f, 5.661f, 0.500f, F32_TILE(96, 64, 1, 2, 2)},
    {64, 64, 4, 1.043f, 0.672f, 4.307f, 0.516f, F32_TILE(64, 64, 2, 2, 1)},
    {32, 64, 6, 0.687f, 0.369f, 3.635f, 1.326f, F32_TILE(32, 64, 1, 2, 2)},
    {32, 32, 5, 0.640f, 0.215f, 3.030f, 1.726f, F32_TILE(32, 32, 1, 1, 4)},
};
#undef F32_TILE
constexpr int kNumF32Tiles = sizeof(kF32Tiles) / sizeof(kF32Tiles[0]), kF32WsTiles = 5;

// Row tiles of height bm (all parity classes of a strided data gradient), and those among them that have
// taps, with their taps summed.
struct F32Rows { long all, busy; double taps; int classes, most; };      // most: taps of a tile
static F32Rows f32_row_tiles(const RowClasses& rows, unsigned bm)
{
    F32Rows out{0, 0, 0., rows.n, 0};
    for (int q = 0; q < rows.n; ++q) {
        const long tiles = (rows.pixels[q] + bm - 1) / bm;
        const int taps = rows.taps[q];
        out.all += tiles;
        if (taps) out.busy += tiles;
        out.taps += (double)tiles * taps;
        if (tiles && taps > out.most) out.most = taps;
    }
    return out;
}

static double f32_us(const RowClasses& classes, int cs, int cd, const F32Tile& t)
{
    const F32Rows rows = f32_row_tiles(classes, t.bm);
    if (rows.busy == 0) return t.fixed;
    const long columns = (cd + t.bn - 1) / t.bn, slabs = (cs + kF32BK - 1) / kF32BK;
    if (rows.classes > 1) {
        // parity classes: tiles of different length fill the units evenly but for the last ones; one that no tap
        // reaches only stores zeros
        const double tiles = (rows.busy + 0.6 * (rows.all - rows.busy)) * columns;
        const double even = (rows.taps * columns * slabs * t.shared + tiles * t.tile / t.per_cu) / 256;
        const double last = (double)rows.most * slabs * t.step + t.tile;
        return t.fixed + (even > 0.5 * last ? even + 0.5 * last : last);
    }
    const double steps = rows.taps / rows.busy * slabs;
    const long fullest = (rows.busy * columns + 255) / 256;    // tiles of one compute unit
    auto round = [&](long n) { return steps * (n * t.shared > t.step ? n * t.shared : t.step) + t.tile; };
    const long rest = fullest % t.per_cu;
    return t.fixed + fullest / t.per_cu * round(t.per_cu) + (rest ? round(rest) : 0.);
}

// Fields that the parameters of both kernels have.
template <typename Params>
static bool f32_fill(const Geom& g, bool dgrad, const RowClasses& rows, const F32Tile& tile, Params* P)
{
    P->NB = g.N;
    if (!dgrad) { P->Hs = g.H; P->Ws = g.W; P->Cs = g.C; P->Hd = g.Ho; P->Wd = g.Wo; P->Cd = g.K; }
    else        { P->Hs = g.Ho; P->Ws = g.Wo; P->Cs = g.K; P->Hd = g.H; P->Wd = g.W; P->Cd = g.C; }
    P->R = g.R; P->S = g.S;
    P->sh = g.sh; P->sw = g.sw; P->ph = g.ph; P->pw = g.pw; P->dh = g.dh; P->dw = g.dw;
    P->sw_cls = dgrad ? g.sw : 1;
    P->b_row_pitch = g.R * g.S * P->Cs;
    P->tiles_n = (P->Cd + tile.bn - 1) / tile.bn;
    long tiles = 0;
    P->nclasses = rows.n;
    for (int q = 0; q <= rows.n; ++q) {
        P->class_tile_start[q] = (int)tiles;
        if (q < rows.n) tiles += (rows.pixels[q] + (unsigned)tile.bm - 1) / tile.bm;
    }
    const long total = tiles * P->tiles_n;
    if (total <= 0 || total > 0x7fffffc0L) return false;
    P->total_tiles = (int)total;
    return true;
}

static hipError_t run_f32_igemm(const Geom& g, bool dgrad, const float* A, const float* B, float* D, hipStream_t st)
{
    const bool ws = f32_byte_offsets_fit_31_bits(g);
    const int first = ws ? 0 : kF32WsTiles;
    int pick = first;
    const RowClasses rows = row_classes(g, dgrad);
    const int cs = dgrad ? g.K : g.C, cd = dgrad ? g.C : g.K;
    double best = f32_us(rows, cs, cd, kF32Tiles[first]);
    for (int i = first + 1; i < kNumF32Tiles; ++i) {
        const double us = f32_us(rows, cs, cd, kF32Tiles[i]);
        if (us < best) { best = us; pick = i; }
    }
    const int forced = forced_f32_tile();
    if (forced >= first && forced < kNumF32Tiles) pick = forced;
    const F32Tile& tile = kF32Tiles[pick];
    if (pick >= kF32WsTiles) {
        F32Params P;
        P.A = A; P.B = B; P.D = D;
        return f32_fill(g, dgrad, rows, tile, &P) ? tile.launch[dgrad](P, st) : hipErrorInvalidValue;
    }
    IgemmParams P{};
    if (!f32_fill(g, dgrad, rows, tile, &P)) return hipErrorInvalidValue;
    P.A = reinterpret_cast<const __half*>(A); P.B = reinterpret_cast<const __half*>(B); P.D = reinterpret_cast<__half*>(D);
    P.Cs *= 2; P.b_row_pitch *= 2;              // counted in halves
    P.mode = dgrad;
    set_taps(g, dgrad, &P);
    return launch_igemm_ws_f32(pick, P, st);
}

hipError_t run_fwd_f32(const Geom& g, const float* x, const float* w, float* y, hipStream_t st)
{
    if (!f32_supported(g)) return launch_direct_fwd_f32(g, x, w, y, st);
    return run_f32_igemm(g, false, x, w, y, st);
}

hipError_t run_dgrad_f32(const Geom& g, const float* dy, const float* w, float* dx, void* ws, hipStream_t st)
{
    if (!f32_supported(g)) return launch_direct_dgrad_f32(g, dy, w, dx, st);
    float* wT = static_cast<float*>(ws);
    dim3 grid((g.C + 31) / 32, (g.K + 31) / 32, g.R * g.S);
    hipLaunchKernelGGL(filter_transpose_f32_kernel, grid, dim3(256), 0, st, w, wT, g.K, g.R * g.S, g.C);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return run_f32_igemm(g, true, dy, wT, dx, st);
}

template <int BM, int BN>
static hipError_t launch_f32_wgrad(const F32WgradParams& P, hipStream_t st)
{
    constexpr size_t lds = 2 * kF32BP * (BM + BN) * sizeof(float);
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_f32_kernel<BM, BN, 2, 2>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    long blocks = (long)P.tiles_c * P.tiles_k * P.R * P.S * P.splits;
    hipLaunchKernelGGL((wgrad_f32_kernel<BM, BN, 2, 2>), dim3((unsigned)blocks), dim3(256), lds, st, P);
    return hipGetLastError();
}

hipError_t run_wgrad_f32(const Geom& g, const F32Plan& plan, const float* x, const float* dy, float* dw, void* ws, hipStream_t st)
{
    if (!f32_supported(g)) return launch_direct_wgrad_f32(g, x, dy, dw, st);
    F32WgradParams P;
    const F32WgradShape& shape = plan.wgrad;
    const int bm = shape.bm, bn = shape.bn;
    P.splits = shape.splits;
    P.steps_per_split = shape.sps;
    P.X = x; P.G = dy;
    P.N = g.N; P.H = g.H; P.W = g.W; P.C = g.C; P.K = g.K; P.R = g.R; P.S = g.S;
    P.sh = g.sh; P.sw = g.sw; P.ph = g.ph; P.pw = g.pw; P.dh = g.dh; P.dw = g.dw;
    P.Ho = g.Ho; P.Wo = g.Wo;
    P.P = g.N * g.Ho * g.Wo;
    P.tiles_k = (g.K + bm - 1) / bm;
    P.tiles_c = (g.C + bn - 1) / bn;
    P.out = P.splits > 1 ? static_cast<float*>(ws) : dw;
    hipError_t e;
    if (shape.ws) e = launch_wgrad_ws_f32(bm, bn, P, st);
    else if (bm == 128 && bn == 128) e = launch_f32_wgrad<128, 128>(P, st);
    else if (bm == 128) e = launch_f32_wgrad<128, 64>(P, st);
    else if (bn == 128) e = launch_f32_wgrad<64, 128>(P, st);
    else e = launch_f32_wgrad<64, 64>(P, st);
    if (e != hipSuccess || P.splits == 1) return e;
    return launch_splitk_reduce(static_cast<const float*>(ws), dw, P.splits, (long)g.K * g.R * g.S * g.C, st);
}

}  // namespace sdconv
