// Weight gradient on binary32 tensors with waves that only fetch: the tiles and LDS layout of wgrad_f32_kernel
// (conv_f32.hip), [pixel][channel] with the columns of odd pixels XOR 32, filled by LDS-DMA through a
// ring of S stages.  The staged kernel divided twice for every load and waited for its loads once a step; here a
// lane divides once a step.  Bound by the matrix pipe in large layers (103-135 TFLOP/s pointwise, 79-109 where pixels
// are gathered), in small ones by the partial sums of its pixel ranges: one workgroup a compute unit keeps the
// pipe as busy as two did, so there are fewer ranges.
// Chains are folded every 64 pixels, or the longer ranges would double the error (res4: 3.2e-7 -> 6.9e-7; now 1.7e-7).
#include "common.h"
#include "dma.h"
#include "wgrad.h"

namespace sdconv {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int BM, int BN, int WGM, int WGN, int S>
__global__ __launch_bounds__(64 * (WGM * WGN + 2)) void wgrad_ws_f32_kernel(F32WgradParams P)
{
    constexpr int NWC = WGM * WGN, NI = 2;              // multiplying and fetching waves
    constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 32, FN = WN / 32;
    constexpr int BP = kF32BP;                          // pixels of a step
    constexpr int NG = BM / 8, NX = BN / 8;             // load instructions of a stage, 1 KiB each: dy rows, then x rows
    constexpr int PG = NG / NI, PX = NX / NI;           // ... and of one fetching wave
    constexpr int GROWS = 256 / BM, XROWS = 256 / BN;   // pixels of a load instruction
    constexpr int STAGE = (NG + NX) * 1024, INFLIGHT = (S - 2) * (PG + PX);
    static_assert(BP * 4 == 128 && NG % NI == 0 && NX % NI == 0 && BM >= 64 && BN >= 64 && BM <= 128 && BN <= 128, "tile shape");
    static_assert(WM % 32 == 0 && WN % 32 == 0 && S >= 2 && INFLIGHT < 64, "pipeline");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    // Every XCD takes a run of consecutive workgroups: the tiles of one pixel range, which read the same
    // pixels, then share an L2.
    const int chunk = gridDim.x >> 3;
    int b = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    if (b >= P.tiles_c * P.tiles_k * P.R * P.S * P.splits) return;
    const int tc = b % P.tiles_c; b /= P.tiles_c;
    const int tk = b % P.tiles_k; b /= P.tiles_k;
    const int tap = b % (P.R * P.S);
    const int split = b / (P.R * P.S);
    const int k0 = tk * BM, c0 = tc * BN;

    const int step0 = split * P.steps_per_split;
    int nk = (P.P + BP - 1) / BP - step0;
    if (nk > P.steps_per_split) nk = P.steps_per_split;

    if (wave >= NWC) {
        // ---- fetching wave: every second load instruction of a stage, S-1 steps ahead ----
        const int fw = wave - NWC;
        const int grow = lane / (BM / 4), xrow = lane / (BN / 4);       // pixel within a load instruction
        const int gcol = k0 + ((lane % (BM / 4)) ^ ((grow & 1) << 3)) * 4;
        const int xcol = c0 + ((lane % (BN / 4)) ^ ((xrow & 1) << 3)) * 4;
        const unsigned goff = gcol < P.K ? (unsigned)((fw * GROWS + grow) * P.K + gcol) * 4u : kOutOfRange;
        const unsigned xoff = xcol < P.C ? (unsigned)((fw * XROWS + xrow) * P.C + xcol) * 4u : kOutOfRange;
        const unsigned gstep = (unsigned)(NI * GROWS * P.K) * 4u, xstep = (unsigned)(NI * XROWS * P.C) * 4u;
        const int oh = (tap / P.S) * P.dh - P.ph, ow = (tap % P.S) * P.dw - P.pw;
        const bool linear = P.R * P.S == 1 && P.sh == 1 && P.sw == 1 && P.ph == 0 && P.pw == 0;
        const int4v rsrcX = make_rsrc(P.X, (unsigned)((long)P.N * P.H * P.W * P.C * 4));
        auto issue = [&](int q, int stage) {
            const int p0 = (step0 + q) * BP;
            const unsigned sbase = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds0 + stage * STAGE + fw * 1024));
            // descriptors that start at the step's first pixel and end with the tensor: pixels past the
            // last one read as zeros
            const int4v rsrcG = make_rsrc(P.G + (long)p0 * P.K, (unsigned)((long)(P.P - p0) * P.K * 4));
            if (linear) {
                const int4v rsrcL = make_rsrc(P.X + (long)p0 * P.C, (unsigned)((long)(P.P - p0) * P.C * 4));
#pragma unroll
                for (int i = 0; i < PG; ++i) dma16(goff == kOutOfRange ? goff : goff + i * gstep, rsrcG, 0, sbase + i * NI * 1024);
#pragma unroll
                for (int i = 0; i < PX; ++i)
                    dma16(xoff == kOutOfRange ? xoff : xoff + i * xstep, rsrcL, 0, sbase + NG * 1024 + i * NI * 1024);
            } else {
                // lane l finds where pixel l % 32 of the step lies in x under this tap; the loads ask it
                const int p = p0 + (lane & 31);
                const int n = p / (P.Ho * P.Wo), rem = p - n * (P.Ho * P.Wo);
                const int ho = rem / P.Wo, wo = rem - ho * P.Wo;
                const int h = ho * P.sh + oh, w = wo * P.sw + ow;
                const bool in = p < P.P && (unsigned)h < (unsigned)P.H && (unsigned)w < (unsigned)P.W;
                const unsigned pix = in ? (unsigned)(((n * P.H + h) * P.W + w) * P.C) * 4u : kOutOfRange;
                unsigned xo[PX];
#pragma unroll
                for (int i = 0; i < PX; ++i) {
                    const unsigned at = (unsigned)__shfl((int)pix, (i * NI + fw) * XROWS + xrow);
                    xo[i] = at == kOutOfRange || xcol >= P.C ? kOutOfRange : at + (unsigned)xcol * 4u;
                }
#pragma unroll
                for (int i = 0; i < PG; ++i) dma16(goff == kOutOfRange ? goff : goff + i * gstep, rsrcG, 0, sbase + i * NI * 1024);
#pragma unroll
                for (int i = 0; i < PX; ++i) dma16(xo[i], rsrcX, 0, sbase + NG * 1024 + i * NI * 1024);
            }
        };
        int is = 0;
#pragma unroll 1
        for (int q = 0; q < nk; ++q) {
            if (q >= S - 1) {
                wait_vmcnt<INFLIGHT>();
                stage_barrier();       // step q-(S-1) is in LDS; the stage before it is free
            }
            issue(q, is);
            is = (is + 1 == S) ? 0 : is + 1;
        }
        for (int it = nk > S - 1 ? nk - (S - 1) : 0; it < nk; ++it) {
            if (it + S - 2 < nk) wait_vmcnt<INFLIGHT>(); else wait_vmcnt<0>();
            stage_barrier();
        }
        return;
    }

    const int wm = wave / WGN, wn = wave % WGN, l32 = lane & 31, lhi = lane >> 5;
    f32x16 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][c][e] = 0.f;
    // what a chain of kFoldSteps steps has added up goes to sums of its own: the rounding errors then do not
    // grow with the number of pixels of a range
    constexpr int kFoldSteps = 2;
    f32x16 sum[FM][FN] = {};
    int cs = 0;
    for (int it = 0; it < nk; ++it) {
        stage_barrier();
        const float* sg = reinterpret_cast<const float*>(smem + cs * STAGE);
        const float* sx = sg + BP * BM;
#pragma unroll
        for (int t = 0; t < BP / 2; ++t) {
            const int row = 2 * t + lhi;            // pixel of the step: parity == lhi
            float fa[FM], fb[FN];
#pragma unroll
            for (int a = 0; a < FM; ++a) fa[a] = sg[row * BM + ((wm * WM + a * 32 + l32) ^ (lhi << 5))];
#pragma unroll
            for (int c = 0; c < FN; ++c) fb[c] = sx[row * BN + ((wn * WN + c * 32 + l32) ^ (lhi << 5))];
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int c = 0; c < FN; ++c)
                    acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[c], fa[a], acc[a][c], 0, 0, 0);
        }
        if (it % kFoldSteps == kFoldSteps - 1) {
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int c = 0; c < FN; ++c)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        sum[a][c][e] += acc[a][c][e];
                        acc[a][c][e] = 0.f;
                    }
        }
        cs = (cs + 1 == S) ? 0 : cs + 1;
    }

#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][c][e] += sum[a][c][e];

    // a lane holds four consecutive channels of a filter: 16-byte stores
    float* out = P.out + (long)split * P.K * P.R * P.S * P.C;
#pragma unroll
    for (int a = 0; a < FM; ++a) {
        const int k = k0 + wm * WM + a * 32 + l32;
        if (k >= P.K) continue;
        float* row = out + ((long)k * P.R * P.S + tap) * P.C;
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = c0 + wn * WN + c * 32 + 8 * q + 4 * lhi;
                if (col < P.C) {
                    const f32x4 v = {acc[a][c][4 * q], acc[a][c][4 * q + 1], acc[a][c][4 * q + 2], acc[a][c][4 * q + 3]};
                    *reinterpret_cast<f32x4*>(row + col) = v;
                }
            }
    }
}

template <int BM, int BN, int WGM, int WGN, int S>
static hipError_t launch_one(const F32WgradParams& P, hipStream_t st)
{
    constexpr size_t lds = (size_t)S * kF32BP * (BM + BN) * sizeof(float);
    static_assert(lds <= 160 * 1024, "LDS budget");
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_ws_f32_kernel<BM, BN, WGM, WGN, S>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    const long blocks = (long)P.tiles_c * P.tiles_k * P.R * P.S * P.splits;
    hipLaunchKernelGGL((wgrad_ws_f32_kernel<BM, BN, WGM, WGN, S>), dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(64 * (WGM * WGN + 2)),
                       lds, st, P);
    return hipGetLastError();
}

hipError_t launch_wgrad_ws_f32(int bm, int bn, const F32WgradParams& P, hipStream_t st)
{
    if (bm == 128 && bn == 128) return launch_one<128, 128, 2, 4, 2>(P, st);
    if (bm == 128 && bn == 64) return launch_one<128, 64, 2, 2, 3>(P, st);
    if (bm == 64 && bn == 128) return launch_one<64, 128, 2, 2, 3>(P, st);
    if (bm == 64 && bn == 64) return launch_one<64, 64, 2, 2, 3>(P, st);
    return hipErrorInvalidValue;
}

}  // namespace sdconv
