// Stride-1 3x3-class forward / data-gradient kernel that keeps the input patch in LDS.
//
// The implicit-GEMM kernels fetch the activation tile once per filter tap: a 3x3 layer reads
// (nearly) the same pixels nine times from L2 and the global->LDS path, not the MFMA pipe,
// sets the pace.  Here a workgroup owns a TH x TW block of output pixels of one image and,
// per 64-channel slab, loads the (TH+2) x (TW+2) input patch ONCE (halo included, pixels
// outside the image zero-filled by the buffer range check = the padding).  The nine taps then
// read their A fragments from the same patch at a per-tap pixel displacement; only the filter
// slab (BN rows x 64 channels per tap) still streams through a ring, one stage per tap.
// Activation traffic drops from 9x to (TH+2)(TW+2)/(TH*TW) = 1.27x (16x16) per slab.
//
// Roles: either the upper half of the waves sends all loads (see igemm_ws.hip for why) and every
// wave multiplies, or extra waves do nothing but fetch (NDW below).  Two patch buffers alternate
// between slabs; the patch of slab kc+1 is requested at the first tap of slab kc and, because
// loads retire in order, has landed by the time the filter stage of its first tap has.
//
// Valid for stride 1, (R-1)*dil_h == 2 and (S-1)*dil_w == 2 (3x3 dilation 1 in particular),
// source channels a multiple of 64.  The data gradient of such a layer is the same kind of
// convolution over dy with displaced taps; it reads the filter as stored, [K][R][S][C], as
// 64-filter x BN-channel tiles that the transposing LDS read turns into fragments (lds_tr.h).
#include "common.h"
#include "igemm.h"
#include "dma.h"
#include "igemm_epilogue.h"
#include "lds_tr.h"

namespace sdconv {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4p __attribute__((ext_vector_type(4)));

// TH*TW need not be a multiple of the MFMA block height: the GEMM rows are padded up to
// WGM*MF and the padding rows are multiplied but never stored.  10 x 14 blocks tile the
// 100 x 168 and 50 x 84 feature maps of the res3 / res4 stages exactly.
// A step of one tap is only 64 deep; on small tiles the barrier and the wait then cost as much as the MFMAs
// between them, so a step covers a whole filter row (TPS taps), and a ring stage holds TPS filter slabs.
// NPB: patch buffers.  Two alternate between channel slabs; a layer with 64 source channels has
// one slab and needs one buffer, which lets two or three workgroups share a compute unit's LDS
// (its 134 400-pixel maps make 546-1050 blocks: at one workgroup per unit they run in 3-4 rounds).
// NDW: waves that only fetch, beside the WGM x WGN multiplying ones (then none of those fetches).
// A wave stalls ~90 cycles in every LDS-DMA instruction it sends; with a dozen per step the
// fetching waves of a small block reach the barrier a thousand cycles after the others
// (timestamps of a 10 x 14 x 64 block: 1500 cycles of multiplying and 1200 of waiting per
// step).  Waves with nothing else to do take the stalls off that path.
constexpr int MF = 16, TPS = 3;     // rows of a v_mfma_f32_16x16x32_f16 block, taps of a step

template <int MODE, int TH, int TW, int BN, int WGM, int WGN, int SB, int NPB, int NDW, bool TAIL>
__global__ __launch_bounds__(64 * (WGM * WGN + NDW)) void conv_patch_kernel(IgemmParams P)
{
    constexpr int EH = 2, EW = 2;                   // extra patch rows / columns
    constexpr int PH = TH + EH, PW = TW + EW, PPX = PH * PW;
    constexpr int NW = WGM * WGN, NI = NDW ? NDW : NW / 2, IW0 = NDW ? NW : NW - NI;
    constexpr int BM = TH * TW;                             // output pixels of the block
    constexpr int BMP = (BM + MF * WGM - 1) / (MF * WGM) * (MF * WGM);   // GEMM rows incl. padding
    constexpr int WM = BMP / WGM, WN = BN / WGN;
    constexpr int FM = WM / MF, FN = WN / MF;
    constexpr int ACCN = 4, KSTEP = 32, CPK = KSTEP / 8;
    constexpr int NPL = (PPX + 8 * NI - 1) / (8 * NI);     // patch loads per fetching lane
    constexpr int PATCHB = NPL * NI * 1024;                // bytes of one patch buffer
    constexpr int PB1 = BN / (8 * NI);                     // filter loads per fetching lane and tap
    constexpr int PB = TPS * PB1;                          // ... and step
    constexpr int BSLAB = BN * 128;                        // one tap's filter slab
    constexpr int BSTAGE = TPS * BSLAB;
    constexpr int D = SB - 1;                              // filter stages in flight
    static_assert(NI >= 1 && (NDW > 0 || NI < NW) && WM % MF == 0 && WN % MF == 0 && BN % (8 * NI) == 0, "tile shape");
    static_assert(SB >= 2 && NPL + D * PB < 64, "loads in flight");   // vmcnt is a 6-bit counter
    static_assert(NPB == 1 || NPB == 2, "patch buffers");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    unsigned char* bring = smem + NPB * PATCHB;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- which tile: runs of 8 consecutive tiles per XCD, runs interleaved over the XCDs ------
    constexpr int kRun = 8;
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int tile = ((idx / kRun) * 8 + xcd) * kRun + (idx % kRun);
    if (tile >= P.total_tiles) return;
    const int tn = tile % P.tiles_n;
    int t2 = tile / P.tiles_n;
    const int tx = t2 % P.tiles_w; t2 /= P.tiles_w;
    const int ty = t2 % P.tiles_h;
    const int n = t2 / P.tiles_h;
    const int h0 = ty * TH, w0 = tx * TW, n0 = tn * BN;

    // source pixel of output pixel (h, w) at tap (r, s): (h + oh, w + ow)
    const int oh_min = (MODE == 0) ? -P.ph : P.ph - (P.R - 1) * P.dh;
    const int ow_min = (MODE == 0) ? -P.pw : P.pw - (P.S - 1) * P.dw;
    const int ntaps = P.R * P.S;
    const int kchunks = P.Cs / 64;
    const int ngroups = ntaps / TPS;                // steps per channel slab
    const int nk = ngroups * kchunks;

    // ---- fetching side ---------------------------------------------------------------------
    const bool fetcher = wave >= IW0;
    const int fw = wave - IW0;
    const int fpix = lane >> 3, fslot = lane & 7;   // pixel (or filter row) within an instruction, chunk slot
    unsigned a_off[NPL], b_off[PB1];
    if (fetcher) {
#pragma unroll
        for (int q = 0; q < NPL; ++q) {
            const int pp = (q * NI + fw) * 8 + fpix;            // patch pixel this lane fetches
            const int kcl = fslot ^ ((pp >> 1) & 7);            // logical chunk that lands in slot fslot
            const int pr = pp / PW, pc = pp - pr * PW;
            const int hs = h0 + oh_min + pr, ws = w0 + ow_min + pc;
            const bool ok = pp < PPX && (unsigned)hs < (unsigned)P.Hs && (unsigned)ws < (unsigned)P.Ws;
            a_off[q] = ok ? (unsigned)((((n * P.Hs + hs) * P.Ws + ws) * P.Cs + kcl * 8) * 2) : kOutOfRange;
        }
#pragma unroll
        for (int p = 0; p < PB1; ++p) {
            if (MODE == 0) {
                const int row = (p * NI + fw) * 8 + fpix;
                const int kcl = fslot ^ ((row >> 1) & 7);
                const int nn = n0 + row;
                b_off[p] = (nn < P.Cd) ? (unsigned)((nn * P.b_row_pitch + kcl * 8) * 2) : kOutOfRange;
            } else {
                // [64 filters][BN channels]: chunk slot (p*NI + fw)*64 + lane of the stage
                const int slot = (p * NI + fw) * 64 + lane;
                const int krow = slot / (BN / 8), pc = slot % (BN / 8);
                const int c = n0 + swizzled_chunk<BN>(krow, pc) * 8;
                b_off[p] = (c < P.Cd) ? (unsigned)((krow * P.b_row_pitch + c) * 2) : kOutOfRange;
            }
        }
    }
    const int4v rsrcA = make_rsrc(P.A, (unsigned)(P.NB * P.Hs * P.Ws * P.Cs) * 2u);
    const int4v rsrcB = make_rsrc(P.B, (unsigned)((MODE == 0 ? P.Cd : P.Cs) * P.b_row_pitch) * 2u);

    auto issue_patch = [&](int kc) {                // slab kc into buffer kc & 1
        const unsigned soff = (unsigned)__builtin_amdgcn_readfirstlane(kc * 128);
        const unsigned base = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds0 + (kc & (NPB - 1)) * PATCHB + fw * 1024));
#pragma unroll
        for (int q = 0; q < NPL; ++q) dma16(a_off[q], rsrcA, soff, base + q * NI * 1024);
    };
    // the step the next issue_filter() fetches: its first tap's byte offset in a filter row, channel slab, stage
    const int bpt = (MODE == 0 ? P.Cs : P.Cd) * 2;
    int nx_grp = 0, nx_kc = 0, nx_stage = 0;
    auto issue_filter = [&]() {
        const int first = nx_grp * TPS * bpt + (MODE == 0 ? nx_kc * 128 : nx_kc * 64 * P.b_row_pitch * 2);
        const int base0 = (int)lds0 + NPB * PATCHB + nx_stage * BSTAGE + fw * 1024;
#pragma unroll
        for (int tt = 0; tt < TPS; ++tt) {
            const unsigned soff = (unsigned)__builtin_amdgcn_readfirstlane(first + tt * bpt);
            const unsigned base = (unsigned)__builtin_amdgcn_readfirstlane(base0 + tt * BSLAB);
#pragma unroll
            for (int p = 0; p < PB1; ++p) dma16(b_off[p], rsrcB, soff, base + p * NI * 1024);
        }
        const int t1 = nx_grp + 1;
        const bool wrap = t1 == ngroups;
        nx_grp = __builtin_amdgcn_readfirstlane(wrap ? 0 : t1);
        nx_kc = __builtin_amdgcn_readfirstlane(wrap ? nx_kc + 1 : nx_kc);
        nx_stage = __builtin_amdgcn_readfirstlane(nx_stage + 1 == SB ? 0 : nx_stage + 1);
    };

    // ---- multiplying side ------------------------------------------------------------------
    const int wm = wave / WGN, wn = wave % WGN;
    const int frow = lane & (MF - 1), lhi = lane / MF;
    int pbase[FM];                                  // patch pixel of this lane's row at displacement 0
#pragma unroll
    for (int b = 0; b < FM; ++b) {
        const int ml = wm * WM + b * MF + frow;
        pbase[b] = (ml < BM) ? (ml / TW) * PW + (ml % TW) : 0;      // padding rows read pixel 0
    }
    float4p acc[FN][FM];
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
        for (int b = 0; b < FM; ++b)
#pragma unroll
            for (int e = 0; e < ACCN; ++e) acc[a][b][e] = 0.f;

    // patch-pixel displacement of the taps in their order, which is that of the filter rows: the data
    // gradient's taps move the other way
    const int po_w = (MODE == 0) ? P.dw : -P.dw, po_h = ((MODE == 0) ? P.dh : -P.dh) * PW - (P.S - 1) * po_w;
    const int po0 = (MODE == 0) ? 0 : (P.R - 1) * P.dh * PW + (P.S - 1) * P.dw;
    int po = po0, po_col = 0, po_tap = 0;           // of the tap whose fragments are read next
    auto next_tap = [&]() {
        const bool last = po_tap + 1 == ntaps, turn = po_col + 1 == P.S;     // (selects: a branch here would part the reads)
        po = last ? po0 : po + (turn ? po_h : po_w);
        po_col = turn ? 0 : po_col + 1;
        po_tap = last ? 0 : po_tap + 1;
    };
    constexpr int KK = 64 / KSTEP, G = TPS * KK;    // groups of KSTEP contraction values in a tap and in a step
    // fragments of group g of a step; the tap moves on behind its last group
    auto load_frags = [&](const unsigned char* pa, int stage, int g, half8 (&fa)[FM], half8 (&fb)[FN]) {
        const unsigned char* sb = bring + stage * BSTAGE + (g / KK) * BSLAB;
        const int kk = g % KK, chunk = kk * CPK + lhi;
#pragma unroll
        for (int b = 0; b < FM; ++b) {
            const int prow = pbase[b] + po;
            fa[b] = *reinterpret_cast<const half8*>(pa + prow * 128 + ((chunk ^ ((prow >> 1) & 7)) << 4));
        }
#pragma unroll
        for (int a = 0; a < FN; ++a) {
            if (MODE == 0) {
                const int row = wn * WN + a * MF + frow;
                fb[a] = *reinterpret_cast<const half8*>(sb + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
            } else {
                fb[a] = lds_frag_tr_16<BN>(sb, kk * 32, wn * WN + a * 16, lane);
            }
        }
        if (kk == KK - 1) next_tap();
    };
    auto multiply = [&](half8 (&fa)[FM], half8 (&fb)[FN]) {
#pragma unroll
        for (int a = 0; a < FN; ++a)
#pragma unroll
            for (int b = 0; b < FM; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[a], fa[b], acc[a][b], 0, 0, 0);
    };

    // ---- pipeline: one step per (slab, group of TPS taps), taps fastest ------------------------------------
    if (fetcher) {
        issue_patch(0);
#pragma unroll 1
        for (int s = 0; s < D && s < nk; ++s) issue_filter();
    }
    int tap = 0, kc = 0, stage = 0;
    // loads retire in order: once the filter stage of step t is in, so is everything sent
    // before it, in particular the patch of its slab (sent at least ntaps - D steps earlier)
    // (the next slab's patch, sent at tap 0 between two filter stages, may stay in flight
    // while it is younger than the stage awaited here)
    auto wait_step = [&](int t) {
        const bool patch_younger = tap >= 1 && tap <= D - 1 && kc + 1 < kchunks;
        if (t + D - 1 >= nk) wait_vmcnt<0>();
        else if (patch_younger) wait_vmcnt<(D - 1) * PB + NPL>();
        else wait_vmcnt<(D - 1) * PB>();
    };
    auto issue_step = [&](int t) {                  // behind the barrier of step t
        if (tap == 0 && kc + 1 < kchunks) issue_patch(kc + 1);      // its buffer was last read in slab kc-1
        if (t + D < nk) issue_filter();
    };
    auto next_step = [&]() {
        stage = (stage + 1 == SB) ? 0 : stage + 1;
        if (++tap == ngroups) { tap = 0; ++kc; }
    };
    if constexpr (NDW > 0) {
        if (wave >= NW) {
            for (int t = 0; t < nk; ++t) {
                wait_step(t);
                stage_barrier();
                issue_step(t);
                next_step();
            }
        } else {
            // The next group's fragments are read while the matrix pipe works on this one's; the barrier of
            // the next step, which waits for the last reads of this one, comes in front of its last matrix
            // instructions.  Within a step the reads go between the matrix instructions, one or two behind each: in front of them all,
            // they keep the matrix pipe waiting while LDS, which the fetching waves fill at the same time, takes them
            // (3x3 256->256 on 2x50x84: 10x14 blocks 15.6 -> 14.9 us, 8x16 24.2 -> 22.4, 8x8 data gradient 26.6 -> 23.6).  The next
            // step's first reads, behind its barrier, are another block of code than the last group's matrix instructions and
            // do go in front of them.
            half8 fa[2][FM], fb[2][FN];
            constexpr int READS = FM + FN * (MODE == 0 ? 1 : 2), EACH = (READS + FM * FN - 1) / (FM * FN);
            auto interleave = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < FM * FN; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);          // a matrix instruction
                    __builtin_amdgcn_sched_group_barrier(0x100, EACH, 0);       // LDS reads
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            static_assert(G % 2 == 0, "fragment buffers alternate");
            stage_barrier();
            load_frags(smem, 0, 0, fa[0], fb[0]);
            for (int t = 0; t < nk; ++t) {
                const unsigned char* pa = smem + (kc & (NPB - 1)) * PATCHB;
#pragma unroll
                for (int g = 0; g + 1 < G; ++g) {
                    load_frags(pa, stage, g + 1, fa[(g + 1) & 1], fb[(g + 1) & 1]);
                    multiply(fa[g & 1], fb[g & 1]);
                    interleave();
                }
                next_step();
                wait_lds_reads();       // on both sides of the branch, or the compiler waits again in each matrix instruction
                if (t + 1 < nk) {
                    stage_barrier();
                    load_frags(smem + (kc & (NPB - 1)) * PATCHB, stage, 0, fa[0], fb[0]);
                }
                multiply(fa[1], fb[1]);
                interleave();
            }
        }
    } else {
        for (int t = 0; t < nk; ++t) {
            if (fetcher) wait_step(t);
            stage_barrier();
            if (fetcher) issue_step(t);
            const unsigned char* pa = smem + (kc & (NPB - 1)) * PATCHB;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                half8 fa[FM], fb[FN];
                load_frags(pa, stage, g, fa, fb);
                multiply(fa, fb);
            }
            next_step();
        }
    }

    // ---- epilogue ------------------------------------------------------------------------------
    static_assert(NW * epilogue_strip_bytes<WN, MF>() <= NPB * PATCHB + SB * TPS * BN * 128,
                  "epilogue strips fit in the patch buffers and the filter ring");
    stage_barrier();                                // everybody is done reading the last patch and filter stage
    if (NDW > 0 && wave >= NW) return;              // no barrier follows
    store_rows_via_lds<FM, FN, MF, TAIL>(acc, smem + wave * epilogue_strip_bytes<WN, MF>(), lane, n0 + wn * WN, P,
                               [&](int r) -> unsigned {
        const int ml = wm * WM + r;
        const int h = h0 + ml / TW, w = w0 + ml % TW;
        if (ml >= BM || h >= P.Hd || w >= P.Wd) return kOutOfRange;
        return (unsigned)(((n * P.Hd + h) * P.Wd + w) * P.Cd) * 2u;
    });
}

template <int MODE, int TH, int TW, int BN, int WGM, int WGN, int SB, int NPB, int NDW, bool TAIL>
static hipError_t launch_patch_variant_impl(const IgemmParams& P, hipStream_t st)
{
    if ((P.R * P.S) % TPS != 0 || (P.R * P.S) / TPS < SB - 1) return hipErrorInvalidValue;
    if (NPB == 1 && P.Cs != 64) return hipErrorInvalidValue;      // one patch buffer = one channel slab
    constexpr int NI = NDW ? NDW : WGM * WGN / 2;
    constexpr int NPL = ((TH + 2) * (TW + 2) + 8 * NI - 1) / (8 * NI);
    constexpr size_t lds = (size_t)NPB * NPL * NI * 1024 + (size_t)SB * TPS * BN * 128;
    static_assert(lds <= 160 * 1024, "LDS budget");
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void*>(&conv_patch_kernel<MODE, TH, TW, BN, WGM, WGN, SB, NPB, NDW, TAIL>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    const int grid = ((P.total_tiles + 63) / 64) * 64;
    hipLaunchKernelGGL((conv_patch_kernel<MODE, TH, TW, BN, WGM, WGN, SB, NPB, NDW, TAIL>), dim3(grid), dim3(64 * (WGM * WGN + NDW)),
                       lds, st, P);
    return hipGetLastError();
}

template <int MODE, int TH, int TW, int BN, int WGM, int WGN, int SB, int NPB, int NDW>
static hipError_t launch_patch_variant(const IgemmParams& P, hipStream_t st)
{
    // the tail has kernels of its own: see store_rows_via_lds
    return P.ep.any() ? launch_patch_variant_impl<MODE, TH, TW, BN, WGM, WGN, SB, NPB, NDW, true>(P, st)
                      : launch_patch_variant_impl<MODE, TH, TW, BN, WGM, WGN, SB, NPB, NDW, false>(P, st);
}

// number - 400, block, filters, multiplying waves, ring stages, patch buffers, fetching waves, name
#define SDCONV_PATCH_VARIANTS(X) \
    X(27, 8, 16, 64, 4, 2, 2, 1, 0, "8x16x64_s2_m16_t3_1p") \
    X(33, 10, 14, 64, 3, 2, 2, 1, 2, "10x14x64_6w2f_s2_m16_t3_1p") \
    X(35, 10, 14, 64, 3, 2, 4, 2, 4, "10x14x64_6w4f_s4_m16_t3") \
    X(36, 8, 16, 64, 2, 2, 3, 2, 4, "8x16x64_4w4f_s3_m16_t3") \
    X(37, 8, 8, 64, 2, 2, 3, 2, 4, "8x8x64_4w4f_s3_m16_t3")

const std::array<PatchVariant, kNumPatchVariants> kPatchVariants = [] {
    std::array<PatchVariant, kNumPatchVariants> v{};
#define SDCONV_PATCH_NAME(idx, TH, TW, BN, WGM, WGN, SB, NPB, NDW, name) \
    v[idx] = {TH, TW, BN, SB, "conv_fwd_patch_" name, "conv_dgrad_patch_" name, NPB == 1};
    SDCONV_PATCH_VARIANTS(SDCONV_PATCH_NAME)
    return v;
}();

template <int MODE> static hipError_t launch_mode(int variant, const IgemmParams& P, hipStream_t st)
{
    switch (variant) {
#define SDCONV_PATCH_CASE(idx, TH, TW, BN, WGM, WGN, SB, NPB, NDW, name) \
        case idx: return launch_patch_variant<MODE, TH, TW, BN, WGM, WGN, SB, NPB, NDW>(P, st);
        SDCONV_PATCH_VARIANTS(SDCONV_PATCH_CASE)
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv_patch(int variant, const IgemmParams& P, hipStream_t st)
{
    return P.mode ? launch_mode<1>(variant, P, st) : launch_mode<0>(variant, P, st);
}

}  // namespace sdconv
