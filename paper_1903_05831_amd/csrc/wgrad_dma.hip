// Weight gradient with an asynchronous global->LDS pipeline (see wgrad.hip for the maths).
//
//   dw[k][r][s][c] = sum_p dy[p][k] * x[src(p; r,s)][c],   p = (n,ho,wo)
//
// One workgroup owns a (filter tile, channel tile, tap, pixel range).  Per contraction step
// it needs BP pixels of dy (rows of BM filters) and the BP matching pixels of x (rows of BN
// channels); both tiles go to LDS as they sit in memory, [pixel][channel], with
// buffer_load_dwordx4 ... lds into a ring of S stages, and the MFMA fragments come from the
// transposing LDS read (four consecutive pixels of one channel per lane).
//
// Addressing: dy rows are consecutive pixels, so a lane's offset is fixed and the buffer
// descriptor's base moves by BP rows per step; its shrinking size makes the hardware range
// check zero the rows past the last pixel.  x rows are gathered: BP lanes decode one pixel
// each per step into an LDS table of byte offsets (out-of-image -> out of range -> zeros), one
// step ahead of the loads that use it; with a 1x1 stride-1 unpadded filter x is addressed like
// dy and the table is skipped (LINEAR).
//
// 64-byte granules of a tile row are XOR-swizzled with the row number (applied on the global
// side by choosing which chunk a lane fetches) so the transposing reads are conflict-free.
#include <type_traits>
#include "common.h"
#include "wgrad.h"
#include "dma.h"

#include "lds_tr.h"

namespace sdconv {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float4w __attribute__((ext_vector_type(4)));

// F: who fetches.  0: every wave its share.  -1: only the upper half of the waves sends the loads (and then multiplies like
// the others); with two waves per SIMD the lower wave keeps the matrix pipe busy while its partner is stalled
// in the burst of LDS-DMA instructions, instead of both stalling at once (see igemm_ws_body.h).  F > 0: so many waves
// do nothing else.  The others then need no registers for addresses, and four waves of 64x64 read a third less of
// LDS than eight of 64x32: 3x3 256->256 on 2x50x84 with its reduction 23.8 -> 22.8 us, 1x1 1024->256 16.1 -> 14.9, 1x1 128->512
// on 2x100x168 16.2 -> 15.0, 3x3 stride 2 on 173x271 16.8 -> 15.4, each at its best number of ranges.
// MF: 32 = v_mfma_f32_32x32x16_f16 blocks, 16 = v_mfma_f32_16x16x32_f16 blocks (measured faster
// on the large tiles).
template <int BM, int BN, int WGM, int WGN, int S, int BP, bool LINEAR, int F, int MF>
__global__ __launch_bounds__(64 * (WGM * WGN + (F > 0 ? F : 0))) void wgrad_dma_kernel(WgradParams P)
{
    constexpr int NW = WGM * WGN;                           // multiplying waves
    constexpr bool HF = F < 0;
    constexpr int NWF = F > 0 ? F : HF ? NW / 2 : NW, NT = 64 * NWF;    // fetching waves / threads
    constexpr int FW0 = F > 0 ? NW : NW - NWF;              // first fetching wave
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int FM = WM / MF, FN = WN / MF;
    constexpr int ACCN = MF == 32 ? 16 : 4, KSTEP = MF == 32 ? 16 : 32;
    constexpr int CRG = BM / 8, CRX = BN / 8;           // 16-byte chunks per tile row
    constexpr int RPG = NT / CRG, RPX = NT / CRX;       // rows one pass of all threads covers
    constexpr int PG = BP / RPG, PX = BP / RPX;         // DMA loads per thread and stage
    constexpr int GBYTES = BP * BM * 2, XBYTES = BP * BN * 2, STAGE = GBYTES + XBYTES;
    constexpr int INFLIGHT = (S - 2) * (PG + PX);
    static_assert((MF == 32 || MF == 16) && WM % MF == 0 && WN % MF == 0 && BP % KSTEP == 0, "wave tile");
    static_assert(PG >= 1 && PX >= 1 && BP % RPG == 0 && BP % RPX == 0, "staging");
    static_assert(F > 0 ? BP == 64 : RPG % 4 == 0 && RPX % 4 == 0, "staging");
    static_assert(S >= 2 && INFLIGHT < 64 && BP % 16 == 0 && BP <= 64 * NW, "pipeline");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    unsigned* xtab = reinterpret_cast<unsigned*>(smem + S * STAGE);     // [S][BP] byte offsets of x pixels

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const bool fetcher = wave >= FW0;
    const int ft = tid - FW0 * 64, fw = wave - FW0;         // index among the fetching threads / waves

    // Which tile: the tiles of one pixel range (all filter tiles, channel tiles and taps of a
    // split) read the same dy and x rows, and each XCD has an L2 of its own, so runs of 8
    // consecutive tiles go to one XCD (workgroup b runs on XCD b % 8) instead of being dealt round
    // over all eight, which made every XCD fetch every operand row again.
    constexpr int kRun = 8;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    int b = ((slot / kRun) * 8 + xcd) * kRun + (slot % kRun);
    if (b >= P.total_blocks) return;
    const int tc = b % P.tiles_c; b /= P.tiles_c;
    const int tk = b % P.tiles_k; b /= P.tiles_k;
    const int tap = b % (P.R * P.S);
    const int split = b / (P.R * P.S);
    const int r = tap / P.S, s = tap % P.S;
    const int k0 = tk * BM, c0 = tc * BN;
    const int oh = r * P.dh - P.ph, ow = s * P.dw - P.pw;

    const int bp_per_64 = 64 / BP;                           // steps_per_split counts 64-pixel units
    const int step0 = split * P.steps_per_split * bp_per_64;
    const int total_steps = (P.P + BP - 1) / BP;
    int nsteps = total_steps - step0;
    if (nsteps > P.steps_per_split * bp_per_64) nsteps = P.steps_per_split * bp_per_64;
    if (nsteps < 0) nsteps = 0;

    if constexpr (F > 0) if (wave >= NW) {
        // ---- a wave that only fetches ----------------------------------------------------------
        // PG consecutive load instructions of a step's dy tile and PX of its x tile, sent in runs (dma.h).  In gathering
        // layers lane l finds the place of pixel l of a step, and the loads ask it by a lane shuffle; that is
        // done before the barrier behind which the loads go out.
        constexpr int LG = BM / 8, LX = BN / 8;             // lanes to a row
        unsigned g_off[PG], x_off[PX], x_out[PX];
        int g_row[PG], x_row[PX];
#pragma unroll
        for (int i = 0; i < PG; ++i) {
            g_row[i] = (fw * PG + i) * (64 / LG) + lane / LG;
            const int k = k0 + swizzled_chunk<BM>(g_row[i], lane % LG) * 8;
            g_off[i] = (k < P.K ? (unsigned)((g_row[i] * P.K + k) * 2) : kOutOfRange) + kRunSlack - run_offset(i);
        }
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            x_row[i] = (fw * PX + i) * (64 / LX) + lane / LX;
            const int c = c0 + swizzled_chunk<BN>(x_row[i], lane % LX) * 8;
            x_out[i] = c < P.C ? 0u : kOutOfRange;
            x_off[i] = (unsigned)((LINEAR ? x_row[i] * P.C + c : c) * 2) + kRunSlack - run_offset(i);
            if (LINEAR) x_off[i] |= x_out[i];
        }
        const int4v rsrcG = make_rsrc(reinterpret_cast<const unsigned char*>(P.G) - kRunSlack, (unsigned)(P.P * P.K) * 2u + kRunSlack);
        const int4v rsrcX = make_rsrc(reinterpret_cast<const unsigned char*>(P.X) - kRunSlack, (unsigned)(P.N * P.H * P.W * P.C) * 2u + kRunSlack);
        const unsigned to_g = lds0 + fw * PG * 1024, to_x = lds0 + GBYTES + fw * PX * 1024;
        const int hw = P.Ho * P.Wo;
        const int adv_n = BP / hw, adv_ho = (BP % hw) / P.Wo, adv_wo = (BP % hw) % P.Wo;
        int left = P.P - step0 * BP;                        // pixels from the step's first to the last
        int n = 0, ho = 0, wo = 0;
        if (!LINEAR) {
            const int px = step0 * BP + lane;
            n = px / hw;
            ho = (px - n * hw) / P.Wo;
            wo = px - n * hw - ho * P.Wo;
        }
        unsigned so_g = (unsigned)(step0 * BP) * P.K * 2, so_x = LINEAR ? (unsigned)(step0 * BP) * P.C * 2 : 0u;
        unsigned v[PX];
        auto place = [&]() __attribute__((always_inline)) {
            if (LINEAR) return;
            const int h = ho * P.sh + oh, w = wo * P.sw + ow;
            unsigned at = (unsigned)((((n * P.H + h) * P.W + w) * P.C) * 2);
            if ((unsigned)h >= (unsigned)P.H || (unsigned)w >= (unsigned)P.W || lane >= left) at = kOutOfRange;
#pragma unroll
            for (int i = 0; i < PX; ++i) v[i] = __shfl(at, x_row[i]);
#pragma unroll
            for (int i = 0; i < PX; ++i) v[i] = (v[i] & kOutOfRange) | x_out[i] | (v[i] + x_off[i]);
            wo += adv_wo;
            int carry = wo >= P.Wo;
            wo -= carry ? P.Wo : 0;
            ho += adv_ho + carry;
            carry = ho >= P.Ho;
            ho -= carry ? P.Ho : 0;
            n += adv_n + carry;
        };
        auto send = [&](int stage) __attribute__((always_inline)) {
            const unsigned sg = __builtin_amdgcn_readfirstlane(so_g), sx = __builtin_amdgcn_readfirstlane(so_x);
            const unsigned lg = __builtin_amdgcn_readfirstlane(to_g + stage * STAGE), lx = __builtin_amdgcn_readfirstlane(to_x + stage * STAGE);
            if (left >= BP) {
                dma16_runs<PG>(g_off, rsrcG, sg, lg);
                if (LINEAR) dma16_runs<PX>(x_off, rsrcX, sx, lx); else dma16_runs<PX>(v, rsrcX, sx, lx);
            } else {                                        // the pixels end within the step
                unsigned vg[PG], vx[PX];
#pragma unroll
                for (int i = 0; i < PG; ++i) vg[i] = g_row[i] < left ? g_off[i] : kOutOfRange;
#pragma unroll
                for (int i = 0; i < PX; ++i) vx[i] = !LINEAR ? v[i] : x_row[i] < left ? x_off[i] : kOutOfRange;
                dma16_runs<PG>(vg, rsrcG, sg, lg);
                dma16_runs<PX>(vx, rsrcX, sx, lx);
            }
            so_g += BP * P.K * 2;
            if (LINEAR) so_x += BP * P.C * 2;
            left -= BP;
        };
        int is = 0;
        place();
#pragma unroll 1
        for (int q = 0; q < nsteps; ++q) {
            if (q >= S - 1) {
                wait_vmcnt<INFLIGHT>();
                stage_barrier();
            }
            send(is);
            is = (is + 1 == S) ? 0 : is + 1;
            place();
        }
        for (int it = nsteps > S - 1 ? nsteps - (S - 1) : 0; it < nsteps; ++it) {
            if (it + S - 2 < nsteps) wait_vmcnt<INFLIGHT>(); else wait_vmcnt<0>();
            stage_barrier();
        }
        return;
    }

    // ---- fixed per-thread parts of the offsets ----------------------------------------------
    unsigned g_off[PG], x_add[PX];
    int x_row[PX];
#pragma unroll
    for (int i = 0; i < PG; ++i) {
        int row = i * RPG + ft / CRG, pc = ft % CRG;
        int lc = swizzled_chunk<BM>(row, pc);
        int k = k0 + lc * 8;
        g_off[i] = (k < P.K) ? (unsigned)((row * P.K + k) * 2) : kOutOfRange;
    }
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        int row = i * RPX + ft / CRX, pc = ft % CRX;
        int lc = swizzled_chunk<BN>(row, pc);
        int c = c0 + lc * 8;
        x_row[i] = row;
        if (LINEAR) x_add[i] = (c < P.C) ? (unsigned)((row * P.C + c) * 2) : kOutOfRange;
        else x_add[i] = (c < P.C) ? (unsigned)(c * 2) : kOutOfRange;
    }
    const int4v rsrcX = make_rsrc(P.X, (unsigned)(P.N * P.H * P.W * P.C) * 2u);

    // x offset table of one step: lane t < BP holds pixel p0 + t.  The steps come in order, so
    // the lane keeps its pixel's (image, row, column) and moves it on by BP pixels per step with
    // two carries instead of dividing again (the divisions cost 5 % of a 3x3 layer's kernel).
    int tb_p = 0, tb_n = 0, tb_ho = 0, tb_wo = 0;
    const int hw = P.Ho * P.Wo;
    const int adv_n = BP / hw, adv_ho = (BP % hw) / P.Wo, adv_wo = (BP % hw) % P.Wo;
    if (!LINEAR && tid < BP) {
        tb_p = step0 * BP + tid;
        tb_n = tb_p / hw;
        const int rem = tb_p - tb_n * hw;
        tb_ho = rem / P.Wo;
        tb_wo = rem - tb_ho * P.Wo;
    }
    auto fill_table = [&](int slot) {
        if (LINEAR) return;
        if (tid < BP) {
            unsigned off = kOutOfRange;
            if (tb_p < P.P) {
                int h = tb_ho * P.sh + oh, w = tb_wo * P.sw + ow;
                if ((unsigned)h < (unsigned)P.H && (unsigned)w < (unsigned)P.W)
                    off = (unsigned)((((tb_n * P.H + h) * P.W + w) * P.C) * 2);
            }
            xtab[slot * BP + tid] = off;
            tb_p += BP;
            tb_wo += adv_wo;
            int carry = tb_wo >= P.Wo;
            tb_wo -= carry ? P.Wo : 0;
            tb_ho += adv_ho + carry;
            carry = tb_ho >= P.Ho;
            tb_ho -= carry ? P.Ho : 0;
            tb_n += adv_n + carry;
        }
    };

    // dy, and x in pointwise layers: the descriptor starts at the step's first pixel and ends with the
    // tensor; the steps come in order, so both move on by BP pixels.
    const unsigned long long gstep = (unsigned long long)BP * P.K * 2, xstep = (unsigned long long)BP * P.C * 2;
    unsigned long long g_at = reinterpret_cast<unsigned long long>(P.G) + step0 * gstep;
    unsigned long long x_at = reinterpret_cast<unsigned long long>(P.X) + step0 * xstep;
    int px_left = P.P - step0 * BP;
    auto issue = [&](int stage) {
        const unsigned sbase = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds0 + stage * STAGE + fw * 1024));
        unsigned xo[PX];
        if (!LINEAR) {
            // all table entries before the first load: the loads are assembly that nothing may pass,
            // and an entry read just before its load would hold the wave up for an LDS access each time
#pragma unroll
            for (int i = 0; i < PX; ++i) xo[i] = xtab[stage * BP + x_row[i]];
        }
        const int4v rsrcG = make_rsrc(reinterpret_cast<const void*>(g_at), (unsigned)(px_left * P.K) * 2u);
#pragma unroll
        for (int i = 0; i < PG; ++i) dma16(g_off[i], rsrcG, 0, sbase + i * RPG * BM * 2);
        if (LINEAR) {
            const int4v rsrcL = make_rsrc(reinterpret_cast<const void*>(x_at), (unsigned)(px_left * P.C) * 2u);
#pragma unroll
            for (int i = 0; i < PX; ++i) dma16(x_add[i], rsrcL, 0, sbase + GBYTES + i * RPX * BN * 2);
        } else {
#pragma unroll
            for (int i = 0; i < PX; ++i) {
                const unsigned voff = (int)(xo[i] | x_add[i]) < 0 ? kOutOfRange : xo[i] + x_add[i];
                dma16(voff, rsrcX, 0, sbase + GBYTES + i * RPX * BN * 2);
            }
        }
        g_at += gstep;
        x_at += xstep;
        px_left -= BP;
    };

    typedef typename std::conditional<MF == 32, float16v, float4w>::type acc_t;
    acc_t acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int e = 0; e < ACCN; ++e) acc[a][c][e] = 0.f;

    // ORDERED: the first portion's fragments are read at once and the next one's between the matrix instructions, where
    // the compiler reads them before their use (256x256 tiles with their reduction, 3x3 512->512 on 25 088 pixels 115.4 ->
    // 111.0 us, 1x1 2048->512 65.2 -> 62.6; 128x128 with fetching waves, 3x3 256->256 on 2x50x84 23.9 -> 22.8).  Waves with
    // smaller tiles have too few matrix instructions to read behind (64x64 tiles 3-4 % slower), and where every wave fetches its
    // share two workgroups on the compute unit fill each other's gaps (128x128 tiles of four waves 0.7 to 0.9 % slower).
    constexpr int NCH = BP / KSTEP;
    constexpr bool ORDERED = F != 0 && MF == 16 && NCH > 1 && WM * WN >= 64 * 64;
    auto compute = [&](int stage) {
        const unsigned char* sg = smem + stage * STAGE;
        const unsigned char* sx = sg + GBYTES;
#pragma unroll
        for (int kk = 0; kk < BP / KSTEP; ++kk) {
            half8 fa[FM], fb[FN];
#pragma unroll
            for (int a = 0; a < FM; ++a) {
                if (MF == 32) fa[a] = lds_frag_tr<BM>(sg, kk * 16, wm * WM + a * 32, lane);
                else fa[a] = lds_frag_tr_16<BM>(sg, kk * 32, wm * WM + a * 16, lane);
            }
#pragma unroll
            for (int c = 0; c < FN; ++c) {
                if (MF == 32) fb[c] = lds_frag_tr<BN>(sx, kk * 16, wn * WN + c * 32, lane);
                else fb[c] = lds_frag_tr_16<BN>(sx, kk * 32, wn * WN + c * 16, lane);
            }
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int c = 0; c < FN; ++c) {
                    if constexpr (MF == 32)
                        acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[c], fa[a], acc[a][c], 0, 0, 0);
                    else
                        acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[c], fa[a], acc[a][c], 0, 0, 0);
                }
        }
        if constexpr (ORDERED) {        // 0x100: LDS reads, 0x008: matrix instructions
            constexpr int FIRST = 2 * (FM + FN), REST = (NCH - 1) * FIRST, MULS = NCH * FM * FN, EACH = (REST + MULS - 1) / MULS;
            __builtin_amdgcn_sched_group_barrier(0x100, FIRST, 0);
#pragma unroll
            for (int i = 0; i < (REST + EACH - 1) / EACH; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, EACH, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, MULS, 0);
        }
    };

    // ---- ring pipeline ---------------------------------------------------------------------------
    if constexpr (F > 0) {
        int cs = 0;
        for (int it = 0; it < nsteps; ++it) {
            stage_barrier();
            compute(cs);
            cs = (cs + 1 == S) ? 0 : cs + 1;
        }
    } else if (nsteps > 0) {
#pragma unroll
        for (int q = 0; q < S; ++q)
            if (q < nsteps) fill_table(q);
        if (!LINEAR) __syncthreads();
        int issued = 0;
#pragma unroll
        for (int q = 0; q < S - 1; ++q)
            if (q < nsteps) { if (fetcher) issue(q); ++issued; }
        int cs = 0, is = (S - 1) % S;
        for (int it = 0; it < nsteps; ++it) {
            if (fetcher) { if (it + S - 2 < nsteps) wait_vmcnt<INFLIGHT>(); else wait_vmcnt<0>(); }
            stage_barrier();        // waits for this wave's table writes too
            if (issued < nsteps) {
                if (fetcher) issue(is);
                ++issued;
                is = (is + 1 == S) ? 0 : is + 1;
            }
            // table of step it+S (read by the issue of the next iteration) reuses the slot of
            // step `it`, whose loads were issued S-1 iterations ago
            if (it + S < nsteps) fill_table(cs);
            compute(cs);
            cs = (cs + 1 == S) ? 0 : cs + 1;
        }
    }

    // ---- store the fp32 tile -------------------------------------------------------------------
    // The products are taken transposed (x fragment first), so a lane holds four consecutive channels of
    // one filter row: 16-byte stores, a quarter of the instructions of the 4-byte ones that the other
    // order needs (a 256x256 tile: 256 instead of 1024 a workgroup; res5 3x3 with its ranges lost
    // 9 us to them).  The range check of the buffer drops filters and channels past the end.  A descriptor
    // starts at the first filter of a block row, so that offsets count the floats of MF filters and not of dw.
    const long pitch = (long)P.R * P.S * P.C;
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    const int lrow = lane & (MF - 1), lhi = lane / MF;
    const unsigned row = (unsigned)(lrow * pitch + (long)tap * P.C) * 4u;
#pragma unroll
    for (int a = 0; a < FM; ++a) {
        const int kb = k0 + wm * WM + a * MF, k = kb + lrow;
        const __amdgpu_buffer_rsrc_t rsrcD =
            __builtin_amdgcn_make_buffer_rsrc(P.out + ((long)split * P.K + kb) * pitch, 0, (int)kOutOfRange, 0x00020000);
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int q = 0; q < ACCN / 4; ++q) {
                const int col = c0 + wn * WN + c * MF + (MF == 32 ? 8 * q : 0) + 4 * lhi;
                const float4w v = {acc[a][c][4 * q], acc[a][c][4 * q + 1], acc[a][c][4 * q + 2], acc[a][c][4 * q + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), rsrcD,
                                                       k < P.K && col < P.C ? row + (unsigned)col * 4u : kOutOfRange, 0, 0);
            }
    }
}

template <int BM, int BN, int WGM, int WGN, int S, int BP, int F, int MF>
static hipError_t launch_wdma(const WgradParams& P0, hipStream_t st)
{
    constexpr size_t lds = (size_t)S * BP * (BM + BN) * 2 + (size_t)S * BP * sizeof(unsigned);
    static_assert(lds <= 160 * 1024, "LDS budget");
    const bool linear = P0.R == 1 && P0.S == 1 && P0.sh == 1 && P0.sw == 1 && P0.ph == 0 && P0.pw == 0;
    static std::atomic<bool> configured{false};   // set once the attribute call has succeeded; a second thread may repeat it, harmlessly
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void*>(&wgrad_dma_kernel<BM, BN, WGM, WGN, S, BP, false, F, MF>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        e = hipFuncSetAttribute(
            reinterpret_cast<const void*>(&wgrad_dma_kernel<BM, BN, WGM, WGN, S, BP, true, F, MF>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    WgradParams P = P0;
    P.total_blocks = P.tiles_c * P.tiles_k * P.R * P.S * P.splits;
    const long blocks = ((long)P.total_blocks + 63) / 64 * 64;     // whole runs of 8 tiles on each of 8 XCDs
    if (linear)
        hipLaunchKernelGGL((wgrad_dma_kernel<BM, BN, WGM, WGN, S, BP, true, F, MF>), dim3((unsigned)blocks),
                           dim3(64 * (WGM * WGN + (F > 0 ? F : 0))), lds, st, P);
    else
        hipLaunchKernelGGL((wgrad_dma_kernel<BM, BN, WGM, WGN, S, BP, false, F, MF>), dim3((unsigned)blocks),
                           dim3(64 * (WGM * WGN + (F > 0 ? F : 0))), lds, st, P);
    return hipGetLastError();
}

// number - 100, tile, multiplying waves, ring stages, pixels of a step, fetching waves (F above), matrix block, name
#define SDCONV_WGRAD_VARIANTS(X) \
    X(4, 64, 128, 1, 4, 3, 64, 0, 32, "wgrad_dma_64x128x64_4w_s3") \
    X(7, 64, 64, 2, 2, 3, 64, 0, 32, "wgrad_dma_64x64x64_4w_s3") \
    X(8, 128, 64, 2, 2, 3, 64, 0, 32, "wgrad_dma_128x64x64_4w_s3") \
    X(12, 128, 128, 2, 4, 3, 64, -1, 32, "wgrad_dma_128x128x64_8w_s3_hf") \
    X(14, 256, 256, 2, 4, 2, 64, -1, 16, "wgrad_dma_256x256x64_8w_s2_hf_m16") \
    X(15, 256, 256, 2, 4, 3, 32, -1, 16, "wgrad_dma_256x256x32_8w_s3_hf_m16") \
    X(16, 128, 128, 2, 4, 3, 64, -1, 16, "wgrad_dma_128x128x64_8w_s3_hf_m16") \
    X(17, 256, 128, 4, 2, 3, 64, -1, 16, "wgrad_dma_256x128x64_8w_s3_hf_m16") \
    X(18, 64, 64, 2, 2, 3, 64, 0, 16, "wgrad_dma_64x64x64_4w_s3_m16") \
    X(19, 128, 128, 2, 2, 2, 64, 0, 16, "wgrad_dma_128x128x64_4w_s2_m16") \
    X(20, 128, 128, 2, 2, 3, 64, 4, 16, "wgrad_dma_128x128x64_4w4f_s3_m16") \
    X(21, 64, 64, 2, 2, 3, 64, 4, 32, "wgrad_dma_64x64x64_4w4f_s3") \
    X(22, 128, 64, 2, 2, 3, 64, 4, 32, "wgrad_dma_128x64x64_4w4f_s3") \
    X(23, 256, 128, 4, 2, 3, 64, 4, 16, "wgrad_dma_256x128x64_8w4f_s3_m16")

const std::array<WgradVariant, kNumWgradDmaVariants> kWgradDmaVariants = [] {
    std::array<WgradVariant, kNumWgradDmaVariants> v{};
#define SDCONV_WGRAD_NAME(idx, BM, BN, WGM, WGN, S, BP, F, MF, name) v[idx] = {BM, BN, name, F > 0};
    SDCONV_WGRAD_VARIANTS(SDCONV_WGRAD_NAME)
    return v;
}();

hipError_t launch_wgrad_dma(int variant, const WgradParams& P, hipStream_t st)
{
    switch (variant) {
#define SDCONV_WGRAD_CASE(idx, BM, BN, WGM, WGN, S, BP, F, MF, name) \
        case idx: return launch_wdma<BM, BN, WGM, WGN, S, BP, F, MF>(P, st);
        SDCONV_WGRAD_VARIANTS(SDCONV_WGRAD_CASE)
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sdconv
