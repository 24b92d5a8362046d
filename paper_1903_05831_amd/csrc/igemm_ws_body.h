// Implicit-GEMM forward / data-gradient kernel with separate fetching and multiplying waves.
//
// Same tiles, LDS layout, swizzle and contraction order as igemm_dma.hip.  What differs is who
// sends the global->LDS loads.  A wave that issues buffer_load ... lds stalls until the texture
// path has taken the instruction (about 16-20 cycles per 1 KiB instruction, per CU), and while
// it stalls it cannot feed the matrix pipe.  When every wave fetches and then multiplies, all
// waves of a SIMD stall together and the fetch time adds to the MFMA time.  Here
//   NP > 0 : NP extra waves do nothing but fetch (they own no part of the tile), the WGM x WGN
//            multiplying waves never touch global memory until the epilogue;
//   NP == 0: the upper half of the multiplying waves fetches for everybody.  With two waves per
//            SIMD (wave w and w + NWC/2 share one) the lower wave multiplies while the upper one
//            is stalled in its burst of loads, then the upper one multiplies.
// One workgroup barrier per contraction step, shared by both kinds of wave, orders the ring.
//
// The data gradient (MODE 1) reads the filter as it is stored, [K][R][S][C]: its B tile is 64
// filters (contraction rows) x BN input channels, kept in LDS in that orientation and turned
// into fragments by the transposing LDS read (lds_tr.h), so no transposed copy of the filter
// is needed.  The forward pass keeps the [row][64 contraction halves] tiles of igemm_dma.hip.
//
// Row addressing is computed once per workgroup by all threads (one tile row each: byte offset
// of the pixel at tap displacement 0 and a bit for every tap outside the image) and handed to
// the fetching waves through LDS; in pointwise layers a row is a pixel of the source and the
// fetching waves know its offset themselves.
#pragma once
#include <type_traits>
#include "common.h"
#include "igemm.h"
#include "dma.h"
#include "igemm_epilogue.h"
#include "lds_tr.h"

namespace sdconv {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float4v_ __attribute__((ext_vector_type(4)));

// Contraction steps before its end at which a tile asks for its shortcut or mask values: their transfer from HBM
// then passes during the loop, not after it.  Fused RoI-head layers with 2: 1x1 512->2048 on 100 RoIs
// 19.6 -> 18.3 us, 256->1024 on 47x84 11.5 -> 10.6, 1024->512 data gradient on 512 RoIs 166.8 -> 161.9.  With 5 and more the
// lines displace operands from L2 (87 -> 93 us on 512->2048, 512 RoIs); strided data gradients, whose lines
// are spread over four classes' tiles, lose 1 % with any.
constexpr int kWarmSteps = 2;

// A value from each line of 64 bytes of the parameters that every tile needs, so that the lines come in one trip: the compiler
// loads them where they are used and nothing ahead of a branch, and by how that falls out a tile waited for two to five trips to cold
// lines before its first operand load, each some 3 % of a small layer.
__device__ __forceinline__ void ask_for_parameters(const IgemmParams& P)
{
    asm volatile("" :: "s"(P.Cs), "s"(P.total_tiles), "s"(P.taps_h[0].count), "s"(P.taps_w[0].count), "s"(P.tap_dh), "s"(P.pointwise));
}

// MF: 32 = v_mfma_f32_32x32x16_f16 blocks; 16 = v_mfma_f32_16x16x32_f16 blocks, for tile heights
// that are a multiple of 16 but not of 32 per wave row (224 = 2 x 112 rows: 25088 = 112 x 224
// pixels of the RoI head then give 224 or 896 tiles instead of 196 or 784 for 256 CUs).
// The work of one workgroup on tile `tile` of a launch (or of a part of one, see
// igemm_ws_mixed_kernel) with `tiles_n` column tiles whose row tiles start at row tile `tm0`.
template <int MODE, int BM, int BN, int WGM, int WGN, int S, int BK, int NP, int MF = 32, bool TAIL = false, bool F32 = false, int KS = 1>
__device__ __forceinline__ void igemm_ws_body(const IgemmParams& P, const int tile, const int tiles_n, const int tm0)
{
    constexpr int NWC = WGM * WGN * KS;             // multiplying waves; KS > 1: they divide each step's contraction too
    constexpr int NW = NWC + NP, NT = 64 * NW;
    constexpr int NI = NP ? NP : NWC / 2;           // fetching waves
    constexpr int IW0 = NP ? NWC : NWC / 2;         // first fetching wave
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int FM = WM / MF, FN = WN / MF;
    constexpr int ACCN = MF == 32 ? 16 : 4;         // accumulator floats per lane and block
    constexpr int ROWB = BK * 2;                    // bytes per tile row: eight 16-byte chunks
    constexpr int NA = BM / 8, NB = BN / 8;         // load instructions of a stage, 1 KiB each: activation rows and filter
    constexpr int PA = (NA + NI - 1) / NI, PB = (NB + NI - 1) / NI, PL = PA + PB;   // ... and of a fetching wave: so many in a row
    constexpr int ABYTES = PA * NI * 1024, STAGE = PL * NI * 1024;
    constexpr int INFLIGHT = (S - 2) * PL;          // loads a fetching wave may leave outstanding
    static_assert((MF == 32 || MF == 16) && WM % MF == 0 && WN % MF == 0 && BM % 8 == 0 && BN % 8 == 0, "tile shape");
    static_assert(S >= 2 && INFLIGHT < 64, "pipeline depth");
    static_assert(BK == 64, "contraction step");
    static_assert(!F32 || (MF == 32 && !TAIL && NP > 0), "binary32 tensors");
    static_assert(KS == 1 || (F32 && 4 % KS == 0), "the waves' sums meet in the binary32 epilogue only");
    constexpr bool KROWS = MODE == 0 || F32;        // the filter's rows are destination channels
    constexpr int DBYTES = F32 ? 4 : 2;             // bytes of a destination element
    static_assert(NI >= 1 && (NP > 0 || NWC % 2 == 0), "fetching waves");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    // row table (gathering layers): byte offset of the pixel at tap displacement 0, a bit per tap that
    // leaves the image, and where the row's result goes (strided data gradients)
    unsigned* row_off = reinterpret_cast<unsigned*>(smem + S * STAGE);      // [BM]
    unsigned* row_lo = row_off + BM;                                        // [BM] taps 0..31
    unsigned* row_hi = row_lo + BM;                                         // [BM] taps 32..63
    unsigned* row_dst = row_hi + BM;                                        // [BM] (MODE 1 only)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int tn = tile % tiles_n;
    int tm = tile / tiles_n + tm0;
    int cls = 0;
    if (MODE == 1) {
        while (cls + 1 < P.nclasses && tm >= P.class_tile_start[cls + 1]) ++cls;
        tm -= P.class_tile_start[cls];
    }
    const int ca = MODE == 1 ? cls / P.sw_cls : 0, cb = MODE == 1 ? cls % P.sw_cls : 0;

    int Hi, Wj, mh, mw, eh, ew;
    if (MODE == 0) { Hi = P.Hd; Wj = P.Wd; mh = P.sh; mw = P.sw; eh = 1; ew = 1; }
    else {
        Hi = (P.Hd - ca + P.sh - 1) / P.sh; Wj = (P.Wd - cb + P.sw - 1) / P.sw;
        mh = 1; mw = 1; eh = P.sh; ew = P.sw;
    }
    const int Mcls = P.NB * Hi * Wj;
    const int m0 = tm * BM, n0 = tn * BN;

    // The taps that reach this class form a grid of th.count x tw.count (common.h: they are evenly
    // spaced along each axis), so their displacements are counted on in scalar registers while the
    // loads go out.  With tap and row tables filled by a first and a second pass over the workgroup,
    // a barrier after each, the first load left 1.1 us after the start of the kernel.
    const AxisTaps th = P.taps_h[ca], tw = P.taps_w[cb];
    const int ntaps = th.count * tw.count;
    if (MODE == 1 && !F32 && ntaps == 0) {
        // a class without taps (three of the four of a 1x1 stride-2 layer): nothing to multiply.  With a tail the result is
        // 0 whatever the mask holds, which is then not read, unless a scale is infinite or NaN or something is added
        // (1x1 stride 2 with scale and mask: 2048->1024 on 512 RoIs of 14x14 205 -> 180 us, 512->256 on 173x271 19.5 -> 14.9).
        bool zero = true;
        if constexpr (TAIL) {
            if (P.ep.bias || P.ep.residual) zero = false;
            else if (P.ep.scale)
                for (int c = n0 + lane; c < n0 + BN && c < P.Cd; c += 64) zero = zero && fabsf(P.ep.scale[c]) < INFINITY;
            zero = __all(zero);
        }
        if (zero) {
            if (wave < NWC)
                store_zero_subtile<WM, WN>(lane, m0 + (wave / WGN) * WM, n0 + (wave % WGN) * WN, Mcls, P, Hi, Wj, eh, ew, ca, cb);
            return;
        }
    }
    const int kchunks = (P.Cs + BK - 1) / BK;
    const int nk = ntaps * kchunks;

    // ---- row table: one tile row per thread (pointwise layers: a row is a source pixel, no table) ----
    if (!P.pointwise) {
        for (int r = tid; r < BM; r += NT) {
            const int m = m0 + r;
            unsigned off = 0, dst = kOutOfRange;
            unsigned long long in = 0ull;
            if (m < Mcls) {
                const int n = m / (Hi * Wj);
                const int rem = m - n * (Hi * Wj);
                const int i = rem / Wj, j = rem - i * Wj;
                const int ih = i * mh, jw = j * mw;
                off = (unsigned)((((n * P.Hs + ih) * P.Ws + jw) * P.Cs) * 2);
                unsigned long long inw = 0ull;
                for (int t = 0; t < tw.count; ++t)
                    if ((unsigned)(jw + tw.disp + t * P.tap_dw) < (unsigned)P.Ws) inw |= 1ull << t;
                for (int t = 0; t < th.count; ++t)
                    if ((unsigned)(ih + th.disp + t * P.tap_dh) < (unsigned)P.Hs) in |= inw << (t * tw.count);
                if (MODE == 1) dst = (unsigned)(((n * P.Hd + (i * eh + ca)) * P.Wd + (j * ew + cb)) * P.Cd) * DBYTES;
            }
            row_off[r] = off;
            row_lo[r] = ~(unsigned)in;
            row_hi[r] = ~(unsigned)(in >> 32);
            if (MODE == 1) row_dst[r] = dst;
        }
        __syncthreads();
    }

    const bool fetcher = wave >= IW0;

    // ---- fetching side ---------------------------------------------------------------------
    // A wave that only fetches takes PA consecutive load instructions of the activations and PB of the filter (one that
    // multiplies too takes every NI-th); where these are more than the tile has, the last ones fetch nothing (into the
    // stage's padding).
    const int fw = wave - IW0;                      // fetching wave index
    constexpr int GAP = NP ? 1 : NI;                // load instructions from one of a wave to its next
    static_assert(NP > 0 || (NA % NI == 0 && NB % NI == 0), "no padding");
    auto a_instr = [&](int p) __attribute__((always_inline)) { return (NP ? fw * PA : fw) + p * GAP; };
    auto b_instr = [&](int p) __attribute__((always_inline)) { return (NP ? fw * PB : fw) + p * GAP; };
    auto chunk_of = [&](int r) __attribute__((always_inline)) { return (lane & 7) ^ ((r >> 1) & 7); };     // logical chunk that lands in this lane's slot of row r
    unsigned off[PL], out[PA];                      // out: bit t: tap t (of 0..31) of this row is outside
    const bool partial = (P.Cs % BK) != 0;          // last channel chunk is short
    if (fetcher) {
#pragma unroll
        for (int p = 0; p < PA; ++p) {
            const int r = a_instr(p) * 8 + (lane >> 3);
            out[p] = 0;
            if (PA * NI > NA && r >= BM) {
                off[p] = kOutOfRange;
                out[p] = ~0u;
            } else if (P.pointwise) {
                off[p] = m0 + r < Mcls ? (unsigned)(((m0 + r) * P.Cs + chunk_of(r) * 8) * 2) : kOutOfRange;
            } else {
                off[p] = row_off[r] + (unsigned)(chunk_of(r) * 16);
                out[p] = row_lo[r];
            }
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int i = b_instr(p);               // instruction of the filter tile
            unsigned o;
            if (KROWS) {
                const int r = i * 8 + (lane >> 3), n = n0 + r;
                o = (n < P.Cd) ? (unsigned)((n * P.b_row_pitch + chunk_of(r) * 8) * 2) : kOutOfRange;
            } else {
                // [64 filters][BN channels]: chunk slot i * 64 + lane of the tile
                const int slot = i * 64 + lane;
                const int krow = slot / (BN / 8), pc = slot % (BN / 8);
                const int c = n0 + swizzled_chunk<BN>(krow, pc) * 8;
                o = (c < P.Cd) ? (unsigned)((krow * P.b_row_pitch + c) * 2) : kOutOfRange;
            }
            off[PA + p] = PB * NI > NB && i >= NB ? kOutOfRange : o;
        }
    }
    const unsigned spanA = (unsigned)(P.NB * P.Hs * P.Ws * P.Cs) * 2u, spanB = (unsigned)((KROWS ? P.Cd : P.Cs) * P.b_row_pitch) * 2u;
    const unsigned to_a = lds0 + (NP ? fw * PA : fw) * 1024, to_b = lds0 + ABYTES + (NP ? fw * PB : fw) * 1024;
    auto uniform = [](int v) __attribute__((always_inline)) { return (unsigned)__builtin_amdgcn_readfirstlane(v); };

    // The contraction step the next loads fetch: tap (counted from the first), its column in the grid of taps, channel
    // chunk, and the tap's byte displacements in the source image (ad) and in a filter row (bo).
    // Taps vary fastest: the taps of a 3x3 re-read nearly the same pixels of one channel slab back to back, while it is
    // still in L2.
    const int bpt = (KROWS ? P.Cs : P.Cd) * 2;                  // filter bytes of a tap
    const int ad0 = (th.disp * P.Ws + tw.disp) * P.Cs * 2, ad_w = P.tap_dw * P.Cs * 2;
    const int ad_h = (P.tap_dh * P.Ws - (tw.count - 1) * P.tap_dw) * P.Cs * 2;
    const int bo0 = (th.first * P.S + tw.first) * bpt, bo_w = P.tap_sw * bpt;
    const int bo_h = (P.tap_sh * P.S - (tw.count - 1) * P.tap_sw) * bpt;
    const int bk = KROWS ? ROWB : BK * P.b_row_pitch * 2;       // filter bytes from one channel chunk to the next
    // Any layer.  What only the last, short channel chunk or a 33rd tap needs is kept off the common path.
    struct Step { int tap, col, kc, ad, bo; };
    const int4v rsrcA0 = make_rsrc(P.A, spanA), rsrcB0 = make_rsrc(P.B, spanB);
    auto issue = [&](int stage, Step& nx) __attribute__((always_inline)) {
        const unsigned cbytes = uniform(nx.kc * ROWB), bsoff = uniform(nx.bo + nx.kc * bk), ad = uniform(nx.ad);
        const unsigned base_a = uniform((int)(to_a + stage * STAGE)), base_b = uniform((int)(to_b + stage * STAGE));
        const int cleft = P.Cs - nx.kc * BK;        // channels left from this chunk's start
        auto load_a = [&](int p, unsigned voff) { dma16(voff, rsrcA0, cbytes, base_a + p * GAP * 1024); };
        auto load_b = [&](int p, unsigned voff) { dma16(voff, rsrcB0, bsoff, base_b + p * GAP * 1024); };
        // (where these waves multiply too, the lane number is read anew in the rare branches: what follows from it is not kept in
        // registers meanwhile)
        if (partial && cleft < BK) {
            int lane = threadIdx.x & 63;
            if constexpr (NP == 0) asm volatile("" : "+v"(lane));
            // Lanes whose chunk is past the last channel: in the row 8 * i + lane / 8 of instruction i it depends on the lane and on
            // whether i is odd.  Worked out for each load it made such layers 6-20 % slower on the tiles without waves that only
            // fetch (3x3 data gradient, 72->256 on 2x50x84, 224x256 tiles 30.1 -> 26.7 us, 256x256 33.6 -> 29.1) and 13-30 % with more than 32 taps.
            const int even = (lane & 7) ^ (lane >> 4);
            const unsigned past[2] = {even * 8 >= cleft ? kOutOfRange : 0u, (even ^ 4) * 8 >= cleft ? kOutOfRange : 0u};
            if (nx.tap < 32) {
                const int sh = 31 - nx.tap;
#pragma unroll
                for (int p = 0; p < PA; ++p)
                    load_a(p, (int)((out[p] << sh) | past[a_instr(p) & 1]) < 0 ? kOutOfRange : off[p] + ad);
            } else {
#pragma unroll
                for (int p = 0; p < PA; ++p) {
                    const int r = a_instr(p) * 8 + (lane >> 3);
                    const unsigned o = PA * NI > NA && r >= BM ? ~0u : row_hi[r];
                    load_a(p, (int)((o << (63 - nx.tap)) | past[a_instr(p) & 1]) < 0 ? kOutOfRange : off[p] + ad);
                }
            }
            // KROWS: the filter's rows are those of the other operand; else instruction i holds contraction rows from i * 512 / BN on
            const int row0 = b_instr(0) * (512 / BN) + lane / (BN / 8);
#pragma unroll
            for (int p = 0; p < PB; ++p)
                load_b(p, (KROWS ? past[b_instr(p) & 1] != 0u : row0 + p * GAP * (512 / BN) >= cleft) ? kOutOfRange : off[PA + p]);
        } else {
            if (P.pointwise) {
#pragma unroll
                for (int p = 0; p < PA; ++p) load_a(p, off[p]);
            } else if (nx.tap < 32) {
                const int sh = 31 - nx.tap;
#pragma unroll
                for (int p = 0; p < PA; ++p) load_a(p, (int)(out[p] << sh) < 0 ? kOutOfRange : off[p] + ad);
            } else {
                int lane = threadIdx.x & 63;
                if constexpr (NP == 0) asm volatile("" : "+v"(lane));
#pragma unroll
                for (int p = 0; p < PA; ++p) {
                    const int r = a_instr(p) * 8 + (lane >> 3);
                    const unsigned o = PA * NI > NA && r >= BM ? ~0u : row_hi[r];
                    load_a(p, (o >> (nx.tap - 32)) & 1u ? kOutOfRange : off[p] + ad);
                }
            }
#pragma unroll
            for (int p = 0; p < PB; ++p) load_b(p, off[PA + p]);
        }
        if (nx.tap + 1 == ntaps) nx = Step{0, 0, nx.kc + 1, ad0, bo0};
        else {
            const bool wrap = nx.col + 1 == tw.count;
            nx = Step{nx.tap + 1, wrap ? 0 : nx.col + 1, nx.kc, nx.ad + (wrap ? ad_h : ad_w), nx.bo + (wrap ? bo_h : bo_w)};
        }
        nx.tap = __builtin_amdgcn_readfirstlane(nx.tap);
        nx.kc = __builtin_amdgcn_readfirstlane(nx.kc);
    };

    if constexpr (NP > 0) if (fetcher) {
        // ---- dedicated fetching wave: S-1 steps ahead of the multipliers ---------------------
        int is = 0;
        auto fetch = [&](int from, int to, auto send) __attribute__((always_inline)) {
#pragma unroll 1
            for (int q = from; q < to; ++q) {
                if (q >= S - 1) {
                    wait_vmcnt<INFLIGHT>();
                    stage_barrier();       // step q-(S-1) is in LDS; the stage before it is free
                }
                send(is);
                is = (is + 1 == S) ? 0 : is + 1;
            }
        };
        if (P.tap_bias < 0) {
            Step nx{0, 0, 0, ad0, bo0};
            fetch(0, nk, [&](int stage) __attribute__((always_inline)) { issue(stage, nx); });
        } else {
            // A wave issues an instruction every four to six cycles and the texture path takes a load in 16, so the number
            // of its instructions is what bounds a fetching wave: a 64x64 tile's step of 16 loads took the time of 64
            // B/ns and compute unit where loads alone reach 130 (one or two waves are enough for that).  So here a run of
            // loads shares one LDS base (dma16_runs) and one scalar offset, in which tap and channel chunk are
            // counted; pointwise layers have nothing else to do, others two vector operations a load that put the
            // taps outside the image past the descriptor's range.  3x3 512->128 on 16x512, 64x64 tiles: 22.9 -> 17.9 us;
            // 3x3 256->256 on 2x50x84, 80x128 tiles, with the order of reads below: 17.4 -> 14.6, data gradient 17.8 -> 15.3.
            const unsigned char* a0 = reinterpret_cast<const unsigned char*>(P.A) - kRunSlack - P.tap_bias;
            const int4v rsrcA = make_rsrc(a0, spanA + kRunSlack + P.tap_bias);
            const int4v rsrcB = make_rsrc(reinterpret_cast<const unsigned char*>(P.B) - kRunSlack, spanB + kRunSlack);
#pragma unroll
            for (int p = 0; p < PA; ++p) off[p] += kRunSlack - run_offset(p);
#pragma unroll
            for (int p = 0; p < PB; ++p) off[PA + p] += kRunSlack - run_offset(p);
            int so_a = P.tap_bias + ad0, so_b = bo0, tap = 0, col = 0;
            const int whole = partial ? nk - ntaps : nk;        // steps with 64 channels
            // a chunk's last tap lies (count_h - 1) rows and (count_w - 1) columns from the next chunk's first
            // (ad_kh, bo_kh: what such a move is more than one to the next row of taps)
            const int ad_kh = ROWB - ((th.count - 1) * P.tap_dh * P.Ws + (tw.count - 1) * P.tap_dw) * P.Cs * 2 - ad_h;
            const int bo_kh = bk - ((th.count - 1) * P.tap_sh * P.S + (tw.count - 1) * P.tap_sw) * bpt - bo_h;
            auto next_tap = [&]() __attribute__((always_inline)) {
                if (++col < tw.count) {
                    ++tap;
                    so_a += ad_w;
                    so_b += bo_w;
                } else {
                    const bool last = tap + 1 == ntaps;
                    col = 0;
                    tap = last ? 0 : tap + 1;
                    so_a += ad_h + (last ? ad_kh : 0);
                    so_b += bo_h + (last ? bo_kh : 0);
                }
            };
            if (P.pointwise) {
                fetch(0, whole, [&](int stage) __attribute__((always_inline)) {
                    dma16_runs<PA>(off, rsrcA, uniform(so_a), uniform((int)(to_a + stage * STAGE)));
                    dma16_runs<PB>(off + PA, rsrcB, uniform(so_b), uniform((int)(to_b + stage * STAGE)));
                    so_a += ROWB;
                    so_b += bk;
                });
            } else {
                fetch(0, whole, [&](int stage) __attribute__((always_inline)) {
                    unsigned v[PA];
                    const int sh = 31 - tap;
#pragma unroll
                    for (int p = 0; p < PA; ++p) v[p] = (out[p] << sh & kOutOfRange) | off[p];
                    dma16_runs<PA>(v, rsrcA, uniform(so_a), uniform((int)(to_a + stage * STAGE)));
                    dma16_runs<PB>(off + PA, rsrcB, uniform(so_b), uniform((int)(to_b + stage * STAGE)));
                    next_tap();
                });
            }
            if (whole < nk) {           // the last channel chunk is short
                const int cleft = P.Cs % BK;
#pragma unroll
                for (int p = 0; p < PA; ++p)
                    if (chunk_of(a_instr(p) * 8 + (lane >> 3)) * 8 >= cleft) { off[p] = kOutOfRange; out[p] = ~0u; }
#pragma unroll
                for (int p = 0; p < PB; ++p) {
                    const int contraction = KROWS ? chunk_of(b_instr(p) * 8 + (lane >> 3)) * 8 : (b_instr(p) * 64 + lane) / (BN / 8);
                    if (contraction >= cleft) off[PA + p] = kOutOfRange;
                }
                fetch(whole, nk, [&](int stage) __attribute__((always_inline)) {
                    unsigned v[PA];
                    const int sh = 31 - tap;
#pragma unroll
                    for (int p = 0; p < PA; ++p) v[p] = (out[p] << sh & kOutOfRange) | off[p];
                    dma16_runs<PA>(v, rsrcA, uniform(so_a), uniform((int)(to_a + stage * STAGE)));
                    dma16_runs<PB>(off + PA, rsrcB, uniform(so_b), uniform((int)(to_b + stage * STAGE)));
                    next_tap();
                });
            }
        }
        for (int it = nk > S - 1 ? nk - (S - 1) : 0; it < nk; ++it) {
            if (it + S - 2 < nk) wait_vmcnt<INFLIGHT>(); else wait_vmcnt<0>();
            stage_barrier();
        }
        return;
    }

    // byte offset in the destination of the pixel that tile row r goes to
    const bool straight = MODE == 0 || (eh == 1 && ew == 1);        // destination pixel index == GEMM row index
    auto dst_off = [&](int r) -> unsigned {
        if (straight) return m0 + r < Mcls ? (unsigned)((m0 + r) * P.Cd) * DBYTES : kOutOfRange;
        return row_dst[r];
    };

    // ---- multiplying side ------------------------------------------------------------------
    const int wk = wave / (WGM * WGN), wmn = wave % (WGM * WGN), wm = wmn / WGN, wn = wmn % WGN;
    typedef typename std::conditional<MF == 32, float16v, float4v_>::type acc_t;
    acc_t acc[FN][FM];
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
        for (int b = 0; b < FM; ++b)
#pragma unroll
            for (int e = 0; e < ACCN; ++e) acc[a][b][e] = 0.f;

    // binary32: what a chain of kFoldSteps steps has added up goes to sums of its own, so that the rounding
    // errors do not grow with the length of the contraction
    constexpr int kFoldSteps = 2;
    acc_t sum[F32 ? FN : 1][F32 ? FM : 1] = {};
    auto fold = [&]() {
        if constexpr (F32) {
#pragma unroll
            for (int a = 0; a < FN; ++a)
#pragma unroll
                for (int b = 0; b < FM; ++b)
#pragma unroll
                    for (int e = 0; e < ACCN; ++e) {
                        sum[a][b][e] += acc[a][b][e];
                        acc[a][b][e] = 0.f;
                    }
        }
    };

    // fragment lane mapping: row (or column) lane % MF of a block, contraction chunk lane / MF
    const int frow = lane & (MF - 1), lhi = lane / MF;
    constexpr int KSTEP = MF == 32 ? 16 : 32;       // contraction values per MFMA
    constexpr int CPK = KSTEP / 8;                  // 16-byte chunks per MFMA step
    constexpr int NCH = BK / KSTEP / KS;            // portions of KSTEP contraction values that a wave takes of a step
    // ORDERED: the fragments of the first portion are read at once and those of the next ones one by one between the matrix
    // instructions, where the compiler on its own reads them just before their use or all in one go, and the matrix pipe
    // waits: 3x3 256->256 on 2x50x84, 96x128 tiles 15.0 -> 13.4 us forward, 16.7 -> 16.2 data gradient, 224x128 23.9 ->
    // 22.4 and 25.7 -> 24.0, 128x128 data gradient 19.1 -> 17.2; 1x1 2048->512 on 25 088 pixels, 224x256, 51.4 -> 47.4.
    // It takes a second set of fragments, and tiles that lose a workgroup or spill for it do not have it (128x128 with
    // two workgroups a compute unit, 1x1 512->128 data gradient: 10.6 us against 14.0); nor do waves with a few matrix blocks,
    // whose reads then wait for them (64x128, 3x3 data gradient: 25.5 against 27.2; 160x256 with waves that fetch too: 1-3 % slower).
    constexpr int PERCU = 160 * 1024 / (S * STAGE + 16 * BM), WAVES = (NW * (PERCU < 1 ? 1 : PERCU) + 3) / 4;     // ... a SIMD
    constexpr bool ORDERED = !F32 && FM >= (NP ? 2 : 7) && WM * WN >= 2048 && FM * FN * ACCN + 8 * (FM + FN) + 24 <= 512 / WAVES;
    auto compute = [&](int stage) __attribute__((always_inline)) {
        const unsigned char* sa = smem + stage * STAGE;
        const unsigned char* sb = sa + ABYTES;
#pragma unroll
        for (int k0 = 0; k0 < NCH; ++k0) {
            const int kk = KS > 1 ? wk * NCH + k0 : k0, chunk = kk * CPK + lhi;
            half8 fa[FM], fb[FN];
#pragma unroll
            for (int b = 0; b < FM; ++b) {
                int row = wm * WM + b * MF + frow;
                fa[b] = *reinterpret_cast<const half8*>(sa + row * ROWB + ((chunk ^ ((row >> 1) & 7)) << 4));
            }
#pragma unroll
            for (int a = 0; a < FN; ++a) {
                if (KROWS) {
                    int row = wn * WN + a * MF + frow;
                    fb[a] = *reinterpret_cast<const half8*>(sb + row * ROWB + ((chunk ^ ((row >> 1) & 7)) << 4));
                } else if (MF == 32) {
                    fb[a] = lds_frag_tr<BN>(sb, kk * 16, wn * WN + a * 32, lane);
                } else {
                    fb[a] = lds_frag_tr_16<BN>(sb, kk * 32, wn * WN + a * 16, lane);
                }
            }
            // binary32: the four floats of a lane's chunk go into four instructions; the filter's lanes do
            // the same, so both sides agree on which contraction index sits in which slot
#pragma unroll
            for (int t = 0; t < (F32 ? 4 : 1); ++t)
#pragma unroll
                for (int a = 0; a < FN; ++a)
#pragma unroll
                    for (int b = 0; b < FM; ++b) {
                        if constexpr (F32)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float4v_, fb[a])[t],
                                                                             __builtin_bit_cast(float4v_, fa[b])[t], acc[a][b], 0, 0, 0);
                        else if constexpr (MF == 32)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[a], fa[b], acc[a][b], 0, 0, 0);
                        else
                            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[a], fa[b], acc[a][b], 0, 0, 0);
                    }
        }
        if constexpr (ORDERED) {        // 0x100: LDS reads, 0x008: matrix instructions
            constexpr int FIRST = FM + FN * (KROWS ? 1 : 2), REST = (NCH - 1) * FIRST, MULS = NCH * FM * FN - FM;
            constexpr int EACH = (REST + MULS - 1) / MULS;
            __builtin_amdgcn_sched_group_barrier(0x100, FIRST, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, FM, 0);
#pragma unroll
            for (int i = 0; i < (REST + EACH - 1) / EACH; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, EACH, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, MULS, 0);
        }
    };

    // TAIL: the lines of the shortcut or mask tensor that the epilogue will read are fetched into L2 before
    // the loop ends, one line a lane and load, by the waves that send no operand loads.
    constexpr int NLINES = BM * BN / 64, WARM = 64 * (NP ? NWC : NWC / 2), NWARM = TAIL ? (NLINES + WARM - 1) / WARM : 1;
    int warm[NWARM] = {};
    const int warm_at = nk > kWarmSteps ? nk - kWarmSteps : 0;
    auto warm_tail = [&]() {
        if constexpr (TAIL) {
            const __half* aux = P.ep.residual ? P.ep.residual : P.ep.mask;
            if (!aux || !straight) return;
            const __amdgpu_buffer_rsrc_t rsrcX = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<__half*>(aux), 0, (int)((unsigned)(P.NB * P.Hd * P.Wd * P.Cd) * 2u), 0x00020000);
#pragma unroll
            for (int i = 0; i < NWARM; ++i) {
                const int line = i * WARM + tid, r = line / (BN / 64), c = n0 + line % (BN / 64) * 64;
                const unsigned o = r < BM ? dst_off(r) : kOutOfRange;
                warm[i] = __builtin_amdgcn_raw_buffer_load_b32(
                    rsrcX, o != kOutOfRange && c < P.Cd ? o + (unsigned)c * 2u : kOutOfRange, 0, 0);
            }
        }
    };

    if (NP > 0) {
        int cs = 0;
        for (int it = 0; it < nk; ++it) {
            if (TAIL && it == warm_at) warm_tail();
            stage_barrier();
            compute(cs);
            if (F32 && it % kFoldSteps == kFoldSteps - 1) fold();
            cs = (cs + 1 == S) ? 0 : cs + 1;
        }
        if constexpr (F32) {
#pragma unroll
            for (int a = 0; a < FN; ++a)
#pragma unroll
                for (int b = 0; b < FM; ++b)
#pragma unroll
                    for (int e = 0; e < ACCN; ++e) acc[a][b][e] += sum[a][b][e];
        }
    } else {
        // upper half of the waves fetches for the whole group, then multiplies its own share
        Step nx{0, 0, 0, ad0, bo0};
        if (fetcher) {
#pragma unroll 1
            for (int s = 0; s < S - 1 && s < nk; ++s) issue(s, nx);
        }
        int cs = 0, is = (S - 1) % S;
        for (int it = 0; it < nk; ++it) {
            if (TAIL && !fetcher && it == warm_at) warm_tail();
            if (fetcher) { if (it + S - 2 < nk) wait_vmcnt<INFLIGHT>(); else wait_vmcnt<0>(); }
            stage_barrier();
            if (fetcher && it + S - 1 < nk) issue(is, nx);
            is = (is + 1 == S) ? 0 : is + 1;
            compute(cs);
            cs = (cs + 1 == S) ? 0 : cs + 1;
        }
    }
    if (TAIL) {
#pragma unroll
        for (int i = 0; i < NWARM; ++i) asm volatile("" :: "v"(warm[i]));
    }

    if constexpr (F32) {
        if constexpr (KS > 1) {     // the groups' sums, added in the order of the groups
            float4v_* sums = reinterpret_cast<float4v_*>(smem);
            static_assert((KS - 1) * BM * BN * 4 <= S * STAGE, "sums fit in the ring");
            auto slot = [&](int group, int a, int b, int q) {
                return ((((group - 1) * WGM * WGN + wmn) * FN + a) * FM + b) * 256 + q * 64 + lane;
            };
            __syncthreads();        // everybody is done reading the last stage
            if (wk > 0) {
#pragma unroll
                for (int a = 0; a < FN; ++a)
#pragma unroll
                    for (int b = 0; b < FM; ++b)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            sums[slot(wk, a, b, q)] = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
            }
            __syncthreads();
            if (wk > 0) return;
#pragma unroll
            for (int group = 1; group < KS; ++group)
#pragma unroll
                for (int a = 0; a < FN; ++a)
#pragma unroll
                    for (int b = 0; b < FM; ++b)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float4v_ v = sums[slot(group, a, b, q)];
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[a][b][4 * q + e] += v[e];
                        }
        }
        // a lane holds four consecutive destination channels of a pixel: stored as they are
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const __amdgpu_buffer_rsrc_t rsrcD =
            __builtin_amdgcn_make_buffer_rsrc(P.D, 0, (int)((unsigned)(P.NB * P.Hd * P.Wd * P.Cd) * 4u), 0x00020000);
#pragma unroll
        for (int b = 0; b < FM; ++b) {
            const unsigned o = dst_off(wm * WM + b * 32 + frow);
#pragma unroll
            for (int a = 0; a < FN; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = n0 + wn * WN + a * 32 + 8 * q + 4 * lhi;
                    const float4v_ v = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
                    __builtin_amdgcn_raw_buffer_store_b128(
                        __builtin_bit_cast(u4, v), rsrcD,
                        o != kOutOfRange && col < P.Cd ? o + (unsigned)col * 4u : kOutOfRange, 0, 0);
                }
        }
        return;
    } else {
    // ---- epilogue: through a per-wave LDS strip into 16-byte NHWC stores --------------------
    static_assert(NWC * epilogue_strip_bytes<WN, MF>() <= S * STAGE, "epilogue strips fit in the ring");
    stage_barrier();                                // everybody is done reading the last stage
    store_rows_via_lds<FM, FN, MF, TAIL, PERCU < 2 ? 256 : 512 / WAVES / 8 * 8>(acc, smem + wave * epilogue_strip_bytes<WN, MF>(), lane, n0 + wn * WN, P,
                                         [&](int r) { return dst_off(wm * WM + r); });
    }
}

// Which tile a workgroup takes: runs of kRun consecutive tiles per XCD (workgroup b runs on XCD
// b % 8), runs interleaved over the XCDs.  Consecutive tiles are the column tiles of one row
// tile, which read the same activation rows: a run keeps them on one L2.  Measured on the
// detector step: runs of 2 beat runs of 1 (every L2 fetches every activation row), and runs of
// 4, 8 and 16 (fewer row tiles per XCD in flight at a time), by 0.5-0.9 %.
__device__ __forceinline__ int xcd_run_tile(int b)
{
    constexpr int kRun = 2;
    const int xcd = b & 7, idx = b >> 3;
    return ((idx / kRun) * 8 + xcd) * kRun + (idx % kRun);
}

// Bytes of the ring: a stage is a whole number of load instructions for each fetching wave.
template <int BM, int BN, int NWC, int S, int NP> constexpr size_t ws_ring_bytes()
{
    constexpr int NI = NP ? NP : NWC / 2;
    return (size_t)S * ((BM / 8 + NI - 1) / NI + (BN / 8 + NI - 1) / NI) * NI * 1024;
}

}  // namespace sdconv
