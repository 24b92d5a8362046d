// Kernel selection: which route and tile variant serves a given geometry and pass.
#include "common.h"
#include "igemm.h"
#include "wgrad.h"
#include "dma.h"
#include "thin.h"
#include "narrow.h"
#include <math.h>
#include <stdlib.h>
#include <map>
#include <numeric>
#include <mutex>
#include <string>

namespace sdconv {

static int env_int(const char* name, int dflt)
{
    const char* e = getenv(name);
    return (e && *e) ? atoi(e) : dflt;
}

// Tuning hooks (used by fit_models.py and by the tests that force every variant): environment
// variables that override the dispatcher, honoured only when SDCONV_TUNE=1 was set before the
// library's first call.  That switch is read once; without it no call touches the environment.
static bool tuning()
{
    static const bool on = env_int("SDCONV_TUNE", 0) != 0;
    return on;
}
static int hook(const char* name, int dflt) { return tuning() ? env_int(name, dflt) : dflt; }

static bool force_direct() { return hook("SDCONV_FORCE_DIRECT", 0) != 0; }
static int forced_variant() { return hook("SDCONV_IGEMM_VARIANT", -1); }
int forced_wgrad_splits() { return hook("SDCONV_WGRAD_SPLITS", -1); }
int forced_f32_tile() { return hook("SDCONV_F32_TILE", -1); }
static int forced_wgrad_variant() { return hook("SDCONV_WGRAD_VARIANT", -1); }

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Weight gradients that keep the choice measured for them, at the measured batch and at half to twice of it.  In
// time the models' choices are as good (a training step of the detector within 0.1 %).  What the entries fix is
// memory: through wgrad_partial_limit they hold these layers, and those with up to seven filters less, whose padded
// copies lie in the workspace too, within the array of conv2d_wgrad_static_scratch, where the rule for
// all layers lets partial sums have more and that call would be refused.
struct WgradEntry { int N, H, W, C, K, stride, variant, splits; };      // 1x1 without padding; splits 0: the model's
static const WgradEntry kWgradEntries[] = {
    {2, 200, 336, 256, 128, 1, 116, 0},
    {2, 200, 336, 256, 512, 2, 112, 0},
    {512, 14, 14, 1024, 512, 1, 114, 32},
    {512, 7, 7, 2048, 512, 1, 115, 12},
};
static const WgradEntry* wgrad_entry(const Geom& g)
{
    if (g.R * g.S != 1 || g.ph || g.pw || g.sh != g.sw || g.dh * g.dw != 1 || hook("SDCONV_NO_TUNED_TABLE", 0)) return nullptr;
    for (const WgradEntry& e : kWgradEntries)
        if (e.C == g.C && e.K == g.K && e.H == g.H && e.W == g.W && e.stride == g.sh && 2 * g.N >= e.N && g.N <= 2 * e.N) return &e;
    return nullptr;
}

// The LDS-DMA kernels address their binary16 operands with 32-bit BYTE offsets and use bit 31
// of the offset as "outside the image / past the tile" (the hardware range check then writes
// zeros).  A tensor of 2^30 elements or more has real data at such offsets, so a masked load
// would fetch it instead of zeros: those layers take the register-staged kernels (igemm.hip,
// wgrad.hip), which index elements and test every load themselves.
static bool byte_offsets_fit_31_bits(const Geom& g)
{
    const long lim = 1L << 30;
    return (long)g.N * g.H * g.W * g.C < lim && (long)g.N * g.Ho * g.Wo * g.K < lim &&
           (long)g.K * g.R * g.S * g.C < lim;
}

// The pipelined weight-gradient kernels store dw and its partial sums, 4 bytes an element, with 32-bit
// offsets of the same kind from the first filter of a matrix block of up to 32; longer filters take the
// register-staged kernels too.
static bool wgrad_offsets_fit_31_bits(const Geom& g)
{
    return byte_offsets_fit_31_bits(g) && (long)(g.K < 32 ? g.K : 32) * g.R * g.S * g.C <= 1L << 29;
}

// Fetching waves of the weight gradient use descriptors that start kRunSlack before their tensor and the same mark.
static bool wgrad_runs_fit(const Geom& g)
{
    const long most = (1L << 31) - kRunSlack;
    return 2L * g.N * g.H * g.W * g.C <= most && 2L * g.N * g.Ho * g.Wo * g.K <= most;
}

// The MFMA route moves 16-byte (8-half) vectors along the channel axis of every tensor.
static bool igemm_ok(const Geom& g)
{
    if (force_direct()) return false;
    if (g.C % 8 || g.K % 8) return false;
    if (g.R * g.S > kMaxTaps) return false;
    return true;
}

RowClasses row_classes(const Geom& g, bool dgrad)
{
    RowClasses c;
    c.n = dgrad ? g.sh * g.sw : 1;
    if (c.n == 1) {
        c.pixels[0] = (unsigned)g.N * (dgrad ? g.H * g.W : g.Ho * g.Wo);
        c.taps[0] = g.R * g.S;
        return c;
    }
    int rows[kMaxClasses], cols[kMaxClasses], taps_h[kMaxClasses] = {}, taps_w[kMaxClasses] = {};
    for (int a = 0; a < g.sh; ++a) rows[a] = g.H > a ? (g.H - a + g.sh - 1) / g.sh : 0;
    for (int b = 0; b < g.sw; ++b) cols[b] = g.W > b ? (g.W - b + g.sw - 1) / g.sw : 0;
    // tap r meets the class a with (a + ph - r * dh) % sh == 0
    for (int r = 0; r < g.R; ++r) ++taps_h[((r * g.dh - g.ph) % g.sh + g.sh) % g.sh];
    for (int t = 0; t < g.S; ++t) ++taps_w[((t * g.dw - g.pw) % g.sw + g.sw) % g.sw];
    for (int a = 0, q = 0; a < g.sh; ++a)
        for (int b = 0; b < g.sw; ++b, ++q) {
            c.pixels[q] = (unsigned)g.N * rows[a] * cols[b];
            c.taps[q] = taps_h[a] * taps_w[b];
        }
    return c;
}

// Row tiles of the fwd/dgrad index space for a tile height bm.
static int row_tiles(const Geom& g, bool dgrad, int bm, int* starts, int* nclasses)
{
    const RowClasses rows = row_classes(g, dgrad);
    int acc = 0;
    for (int q = 0; q < rows.n; ++q) {
        starts[q] = acc;
        acc += (rows.pixels[q] + bm - 1) / bm;
    }
    starts[rows.n] = acc;
    *nclasses = rows.n;
    return acc;
}

static const IgemmVariant& igemm_variant(int v)
{
    if (v >= 300) return kIgemmWsVariants[v - 300];
    return v >= 100 ? kIgemmDmaVariants[v - 100] : kIgemmVariants[v];
}

// The patch kernels take stride-1 layers whose taps span exactly two extra rows and columns
// (3x3, dilation 1) and whose contraction channels come in whole 64-channel slabs.
static bool patch_ok(const Geom& g, bool dgrad)
{
    int cs = dgrad ? g.K : g.C;
    return g.sh == 1 && g.sw == 1 && (g.R - 1) * g.dh == 2 && (g.S - 1) * g.dw == 2 && cs % 64 == 0 &&
           g.R * g.S >= 4;
}

static bool patch_variant_ok(const Geom& g, bool dgrad, int v)
{
    const PatchVariant& pv = kPatchVariants[v - 400];
    const int taps = g.R * g.S;
    if (!pv.fwd_name || (pv.one_slab && (dgrad ? g.K : g.C) != 64)) return false;
    return patch_ok(g, dgrad) && taps % 3 == 0 && taps / 3 >= pv.stages - 1;
}

static const char* igemm_name(int v, bool dgrad)
{
    if (v >= 400) return dgrad ? kPatchVariants[v - 400].dgrad_name : kPatchVariants[v - 400].fwd_name;
    return dgrad ? igemm_variant(v).dgrad_name : igemm_variant(v).fwd_name;
}

// The launch with two tile widths (324) takes undivided images only: a strided data gradient
// with its parity classes runs as the plain 224 x 256 variant.
static int ws_variant_for(const Geom& g, bool dgrad, int v)
{
    if (v == 324 && dgrad && g.sh * g.sw > 1) return 310;
    return v;
}

// Time of a forward or data-gradient pass under each tile variant.  A workgroup takes `step` us per 64 contraction channels of a tap (where several share a
// compute unit `shared` us times their number, if that is more), and `tile` us per tile besides; launch
// and first loads are `fixed`; the operands move at `hbm` MB/us meanwhile.  What decides is mostly how the
// tiles of a variant divide by 256 compute units.  Three sets of constants: pointwise layers, layers that
// gather, and strided data gradients, whose parity classes have tiles of different length (a step is that of
// gathering).  The constants are what fit_models.py makes of the timings in profiles/: least-squares fits to those
// from before the fetching waves sent runs (1444 layers), bounded by the measured rates of matrix instructions alone (2.06 PFLOP/s)
// and of streaming (6.1 TB/s; 3.5 at least) and by a start of 0.5 us; then, past these bounds, those of gathering layers scaled by the median
// of measured over predicted time (`hbm` by its inverse) where a variant is within 20 % of the fastest on the present timings of 1991 layers
// (0.8 to 1.1), and two 64x64 tiles (327 and 328), alike but for the matrix block, fitted to those for pointwise layers: long
// contractions took the slower one.  (A `step` no longer than `shared` never counts.)  Not scaled are the kernels without runs of loads
// but 101 and 427: near the fastest, their median is below one by the choice of layers alone.  On some 1000 passes of random layers whose
// kernel this changes, times fell by 5 to 8 % (112 took layers of one channel chunk from 101 that it reads twice as often: 54 -> 86 us).
// On layers left out of the scaling the choice is 1.21 % slower than the fastest of 27 measured variants (3.8 % at the 90th percentile, 19 %
// at the 99th), with all kernels scaled 1.23 %, without any scaling 1.33 % (4.3 %, 21 %), under a fit to the present timings 1.55 %
// (5.4 %, 21 %); rules by row counts were 17 % (57 %) slower.
struct RowCost { float fixed, step, shared, tile, hbm; };
struct RowModel { int variant, per_cu; RowCost pointwise, gather, strided; };   // step 0: not taken
static const RowModel kRowModels[] = {
    {101, 3, {2.626f, 0.768f, 0.611f, 1.227f, 4.342f}, {2.810f, 0.781f, 0.564f, 1.025f, 3.845f}, {}},
    {112, 5, {2.829f, 0.782f, 0.457f, 0.543f, 3.500f}, {3.552f, 0.782f, 0.437f, 0.000f, 3.500f}, {}},
    {310, 1, {0.864f, 1.208f, 0.000f, 4.512f, 4.162f}, {0.552f, 1.294f, 0.000f, 5.334f, 3.168f}, {0.500f, 1.171f, 0.000f, 6.070f, 3.500f}},
    {311, 1, {0.687f, 1.352f, 0.000f, 5.017f, 4.024f}, {0.551f, 1.427f, 0.000f, 5.654f, 3.174f}, {0.500f, 1.294f, 0.000f, 6.539f, 3.500f}},
    {316, 1, {0.960f, 0.788f, 0.000f, 3.781f, 4.578f}, {0.500f, 0.815f, 0.000f, 4.163f, 3.500f}, {0.500f, 0.815f, 0.000f, 5.306f, 3.500f}},
    {325, 1, {1.738f, 0.424f, 0.000f, 2.271f, 3.864f}, {1.534f, 0.384f, 0.000f, 2.409f, 3.679f}, {1.856f, 0.404f, 0.000f, 3.081f, 3.500f}},
    {326, 1, {1.820f, 0.956f, 0.000f, 3.075f, 4.274f}, {1.407f, 0.910f, 0.000f, 3.038f, 3.514f}, {0.525f, 0.914f, 0.000f, 5.403f, 3.500f}},
    {327, 2, {1.967f, 0.227f, 0.227f, 1.500f, 4.543f}, {1.920f, 0.239f, 0.175f, 1.251f, 3.934f}, {1.472f, 0.269f, 0.197f, 2.552f, 3.500f}},
    {328, 2, {1.943f, 0.225f, 0.225f, 1.474f, 4.453f}, {1.879f, 0.236f, 0.170f, 1.205f, 3.968f}, {1.507f, 0.268f, 0.193f, 2.561f, 3.500f}},
    {329, 1, {1.638f, 0.353f, 0.000f, 2.045f, 4.331f}, {1.464f, 0.310f, 0.000f, 2.034f, 3.789f}, {1.785f, 0.331f, 0.000f, 2.613f, 3.908f}},
    {330, 1, {1.692f, 0.469f, 0.000f, 2.452f, 4.279f}, {1.053f, 0.449f, 0.000f, 3.106f, 3.349f}, {1.500f, 0.430f, 0.000f, 3.323f, 3.578f}},
    {331, 1, {1.288f, 0.726f, 0.000f, 3.638f, 4.327f}, {0.557f, 0.738f, 0.000f, 4.697f, 3.141f}, {0.500f, 0.662f, 0.000f, 5.317f, 3.500f}},
    {332, 1, {1.523f, 0.664f, 0.000f, 3.382f, 4.467f}, {0.520f, 0.639f, 0.000f, 4.251f, 3.363f}, {0.807f, 0.614f, 0.000f, 4.943f, 3.500f}},
    {333, 1, {1.682f, 0.424f, 0.000f, 2.358f, 4.323f}, {1.394f, 0.350f, 0.000f, 2.325f, 3.850f}, {1.736f, 0.384f, 0.000f, 3.063f, 3.885f}},
    {334, 1, {1.710f, 0.392f, 0.000f, 2.198f, 4.350f}, {1.428f, 0.347f, 0.000f, 2.221f, 4.006f}, {1.818f, 0.378f, 0.000f, 2.915f, 4.006f}},
    {335, 1, {1.776f, 0.541f, 0.000f, 2.687f, 4.484f}, {1.156f, 0.507f, 0.000f, 3.194f, 3.434f}, {1.409f, 0.497f, 0.000f, 3.818f, 3.503f}},
    {336, 1, {1.686f, 0.604f, 0.000f, 3.000f, 4.519f}, {0.665f, 0.581f, 0.000f, 3.928f, 3.416f}, {1.211f, 0.553f, 0.000f, 4.326f, 3.500f}},
    {337, 1, {1.659f, 0.306f, 0.000f, 1.938f, 3.844f}, {1.495f, 0.271f, 0.000f, 1.839f, 3.957f}, {1.950f, 0.306f, 0.000f, 2.435f, 3.500f}},
    {338, 1, {1.545f, 1.019f, 0.000f, 3.132f, 4.382f}, {0.965f, 1.082f, 0.000f, 4.151f, 3.161f}, {0.500f, 0.977f, 0.000f, 5.238f, 3.500f}},
    {339, 2, {2.285f, 0.719f, 0.487f, 1.626f, 4.446f}, {2.869f, 0.707f, 0.440f, 0.744f, 3.427f}, {0.500f, 0.692f, 0.431f, 4.074f, 3.500f}},
    {340, 3, {1.952f, 0.605f, 0.340f, 1.470f, 3.831f}, {3.208f, 0.586f, 0.314f, 0.000f, 3.543f}, {0.500f, 0.593f, 0.318f, 3.724f, 3.500f}},
    {427, 2, {}, {2.317f, 0.219f, 0.219f, 1.607f, 3.493f}, {}},
    {433, 2, {}, {2.703f, 0.280f, 0.280f, 1.511f, 3.500f}, {}},
    {435, 1, {}, {1.361f, 0.324f, 0.000f, 2.480f, 3.500f}, {}},
    {436, 1, {}, {1.404f, 0.268f, 0.000f, 2.407f, 3.500f}, {}},
    {437, 1, {}, {1.595f, 0.177f, 0.000f, 1.923f, 3.500f}, {}},
};
constexpr float kEmptyTile = 0.6f;      // of `tile`: a tile of a class that no tap reaches only stores zeros

// Two resources at work together: near the larger time, more where they are alike.
static float both(float a, float b)
{
    return sqrtf(a * a + b * b);
}

// Time until the last tile is done when `slots` workgroups take the tiles in order, class by class.
struct TileClass { long tiles; float us; };
static float makespan(const TileClass* classes, int n, long slots)
{
    struct { float at; long slots; } free[kMaxClasses + 2] = {{0.f, slots}};    // sorted; a class adds at most one group
    int groups = 1;
    for (int q = 0; q < n; ++q) {
        long m = classes[q].tiles;
        const float us = classes[q].us;
        if (m > 4 * slots) {                // whole rounds move every slot alike
            const long rounds = m / slots - 2;
            for (int i = 0; i < groups; ++i) free[i].at += rounds * us;
            m -= rounds * slots;
        }
        while (m > 0) {
            const long take = free[0].slots < m ? free[0].slots : m;
            const float done = free[0].at + us;
            m -= take;
            free[0].slots -= take;
            if (free[0].slots == 0) {
                --groups;
                for (int i = 0; i < groups; ++i) free[i] = free[i + 1];
            }
            int i = groups;
            while (i > 0 && free[i - 1].at > done) --i;
            if (i > 0 && free[i - 1].at == done) {
                free[i - 1].slots += take;
                continue;
            }
            for (int j = groups; j > i; --j) free[j] = free[j - 1];
            free[i] = {done, take};
            ++groups;
        }
    }
    return free[groups - 1].at;
}

// Tiles of one length: the fullest compute unit sets the time.
static float rounds_us(unsigned tiles, float steps, int per_cu, const RowCost& c)
{
    auto round = [&](unsigned n) { return steps * (n * c.shared > c.step ? n * c.shared : c.step) + c.tile; };
    const unsigned fullest = (tiles + 255) / 256, full = fullest / per_cu, rest = fullest - full * per_cu;
    return (float)full * round(per_cu) + (rest ? round(rest) : 0.f);
}

static const RowModel& row_model(int variant)
{
    const RowModel* m = kRowModels;
    while (m->variant != variant) ++m;
    return *m;
}

// What the times of one pass under all variants have in common.  A call is planned anew each time, in front of a
// kernel of a few us, so nothing is computed for every variant that need not be, and a variant is dropped as
// soon as a lower bound of its time is above the best one: strided data gradients are planned in 0.8-1.1 us where
// it took 2.5-2.7, other passes in 0.36 where it took 0.61, with the same choices.
struct RowShape {
    bool pointwise;
    RowClasses rows;
    int cd, Hd, Wd, N;
    float slabs[2];                         // 64-channel steps a tap takes with steps of 64 and of 32 channels
    float mb;
};

static RowShape row_shape(const Geom& g, bool dgrad)
{
    RowShape s;
    s.pointwise = g.R * g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
    s.N = g.N;
    s.cd = dgrad ? g.C : g.K;
    s.Hd = dgrad ? g.H : g.Ho;
    s.Wd = dgrad ? g.W : g.Wo;
    const int cs = dgrad ? g.K : g.C;
    s.slabs[0] = (float)((cs + 63) / 64);
    s.slabs[1] = (float)((cs + 31) / 32) / 2;
    s.rows = row_classes(g, dgrad);
    const float x = 2e-6f * g.N * g.H * g.W * g.C / (g.R * g.S == 1 && !dgrad ? g.sh * g.sw : 1);    // MB
    s.mb = x + 2e-6f * g.N * g.Ho * g.Wo * g.K + 2e-6f * g.K * g.R * g.S * g.C;
    return s;
}

// Time of a variant if that is less than `best`; otherwise `best` or more, or less than 0 if it is not taken.
static float row_us(const RowShape& s, const RowModel& m, float best)
{
    const RowClasses& R = s.rows;
    const bool strided = R.n > 1, mixed = m.variant == 324;
    auto cost = [&](const RowModel& r) -> const RowCost& { return s.pointwise ? r.pointwise : strided ? r.strided : r.gather; };
    const RowModel& wide = mixed ? row_model(310) : m;
    const RowCost& c = cost(wide);
    if (c.step == 0.f || (mixed && strided)) return -1.f;
    const float slabs = s.slabs[m.variant < 300], move = s.mb / c.hbm;
    if (c.fixed + move >= best) return best;
    float work;
    if (m.variant >= 400) {
        const PatchVariant& v = kPatchVariants[m.variant - 400];
        work = rounds_us((unsigned)s.N * ((s.Hd + v.th - 1) / v.th) * ((s.Wd + v.tw - 1) / v.tw) * ((s.cd + v.bn - 1) / v.bn),
                         R.taps[0] * slabs, m.per_cu, c);
    } else {
        const IgemmVariant& v = igemm_variant(m.variant);
        const unsigned columns = (s.cd + v.bn - 1) / v.bn, bm = v.bm;
        const float steps = R.taps[0] * slabs;
        if (mixed) {                // as its launcher divides the rows: 224x256 tiles, then 224x128 ones
            const long rows = (R.pixels[0] + bm - 1) / bm, whole = mixed_wide_rows(rows, columns);
            work = rounds_us(whole * columns, steps, 1, c);
            if (whole < rows) work += rounds_us((rows - whole) * ((s.cd + 127) / 128), steps, 1, cost(row_model(316)));
        } else if (!strided) {
            work = rounds_us((R.pixels[0] + bm - 1) / bm * columns, steps, m.per_cu, c);
        } else {
            TileClass classes[kMaxClasses];
            unsigned tiles = 0;
            for (int q = 0; q < R.n; ++q) tiles += classes[q].tiles = (R.pixels[q] + bm - 1) / bm * columns;
            const unsigned fullest = (tiles + 255) / 256, crowd = fullest < (unsigned)m.per_cu ? fullest : m.per_cu;
            const float step = crowd * c.shared > c.step ? crowd * c.shared : c.step;
            float sum = 0.f;
            for (int q = 0; q < R.n; ++q) {
                classes[q].us = R.taps[q] * slabs * step + (R.taps[q] ? c.tile : kEmptyTile * c.tile);
                sum += classes[q].tiles * classes[q].us;
            }
            // the slots are busy for the sum at least (less what the rounding of either may add)
            if (c.fixed + both(sum / (256 * m.per_cu), move) * 0.9999f >= best) return best;
            work = makespan(classes, R.n, 256L * m.per_cu);
        }
    }
    return c.fixed + both(work, move);
}

static int pick_variant(const Geom& g, bool dgrad)
{
    if (!byte_offsets_fit_31_bits(g)) return (dgrad ? g.C : g.K) <= 64 ? 3 : 0;
    const int fv = forced_variant();
    if (fv >= 400 && fv < 400 + kNumPatchVariants && patch_variant_ok(g, dgrad, fv)) return fv;
    const bool known = (fv >= 0 && fv < kNumIgemmVariants) || (fv >= 100 && fv < 100 + kNumIgemmDmaVariants) ||
                       (fv >= 300 && fv < 300 + kNumIgemmWsVariants);
    if (known && (dgrad ? igemm_variant(fv).dgrad_name : igemm_variant(fv).fwd_name)) return ws_variant_for(g, dgrad, fv);
    int best = -1;
    float best_us = INFINITY;
    const RowShape shape = row_shape(g, dgrad);
    auto consider = [&](const RowModel& m) {
        const float us = row_us(shape, m, best_us);
        if (us >= 0.f && us < best_us) { best = m.variant; best_us = us; }
    };
    // the variants below 300 are forward kernels: a data gradient of that kind wants a filter copy in the
    // workspace, and was faster by 0.5 % over layers of any channel counts (by 0.02 % over a detector's)
    for (const RowModel& m : kRowModels)
        if (m.variant < 300 ? !dgrad : m.variant < 400 || patch_variant_ok(g, dgrad, m.variant)) consider(m);
    static const RowModel kMixed = {324, 1, {}, {}, {}};        // its costs are those of its halves
    consider(kMixed);
    return ws_variant_for(g, dgrad, best);
}

static bool thin_ok(const Geom& g) { return !force_direct() && g.C <= 4 && thin_supported(g); }

// Filter counts that are not a multiple of 8 (with channels that are): the layer runs as one with
// the filter count rounded up, on padded copies of the filter and of the K-channel tensor that
// live in the workspace (padk.hip).
static bool padk_ok(const Geom& g)
{
    if (force_direct() || hook("SDCONV_NO_PADK", 0)) return false;
    if (g.K % 8 == 0 || g.C % 8 != 0 || g.R * g.S > kMaxTaps || g.sh * g.sw > kMaxClasses) return false;
    // the padded copies must stay below 2^31 elements like every other tensor
    const long kp = (g.K + 7) / 8 * 8, lim = 0x7fffffffL;
    return (long)g.N * g.Ho * g.Wo * kp <= lim && kp * g.R * g.S * g.C <= lim;
}
// Of these the pointwise layers with few filters have kernels that need no copies, where those are the
// faster ones (narrow.hip).
static bool narrow_ok(const Geom& g, int pass) { return padk_ok(g) && narrow_supported(g, pass); }
static Geom padded_k(const Geom& g) { Geom p = g; p.K = (g.K + 7) / 8 * 8; return p; }
static size_t padk_filter_bytes(const Geom& gp) { return align256((size_t)gp.K * gp.R * gp.S * gp.C * sizeof(__half)); }
static size_t padk_act_bytes(const Geom& gp) { return align256((size_t)gp.N * gp.Ho * gp.Wo * gp.K * sizeof(__half)); }
static size_t padk_dw_bytes(const Geom& gp) { return align256((size_t)gp.K * gp.R * gp.S * gp.C * sizeof(float)); }

// "padk+<inner kernel name>", kept for the life of the process
static const char* padk_name(const char* inner)
{
    static std::mutex mu;
    static std::map<std::string, std::string> names;
    std::lock_guard<std::mutex> lock(mu);
    auto it = names.find(inner);
    if (it == names.end()) it = names.emplace(inner, std::string("padk+") + inner).first;
    return it->second.c_str();
}

Plan plan_fwd(const Geom& g)
{
    if (narrow_ok(g, SDCONV_FWD)) return Plan{ROUTE_NARROW, 0, 1, 0, "narrow_fwd"};
    if (padk_ok(g)) {
        const Geom gp = padded_k(g);
        const Plan in = plan_fwd(gp);
        return Plan{ROUTE_PADK, in.variant, 1, padk_filter_bytes(gp) + padk_act_bytes(gp) + in.workspace_bytes,
                    padk_name(in.name)};
    }
    if (thin_ok(g)) return Plan{ROUTE_THIN, 0, 1, align256(thin_packed_filter_bytes(g)), "thin_fwd"};
    if (!igemm_ok(g)) return Plan{ROUTE_DIRECT, 0, 1, 0, "direct_fwd"};
    int v = pick_variant(g, false);
    return Plan{ROUTE_IGEMM, v, 1, 0, igemm_name(v, false)};
}

Plan plan_dgrad(const Geom& g)
{
    if (narrow_ok(g, SDCONV_DGRAD)) return Plan{ROUTE_NARROW, 0, 1, 0, "narrow_dgrad"};
    if (padk_ok(g)) {
        const Geom gp = padded_k(g);
        const Plan in = plan_dgrad(gp);
        return Plan{ROUTE_PADK, in.variant, 1, padk_filter_bytes(gp) + padk_act_bytes(gp) + in.workspace_bytes,
                    padk_name(in.name)};
    }
    if (!force_direct() && g.C <= 4 && thin_dgrad_mfma_supported(g) && byte_offsets_fit_31_bits(g) &&
        !hook("SDCONV_NO_THIN_MFMA_DGRAD", 0))
        return Plan{ROUTE_THIN, 1, 1, align256(thin_dgrad_mfma_workspace_bytes(g)), "thin_dgrad_mfma"};
    if (!force_direct() && g.C <= 4 && g.K % 8 == 0 && g.sh * g.sw <= kMaxClasses &&
        thin_dgrad_lds_bytes(g) <= 64 * 1024)
        return Plan{ROUTE_THIN, 0, 1, align256((size_t)g.K * g.R * g.S * g.C * sizeof(__half)), "thin_dgrad"};
    if (!igemm_ok(g) || g.sh * g.sw > kMaxClasses) return Plan{ROUTE_DIRECT, 0, 1, 0, "direct_dgrad"};
    int v = pick_variant(g, true);
    // the register-staged kernels want the filter transposed to [C][R][S][K] in the workspace; the
    // split-role and patch kernels read it as stored
    size_t ws = v >= 300 ? 0 : align256((size_t)g.K * g.R * g.S * g.C * sizeof(__half));
    return Plan{ROUTE_IGEMM, v, 1, ws, igemm_name(v, true)};
}

static const WgradVariant& wgrad_variant(int v)
{
    return v >= 100 ? kWgradDmaVariants[v - 100] : kWgradVariants[v];
}

// Time of a weight gradient as a function of the tile variant and the number of pixel ranges, from
// which both are chosen.  A workgroup takes `step` us per 64-pixel step (where several share a compute unit
// `shared` us times their number, if that is more), and `tile` us per tile besides; launch and first loads are
// `fixed`; the operands move at `hbm` MB/us meanwhile, and the sums leave at `store` MB/us after the loop.
// The constants are fits to the present timings (fit_models.py; no less than the matrix instructions alone take).  The time has a narrow
// minimum between too few workgroups and the traffic of too many partial sums: rules by channel counts
// with one number of ranges for all lost 48 % over layers of random size.  The choice is 1.5 % slower than
// the fastest measured (variant, ranges) pair on layers left out of the fit (5.5 % at the 90th percentile).  300 of the 802 layers
// have 12 to 700 pixels and filters of up to 7x7: a fit to the others alone (200 pixels and more, 2.0 % slower; 3.7 % without the variants
// that have fetching waves, 120 and up) chose 2.5 % slower ones on 1000 more layers of that kind (8.9 %, 17 %; now 1.1 %, 3.8 %, 15 %):
// 256x256 tiles for a large dw (3x3 stride 2, 1984->896 on 17x11: 17.5 -> 26.9 us).
struct WgradCost { float fixed, step, shared, tile, store, hbm; };
struct WgradModel { int variant, per_cu; WgradCost linear, gather; };   // per_cu: workgroups a compute unit holds
static const WgradModel kWgradModels[] = {
    {104, 2, {2.710f, 0.429f, 0.423f, 0.000f, 2.541f, 5.669f}, {2.846f, 0.581f, 0.388f, 0.000f, 3.175f, 2.393f}},
    {107, 3, {2.285f, 0.340f, 0.294f, 0.000f, 2.701f, 4.530f}, {2.690f, 0.397f, 0.259f, 0.000f, 3.343f, 2.423f}},
    {108, 2, {2.667f, 0.430f, 0.377f, 0.000f, 2.590f, 5.105f}, {2.871f, 0.531f, 0.358f, 0.000f, 3.078f, 2.426f}},
    {112, 1, {1.154f, 0.529f, 0.000f, 2.305f, 2.761f, 6.010f}, {2.708f, 0.554f, 0.000f, 0.881f, 3.018f, 2.486f}},
    {114, 1, {1.772f, 1.256f, 0.000f, 4.186f, 3.922f, 5.405f}, {4.026f, 1.319f, 0.000f, 1.849f, 4.437f, 3.048f}},
    {115, 1, {2.383f, 1.377f, 0.000f, 3.986f, 4.322f, 6.100f}, {4.045f, 1.581f, 0.000f, 1.386f, 4.767f, 3.341f}},
    {116, 1, {1.339f, 0.527f, 0.000f, 2.239f, 2.846f, 6.100f}, {2.799f, 0.628f, 0.000f, 0.722f, 3.212f, 2.589f}},
    {117, 1, {2.312f, 0.865f, 0.000f, 2.456f, 3.207f, 6.100f}, {3.312f, 0.867f, 0.000f, 1.214f, 3.706f, 2.646f}},
    {118, 3, {2.328f, 0.343f, 0.295f, 0.000f, 2.905f, 4.558f}, {2.725f, 0.401f, 0.258f, 0.000f, 3.387f, 2.413f}},
    {119, 2, {2.671f, 0.749f, 0.496f, 0.000f, 2.962f, 4.981f}, {3.074f, 0.746f, 0.462f, 0.000f, 3.496f, 2.406f}},
    {120, 1, {1.324f, 0.458f, 0.000f, 1.996f, 2.612f, 5.114f}, {2.846f, 0.506f, 0.000f, 1.147f, 3.262f, 2.659f}},
    {121, 3, {2.375f, 0.314f, 0.290f, 0.000f, 2.580f, 4.192f}, {2.987f, 0.327f, 0.254f, 0.000f, 3.215f, 2.661f}},
    {122, 2, {2.831f, 0.400f, 0.374f, 0.000f, 2.564f, 4.821f}, {3.390f, 0.420f, 0.340f, 0.000f, 3.051f, 2.679f}},
    {123, 1, {2.099f, 0.686f, 0.000f, 3.079f, 3.317f, 6.059f}, {3.405f, 0.795f, 0.000f, 1.719f, 3.916f, 2.991f}},
};
constexpr float kWorthScratch = 1.15f;      // see choose_wgrad; with 1.1 one of 300 000 random layers that were served was refused under the present fit
constexpr float kReduceFixed = 2.5f, kReduceRate = 6.0f;    // us with the gap between the kernels, MB/us

static long wgrad_steps(const Geom& g) { return ((long)g.N * g.Ho * g.Wo + 63) / 64; }
static long wgrad_tiles(const Geom& g, const WgradVariant& v)
{
    return (long)((g.K + v.bm - 1) / v.bm) * ((g.C + v.bn - 1) / v.bn) * g.R * g.S;
}

// Bytes that the partial sums of a layer may take beside `copies` bytes of padded operands in the
// workspace.  conv2d_wgrad_static_scratch has SDCONV_STATIC_SCRATCH_BYTES for both and runs the same plan, so the
// partial sums stay within what is left of it: every layer whose copies fit is served.  Layers that need
// more for 384 workgroups of the plain tile may have that much: one range or two would leave most of the
// chip idle for long (3x3 1024 -> 1024 on 8x56x56: 562 us with the 75 MB of two ranges, 465 with three).
static size_t wgrad_partial_limit(const Geom& g, size_t copies)
{
    const long pixels = (long)g.N * g.Ho * g.Wo, steps = wgrad_steps(g);
    const int side = g.K >= 512 && g.C >= 512 && pixels >= 20000 && wgrad_offsets_fit_31_bits(g) ? 256 : 128;
    const int bm = g.K <= 64 ? 64 : side, bn = g.C <= 64 && wgrad_offsets_fit_31_bits(g) ? 64 : side;
    const long tiles = (long)((g.K + bm - 1) / bm) * ((g.C + bn - 1) / bn) * g.R * g.S;
    long ranges = (384 + tiles - 1) / tiles;
    if (ranges > steps / 4) ranges = steps / 4;
    const size_t demand = ranges > 1 ? ranges * (size_t)4 * g.K * g.R * g.S * g.C : 0;
    const size_t scratch = SDCONV_STATIC_SCRATCH_BYTES, left = copies < scratch ? scratch - copies : 0;
    if (left && wgrad_entry(g)) return left;
    return demand > left ? demand : left;
}

struct WgradChoice { int variant, splits; float us; };

// What the times of one weight gradient under all variants have in common, as RowShape for the other passes.  The numbers of
// pixel ranges to try follow from the tile alone, of which the variants share six: they are worked out once a tile, and a time
// only where its lower bounds are below the best one.  A plan of 1.1 to 1.4 us (a forward pass's: 0.6) took 2.1 to 2.5 where each
// of the 14 variants worked its ranges out for itself, with the same choices.
struct WgradRanges {
    unsigned ranges, fullest;               // workgroups of the fullest compute unit
    float n, steps, busy, reduce;           // ranges, steps of one, steps of the fullest unit's workgroups; us of the reduction
};
struct WgradTile { unsigned tiles; int n; WgradRanges at[14]; };    // n < 0: not worked out yet
struct WgradShape {
    bool linear;
    unsigned total;                         // 64-pixel steps
    size_t dw_bytes;
    float dw, mb;                           // MB of dw, of x and dy
    WgradTile of[3][3];                     // by tile height and width 64, 128, 256
};

static void wgrad_shape(const Geom& g, WgradShape* s)
{
    s->linear = g.R * g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
    s->total = (unsigned)wgrad_steps(g);
    s->dw_bytes = (size_t)4 * g.K * g.R * g.S * g.C;
    s->dw = 4e-6f * g.K * g.R * g.S * g.C;
    const float x = 2e-6f * g.N * g.H * g.W * g.C / (g.R * g.S == 1 ? g.sh * g.sw : 1);
    s->mb = x + 2e-6f * g.N * g.Ho * g.Wo * g.K;
    unsigned up[2][3];                      // tiles along K and C
    for (int i = 0; i < 3; ++i) {
        up[0][i] = ((unsigned)g.K + (64u << i) - 1) >> (6 + i);
        up[1][i] = ((unsigned)g.C + (64u << i) - 1) >> (6 + i);
    }
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            s->of[i][j].tiles = up[0][i] * up[1][j] * g.R * g.S;
            s->of[i][j].n = -1;
        }
}

// The numbers of ranges that make the workgroups a little fewer than a multiple of the compute units, and the smallest; those
// whose partial sums take no more than `limit`.
static void wgrad_ranges(const WgradShape& s, size_t limit, WgradTile* t)
{
    static const int candidates[] = {1, 2, 3, -40, -64, -96, -128, -192, -256, -320, -384, -512, -768, -1024};
    unsigned last = 0;
    t->n = 0;
    for (int cand : candidates) {                           // ranges, or minus the workgroups to make
        unsigned n = cand > 0 ? (unsigned)cand : (unsigned)-cand / t->tiles;
        if (n > s.total / 2) n = s.total / 2;
        if (n < 1) n = 1;
        if (n <= last) continue;                            // (the next lines only make it smaller)
        const unsigned steps = (s.total + n - 1) / n;
        n = (s.total + steps - 1) / steps;                  // ranges that are not empty
        if (n <= last) continue;
        if (n > 1 && n * s.dw_bytes > limit) return;
        last = n;
        const unsigned fullest = (t->tiles * n + 255) / 256;
        t->at[t->n++] = WgradRanges{n, fullest, (float)n, (float)steps, (float)steps * fullest,
                                    n > 1 ? n * s.dw / kReduceRate + kReduceFixed : 0.f};
    }
}

// The fastest number of ranges for one variant whose partial sums take no more than `limit`, if faster than `best`; and, where
// that is asked for, the fastest whose sums take no more than `left`, unless it is too slow to be taken (choose_wgrad).
static void wgrad_best_splits(WgradShape* s, const WgradModel& m, size_t limit, WgradChoice* best, size_t left, WgradChoice* within)
{
    const WgradCost& c = s->linear ? m.linear : m.gather;
    const WgradVariant& v = kWgradDmaVariants[m.variant - 100];
    WgradTile* t = &s->of[v.bm >> 7][v.bn >> 7];
    const float move = s->mb / c.hbm, store = s->dw / c.store;
    auto late = [&](float us) {
        return us >= best->us && (!within || us >= within->us || us >= kWorthScratch * 1.0001f * best->us);
    };
    // No compute unit takes less than an even share of all steps, at its best rate, and more ranges store more; nor does the
    // fullest one take its own steps faster.  (0.9999: what the rounding of either side may add.)
    const float rate = c.shared > c.step / m.per_cu ? c.shared : c.step / m.per_cu;
    const float even = (c.fixed + both((float)t->tiles * s->total * rate / 256, move)) * 0.9999f;
    if (late(even + store)) return;
    if (t->n < 0) wgrad_ranges(*s, limit, t);
    for (const WgradRanges* r = t->at; r < t->at + t->n; ++r) {
        if (late(even + r->n * store)) break;
        const float rest_us = r->n * store + r->reduce;
        if (late((c.fixed + r->busy * rate + rest_us) * 0.9999f)) continue;
        auto round = [&](unsigned n) { return r->steps * (n * c.shared > c.step ? n * c.shared : c.step) + c.tile; };
        const unsigned full = r->fullest / m.per_cu, rest = r->fullest - full * m.per_cu;
        const float work = (float)full * round(m.per_cu) + (rest ? round(rest) : 0.f);
        const float us = c.fixed + both(work, move) + r->n * store + r->reduce;
        if (us < best->us) *best = WgradChoice{m.variant, (int)r->ranges, us};
        if (within && us < within->us && (r->ranges == 1 || r->ranges * s->dw_bytes <= left))
            *within = WgradChoice{m.variant, (int)r->ranges, us};
    }
}

// Tile variant and pixel ranges.  A layer with an entry takes its variant and, at the measured batch, its
// ranges if it has any; else the model's for that variant.
static WgradChoice choose_wgrad(const Geom& g, size_t copies)
{
    const size_t partial_limit = wgrad_partial_limit(g, copies);
    const int fv = forced_wgrad_variant();
    const bool runs = wgrad_runs_fit(g);
    const bool forced = (fv >= 0 && fv < kNumWgradVariants) || (fv >= 100 && fv < 100 + kNumWgradDmaVariants && wgrad_variant(fv).name && (runs || !wgrad_variant(fv).runs));
    int only = forced ? fv : -1;
    const WgradEntry* e = nullptr;
    if (!wgrad_offsets_fit_31_bits(g)) only = g.K <= 64 ? 1 : 0;
    else if (!forced && (e = wgrad_entry(g))) only = e->variant;
    const WgradChoice none{-1, 1, INFINITY};
    WgradChoice c = none;
    if (!(e && e->splits > 0 && e->N == g.N)) {
        // Partial sums that outgrow the static scratch have to be worth it: the models are off by some per cent, and
        // conv2d_wgrad_static_scratch refuses the layer for them.
        const size_t scratch = SDCONV_STATIC_SCRATCH_BYTES, left = copies < scratch ? scratch - copies : 0;
        const bool outgrow = left < partial_limit;
        WgradChoice within = none;
        WgradShape shape;
        wgrad_shape(g, &shape);
        for (const WgradModel& m : kWgradModels)
            if (only < 0 ? runs || !wgrad_variant(m.variant).runs : m.variant == only)
                wgrad_best_splits(&shape, m, partial_limit, &c, left, outgrow ? &within : nullptr);
        if (outgrow && c.splits > 1 && c.splits * shape.dw_bytes > left && within.us <= kWorthScratch * c.us) c = within;
    }
    if (c.variant < 0) {
        long want;
        if (e) {
            want = e->splits;
        } else {            // forced, or indexed by elements: enough workgroups to fill the chip
            const long tiles = wgrad_tiles(g, wgrad_variant(only)), most = wgrad_steps(g) / 4;
            want = (384 + tiles - 1) / tiles;
            if (want > most) want = most;
        }
        const size_t dw_bytes = (size_t)4 * g.K * g.R * g.S * g.C;
        if (want > 1 && want * dw_bytes > partial_limit) want = (long)(partial_limit / dw_bytes);
        c = WgradChoice{only, (int)(want < 1 ? 1 : want), 0.f};
    }
    if (const int fs = forced_wgrad_splits(); fs > 0) {
        const long cap = wgrad_steps(g) / 2;
        c.splits = fs < cap ? fs : (cap < 1 ? 1 : (int)cap);
    }
    return c;
}

// `copies`: bytes of padded operands that the plan's workspace lies behind
static Plan plan_wgrad_beside(const Geom& g, size_t copies)
{
    if (narrow_ok(g, SDCONV_WGRAD))
        return Plan{ROUTE_NARROW, 0, narrow_wgrad_ranges(g), align256(narrow_wgrad_partial_bytes(g)), "narrow_wgrad"};
    if (padk_ok(g)) {
        const Geom gp = padded_k(g);
        const size_t padded = padk_act_bytes(gp) + padk_dw_bytes(gp);
        const Plan in = plan_wgrad_beside(gp, padded);
        return Plan{ROUTE_PADK, in.variant, in.splits, padded + in.workspace_bytes, padk_name(in.name)};
    }
    if (thin_ok(g)) return Plan{ROUTE_THIN, 0, 1, align256(thin_wgrad_partial_bytes(g)), "thin_wgrad"};
    if (!igemm_ok(g)) return Plan{ROUTE_DIRECT, 0, 1, 0, "direct_wgrad"};
    const WgradChoice c = choose_wgrad(g, copies);
    const int v = c.variant;
    const long total_steps = wgrad_steps(g), sps = (total_steps + c.splits - 1) / c.splits;
    const int splits = (int)((total_steps + sps - 1) / sps);
    size_t ws = splits > 1 ? align256((size_t)splits * g.K * g.R * g.S * g.C * sizeof(float)) : 0;
    Plan p{ROUTE_IGEMM, v, splits, ws, wgrad_variant(v).name};
    p.steps_per_split = (int)sps;
    return p;
}

Plan plan_wgrad(const Geom& g) { return plan_wgrad_beside(g, 0); }

// Taps of one axis that meet class c of a data gradient with stride s: those with c + pad - tap * dil a
// multiple of s, every s / gcd(s, dil)-th one.  A forward pass is s = 1 with its taps the other way round.
static AxisTaps axis_taps(int c, int taps, int s, int pad, int dil)
{
    AxisTaps t{0, 0, 0};
    for (int r = taps - 1; r >= 0; --r)
        if ((c + pad - r * dil) % s == 0) {
            t.first = r;
            t.disp = (c + pad - r * dil) / s;
            ++t.count;
        }
    return t;
}

void set_taps(const Geom& g, bool dgrad, IgemmParams* P)
{
    if (!dgrad) {
        P->taps_h[0] = AxisTaps{0, g.R, -g.ph};
        P->taps_w[0] = AxisTaps{0, g.S, -g.pw};
        P->tap_sh = P->tap_sw = 1;
        P->tap_dh = g.dh;
        P->tap_dw = g.dw;
    } else {
        for (int a = 0; a < g.sh; ++a) P->taps_h[a] = axis_taps(a, g.R, g.sh, g.ph, g.dh);
        for (int b = 0; b < g.sw; ++b) P->taps_w[b] = axis_taps(b, g.S, g.sw, g.pw, g.dw);
        P->tap_sh = g.sh / std::gcd(g.sh, g.dh);
        P->tap_sw = g.sw / std::gcd(g.sw, g.dw);
        P->tap_dh = -(P->tap_sh * g.dh / g.sh);
        P->tap_dw = -(P->tap_sw * g.dw / g.sw);
    }
    P->pointwise = g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
}

static hipError_t run_igemm(const Geom& g, const Plan& p, bool dgrad, const __half* A, const __half* B,
                            __half* D, hipStream_t st, const Epilogue& ep)
{
    IgemmParams P;
    P.ep = ep;
    P.A = A; P.B = B; P.D = D;
    P.NB = g.N;
    if (!dgrad) { P.Hs = g.H; P.Ws = g.W; P.Cs = g.C; P.Hd = g.Ho; P.Wd = g.Wo; P.Cd = g.K; }
    else        { P.Hs = g.Ho; P.Ws = g.Wo; P.Cs = g.K; P.Hd = g.H; P.Wd = g.W; P.Cd = g.C; }
    P.R = g.R; P.S = g.S;
    P.sh = g.sh; P.sw = g.sw; P.ph = g.ph; P.pw = g.pw; P.dh = g.dh; P.dw = g.dw;
    P.mode = dgrad ? 1 : 0;
    P.sw_cls = dgrad ? g.sw : 1;
    set_taps(g, dgrad, &P);
    // elements between consecutive rows of the filter matrix the kernel reads: [Cd][R][S][Cs]
    // (forward, and the transposed copy of the register-staged data gradient), or the filter as
    // stored, [K = Cs][R][S][C = Cd], for the data gradient of the split-role and patch kernels
    P.b_row_pitch = g.R * g.S * ((dgrad && p.variant >= 300) ? P.Cd : P.Cs);
    P.tiles_h = P.tiles_w = 0;
    if (p.variant >= 400) {
        const PatchVariant& pv = kPatchVariants[p.variant - 400];
        P.nclasses = 1;
        P.class_tile_start[0] = 0;
        P.tiles_h = (P.Hd + pv.th - 1) / pv.th;
        P.tiles_w = (P.Wd + pv.tw - 1) / pv.tw;
        P.tiles_n = (P.Cd + pv.bn - 1) / pv.bn;
        P.total_tiles = P.NB * P.tiles_h * P.tiles_w * P.tiles_n;
        P.class_tile_start[1] = P.total_tiles;
        return launch_conv_patch(p.variant - 400, P, st);
    }
    const IgemmVariant& v = igemm_variant(p.variant);
    int tiles_m = row_tiles(g, dgrad, v.bm, P.class_tile_start, &P.nclasses);
    P.tiles_n = (P.Cd + v.bn - 1) / v.bn;
    P.total_tiles = tiles_m * P.tiles_n;
    if (p.variant >= 300) return launch_igemm_ws(p.variant - 300, P, st);
    if (p.variant >= 100) return launch_igemm_dma(p.variant - 100, P, st);
    return launch_igemm(p.variant, P, P.total_tiles, st);
}

hipError_t run_fwd(const Geom& g, const Plan& p, const __half* x, const __half* w, __half* y, void* ws, hipStream_t st,
                   const Epilogue& ep)
{
    if (p.route == ROUTE_PADK) {
        // zero filters behind the real ones; the padded result goes to the workspace and its real
        // channels are copied out (with the tail, if any: it sees the rounded result there)
        const Geom gp = padded_k(g);
        unsigned char* base = static_cast<unsigned char*>(ws);
        __half* wp = reinterpret_cast<__half*>(base);
        __half* yp = reinterpret_cast<__half*>(base + padk_filter_bytes(gp));
        void* inner_ws = base + padk_filter_bytes(gp) + padk_act_bytes(gp);
        const long wn = (long)g.K * g.R * g.S * g.C, wpn = (long)gp.K * g.R * g.S * g.C;
        hipError_t e = launch_pad_rows(w, wp, wn, wpn, st);
        if (e != hipSuccess) return e;
        e = run_fwd(gp, plan_fwd(gp), x, wp, yp, inner_ws, st, no_epilogue());
        if (e != hipSuccess) return e;
        return launch_unpad_channels(yp, y, (long)g.N * g.Ho * g.Wo, g.K, gp.K, ep, st);
    }
    if (p.route == ROUTE_NARROW) return launch_narrow_fwd(g, x, w, y, st, ep);
    if (p.route == ROUTE_DIRECT) return launch_direct_fwd(g, x, w, y, st, ep);
    if (p.route == ROUTE_THIN) return launch_thin_fwd(g, x, w, y, ws, st, ep);
    return run_igemm(g, p, false, x, w, y, st, ep);
}

hipError_t run_dgrad(const Geom& g, const Plan& p, const __half* dy, const __half* w, __half* dx, void* ws, hipStream_t st,
                     const Epilogue& ep)
{
    if (p.route == ROUTE_PADK) {
        // zero gradient channels and zero filters behind the real ones; dx comes out in place
        const Geom gp = padded_k(g);
        unsigned char* base = static_cast<unsigned char*>(ws);
        __half* wp = reinterpret_cast<__half*>(base);
        __half* gpad = reinterpret_cast<__half*>(base + padk_filter_bytes(gp));
        void* inner_ws = base + padk_filter_bytes(gp) + padk_act_bytes(gp);
        const long wn = (long)g.K * g.R * g.S * g.C, wpn = (long)gp.K * g.R * g.S * g.C;
        hipError_t e = launch_pad_rows(w, wp, wn, wpn, st);
        if (e != hipSuccess) return e;
        e = launch_pad_channels(dy, gpad, (long)g.N * g.Ho * g.Wo, g.K, gp.K, st);
        if (e != hipSuccess) return e;
        return run_dgrad(gp, plan_dgrad(gp), gpad, wp, dx, inner_ws, st, ep);
    }
    if (p.route == ROUTE_NARROW) return launch_narrow_dgrad(g, dy, w, dx, st, ep);
    if (p.route == ROUTE_DIRECT) return launch_direct_dgrad(g, dy, w, dx, st, ep);
    if (p.route == ROUTE_THIN && p.variant == 1) return launch_thin_dgrad_mfma(g, dy, w, dx, ws, st, ep);
    if (p.route == ROUTE_IGEMM && p.variant >= 300) return run_igemm(g, p, true, dy, w, dx, st, ep);
    __half* wT = static_cast<__half*>(ws);
    hipError_t e = launch_filter_transpose(w, wT, g.K, g.R * g.S, g.C, st);
    if (e != hipSuccess) return e;
    if (p.route == ROUTE_THIN) return launch_thin_dgrad(g, dy, wT, dx, st, ep);
    return run_igemm(g, p, true, dy, wT, dx, st, ep);
}

hipError_t run_wgrad(const Geom& g, const Plan& p, const __half* x, const __half* dy, float* dw, void* ws, hipStream_t st)
{
    if (p.route == ROUTE_PADK) {
        // zero gradient channels behind the real ones; the first K filters of the padded result are dw
        const Geom gp = padded_k(g);
        unsigned char* base = static_cast<unsigned char*>(ws);
        __half* gpad = reinterpret_cast<__half*>(base);
        float* dwp = reinterpret_cast<float*>(base + padk_act_bytes(gp));
        void* inner_ws = base + padk_act_bytes(gp) + padk_dw_bytes(gp);
        hipError_t e = launch_pad_channels(dy, gpad, (long)g.N * g.Ho * g.Wo, g.K, gp.K, st);
        if (e != hipSuccess) return e;
        e = run_wgrad(gp, plan_wgrad_beside(gp, padk_act_bytes(gp) + padk_dw_bytes(gp)), x, gpad, dwp, inner_ws, st);
        if (e != hipSuccess) return e;
        return launch_copy_f32(dwp, dw, (long)g.K * g.R * g.S * g.C, st);
    }
    if (p.route == ROUTE_NARROW) {
        hipError_t e = launch_narrow_wgrad(g, x, dy, p.splits > 1 ? static_cast<float*>(ws) : dw, st);
        if (e != hipSuccess || p.splits == 1) return e;
        return launch_splitk_reduce(static_cast<const float*>(ws), dw, p.splits, (long)g.K * g.C, st);
    }
    if (p.route == ROUTE_DIRECT) return launch_direct_wgrad(g, x, dy, dw, st);
    if (p.route == ROUTE_THIN) return launch_thin_wgrad(g, x, dy, dw, ws, st);
    const WgradVariant& v = wgrad_variant(p.variant);
    WgradParams P;
    P.X = x; P.G = dy;
    P.N = g.N; P.H = g.H; P.W = g.W; P.C = g.C; P.K = g.K; P.R = g.R; P.S = g.S;
    P.sh = g.sh; P.sw = g.sw; P.ph = g.ph; P.pw = g.pw; P.dh = g.dh; P.dw = g.dw;
    P.Ho = g.Ho; P.Wo = g.Wo;
    P.P = g.N * g.Ho * g.Wo;
    P.splits = p.splits;
    P.steps_per_split = p.steps_per_split;
    P.tiles_k = (g.K + v.bm - 1) / v.bm;
    P.tiles_c = (g.C + v.bn - 1) / v.bn;
    P.out = (P.splits > 1) ? static_cast<float*>(ws) : dw;
    hipError_t e = p.variant >= 100 ? launch_wgrad_dma(p.variant - 100, P, st) : launch_wgrad(p.variant, P, st);
    if (e != hipSuccess || P.splits == 1) return e;
    return launch_splitk_reduce(static_cast<const float*>(ws), dw, P.splits, (long)g.K * g.R * g.S * g.C, st);
}

}  // namespace sdconv
