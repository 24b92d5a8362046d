"""Timings of the kernel variants on layers of random size, and the constants of the time models in
csrc/dispatch.hip and csrc/conv_f32.hip fitted to them.

    python -m paper_1903_05831_amd.fit_models measure --what rows|wgrad|f32|f32wgrad --seed 1 --seconds 100 --out t.jsonl.gz
    python -m paper_1903_05831_amd.fit_models fit --timings profiles/layer_timings.jsonl.gz --before profiles/layer_timings_before_runs.jsonl.gz

``measure`` needs the GPU: every variant (and, for the weight gradient, every sensible number of
pixel ranges) of each layer, as HIP graphs of many calls on tensors that do not fit the caches, the best
of three runs, variants in turn.  ``fit`` runs anywhere.  It prints the constants of kRowModels, kWgradModels, kF32Tiles and kF32WgradTiles and,
by threefold cross-validation over the layers, how much slower than the fastest measured variant the model's
choice is on layers that it was not fitted to.  Constants are bounded by what the hardware can do: a step
takes no less than the matrix instructions alone (2.06 PFLOP/s measured over 256 compute units),
nothing moves faster than 6.1 MB/us (HBM streaming as measured), and a forward or data-gradient kernel moves
its operands at 3.5 MB/us at least and starts in 0.5 us at least: most tiles of 128 rows and more sit at
those two, their layers being bound by the steps.

``--before``: timings of the same variants from before their fetching waves sent runs of loads.  kRowModels is the fit to
those, with two corrections from the present ones (row_models), which move constants past the bounds above; kF32Tiles
is the fit to those as it is.  Without it both are fits to the present timings, which choose slightly worse forward and
data-gradient kernels.
"""
from __future__ import annotations

import argparse
import gzip
import json
import math
import os
import random
import sys
import time

# ---- layers ------------------------------------------------------------------------------------

# (C, K, R, stride) of ResNet-50 bottleneck blocks, pyramid and box-head layers
DETECTOR_LAYERS = [
    (64, 64, 1, 1), (64, 64, 3, 1), (64, 256, 1, 1), (256, 64, 1, 1), (256, 128, 1, 1), (128, 128, 3, 2),
    (128, 512, 1, 1), (256, 512, 1, 2), (512, 128, 1, 1), (128, 128, 3, 1), (512, 256, 1, 1), (256, 256, 3, 2),
    (256, 1024, 1, 1), (512, 1024, 1, 2), (1024, 256, 1, 1), (256, 256, 3, 1), (1024, 512, 1, 1), (512, 512, 3, 2),
    (512, 2048, 1, 1), (1024, 2048, 1, 2), (2048, 512, 1, 1), (512, 512, 3, 1), (256, 256, 1, 1), (1024, 512, 3, 1),
    (12544, 1024, 1, 1), (1024, 1024, 1, 1)]


def random_layers(seed: int, count: int, few_pixels: bool = False):
    """Geometries (N, H, W, C, K, R, stride, pad, dilation): half of them with the channels of a
    detector's layer on maps of random size and number, half with any channels (in eights).  Or layers of 12 to 700 pixels, with
    any channels and filters of up to 7x7: a weight gradient of few steps."""
    rng = random.Random(seed)
    out = []
    while few_pixels and len(out) < count:
        C, K = (8 * int(math.exp(rng.uniform(0, math.log(256)))) for _ in range(2))
        R, stride, N = rng.choice([1, 1, 3, 3, 5, 7]), rng.choice([1, 1, 2]), rng.choice([1, 1, 2, 4])
        px = int(math.exp(rng.uniform(math.log(12), math.log(700))))
        H = max(3, int((px / N) ** 0.5 * rng.uniform(0.6, 1.0)))
        if C * K * R * R <= 1 << 26:
            out.append((N, H * stride, max(3, px // (N * H)) * stride, C, K, R, stride, R // 2, 1))
    while len(out) < count:
        if rng.random() < 0.5:
            C, K, R, stride = rng.choice(DETECTOR_LAYERS)
        else:
            C, K = (8 * int(math.exp(rng.uniform(0, math.log(256)))) for _ in range(2))
            R, stride = rng.choice([1, 1, 3]), rng.choice([1, 1, 2])
        px = int(math.exp(rng.uniform(math.log(200), math.log(150_000))))
        H = max(3, int(px ** 0.5 * rng.uniform(0.6, 1.0)))
        N, H, W = 1, H, max(3, px // H)
        if rng.random() < 0.2:                              # regions of interest
            H = W = rng.choice([7, 14])
            N = max(1, px // (H * W))
        if max(C, K) * px <= 1.2e8 and C * K * R * R * px <= 3e11:
            out.append((N, H, W, C, K, R, stride, R // 2, 1))
    return out


def out_hw(k):
    N, H, W, C, K, R, s, pad, dil = k
    return tuple((n + 2 * pad - dil * (R - 1) - 1) // s + 1 for n in (H, W))


# ---- measurement -------------------------------------------------------------------------------

ROW_VARIANTS = [101, 112, 310, 311, 316, 324] + list(range(325, 341)) + [427, 433, 435, 436, 437]
# variants with a row in the models (324 has those of its two halves)
ROW_MODELS = [v for v in ROW_VARIANTS if v != 324]
WGRAD_MODELS = WGRAD_VARIANTS = [104, 107, 108, 112, 114, 115, 116, 117, 118, 119, 120, 121, 122, 123]
# kernels that the runs of loads do not reach and whose constants for gathering layers stay (row_models)
UNSCALED = (112, 433, 435, 436, 437)
ONE_SLAB = {427, 433}                    # one patch buffer: 64 contraction channels only
WORKGROUPS = (40, 64, 96, 128, 192, 256, 320, 384, 512, 768, 1024)


def measure(what: str, seed: int, seconds: float, path: str, few_pixels: bool = False) -> None:
    os.environ["SDCONV_TUNE"] = "1"             # before the first library call
    os.environ["SDCONV_NO_TUNED_TABLE"] = "1"      # nor the entries of four weight gradients
    import torch
    import paper_1903_05831_amd as sd

    pool = 3 << 30
    src = torch.empty(pool // 2, dtype=torch.float16, device="cuda")
    for i in range(0, src.numel(), 1 << 26):
        src[i:i + (1 << 26)].normal_(0, 0.5)
    dst, wsp = torch.empty_like(src), torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()
    f32 = what.startswith("f32")
    calls = ((sd.conv2d_fwd_f32, sd.conv2d_dgrad_f32, sd.conv2d_wgrad_f32) if f32 else
             (sd.conv2d_fwd, sd.conv2d_dgrad, sd.conv2d_wgrad))
    need_bytes = sd.conv2d_workspace_bytes_f32 if f32 else sd.conv2d_workspace_bytes

    def graph(d, p, nbytes, us):
        na, nb, no = (-(-n // 256) * 256 for n in nbytes)
        copies = max(1, min(pool // (na + nb), pool // no, -(-(700 << 20) // (na + nb + no)), 48))
        count = max(6, min(60, int(400 / us)))
        need = need_bytes(d, p)
        assert need <= wsp.numel()
        ws = wsp[:max(need, 256)]

        def one(i):
            a = src.data_ptr() + i % copies * (na + nb)
            calls[p](d, a, a + na, dst.data_ptr() + i % copies * no, ws, stream.cuda_stream)
        with torch.cuda.stream(stream):
            one(0)
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            for i in range(count):
                one(i)
        return g, count

    def best_times(graphs):
        best = [1e30] * len(graphs)
        ev = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in graphs]
        with torch.cuda.stream(stream):
            for _ in range(4):
                for (g, _), (a, b) in zip(graphs, ev):
                    a.record()
                    g.replay()
                    b.record()
                stream.synchronize()
                best = [min(t, a.elapsed_time(b) * 1e3 / n) for t, (_, n), (a, b) in zip(best, graphs, ev)]
        return best

    def force(**env):
        for name in ("SDCONV_IGEMM_VARIANT", "SDCONV_WGRAD_VARIANT", "SDCONV_WGRAD_SPLITS", "SDCONV_F32_TILE"):
            os.environ.pop(name, None)
        os.environ.update({k: str(v) for k, v in env.items()})

    start, done = time.time(), 0
    with gzip.open(path, "wt") as out:
        for k in random_layers(seed, 2000, few_pixels):
            if time.time() - start > seconds:
                break
            N, H, W, C, K, R, s, pad, dil = k
            d = sd.make_desc(N, H, W, C, K, R, R, (s, s), (pad, pad), (dil, dil))
            ho, wo = out_hw(k)
            e = 4 if f32 else 2
            x, w, y, dw = e * N * H * W * C, e * K * R * R * C, e * N * ho * wo * K, 4 * K * R * R * C
            us = max(5.0, 2e6 * N * ho * wo * K * R * R * C / (80e12 if f32 else 0.6e15), (x + w + y) / 3.5e6)
            for p in ((2,) if what.endswith("wgrad") else (0, 1)):
                nbytes = ((x, w, y), (y, w, x), (x, y, dw))[p]
                graphs, labels = [], []
                if what == "rows":
                    for v in ROW_VARIANTS:
                        if p == 1 and v < 300:
                            continue
                        force(SDCONV_IGEMM_VARIANT=v)
                        if v >= 400 and ("patch" not in sd.kernel_name(d, p) or
                                         v in ONE_SLAB and (K if p else C) != 64):
                            continue
                        graphs.append(graph(d, p, nbytes, us))
                        labels.append(v)
                elif what == "f32wgrad":
                    total = -(-N * ho * wo // 32)
                    for v, (bm, bn, _) in enumerate(F32_WGRAD_TILES):
                        tiles = -(-K // bm) * -(-C // bn) * R * R
                        for ranges in sorted({ranges_made(total, r) for r in [1, 2] + [n // tiles for n in WORKGROUPS[3:]]}):
                            if ranges * dw <= 256 << 20:
                                force(SDCONV_F32_TILE=100 + v, SDCONV_WGRAD_SPLITS=ranges)
                                graphs.append(graph(d, p, nbytes, us))
                                labels.append((v, ranges))
                elif f32:
                    for v in range(len(F32_TILES)):
                        force(SDCONV_F32_TILE=v)
                        graphs.append(graph(d, p, nbytes, us))
                        labels.append(v)
                else:
                    total = -(-N * ho * wo // 64)
                    for v in WGRAD_VARIANTS:
                        bm, bn, _ = WGRAD_TILES[v]
                        tiles = -(-K // bm) * -(-C // bn) * R * R
                        for ranges in sorted({ranges_made(total, r) for r in
                                              [1, 2, 3] + [n // tiles for n in WORKGROUPS]}):
                            if ranges * dw <= 256 << 20:
                                force(SDCONV_WGRAD_VARIANT=v, SDCONV_WGRAD_SPLITS=ranges)
                                graphs.append(graph(d, p, nbytes, us))
                                labels.append((v, ranges))
                best = best_times(graphs)
                out.write(json.dumps({"what": what, "k": k, "p": p,
                                      "us": [(v, round(t, 2)) for v, t in zip(labels, best)]}) + "\n")
                del graphs
            done += 1
            if done % 20 == 0:
                print(what, done, "layers", round(time.time() - start), "s", flush=True)
    print("wrote", path, done, "layers", flush=True)


# ---- the models, as in csrc/dispatch.hip -----------------------------------------------------------

F32_MATRIX = 157.3e6                # flop/us, the fp32 matrix peak
MATRIX, STREAM = 2.06e9, 6.1        # flop/us over the chip with matrix instructions alone; MB/us
TILES = {101: (128, 128), 112: (128, 64), 310: (224, 256), 311: (256, 256), 316: (224, 128),
         325: (144, 64), 326: (144, 256), 327: (64, 64), 328: (64, 64), 329: (64, 128), 330: (128, 128), 331: (256, 128),
         332: (224, 128), 333: (96, 128), 334: (80, 128), 335: (160, 128), 336: (192, 128), 337: (96, 64), 338: (160, 256),
         339: (128, 128), 340: (128, 64)}
PATCHES = {427: (8, 16, 64), 433: (10, 14, 64), 435: (10, 14, 64), 436: (8, 16, 64), 437: (8, 8, 64)}
PER_CU = {101: 3, 112: 5, 327: 2, 328: 2, 339: 2, 340: 3, 427: 2, 433: 2}
WGRAD_TILES = {100: (128, 128, 2), 104: (64, 128, 2), 107: (64, 64, 3), 108: (128, 64, 2), 109: (256, 256, 1),
               112: (128, 128, 1), 113: (256, 128, 1), 114: (256, 256, 1), 115: (256, 256, 1), 116: (128, 128, 1),
               117: (256, 128, 1), 118: (64, 64, 3), 119: (128, 128, 2), 120: (128, 128, 1), 121: (64, 64, 3), 122: (128, 64, 2), 123: (256, 128, 1)}
FILTER_COPY = 3.2                   # us: the data gradient of the variants below 300 transposes the filter first
EMPTY_TILE = 0.6                    # of `tile`: a tile of a parity class without taps only stores zeros
REDUCE_FIXED, REDUCE_RATE = 2.5, 6.0
POINTWISE, GATHER, STRIDED = range(3)


def kind(k, p):
    if k[5] == 1 and k[6] == 1 and k[7] == 0:
        return POINTWISE
    return STRIDED if p == 1 and k[6] > 1 else GATHER


def tile_classes(k, p, v):
    """[(tiles, 64-channel steps of each)] of the pass, in the order of their launch ("f32": taps of each)."""
    N, H, W, C, K, R, s, pad, dil = k
    cs, cd = (K, C) if p else (C, K)
    hd, wd = (H, W) if p else out_hw(k)
    bk = 32 if v == "f32" or v < 300 else 64
    slabs = 1 if v == "f32" else -(-cs // bk) * bk / 64
    if v in PATCHES:
        th, tw, bn = PATCHES[v]
        return [(N * -(-hd // th) * -(-wd // tw) * -(-cd // bn), R * R * slabs)]
    bm, bn = TILES[v]
    columns = -(-cd // bn)
    if p == 0 or s == 1:
        return [(-(-N * hd * wd // bm) * columns, R * R * slabs)]
    out = []
    for q in range(s * s):
        a, b = divmod(q, s)
        taps = [sum((o + pad - r * dil) % s == 0 for r in range(R)) for o in (a, b)]
        rows = N * max(0, (H - a + s - 1) // s) * max(0, (W - b + s - 1) // s)
        out.append((-(-rows // bm) * columns, taps[0] * taps[1] * slabs))
    return out


def makespan(classes, slots):
    """Tiles taken in order by whichever of the slots is free first: [(tiles, us each)] -> us."""
    free = [[0.0, slots]]                       # (time, slots free from then on), sorted
    for m, d in classes:
        if m > 4 * slots:                       # whole rounds move every slot alike
            rounds = m // slots - 2
            free = [[t + rounds * d, n] for t, n in free]
            m -= rounds * slots
        while m > 0:
            t, n = free.pop(0)
            q = min(n, m)
            m -= q
            if n > q:
                free.insert(0, [t, n - q])
            i = len(free)
            while i and free[i - 1][0] > t + d:
                i -= 1
            if i and free[i - 1][0] == t + d:
                free[i - 1][1] += q
            else:
                free.insert(i, [t + d, q])
    return free[-1][0]


def compute_us(classes, per_cu, c):
    fixed, step, shared, tile, hbm = c
    if len(classes) > 1:
        crowd = min(per_cu, -(-sum(m for m, _ in classes) // 256))
        return makespan([(m, s * max(step, crowd * shared) + (tile if s else EMPTY_TILE * tile))
                         for m, s in classes], 256 * per_cu)
    n, steps = classes[0]
    fullest = -(-n // 256)
    full, rest = divmod(fullest, per_cu)
    t = full * (steps * max(step, per_cu * shared) + tile)
    return t + (steps * max(step, rest * shared) + tile if rest else 0.0)


def megabytes(k, p):
    N, H, W, C, K, R, s, pad, dil = k
    ho, wo = out_hw(k)
    return 2e-6 * (N * H * W * C / (s * s if R == 1 and p == 0 else 1) + N * ho * wo * K + K * R * R * C)


def both(a, b):
    """Two resources at work together: near the larger, more where they are alike."""
    return math.hypot(a, b)


def row_us(models, k, p, v):
    if p == 1 and v < 300:
        return None                 # these want a filter copy in the workspace: measured layers only
    c = models.get((310 if v == 324 else v, kind(k, p)))
    if c is None or v == 324 and kind(k, p) == STRIDED:
        return None
    if v == 324:        # whole rounds of 224x256 tiles, the rest as 224x128 ones
        half = models[316, kind(k, p)]
        (n, steps), = tile_classes(k, p, 310)
        columns = -(-(k[3] if p else k[4]) // 256)
        rows = n // columns
        wide = rows if 2 * (n % 256) > 256 + columns else n // 256 * 256 // columns
        narrow = (rows - wide) * -(-(k[3] if p else k[4]) // 128)
        work = sum(compute_us([(m, steps)], 1, q) for m, q in ((wide * columns, c), (narrow, half)) if m)
    else:
        work = compute_us(tile_classes(k, p, v), PER_CU.get(v, 1), c)
    return c[0] + both(work, megabytes(k, p) / c[4])


def ranges_made(total_steps, ranges):
    ranges = max(1, min(ranges, total_steps // 2))
    return -(-total_steps // -(-total_steps // ranges))


def wgrad_us(models, k, v, ranges):
    N, H, W, C, K, R, s, pad, dil = k
    fixed, step, shared, tile, store, hbm = models[v, min(kind(k, 2), GATHER)]
    bm, bn, per_cu = WGRAD_TILES[v]
    ho, wo = out_hw(k)
    steps = -(-(-(-N * ho * wo // 64)) // ranges)
    fullest = -(-(-(-K // bm) * -(-C // bn) * R * R * ranges) // 256)
    full, rest = divmod(fullest, per_cu)
    work = full * (steps * max(step, per_cu * shared) + tile) + (steps * max(step, rest * shared) + tile if rest else 0)
    dw = 4e-6 * K * R * R * C
    x = 2e-6 * N * H * W * C / (s * s if R == 1 else 1) + 2e-6 * N * ho * wo * K
    t = fixed + both(work, x / hbm) + ranges * dw / store
    return t + (ranges * dw / REDUCE_RATE + REDUCE_FIXED if ranges > 1 else 0.0)


# split-role kernels, then register-staged ones; with a unit's workgroups
F32_TILES = [(128, 128, 1), (128, 64, 2), (64, 64, 3), (64, 32, 4), (32, 32, 6),
             (128, 128, 2), (128, 64, 3), (96, 64, 3), (64, 64, 4), (32, 64, 6), (32, 32, 5)]
F32_WGRAD_TILES = [(128, 128, 2), (128, 64, 2), (64, 128, 2), (64, 64, 3)]


def f32_us(models, k, p, tile):
    step, shared, per_tile, fixed = models[tile]
    bm, bn, per_cu = F32_TILES[tile]
    TILES["f32"] = bm, bn
    chunks = -(-(k[4] if p else k[3]) // 32)        # 32 contraction floats a step
    classes = tile_classes(k, p, "f32")
    busy = [(n, steps) for n, steps in classes if steps]
    tiles = sum(n for n, _ in busy)
    if not tiles:
        return fixed
    total, longest = sum(n * taps for n, taps in busy) * chunks, max(taps for _, taps in busy) * chunks
    if len(classes) > 1:        # parity classes: tiles of different length fill the units evenly but for the last ones
        empty = sum(n for n, steps in classes if not steps)
        even = (total * shared + (tiles + EMPTY_TILE * empty) * per_tile / per_cu) / 256
        last = longest * step + per_tile
        return fixed + max(even + 0.5 * last, last)
    steps = total / tiles
    full, rest = divmod(-(-tiles // 256), per_cu)
    t = full * (steps * max(step, per_cu * shared) + per_tile)
    return fixed + t + (steps * max(step, rest * shared) + per_tile if rest else 0.0)


def f32_wgrad_us(models, k, v, ranges):
    N, H, W, C, K, R, s, pad, dil = k
    step, shared, per_tile, fixed, store = models[v]
    bm, bn, per_cu = F32_WGRAD_TILES[v]
    ho, wo = out_hw(k)
    tiles = -(-K // bm) * -(-C // bn) * R * R
    steps = -(-(-(-N * ho * wo // 32)) // ranges)
    full, rest = divmod(-(-tiles * ranges // 256), per_cu)
    t = full * (steps * max(step, per_cu * shared) + per_tile) + (steps * max(step, rest * shared) + per_tile if rest else 0.0)
    dw = 4e-6 * K * R * R * C
    return fixed + t + ranges * dw / store + (ranges * dw / REDUCE_RATE + REDUCE_FIXED if ranges > 1 else 0.0)


# ---- the fits --------------------------------------------------------------------------------------

def least_squares_log(predict, samples, lo, hi, start):
    import numpy as np
    from scipy.optimize import least_squares
    lo, hi = np.array(lo), np.array(hi)
    free = hi > lo

    def residuals(th):
        full = lo.copy()
        full[free] = th
        return [math.log(predict(full, s) / s[-1]) for s in samples]
    r = least_squares(residuals, np.clip(np.array(start), lo, hi)[free], bounds=(lo[free], hi[free]),
                      diff_step=1e-4, max_nfev=40)
    out = lo.copy()
    out[free] = r.x
    return tuple(float(t) for t in out)


def fit_rows(rows, variants=ROW_MODELS, kinds=(POINTWISE, GATHER, STRIDED)):
    models = {}
    for v in variants:
        area = TILES[v][0] * TILES[v][1] if v < 400 else math.prod(PATCHES[v])
        least = 2.0 * area * 64 * 256 / MATRIX
        per_cu = PER_CU.get(v, 1)
        for c in kinds:
            if v >= 400 and c != GATHER or v < 300 and c == STRIDED:
                continue
            samples = [(tuple(x["k"]), x["p"], dict(x["us"])[v]) for x in rows
                       if v in dict(x["us"]) and kind(x["k"], x["p"]) == c]
            samples = [(tile_classes(k, p, v), megabytes(k, p), FILTER_COPY if p == 1 and v < 300 else 0.0, us)
                       for k, p, us in samples]

            def predict(th, s):
                return th[0] + s[2] + both(compute_us(s[0], per_cu, th), s[1] / th[4])
            lo = [0.5, least, least if per_cu > 1 else 0.0, 0.0, 3.5]
            hi = [10.0, 6 * least, 6 * least if per_cu > 1 else 0.0, 20.0, STREAM]
            if c == STRIDED:        # a step is the same work as in any gathering layer
                lo[1:3] = hi[1:3] = models[v, GATHER][1:3]
            th = least_squares_log(predict, samples, lo, hi, [2.0, 1.5 * least, 1.2 * least, 3.0, 4.0])
            # A step below `shared` never counts, and what the solver makes of it, and of the others on its way there, depends on
            # the processor: fitted on without it.
            if th[1] < th[2] and c != STRIDED:
                lo[1] = hi[1] = 0.0
                th = least_squares_log(predict, samples, lo, hi, th)
                th = (th[0], th[2], *th[2:])
            models[v, c] = th
    return models


def rescaled(models, rows, c, near=1.2):
    """The constants of layers of kind `c` times the median of measured over predicted time (`hbm` by its inverse), over the
    passes in which the variant is within 20 % of the fastest."""
    out = dict(models)
    for v in ROW_MODELS:
        if (v, c) not in models or v in UNSCALED:
            continue
        ratios = sorted(dict(x["us"])[v] / row_us(models, x["k"], x["p"], v) for x in rows
                        if kind(x["k"], x["p"]) == c and v in dict(x["us"]) and (x["p"] == 0 or v >= 300)
                        and dict(x["us"])[v] < near * min(t for _, t in x["us"]))
        if len(ratios) >= 20:
            q, th = ratios[len(ratios) // 2], models[v, c]
            out[v, c] = (*(t * q for t in th[:4]), th[4] / q)
    return out


def fit_before(rows):
    """The fit to timings from before the runs, with the digits that the table had."""
    return {k: tuple(round(t, 3) for t in c) for k, c in fit_rows(rows).items()}


def row_models(before, rows):
    """kRowModels: the fit to `before`; gathering layers rescaled to `rows`; the two 64x64 tiles that differ in their matrix block
    only (327, 328) fitted to `rows` for pointwise layers, of which the long ones took the slower tile.  Strided data
    gradients stay: rescaled they choose 0.1 to 0.5 % slower kernels.  So do kernels without runs of loads, for which a ratio taken near
    the fastest is below one by the choice of layers alone: rescaled, the 128x64 tile (112) took strided 1x1 layers with one channel chunk
    from the 128x128 one (54 -> 86 us), and the patch blocks a few per cent of 3x3 layers at 4 to 8 % more.  (101 and 427 choose as well or
    better rescaled: 0.97 and 1.00.)"""
    return {**rescaled(before, rows, GATHER), **fit_rows(rows, (327, 328), (POINTWISE,))}


def fit_wgrad(rows):
    models = {}
    for v in WGRAD_MODELS:
        bm, bn, per_cu = WGRAD_TILES[v]
        least = 2.0 * bm * bn * 64 * 256 / MATRIX
        for c in (POINTWISE, GATHER):
            samples = [(tuple(x["k"]), r, us) for x in rows for (vv, r), us in x["us"]
                       if vv == v and min(kind(x["k"], 2), GATHER) == c]
            models[v, c] = least_squares_log(
                lambda th, s: wgrad_us({(v, c): th}, s[0], v, s[1]), samples,
                [1.0, least, least if per_cu > 1 else 0.0, 0.0, 1.0, 1.5],
                [15.0, 10 * least, 10 * least if per_cu > 1 else 0.0, 15.0, STREAM, STREAM],
                [4.0, 2 * least, 1.5 * least, 2.0, 4.0, 4.5])
    return models


def fit_f32(rows):
    models = {}
    for i, (bm, bn, per_cu) in enumerate(F32_TILES):
        least = 2.0 * bm * bn * 32 * 256 / F32_MATRIX
        samples = [(tuple(x["k"]), x["p"], dict(x["us"])[i]) for x in rows]
        models[i] = least_squares_log(lambda th, s: f32_us({i: th}, s[0], s[1], i), samples,
                                      [least, least, 0.0, 0.5], [6 * least, 6 * least, 10.0, 10.0],
                                      [1.3 * least, 1.2 * least, 2.0, 2.0])
    return models


def fit_f32_wgrad(rows):
    models = {}
    for i, (bm, bn, per_cu) in enumerate(F32_WGRAD_TILES):
        least = 2.0 * bm * bn * 32 * 256 / F32_MATRIX
        samples = [(tuple(x["k"]), r, t) for x in rows for (v, r), t in x["us"] if v == i]
        models[i] = least_squares_log(lambda th, s: f32_wgrad_us({i: th}, s[0], i, s[1]), samples,
                                      [least, least, 0.0, 0.5, 1.0], [6 * least, 6 * least, 10.0, 10.0, STREAM],
                                      [1.3 * least, 1.2 * least, 2.0, 2.0, 4.0])
    return models


def f32_wgrad_choice(models, x):
    return min((f32_wgrad_us(models, x["k"], v, r), (v, r)) for (v, r), _ in x["us"])[1]


def f32_choice(models, x):
    return min(range(len(F32_TILES)), key=lambda i: f32_us(models, x["k"], x["p"], i))


def row_choice(models, x):
    times = dict(x["us"])
    return min((t, v) for v in times if (t := row_us(models, x["k"], x["p"], v)) is not None)[1]


def wgrad_choice(models, x):
    return min((wgrad_us(models, x["k"], v, r), (v, r)) for (v, r), _ in x["us"] if v in WGRAD_MODELS)[1]


def held_out(rows, fit, choice, folds=3):
    """Slow-down of the choice against the fastest measured variant, each layer under a model that was
    fitted without it."""
    rng = random.Random(0)
    fold = {k: rng.randrange(folds) for k in sorted({tuple(x["k"]) for x in rows})}
    loss = []
    for f in range(folds):
        models = fit([x for x in rows if fold[tuple(x["k"])] != f])
        for x in rows:
            if fold[tuple(x["k"])] == f:
                times = dict(x["us"])
                loss.append((times[choice(models, x)] / min(times.values()), x["k"], x["p"]))
    return sorted(loss)


def report(name, loss):
    q = [t for t, _, _ in loss]
    print(f"// {name}: {len({tuple(k) for _, k, _ in loss})} layers, choice on layers left out of the fit "
          f"{100 * (math.exp(sum(map(math.log, q)) / len(q)) - 1):.2f} % slower than the fastest variant "
          f"(90th percentile {100 * (q[int(0.9 * len(q))] - 1):.1f} %, 99th {100 * (q[int(0.99 * len(q))] - 1):.1f} %)")


def load(paths):
    rows = []
    for path in paths:
        with gzip.open(path, "rt") as f:
            for line in f:
                x = json.loads(line)
                x["k"] = tuple(x["k"])
                x["us"] = [(tuple(v) if isinstance(v, list) else v, t) for v, t in x["us"]]
                rows.append(x)
    return rows


def fit(paths, before_paths, cross_validate):
    def parts(paths):
        rows = load(paths)
        return {what: [x for x in rows if x["what"] == what] for what in ("rows", "wgrad", "f32", "f32wgrad")}
    now, fit_all = parts(paths), fit_rows
    f32 = now["f32"]
    if before_paths:
        old = parts(before_paths)
        before, f32 = fit_before(old["rows"]), old["f32"]
        fit_all = lambda rows: row_models(before, rows)
    if cross_validate:
        report("rows", held_out(now["rows"], fit_all, row_choice))
        report("wgrad", held_out(now["wgrad"], fit_wgrad, wgrad_choice))
        report("f32", held_out(f32, fit_f32, f32_choice))
        report("f32wgrad", held_out(now["f32wgrad"], fit_f32_wgrad, f32_wgrad_choice))

    def cost(c):
        return "{}" if c is None else "{" + ", ".join(f"{t:.3f}f" for t in c) + "}"
    models = fit_all(now["rows"])
    for v in ROW_MODELS:
        print(f"    {{{v}, {PER_CU.get(v, 1)}, " + ", ".join(cost(models.get((v, c))) for c in range(3)) + "},")
    models = fit_wgrad(now["wgrad"])
    for v in WGRAD_MODELS:
        print(f"    {{{v}, {WGRAD_TILES[v][2]}, " + ", ".join(cost(models[v, c]) for c in range(2)) + "},")
    models = fit_f32(f32)
    for i, (bm, bn, per_cu) in enumerate(F32_TILES):
        print(f"    {{{bm}, {bn}, {per_cu}, {cost(models[i])[1:-1]}, ...}},")
    models = fit_f32_wgrad(now["f32wgrad"])
    for i, (bm, bn, per_cu) in enumerate(F32_WGRAD_TILES):
        print(f"    {{{bm}, {bn}, {per_cu}, {cost(models[i])[1:-1]}}},")


def main() -> int:
    ap = argparse.ArgumentParser()
    sub = ap.add_subparsers(dest="command", required=True)
    m = sub.add_parser("measure")
    m.add_argument("--what", choices=("rows", "wgrad", "f32", "f32wgrad"), required=True)
    m.add_argument("--seed", type=int, default=1)
    m.add_argument("--seconds", type=float, default=100)
    m.add_argument("--out", required=True)
    m.add_argument("--few-pixels", action="store_true", help="layers of 12 to 700 pixels")
    f = sub.add_parser("fit")
    f.add_argument("--timings", nargs="+", required=True)
    f.add_argument("--before", nargs="+", default=[])
    f.add_argument("--no-cross-validation", action="store_true")
    args = ap.parse_args()
    if args.command == "measure":
        measure(args.what, args.seed, args.seconds, args.out, args.few_pixels)
    else:
        fit(args.timings, args.before, not args.no_cross_validation)
    return 0


if __name__ == "__main__":
    sys.exit(main())
