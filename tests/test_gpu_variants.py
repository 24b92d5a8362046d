"""GPU parity of every tile variant of the pipelined kernels, forced one by one through the
dispatcher's environment hooks (read per call), against the fp64 CPU oracle on full tensors.
The shapes give ragged row / spatial tiles, several images, filter-count tails and more than
one 64-channel slab, so every variant sees partial tiles on each axis."""
import os

import numpy as np
import pytest
import torch

import paper_1903_05831_amd as sd

from gpu_harness import check_all_passes, check_fused, say

pytestmark = pytest.mark.gpu


def _rand_case(N, H, W, C, K, R, S, stride, pad, dil, seed):
    d = sd.make_desc(N, H, W, C, K, R, S, stride, pad, dil)
    ho, wo = sd.conv2d_out_shape(d)
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((N, H, W, C), dtype=np.float32).astype(np.float16)
    w = (rng.standard_normal((K, R, S, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (R * S * C)))).astype(np.float16)
    g = rng.standard_normal((N, ho, wo, K), dtype=np.float32).astype(np.float16)
    return d, x, w, g


class forced:
    def __init__(self, **env):
        self.env = {k: str(v) for k, v in env.items()}

    def __enter__(self):
        self.old = {k: os.environ.get(k) for k in self.env}
        os.environ.update(self.env)

    def __exit__(self, *exc):
        for k, v in self.old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v


# stride-1 layers the patch kernels accept (taps span two extra rows and columns, contraction
# channels in whole 64-channel slabs on both the forward and the data-gradient side)
PATCH_SHAPES = [
    # N  H   W   C    K   R  S  stride  pad     dil
    (2, 21, 37, 64, 64, 3, 3, (1, 1), (1, 1), (1, 1)),      # ragged tiles both ways, two images
    (1, 19, 18, 128, 192, 3, 3, (1, 1), (1, 1), (1, 1)),    # two slabs, filter tail (192 = 128 + 64)
    (1, 17, 33, 64, 128, 3, 3, (1, 1), (0, 0), (1, 1)),     # no padding: output smaller than input
    (1, 12, 20, 64, 64, 3, 3, (1, 1), (2, 2), (1, 1)),      # padding 2: output larger than input
    (1, 9, 40, 64, 64, 3, 2, (1, 1), (1, 1), (1, 2)),       # 3x2 taps, dilation 1x2
]
# they take three taps per pipeline step: R*S must be a multiple of 3 and give at least
# (ring stages - 1) steps per channel slab; variant -> ring stages
THREE_TAP_STEP = {427: 2, 433: 2, 435: 4, 436: 3, 437: 3}
PATCH_VARIANTS = list(THREE_TAP_STEP)
# these have a single patch buffer: one 64-channel slab on the contraction side of both passes
ONE_SLAB = {427, 433}


@pytest.mark.parametrize("variant", PATCH_VARIANTS)
def test_patch_kernel_variants(variant):
    for case in PATCH_SHAPES:
        taps = case[5] * case[6]
        if taps % 3 or taps // 3 < THREE_TAP_STEP[variant] - 1:
            continue        # the dispatcher (rightly) does not hand such a layer to this variant
        if variant in ONE_SLAB and (case[3] != 64 or case[4] != 64):
            continue
        say(f"patch variant {variant} case {case}")
        d, x, w, g = _rand_case(*case, seed=variant * 31 + len(case))
        with forced(SDCONV_IGEMM_VARIANT=variant, SDCONV_NO_TUNED_TABLE=1):
            assert "patch" in sd.kernel_name(d, sd.FWD), "shape must reach the patch kernel"
            assert "patch" in sd.kernel_name(d, sd.DGRAD)
            check_all_passes(d, x, w, g, f"patch{variant}{case}")


WS_SHAPES = [
    (2, 23, 29, 64, 72, 3, 3, (2, 2), (1, 1), (1, 1)),      # strided: parity classes in the data gradient
    (1, 31, 37, 136, 200, 3, 3, (1, 1), (1, 1), (1, 1)),    # short last channel slab, filter tail
    (1, 31, 37, 128, 264, 1, 1, (1, 1), (0, 0), (1, 1)),    # 1x1, more than one 256-wide column tile
    (2, 23, 29, 72, 64, 1, 1, (2, 2), (0, 0), (1, 1)),      # 1x1 stride 2, odd image: three parity classes of the data gradient are all zeros
    (1, 21, 27, 64, 64, 1, 3, (2, 2), (0, 1), (1, 1)),      # 1x3 stride 2: the odd-row classes have no taps, both even-row classes do
]
WS_VARIANTS = [310, 311, 316] + list(range(324, 341))


@pytest.mark.parametrize("variant", WS_VARIANTS)
def test_split_role_kernel_variants(variant):
    for case in WS_SHAPES:
        say(f"ws variant {variant} case {case}")
        d, x, w, g = _rand_case(*case, seed=variant * 17 + 3)
        with forced(SDCONV_IGEMM_VARIANT=variant, SDCONV_NO_TUNED_TABLE=1):
            assert "_ws_" in sd.kernel_name(d, sd.FWD)
            check_all_passes(d, x, w, g, f"ws{variant}{case}")


# How the split-role kernels count through the taps that meet a parity class: more than 32 taps (with a
# short last channel slab, and in classes of 9 to 16 taps), strides and dilations with and without a common
# factor (classes with no taps along one axis, or with every other one), a 1x1 filter that is
# padded or has a short slab.  Tiles without waves that only fetch (310), with such waves that divide the activation
# and the filter loads of a stage evenly (327, 337, 340), and with four of them for the 18 or 10 activation loads of 144 and 80
# rows, where the last waves have loads that fetch nothing (325, 326, 334).
TAP_GRIDS = [
    (1, 17, 19, 72, 64, 7, 7, (1, 1), (3, 3), (1, 1)),
    (1, 17, 19, 64, 72, 7, 7, (2, 2), (3, 3), (1, 1)),
    (1, 20, 23, 64, 64, 3, 3, (2, 2), (2, 2), (2, 2)),
    (1, 20, 23, 64, 64, 3, 5, (3, 2), (1, 2), (2, 3)),
    (1, 20, 23, 64, 64, 4, 3, (4, 4), (1, 0), (6, 2)),
    (2, 9, 11, 72, 64, 1, 1, (1, 1), (1, 1), (1, 1)),
    (2, 9, 11, 72, 136, 1, 1, (1, 1), (0, 0), (1, 1)),
]


@pytest.mark.parametrize("variant", [310, 325, 326, 327, 334, 337, 340])
def test_tap_grids_of_split_role_kernels(variant):
    for case in TAP_GRIDS:
        say(f"tap grid variant {variant} case {case}")
        d, x, w, g = _rand_case(*case, seed=variant * 23 + case[5])
        with forced(SDCONV_IGEMM_VARIANT=variant, SDCONV_NO_TUNED_TABLE=1):
            assert "_ws_" in sd.kernel_name(d, sd.FWD) and "_ws_" in sd.kernel_name(d, sd.DGRAD)
            check_all_passes(d, x, w, g, f"taps{variant}{case}")
            check_fused(d, x, w, g, f"taps_fused{variant}{case}")


@pytest.mark.parametrize("dgrad", [False, True])
@pytest.mark.parametrize("variant,R,short,whole", [(v, 3, 72, 128) for v in (310, 311, 316, 338)] + [(v, 7, 40, 64) for v in (328, 334, 337)])
def test_a_short_last_channel_chunk_takes_no_longer_than_a_whole_one(variant, R, short, whole, dgrad):
    """Tiles whose multiplying waves fetch too, and more than 32 taps on tiles with waves that only fetch: as many chunks, the short one
    with less to move: 0.99 to 1.02 and 0.96 to 1.10 times the time, 1.13 to 1.22 and 1.29 to 1.59 where its lanes were told apart
    load by load."""
    stream, graphs, best = torch.cuda.Stream(), [], [1e9, 1e9]
    for cs in (short, whole):
        C, K = (256, cs) if dgrad else (cs, 256)
        d = sd.make_desc(2, 50, 84, C, K, R, R, (1, 1), (R // 2, R // 2))
        src = torch.randn(2, 50, 84, cs, device="cuda").half()
        w = torch.randn(K, R, R, C, device="cuda").mul_(0.05).half()
        out = torch.empty(2, 50, 84, 256, dtype=torch.float16, device="cuda")
        with forced(SDCONV_IGEMM_VARIANT=variant):
            assert ("8w0f" if R == 3 else "4w4f") in sd.kernel_name(d, sd.DGRAD if dgrad else sd.FWD)
            call = sd.conv2d_dgrad if dgrad else sd.conv2d_fwd
            stream.wait_stream(torch.cuda.current_stream())
            call(d, src, w, out, None, stream.cuda_stream)
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                for _ in range(12):
                    call(d, src, w, out, None, stream.cuda_stream)
        graphs.append((graph, src, w, out))
    for _ in range(20):
        for i, (graph, *_) in enumerate(graphs):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            with torch.cuda.stream(stream):
                a.record()
                graph.replay()
                b.record()
            stream.synchronize()
            best[i] = min(best[i], a.elapsed_time(b))
    say(f"variant {variant} {R}x{R} {'data gradient' if dgrad else 'forward'}: {short} / {whole} channels {best[0] / best[1]:.3f}")
    assert best[0] < (1.09 if R == 3 else 1.2) * best[1], best


def test_two_tile_widths_in_one_launch():
    """Variant 324 on a layer with 71 x 4 tiles of 224 x 256 (15 700 = 70 x 224 + 20 rows, so the
    last row tile is ragged): 256 of them stay that wide, the last seven row tiles are cut into 56
    tiles of 224 x 128; the data gradient of the same layer has 71 x 1 tiles and runs them all half
    as wide."""
    case = (1, 100, 157, 64, 1024, 1, 1, (1, 1), (0, 0), (1, 1))
    d, x, w, g = _rand_case(*case, seed=324)
    with forced(SDCONV_IGEMM_VARIANT=324, SDCONV_NO_TUNED_TABLE=1):
        assert "tail128" in sd.kernel_name(d, sd.FWD)
        check_all_passes(d, x, w, g, f"mixed{case}")


@pytest.mark.parametrize("variant", [327, 334])
def test_taps_outside_every_image(variant):
    """3x3 of dilation 9 on 4x4 images: eight taps lie further away than the source is long.  Their offsets must not
    leave the descriptors of the fetching waves' runs, so such layers take the general loop."""
    case = (2, 4, 4, 1024, 136, 3, 3, (1, 1), (9, 9), (9, 9))
    say(f"taps outside, variant {variant} case {case}")
    d, x, w, g = _rand_case(*case, seed=variant)
    with forced(SDCONV_IGEMM_VARIANT=variant, SDCONV_NO_TUNED_TABLE=1):
        check_all_passes(d, x, w, g, f"outside_v{variant}")


# the forward kernels in which every wave fetches its own share (igemm_dma.hip, 101 and 112) and the
# register-staged ones (igemm.hip, 0 and 3), whose data gradient takes a transposed filter copy
DMA_VARIANTS = [0, 3, 101, 112]


@pytest.mark.parametrize("variant", DMA_VARIANTS)
def test_all_wave_fetch_kernel_variants(variant):
    for case in WS_SHAPES:
        say(f"dma variant {variant} case {case}")
        d, x, w, g = _rand_case(*case, seed=variant * 19 + 5)
        with forced(SDCONV_IGEMM_VARIANT=variant, SDCONV_NO_TUNED_TABLE=1):
            assert "_ws_" not in sd.kernel_name(d, sd.FWD) and "patch" not in sd.kernel_name(d, sd.FWD)
            assert variant >= 100 or "_ws_" not in sd.kernel_name(d, sd.DGRAD)
            check_all_passes(d, x, w, g, f"dma{variant}{case}")


WGRAD_SHAPES = [
    (2, 23, 29, 64, 72, 3, 3, (2, 2), (1, 1), (1, 1)),      # strided, gathered x rows, filter tail
    (1, 31, 37, 136, 200, 3, 3, (1, 1), (1, 1), (1, 1)),    # channel and filter tails
    (1, 31, 37, 128, 264, 1, 1, (1, 1), (0, 0), (1, 1)),    # 1x1 unpadded: linear x addressing
    # images of 49 pixels: a step of 64 ends in the next one; 441 pixels are seven steps, the last of three ranges has one
    (9, 7, 7, 72, 136, 3, 3, (1, 1), (1, 1), (1, 1)),
    (30, 3, 3, 64, 72, 3, 3, (1, 1), (1, 1), (1, 1)),       # seven images to a step
    (5, 1, 1, 64, 72, 1, 1, (1, 1), (0, 0), (1, 1)),        # five pixels: the first step is the last, and short
    (1, 5, 7, 72, 64, 3, 3, (1, 1), (2, 2), (2, 2)),        # dilation, fewer pixels than a step
    (2, 19, 24, 72, 80, 3, 3, (2, 1), (1, 1), (1, 1)),      # strides that differ
    (3, 11, 13, 88, 136, 1, 1, (1, 1), (0, 0), (1, 1)),     # linear, channels and filters end within a tile
]
WGRAD_VARIANTS = [0, 1, 104, 107, 108, 112] + list(range(114, 124))      # 0, 1: the register-staged kernels of wgrad.hip


@pytest.mark.parametrize("variant", WGRAD_VARIANTS)
def test_wgrad_kernel_variants(variant):
    for splits in (1, 3):
        for case in WGRAD_SHAPES:
            say(f"wgrad variant {variant} splits {splits} case {case}")
            d, x, w, g = _rand_case(*case, seed=variant * 13 + splits)
            with forced(SDCONV_WGRAD_VARIANT=variant, SDCONV_WGRAD_SPLITS=splits, SDCONV_NO_TUNED_TABLE=1):
                check_all_passes(d, x, w, g, f"wgrad{variant}s{splits}{case}")


# pointwise layers with few filters: pixel counts around the 16 of a wave, the 64 of a workgroup, the
# weight gradient's 256 of a pixel range, and past the 65 536 that the persistent workgroups take in one
# turn, or for which the weight gradient takes three steps a wave; channels below, at and past one
# 256-channel load and one 128-channel tile; filters around each multiple of 16, odd and in fours; the
# longest filters accepted, and longer ones on padded copies
NARROW_SHAPES = [
    # N  H   W   C     K
    (1, 1, 1, 8, 1),
    (1, 3, 5, 32, 3),
    (1, 4, 4, 40, 4),
    (2, 8, 16, 256, 12),
    (1, 16, 16, 128, 15),
    (1, 1, 257, 136, 17),
    (2, 13, 21, 264, 28),
    (1, 7, 9, 512, 33),
    (1, 31, 33, 96, 47),
    (1, 25, 42, 512, 60),
    (1, 9, 7, 576, 63),
    (3, 50, 84, 256, 3),
    (1, 9, 7, 256, 63),
    (1, 5, 7, 1024, 12),
    (1, 7, 9, 512, 30),
    (1, 16, 16, 128, 31),
    (1, 33, 32, 72, 20),
    (1, 257, 259, 64, 15),
    (1, 257, 259, 64, 28),
    (1, 257, 259, 64, 47),
    (1, 257, 259, 64, 60),
    (1, 257, 259, 256, 12),
    (1, 363, 367, 16, 28),
]


def _narrow_passes(pixels, C, K):
    tiles = -(-K // 16)
    wgrad = tiles == 1 or (tiles == 2 and C <= 128 and not 256 < pixels < 1024)
    return [tiles * C <= 1024, tiles * C <= 1024, wgrad]


@pytest.mark.parametrize("shape", NARROW_SHAPES)
def test_narrow_pointwise_kernels(shape):
    N, H, W, C, K = shape
    say(f"narrow pointwise {shape}")
    d, x, w, g = _rand_case(N, H, W, C, K, 1, 1, (1, 1), (0, 0), (1, 1), seed=C * 64 + K)
    for p, name, narrow in zip((sd.FWD, sd.DGRAD, sd.WGRAD), ("fwd", "dgrad", "wgrad"), _narrow_passes(N * H * W, C, K)):
        assert sd.kernel_name(d, p) == "narrow_" + name if narrow else sd.kernel_name(d, p).startswith("padk+")
    check_all_passes(d, x, w, g, f"narrow{shape}")
    check_fused(d, x, w, g, f"narrow_fused{shape}")


def test_narrow_pointwise_route_borders():
    def names(*geom):
        d = sd.make_desc(*geom)
        return [sd.kernel_name(d, p).startswith("narrow") for p in (sd.FWD, sd.DGRAD, sd.WGRAD)]
    one, zero = (1, 1), (0, 0)
    assert names(1, 9, 7, 256, 63, 1, 1, one, zero, one) == [True, True, False]
    assert names(1, 9, 7, 1024, 15, 1, 1, one, zero, one) == [True, True, True]
    assert names(1, 16, 16, 128, 31, 1, 1, one, zero, one) == [True, True, True]
    assert names(1, 1, 257, 128, 31, 1, 1, one, zero, one) == [True, True, False]
    assert names(1, 32, 32, 128, 31, 1, 1, one, zero, one) == [True, True, True]
    assert names(1, 32, 32, 136, 31, 1, 1, one, zero, one) == [True, True, False]
    assert names(1, 9, 7, 1032, 15, 1, 1, one, zero, one) == [False, False, True]
    for geom in [(1, 9, 7, 264, 63, 1, 1, one, zero, one),      # faster on padded copies
                 (1, 9, 7, 64, 65, 1, 1, one, zero, one),       # too many filters
                 (1, 9, 7, 64, 16, 1, 1, one, zero, one),       # a multiple of 8
                 (1, 9, 7, 60, 12, 1, 1, one, zero, one),       # channels not in eights
                 (1, 9, 7, 64, 12, 1, 1, (2, 2), zero, one), (1, 9, 7, 64, 12, 1, 1, one, one, one),
                 (1, 9, 7, 64, 12, 3, 3, one, one, one)]:
        assert names(*geom) == [False] * 3, geom
