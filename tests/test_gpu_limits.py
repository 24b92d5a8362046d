"""Largest sizes the interface accepts: an activation tensor just below 2^31 elements (its last
byte offsets need all 32 bits of the kernels' offsets) through all three passes, and a gradient
buffer of more than 2^31 elements through grad_unscale_check (64-bit indexing).  Outputs are
checked on seeded samples that the oracle computes one by one, the same bar as everywhere."""
import numpy as np
import pytest
import torch

import oracle
import paper_1903_05831_amd as sd
from paper_1903_05831_amd import workloads

from gpu_harness import check_all_passes, say

pytestmark = pytest.mark.gpu


def test_activation_tensor_just_below_2_31_elements():
    """1x1 convolution 128 -> 8 channels on one 4096 x 4080 image: x and dx hold 2 139 095 040
    elements (99.6 % of 2^31); y, dy and dw are small, so the oracle's sampled sums stay cheap."""
    l = workloads.ConvLayer("limit", 1, 4096, 4080, 128, 8, 1, 1, 1, 0, 4096, 4080)
    assert l.N * l.H * l.W * l.C < 2 ** 31 <= l.N * l.H * (l.W + 16) * l.C
    d = sd.desc_of(l)
    say(f"limit layer {l.x_shape} -> {l.y_shape}")
    x, w, g = workloads.make_x(l, 9, 0), workloads.make_w(l, 9, 0), workloads.make_g(l, 9, 0)
    check_all_passes(d, x, w, g, "limit", sample=3000, seed=900)
    del x, w, g
    torch.cuda.empty_cache()


def test_padded_3x3_on_a_tensor_of_more_than_2_30_elements():
    """3x3, pad 1, 2048 -> 8 channels on one 724 x 725 image: x and dx hold 1 075 001 600 elements,
    so their byte offsets pass 2^31 -- the value the LDS-DMA kernels use to mark a load as masked
    (padding taps, ragged rows).  Such layers must take the kernels that index elements instead.
    The samples include the image corners and pixels on both sides of the 2 GiB byte offset.
    (Many channels rather than many pixels: the weight gradient then sums 524 900 pixels, as in the
    detector workload, and binary32 accumulation stays inside the parity bar.)"""
    l = workloads.ConvLayer("limit3x3", 1, 724, 725, 2048, 8, 3, 3, 1, 1, 724, 725)
    assert 2 ** 30 < l.N * l.H * l.W * l.C < 2 ** 31
    d = sd.desc_of(l)
    for p in (sd.FWD, sd.DGRAD, sd.WGRAD):
        name = sd.kernel_name(d, p)
        assert "dma" not in name and "_ws_" not in name and "patch" not in name, name
    say(f"limit layer {l.x_shape} -> {l.y_shape} 3x3 pad 1")
    x, w, g = workloads.make_x(l, 9, 1), workloads.make_w(l, 9, 1), workloads.make_g(l, 9, 1)
    # flat indices worth looking at: corners, last elements, both sides of byte offset 2^31
    pix_2g = (2 ** 31 // 2) // l.C
    extra_x = [0, l.C * (l.W - 1), l.C * l.W * (l.H - 1), l.C * (l.W * l.H - 1), l.C * l.W * l.H - 1] + \
              [l.C * (pix_2g + o) + c for o in (-l.W - 1, -1, 0, 1, 300) for c in (0, l.C - 1)]
    assert max(extra_x) < l.N * l.H * l.W * l.C
    # y is small; its pixels next to the x pixels at the 2 GiB offset read across that offset
    extra_y = [0, l.K * (l.Wo - 1), l.K * l.Wo * (l.Ho - 1), l.K * l.Wo * l.Ho - 1] + \
              [l.K * (pix_2g + o) + k for o in (-l.Wo - 1, -1, 0, 1, 300) for k in (0, l.K - 1)]
    check_all_passes(d, x, w, g, "limit3x3", sample=3000, seed=910,
                     extra={sd.FWD: extra_y, sd.DGRAD: extra_x})
    del x, w, g
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dgrad", [False, True])
@pytest.mark.parametrize("H", [4094, 4095])
def test_source_that_ends_just_below_2_31_bytes(H, dgrad, monkeypatch):
    """3x3 on an H x 4096 x 64 source: with the rows that its taps reach before the first pixel, 4094 rows are the most
    whose offsets stay below 2^31, and 4095 take the fetching waves' general loop.  The last rows of the result are
    those of the same layer on a copy of the last rows of the source, whose sums have the same order: every bit."""
    monkeypatch.setenv("SDCONV_IGEMM_VARIANT", "334")
    W, few, rows = 4096, 8, 6
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H)
    src = torch.empty(1, H, W, 64, dtype=torch.float16, device="cuda").normal_(generator=gen)
    w = torch.empty((64, 3, 3, few) if dgrad else (few, 3, 3, 64), dtype=torch.float16, device="cuda").normal_(0, 0.1, generator=gen)
    st = torch.cuda.current_stream().cuda_stream

    def run(s):
        h = s.shape[1]
        d = sd.make_desc(1, h, W, *((few, 64) if dgrad else (64, few)), 3, 3, (1, 1), (1, 1))
        assert "80x128" in sd.kernel_name(d, sd.DGRAD if dgrad else sd.FWD)
        out = torch.full((1, h, W, few), float("nan"), dtype=torch.float16, device="cuda")
        (sd.conv2d_dgrad if dgrad else sd.conv2d_fwd)(d, s, w, out, None, st)
        return out

    say(f"source 1x{H}x{W}x64, {'data gradient' if dgrad else 'forward'}")
    whole, first, last = run(src), run(src[:, :rows].contiguous()), run(src[:, -rows:].contiguous())
    torch.cuda.synchronize()
    assert torch.equal(whole[:, :rows - 1], first[:, :-1]) and torch.equal(whole[:, 1 - rows:], last[:, 1:])
    assert not torch.isnan(whole).any()
    del src, whole
    torch.cuda.empty_cache()


@pytest.mark.parametrize("C,K,R", [(64, 8, 3), (64, 8, 1), (8, 64, 3)])
def test_weight_gradient_with_fetching_waves_on_offsets_up_to_2_31(C, K, R, monkeypatch):
    """x or dy of 4095 x 4096 x 64: their last row ends 512 KB below 2^31 bytes, of which the fetching waves' descriptors take
    another 3 KB.  dy is zero but in the last rows, so dw is that of a copy of the last rows under the register-staged kernel.
    Products and sums of small whole numbers are exact, so every element is compared."""
    H, W, rows = 4095, 4096, 6
    gen = torch.Generator(device="cuda")
    gen.manual_seed(C + R)
    x = torch.randint(-4, 5, (1, H, W, C), dtype=torch.float16, device="cuda", generator=gen)
    g = torch.zeros(1, H, W, K, dtype=torch.float16, device="cuda")
    g[:, 1 - rows:] = torch.randint(-4, 5, (1, rows - 1, W, K), dtype=torch.float16, device="cuda", generator=gen)

    def run(variant, x, g):
        d = sd.make_desc(1, x.shape[1], W, C, K, R, R, (1, 1), (R // 2, R // 2))
        monkeypatch.setenv("SDCONV_WGRAD_VARIANT", str(variant))
        name, need = sd.kernel_name(d, sd.WGRAD), sd.conv2d_workspace_bytes(d, sd.WGRAD)
        say(f"weight gradient of {tuple(x.shape)} to {K} channels, {R}x{R}: {name}, workspace {need}")
        assert ("4w4f" in name) == (variant == 121)
        dw, ws = torch.full((K, R, R, C), float("nan"), device="cuda"), torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
        sd.conv2d_wgrad(d, x, g, dw, ws, torch.cuda.current_stream().cuda_stream)
        return dw

    whole, last = run(121, x, g), run(1, x[:, -rows:].contiguous(), g[:, -rows:].contiguous())
    torch.cuda.synchronize()
    assert last.abs().max() > 0 and torch.equal(whole, last)
    del x, g
    torch.cuda.empty_cache()


@pytest.mark.parametrize("ranges", [1, 2])
def test_weight_gradient_of_more_than_2_29_elements(ranges, monkeypatch):
    """1x1, 8192 -> 73 728 channels on 256 pixels: the 2.4 GB of dw, and twice that of partial sums, lie past the
    2^31 bytes that a store's offset reaches from the first filter.  Products and sums of small whole numbers
    are exact, so every element is compared."""
    K, C, px = 73728, 8192, 256
    d = sd.make_desc(1, 8, px // 8, C, K, 1, 1, (1, 1), (0, 0))
    monkeypatch.setenv("SDCONV_WGRAD_SPLITS", str(ranges))
    name, need = sd.kernel_name(d, sd.WGRAD), sd.conv2d_workspace_bytes(d, sd.WGRAD)
    say(f"weight gradient {K} x {C}, {ranges} ranges: {name}, workspace {need}")
    assert "dma" in name and need == (0 if ranges == 1 else ranges * 4 * K * C) and 4 * K * C > 2 ** 31
    gen = torch.Generator(device="cuda")
    gen.manual_seed(29 + ranges)
    x = torch.randint(-4, 5, (px, C), device="cuda", generator=gen).half()
    g = torch.randint(-4, 5, (px, K), device="cuda", generator=gen).half()
    dw = torch.full((K, C), float("nan"), device="cuda")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    sd.conv2d_wgrad(d, x, g, dw, ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for k in range(0, K, 8192):
        assert torch.equal(dw[k:k + 8192], g[:, k:k + 8192].float().t() @ x.float()), k
    del dw, ws
    torch.cuda.empty_cache()


def test_unscale_more_than_2_31_elements():
    """n = 2^31 + 12345 fp32 gradients (8.6 GB), values from a seeded generator on the device
    (the host copy of each checked window is taken before the call and handed to the oracle):
    bit-exact results in windows at the start, around the 4 GiB and 8 GiB byte offsets and at
    the end; the flag is 0 without and 1 with a single +inf in the very last element."""
    n = 2 ** 31 + 12345
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(workloads.BASE_SEED + 31)
    g = torch.empty(n, dtype=torch.float32, device=dev)
    step = 1 << 28
    for s in range(0, n, step):
        e = min(n, s + step)
        g[s:e] = torch.randn(e - s, generator=gen, device=dev, dtype=torch.float32) * 1000.0
    windows = [(0, 1 << 16), (2 ** 30 - 4096, 2 ** 30 + 4096), (2 ** 31 - 4096, 2 ** 31 + 4096), (n - 12345 - 64, n)]
    before = [g[a:b].cpu().numpy().copy() for a, b in windows]
    flag = torch.full((1,), -1, dtype=torch.int32, device=dev)
    st = torch.cuda.current_stream().cuda_stream
    inv = float(np.float32(1.0 / 1024.0))
    say(f"unscale n={n}")
    sd.grad_unscale_check(g, n, inv, flag, st)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    for (a, b), src in zip(windows, before):
        want, want_flag = oracle.unscale_check(src, inv)
        assert want_flag == 0
        got = g[a:b].cpu().numpy()
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), f"window {a}:{b}"
    g[n - 1] = float("inf")
    sd.grad_unscale_check(g, n, inv, flag, st)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1
    assert bool(torch.isinf(g[n - 1]))
    del g
    torch.cuda.empty_cache()
