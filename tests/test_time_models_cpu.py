"""The time models of the dispatcher against the committed timings: the variant that the library picks
must be about as fast as the fastest one measured."""
import ctypes
import math
import os
import re
import time

import pytest

import paper_1903_05831_amd as sd
from paper_1903_05831_amd import fit_models

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TIMINGS = os.path.join(ROOT, "profiles", "layer_timings.jsonl.gz")
BEFORE = os.path.join(ROOT, "profiles", "layer_timings_before_runs.jsonl.gz")      # fetching waves sent each load by itself


def _desc(k):
    N, H, W, C, K, R, s, pad, dil = k
    return sd.make_desc(N, H, W, C, K, R, R, (s, s), (pad, pad), (dil, dil))


@pytest.fixture(scope="module")
def variants():
    """Variant of each kernel name (the overrides are honoured: conftest.py sets SDCONV_TUNE)."""
    d, out = sd.make_desc(1, 28, 28, 64, 64, 3, 3, (1, 1), (1, 1)), {}
    for name, known, passes in (("SDCONV_IGEMM_VARIANT", fit_models.ROW_VARIANTS, (sd.FWD, sd.DGRAD)),
                                ("SDCONV_WGRAD_VARIANT", fit_models.WGRAD_VARIANTS, (sd.WGRAD,))):
        for v in known:
            os.environ[name] = str(v)
            out.update({sd.kernel_name(d, p): v for p in passes})
        del os.environ[name]
    return out


def _quality(loss):
    loss = sorted(loss)
    return math.exp(sum(map(math.log, loss)) / len(loss)) - 1, loss[int(0.99 * len(loss))] - 1


def test_forward_and_data_gradient_tiles(variants):
    losses = {}
    for x in fit_models.load([TIMINGS]):
        if x["what"] == "rows":
            # data gradients of the variants below 300 want workspace for a filter copy: measured layers only
            times = {v: us for v, us in x["us"] if x["p"] == 0 or v >= 300}
            losses.setdefault(fit_models.kind(x["k"], x["p"]), []).append(
                times[variants[sd.kernel_name(_desc(x["k"]), x["p"])]] / min(times.values()))
    mean, worst = _quality(sum(losses.values(), []))
    assert sum(map(len, losses.values())) > 1000 and mean < 0.02 and worst < 0.22, (mean, worst)
    # by kind of layer, so that one kind's gain does not hide another's loss: 1.11, 0.80 and 2.61 % here; 1.15 % (gathering)
    # with the constants before their scaling, 2.80 % (strided) with scaled ones
    for kind, most in ((fit_models.POINTWISE, 0.013), (fit_models.GATHER, 0.010), (fit_models.STRIDED, 0.027)):
        assert _quality(losses[kind])[0] < most, (kind, _quality(losses[kind]))


def test_constants_are_those_of_the_fits():
    """What `fit_models fit` makes of the committed timings for forward and data-gradient passes is the table in use."""
    before, now = ([x for x in fit_models.load([path]) if x["what"] == "rows"] for path in (BEFORE, TIMINGS))
    table = {}
    with open(os.path.join(ROOT, "paper_1903_05831_amd", "csrc", "dispatch.hip")) as f:
        text = f.read().split("kRowModels[] = {")[1].split("\n};")[0]
    for line in text.strip().splitlines():
        variant = int(line.split(",")[0].strip(" {"))
        for c, cost in enumerate(re.findall(r"\{([^{}]*)\}", line)):
            if cost:
                table[variant, c] = [float(t.strip().rstrip("f")) for t in cost.split(",")]
    models = fit_models.row_models(fit_models.fit_before(before), now)
    assert models.keys() == table.keys()
    for key, cost in models.items():
        # three digits stand in the table, and other versions of the solver may end a little elsewhere
        assert all(abs(a - b) <= 0.002 + 0.001 * abs(b) for a, b in zip(cost, table[key], strict=True)), (key, cost, table[key])


def test_two_tile_widths_cost_what_their_launch_makes():
    """150 tiles of 224x256 all run at full width in the launch with two tile widths: it is the kernel of the
    plain tiles there (59-60 us and 51 us for these layers) and must not be preferred as a cheaper one."""
    for geom in [(2, 200, 336, 256, 256, 3, 3, (2, 2), (1, 1)), (2, 100, 168, 256, 256, 3, 3, (1, 1), (2, 2), (2, 2))]:
        assert "tail128" not in sd.kernel_name(sd.make_desc(*geom), sd.FWD)
    # 600 tiles: two rounds at full width, the third in halves
    d = sd.make_desc(2, 200, 336, 512, 256, 1, 1, (1, 1), (0, 0))
    assert "tail128" in sd.kernel_name(d, sd.FWD)


@pytest.mark.parametrize("geom,slower", [
    ((512, 55, 40, 32, 272, 1, 1, (2, 2), (0, 0)), "dma_128x64x32"),      # 54.2 us with 128x128 tiles, 85.9 with these
    ((100, 337, 7, 24, 1104, 1, 1, (2, 2), (0, 0)), "dma_128x64x32"),     # 56.7, 84.7
    ((512, 171, 12, 8, 176, 1, 1, (2, 2), (0, 0)), "dma_128x64x32"),      # 31.3, 47.0
])
def test_kernels_whose_constants_were_scaled_by_chance(geom, slower):
    """Layers of one channel chunk, which are bound by their results: a 128x64 tile reads the activations twice as often as a 128x128 one."""
    assert slower not in sd.kernel_name(sd.make_desc(*geom), sd.FWD)


def test_weight_gradient_tiles_and_ranges(variants):
    loss, unmeasured = [], 0
    for x in fit_models.load([TIMINGS]):
        if x["what"] != "wgrad":
            continue
        d, times = _desc(x["k"]), dict(x["us"])
        dw_bytes = 4 * d.K * d.R * d.S * d.C
        pair = variants[sd.kernel_name(d, sd.WGRAD)], max(1, sd.conv2d_workspace_bytes(d, sd.WGRAD) // dw_bytes)
        if pair in times:
            loss.append(times[pair] / min(times.values()))
        else:
            unmeasured += 1
    mean, worst = _quality(loss)
    assert len(loss) > 390 and unmeasured < 5 and mean < 0.025, (mean, worst, unmeasured)
    assert worst < 0.16, worst


@pytest.mark.parametrize("geom,slower", [
    ((1, 17, 11, 1984, 896, 3, 3, (2, 2), (1, 1)), "256x256"),      # 17.5 us with 128x128 tiles, 26.9 with these
    ((2, 8, 15, 384, 1536, 7, 7, (1, 1), (3, 3)), "256x256"),       # 36.1, 52.5
    ((1, 11, 10, 640, 1024, 5, 5, (1, 1), (2, 2)), "256x256"),      # 21.3 (256x128), 27.6
    ((1, 12, 7, 64, 64, 1, 1, (1, 1), (0, 0)), "4w4f"),             # 3.2 without waves that only fetch, 3.3 with them
])
def test_weight_gradients_of_a_few_steps(geom, slower):
    """Of few pixels: what counts is the stores of a large dw from enough tiles, or the start of the launch."""
    assert slower not in sd.kernel_name(sd.make_desc(*geom), sd.WGRAD)


def test_layers_with_an_entry_keep_the_measured_ranges():
    """Entries with a number of pixel ranges: it was measured with that tile variant."""
    for geom, name, ranges in [((512, 14, 14, 1024, 512, 1, 1, (1, 1), (0, 0)), "256x256x64_8w_s2_hf_m16", 32),
                               ((512, 7, 7, 2048, 512, 1, 1, (1, 1), (0, 0)), "256x256x32_8w_s3_hf_m16", 12)]:
        d = sd.make_desc(*geom)
        assert sd.kernel_name(d, sd.WGRAD) == "wgrad_dma_" + name
        assert sd.conv2d_workspace_bytes(d, sd.WGRAD) == ranges * 4 * d.K * d.R * d.S * d.C
        assert sd.kernel_name(sd.make_desc(geom[0] // 2, *geom[1:]), sd.WGRAD) == "wgrad_dma_" + name


def _plan_us(geom, *passes):
    """Microseconds of planning for each pass, the best of many, in turn; less those of a call that plans nothing."""
    call, d, best = sd.lib().conv2d_workspace_bytes, ctypes.byref(sd.make_desc(*geom)), {}
    for _ in range(60):
        for p in (*passes, 99):
            t = time.perf_counter()
            for _ in range(100):
                call(d, p)
            best[p] = min(best.get(p, 1e9), (time.perf_counter() - t) * 1e4)
    return [best[p] - best[99] for p in passes]


@pytest.mark.parametrize("geom", [(1, 56, 56, 64, 64, 3, 3, (1, 1), (1, 1)), (2, 50, 84, 256, 256, 3, 3, (1, 1), (1, 1)),
                                  (2, 50, 84, 1024, 256, 1, 1, (1, 1), (0, 0)), (1, 173, 271, 128, 128, 3, 3, (2, 2), (1, 1))])
def test_a_weight_gradient_is_planned_in_a_few_forward_passes(geom):
    """Every call is planned anew.  The models of 14 weight-gradient variants, each with a dozen numbers of pixel ranges:
    1.6 to 2.3 times a forward pass's plan, 3.3 to 4.3 times where the ranges were worked out for each variant."""
    fwd, wgrad = _plan_us(geom, sd.FWD, sd.WGRAD)
    assert wgrad < 2.8 * fwd, (wgrad, fwd)


@pytest.mark.parametrize("geom", [(1, 173, 271, 128, 128, 3, 3, (2, 2), (1, 1)), (1, 173, 271, 256, 512, 1, 1, (2, 2), (0, 0))])
def test_a_strided_data_gradient_is_planned_in_a_few_forward_passes(geom):
    """The parity classes of a strided data gradient must not be divided out, and their makespan not be computed, for every
    variant: 1.8 to 2.2 times a forward pass's plan, more than 4 times with that."""
    fwd, dgrad = _plan_us(geom, sd.FWD, sd.DGRAD)
    assert dgrad < 3 * fwd, (dgrad, fwd)
