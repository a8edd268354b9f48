"""Host side of the bf16-piece kernels and of the fp32 kernel of three-channel layers (no GPU): the two calls of a layer always take the same instance, whatever the
sizes, what the plan asks for fits the chip, and the GPU tests run every instance that the plan selects, of these kernels and of the fp32 pipeline."""
import ctypes
import random
import time

import pytest

import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import binding
from perf import cases
from test_gpu_few_tiles import SHAPES as FEW_TILE_SHAPES
from test_gpu_parity import ASYMMETRIC_SHAPES, HALF_TILE_SHAPES, LEFTOVER_TILE_SHAPES, MANY_TILE_SHAPES, ONE_BY_ONE_SHAPES, PIPELINE_SHAPES
from test_gpu_shallow import SHAPES as SHALLOW_SHAPES
from test_gpu_shallow import instance_name
from test_gpu_split import SHAPES
from test_gpu_split_1x1 import SHAPES as PIECE_1X1_SHAPES
from test_gpu_split_stem import SHAPES as STEM_SHAPES

FILTERS = [(3, 3), (5, 5), (7, 7), (1, 7), (7, 1), (1, 3), (3, 1), (4, 4)]


def _tf(*flags):
    return tuple("true" if f else "false" for f in flags)


def _listed():
    """(layer, the kernel of the two-call path, of the workspace-free call) as the lists of the GPU tests have them, or as far as they
    have them.  The GPU tests compare numbers alone, so that they hold for any rule of the dispatch."""
    for shape, cfg in SHAPES:
        yield shape, *("conv_split_kernel<%d, %d, %d, %s>" % (*shape[5:7], cfg, *_tf(w)) for w in (False, True))
    for shape, runs in PIECE_1X1_SHAPES:
        yield shape, *("conv_split_1x1_kernel<%d, %s, %s>" % (runs, *_tf(shape[1] % 8, w)) for w in (False, True))
    for shape, instance in STEM_SHAPES:
        yield shape, *("conv_split_stem_kernel<%d, %d, %d, %d, %d, %s>" % (shape[5], *instance, *_tf(w)) for w in (False, True))
    for shape, instance in SHALLOW_SHAPES:
        yield shape, *(instance_name(shape[5], instance, w) for w in (False, True))
    for shape, kernel in FEW_TILE_SHAPES + PIPELINE_SHAPES:
        yield shape, kernel, kernel.split("<")[0] + "<"


@pytest.mark.parametrize("shape,two_call,workspace_free", _listed(), ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_the_layers_of_the_gpu_tests_run_the_instances_they_list(shape, two_call, workspace_free):
    for w, want in ((False, two_call), (True, workspace_free)):
        name = im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"]
        assert name.startswith(want), (name, want)


@pytest.mark.parametrize("shape,pipelined", ASYMMETRIC_SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_which_filters_run_the_fp32_pipeline(shape, pipelined):
    """(Few tiles run it as quarter tiles.)"""
    name = im2win.conv2d_im2win_fwd_launch_info(*shape)["kernel"]
    assert name.startswith(tuple("conv_mfma_%s_kernel<%d, %d," % (k, *shape[5:7]) for k in ("fast", "quarter"))) == pipelined, name


@pytest.mark.parametrize("dims,form", ONE_BY_ONE_SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_which_1x1_layers_run_the_fp32_1x1_kernel(dims, form):
    N, Ci, Hi, Wi, Co, s = dims
    name = im2win.conv2d_im2win_fwd_launch_info(N, Ci, Hi, Wi, Co, 1, 1, s, 0)["kernel"]
    assert name.startswith("conv_mfma_1x1_kernel<") == (form is not None), name
    assert form is None or {"x4": ", false, ", "gather": ", true, "}[form] in name, name


@pytest.mark.parametrize("filt", FILTERS, ids=lambda f: "%dx%d" % f)
def test_both_calls_take_the_same_instance(filt):
    Hf, Wf = filt
    rng = random.Random(100 * Hf + Wf)
    split = 0
    for _ in range(1500):
        s, p = rng.choice([1, 1, 2, 3, 5]), rng.randint(0, 4)
        Hi, Wi = rng.randint(1, 120), rng.choice([rng.randint(1, 60), rng.randint(1, 600)])
        Ci, Co, N = rng.choice([8, 9, 16, 17, 40, 64, 100, 256]), rng.choice([1, 32, 65, 128, 300]), rng.randint(1, 64)
        if Hi + 2 * p < Hf or Wi + 2 * p < Wf or N * Ci * (Hi + 2 * p) * Hf * (Wi + 2 * p) >= 2 ** 31:
            continue
        shape = (N, Ci, Hi, Wi, Co, Hf, Wf, s, p)
        plans = [im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w) for w in (False, True)]
        is_split = [i["kernel"].startswith("conv_split_kernel<") for i in plans]
        assert is_split[0] == is_split[1], shape
        if not is_split[0]:
            continue
        split += 1
        a, b = (i["kernel"].rstrip(">").split(", ") for i in plans)
        assert a[3] == "false" and b[3] == "true" and a[:3] == b[:3], (shape, a, b)
        assert plans[0]["grid"] == plans[1]["grid"] and plans[0]["lds_bytes"] == plans[1]["lds_bytes"] <= 160 * 1024
    # images whose strips pass the 4 GiB that the fp32 pipeline can address, or whose tensors do
    for shape in ((1, 64, 1400, 1400, 64, Hf, Wf, 1, 0), (1, 32, 2048, 2048, 64, Hf, Wf, 1, 0), (1, 16, 2048, 2048, 64, Hf, Wf, 2, 0),
                  (2, 500, 400, 400, 64, Hf, Wf, 1, 0)):
        if shape[0] * shape[1] * (shape[2] - Hf + 1) * shape[3] * Hf >= 2 ** 31:
            continue
        plans = [im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"] for w in (False, True)]
        assert plans[0].startswith("conv_split") == plans[1].startswith("conv_split"), (shape, plans)
    assert split > 100


def test_every_selected_instance_has_a_gpu_test():
    """Plans layers at random over a wide range and over that of the performance cases."""
    tested = {(*shape[5:7], cfg) for shape, cfg in SHAPES}
    rng, seen = random.Random(5), set()
    for i in range(80000):
        if i % 4 == 0:
            c = cases.draw(rng)
            shape = tuple(c[k] for k in ("N", "Ci", "Hi", "Wi", "Co", "Hf", "Wf", "stride", "pad"))
        else:
            Hf, Wf = rng.choice(FILTERS)
            Hi, s, p = int(2 ** rng.uniform(2, 8)), rng.choice([1, 1, 1, 2, 3]), rng.randint(0, 4)
            Wi = Hi if rng.random() < 0.5 else int(2 ** rng.uniform(2, 8))
            shape = (int(2 ** rng.uniform(0, 8)), int(2 ** rng.uniform(1, 10)), Hi, Wi, rng.choice([1, 20, 33, 65, 100, 130, 300]), Hf, Wf, s, p)
            if Hi + 2 * p < Hf or Wi + 2 * p < Wf or shape[0] * max(shape[1], shape[4]) * (Hi + 2 * p) * Hf * (Wi + 2 * p) >= 2 ** 31:
                continue
        name = im2win.conv2d_im2win_fwd_launch_info(*shape)["kernel"]
        if name.startswith("conv_split_kernel<"):
            seen.add(tuple(int(v) for v in name[len("conv_split_kernel<"):].split(", ")[:3]))
    assert len(seen) >= 28 and seen <= tested, (len(seen), sorted(seen - tested))


def test_every_selected_fp32_pipeline_instance_has_a_gpu_test():
    """The same for the fp32 pipeline: whole tiles, several to a workgroup, halves, sixteenths, quarters, ragged channel counts."""
    def plan(shape):
        return im2win.conv2d_im2win_fwd_launch_info(*shape)["kernel"]

    tested = {plan(s) for s in [s for s, _ in FEW_TILE_SHAPES + PIPELINE_SHAPES + ASYMMETRIC_SHAPES] + MANY_TILE_SHAPES + LEFTOVER_TILE_SHAPES + HALF_TILE_SHAPES}
    rng, seen = random.Random(23), {}
    for i in range(150000):
        if i % 3 == 0:
            c = cases.draw(rng)
            shape = tuple(c[k] for k in ("N", "Ci", "Hi", "Wi", "Co", "Hf", "Wf", "stride", "pad"))
        else:
            Hf, Wf = rng.choice(FILTERS + [(2, 2)])
            Hi, s, p = int(2 ** rng.uniform(2, 8)), rng.choice([1, 1, 1, 2, 3]), rng.randint(0, 4)
            Wi = Hi if rng.random() < 0.5 else int(2 ** rng.uniform(2, 8))
            Ci = rng.choice([8, 16, 24, 32, 48, 64, 128, 256, int(2 ** rng.uniform(1, 10))])
            shape = (int(2 ** rng.uniform(0, 8)), Ci, Hi, Wi, rng.choice([1, 20, 33, 64, 65, 100, 128, 130, 256, 300]), Hf, Wf, s, p)
            if Hi + 2 * p < Hf or Wi + 2 * p < Wf or shape[0] * max(Ci, shape[4]) * (Hi + 2 * p) * Hf * (Wi + 2 * p) >= 2 ** 31:
                continue
        seen.setdefault(plan(shape), shape)
    seen = {k: v for k, v in seen.items() if k.startswith(("conv_mfma_fast_kernel<", "conv_mfma_quarter_kernel<"))}
    assert len(seen) >= 58 and set(seen) <= tested, (len(seen), {k: v for k, v in seen.items() if k not in tested})


def test_layers_that_stay_on_the_fp32_pipeline_are_planned_as_fast_as_any():
    """The rule looks for patches only where an estimate can win; a search for every configuration took 1.5 us of each call."""
    lib, info = im2win.load_library(), binding.LaunchInfo()

    def best(*dims):
        t = []
        for _ in range(60):
            t0 = time.perf_counter()
            for _ in range(200):
                lib.conv2d_im2win_fwd_launch_info(*dims, 0, 0, ctypes.byref(info))
            t.append(time.perf_counter() - t0)
        return min(t)

    few, some = best(1, 64, 56, 56, 64, 3, 3, 1, 1), best(16, 64, 28, 28, 64, 3, 3, 1, 1)   # (no search at all: quarter tiles)
    assert info.kernel.startswith(b"conv_mfma_fast_kernel<") and some < 1.3 * few, (few, some)   # (1.05 times; 1.6 to 2.1 with the searches)


# (layer, form): layers of few tiles on both sides of the lines between quarters and sixteenths or halves of a tile.  In us, the sixteenths or
# halves in two calls / workspace-free, quarters likewise:
FEW_TILE_LINES = [
    ((6, 608, 36, 36, 1, 3, 3, 2, 0), "sixteenths"),   # 16.5 / 32, 41 / 50: of 512 pieces 109 have outputs
    ((9, 304, 21, 8, 51, 3, 3, 1, 0), "sixteenths"),   # 14.5 / 18.8, 21 / 27
    ((9, 272, 13, 13, 52, 3, 3, 1, 0), "sixteenths"),  # channels an odd multiple of 16
    ((5, 192, 15, 15, 262, 3, 3, 2, 0), "sixteenths"),  # 13.2 / 23.2, 14.9 / 18.3: two strip words per thread
    ((1, 128, 16, 16, 256, 3, 3, 1, 0), "sixteenths"),  # a unit for every piece
    ((10, 256, 9, 11, 120, 3, 3, 1, 0), "quarters"),   # 16.5 / 23.5, 14.7 / 17.0
    ((3, 576, 21, 21, 39, 3, 3, 1, 0), "quarters"),    # 33 / 45, 29 / 34
    ((1, 64, 56, 56, 64, 3, 3, 1, 1), "quarters"),
    ((2, 12, 65, 65, 7, 5, 5, 2, 0), "halves"),        # 6.0 / 6.5, 6.9 / 7.0
    ((2, 20, 65, 65, 7, 5, 5, 2, 0), "quarters"),
]


@pytest.mark.parametrize("shape,form", FEW_TILE_LINES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_lines_between_the_forms_of_few_tiles(shape, form):
    for w in (False, True):
        name, _, args = im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"].partition("<")
        tail, half = args.split(", ")[8:10] if name == "conv_mfma_fast_kernel" else (None, None)
        assert {"conv_mfma_quarter_kernel": "quarters"}.get(name, "sixteenths" if tail == "true" else "halves" if half == "true" else name) == form, name


# (layer, what follows the filter in the kernel's name): halves with two and with three workgroups per compute unit, ragged channel counts
# in halves and in whole tiles
HALF_TILE_LINES = [
    ((7, 8, 41, 43, 190, 3, 3, 1, 1), "8, 1, 4, 3, {}, false, false, true, false"),     # 579 tiles, 67 left; one K block
    ((4, 8, 41, 43, 190, 3, 3, 1, 1), "8, 1, 4, 2, {}, false, false, true, false"),     # two tiles to a unit at most
    ((7, 24, 41, 43, 190, 3, 3, 1, 1), "8, 1, 4, 2, {}, false, false, true, false"),    # three K blocks
    ((19, 32, 30, 31, 100, 3, 3, 1, 1), "8, 1, 4, 3, {}, false, false, true, false"),   # four
    ((8, 40, 41, 43, 180, 3, 3, 1, 0), "8, 1, 4, 2, {}, false, false, true, false"),    # five
    ((9, 32, 50, 50, 128, 3, 3, 1, 0), "8, 1, 4, 3, {}, false, true, true, false"),     # with sixteenths
    ((9, 320, 38, 38, 134, 3, 3, 2, 1), "8, 2, 4, 2, {}, false, true, true, false"),    # two strip words per thread
    ((7, 20, 43, 42, 190, 3, 3, 1, 1), "8, 1, 4, 3, {}, false, false, false, true"),    # ragged, 594 tiles, 82 left
    ((7, 27, 43, 42, 190, 3, 3, 1, 1), "8, 1, 4, 2, {}, false, false, true, true"),
    ((4, 20, 43, 42, 190, 3, 3, 1, 1), "8, 1, 4, 2, {}, false, false, true, true"),
]


@pytest.mark.parametrize("shape,args", HALF_TILE_LINES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_lines_between_the_forms_of_half_tiles(shape, args):
    for w in (False, True):
        name = im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"]
        assert name == "conv_mfma_fast_kernel<3, 3, %s>" % args.format(*_tf(w)), name


@pytest.mark.parametrize("shape,pieces", [
    ((106, 16, 123, 123, 64, 1, 7, 2, 4), False),   # fp32 pipeline / pieces, two calls and workspace-free: 64 / 71, 68 / 82
    ((86, 32, 28, 28, 65, 1, 7, 2, 1), False),      # 11.3 / 10.8, 11.3 / 12.2
    ((51, 48, 69, 69, 64, 1, 7, 2, 0), True),       # 1.41 and 1.21 times as fast in pieces
    ((137, 32, 6, 84, 300, 1, 7, 2, 4), True),      # 1.17, 1.03
    ((78, 8, 45, 45, 23, 3, 3, 1, 0), False),       # 18.4 / 20.7, 19.1 / 19.8
    ((50, 8, 45, 45, 20, 3, 3, 1, 0), False),       # 13.1 / 15.1, 13.2 / 14.4
    ((120, 8, 36, 5, 20, 3, 3, 1, 4), True),        # 10.2 / 9.7, 10.3 / 9.3: 867 tiles
    ((22, 8, 62, 192, 387, 3, 3, 1, 0), True),      # 221 / 184
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_lines_between_the_fp32_pipeline_and_the_pieces(shape, pieces):
    for w in (False, True):
        name = im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"]
        assert name.startswith("conv_split_kernel<") == pieces, name


def test_a_kernel_name_is_one_kernel():
    """A profiler's kernel name is the name the plan gives, so it has to tell the two bodies apart: the ragged fp32
    instance and the bf16-piece kernel once had the same one."""
    rng, blocks = random.Random(7), {}
    for shape in [(3, 13, 12, 12, 96, 3, 3, 1, 0), (32, 64, 56, 56, 64, 3, 3, 1, 1)] + [
            (rng.randint(1, 64), rng.choice([8, 13, 40, 64, 100]), rng.randint(7, 60), rng.randint(7, 60), 64, *rng.choice(FILTERS), 1, 0)
            for _ in range(2000)]:
        for w in (False, True):
            i = im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)
            assert blocks.setdefault(i["kernel"], i["block"]) == i["block"], (shape, i)


def test_three_channel_layers():
    """The stem kernel: both calls take the same instance, it fits the chip, the GPU tests run every instance selected, and layers it
    turns away run what they ran."""
    tested = {(shape[5], *instance) for shape, instance in STEM_SHAPES}
    rng, seen = random.Random(11), set()
    for shape in ((1, 3, 67, 67, 64, 7, 7, 2, 0), (8, 3, 61, 61, 32, 7, 7, 2, 3)):   # 31 outputs a row: four rows to the fp32 kernel's tile
        for w in (False, True):
            assert im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"].startswith("conv_split_stem_kernel<7"), shape
    for i in range(40000):
        f, s = rng.choice([(3, 1), (3, 2), (3, 3), (7, 2), (7, 2), (11, 4), (11, 4), (7, 1), (7, 3), (11, 2), (11, 8)])
        Hi, p = int(2 ** rng.uniform(2, 10)), rng.randint(0, 6)
        Wi = Hi if rng.random() < 0.5 else int(2 ** rng.uniform(2, 10))
        shape = (int(2 ** rng.uniform(0, 8)), 3, Hi, Wi, rng.choice([1, 24, 32, 33, 64, 65, 96, 97, 200]), f, f, s, p)
        if Hi + 2 * p < f or Wi + 2 * p < f or shape[0] * 96 * (Hi + 2 * p) * f * (Wi + 2 * p) >= 2 ** 31:
            continue
        plans = [im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w) for w in (False, True)]
        a, b = (q["kernel"].rstrip(">").split(", ") for q in plans)
        assert a[0].startswith("conv_split_stem") == b[0].startswith("conv_split_stem"), (shape, a, b)
        if not a[0].startswith("conv_split_stem"):
            # images of fewer columns do not fit its stage; small 7x7 layers go to the fp32 kernel of such layers, where that takes them
            assert (f, s) not in ((7, 2), (11, 4)) or Wi + 2 * p < 34 + f or (f == 7 and shape[4] <= 64 and a[0].startswith("conv_mfma_shallow")), (shape, a)
            continue
        assert a[:5] == b[:5] and a[5] == "false" and b[5] == "true" and plans[0]["grid"] == plans[1]["grid"], (shape, a, b)
        assert plans[0]["lds_bytes"] <= 160 * 1024 and ((f == 3 and s <= 2) or (f, s) in ((7, 2), (11, 4)))
        seen.add((int(a[0].split("<")[1]), *(int(v) for v in a[1:5])))
    assert seen == tested, (seen ^ tested)


# (layer, the kernel its plan starts with): both sides of the lines between the kernels of three-channel layers, on 256 units
LINES = [
    ((201, 3, 54, 54, 32, 3, 3, 1, 1), "conv_mfma_shallow_kernel<3"),          # 2290 pixels per unit, no channel missing
    ((300, 3, 54, 54, 32, 3, 3, 1, 1), "conv_split_stem_kernel<3, 1, 1, 4, 4"),
    ((201, 3, 54, 54, 31, 3, 3, 1, 1), "conv_split_stem_kernel<3, 1, 1, 4, 4"),
    ((201, 3, 54, 54, 96, 3, 3, 1, 1), "conv_split_stem_kernel<3, 1, 1, 4, 4"),
    ((8, 3, 51, 51, 96, 3, 3, 2, 1), "conv_split_stem_kernel<3, 1, 1, 4, 1"),     # 43 tiles of three blocks
    ((3, 3, 129, 129, 96, 3, 3, 2, 1), "conv_split_stem_kernel<3, 2, 1, 4, 1"),   # 100: pairs have a unit each
    ((18, 3, 66, 66, 96, 3, 3, 2, 1), "conv_split_stem_kernel<3, 1, 1, 4, 1"),    # 154: single ones run in one round
    ((1, 3, 313, 313, 160, 3, 3, 2, 0), "conv_split_stem_kernel<3, 2, 1, 4, 1"),
    ((35, 3, 191, 191, 96, 3, 3, 2, 0), "conv_split_stem_kernel<3, 1, 1, 4, 1"),  # fifteen rounds
    ((35, 3, 191, 191, 97, 3, 3, 2, 0), "conv_split_stem_kernel<3, 2, 1, 4, 1"),
    ((9, 3, 261, 261, 32, 11, 11, 4, 5), "conv_split_stem_kernel<11, 2, 4, 1, 1"),   # five rounds
    ((9, 3, 261, 261, 24, 11, 11, 4, 5), "conv_split_stem_kernel<11, 1, 4, 2, 1"),
    ((22, 3, 191, 191, 32, 11, 11, 4, 0), "conv_split_stem_kernel<11, 1, 4, 2, 1"),
]


@pytest.mark.parametrize("shape,kernel", LINES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_lines_between_the_kernels_of_three_channel_layers(shape, kernel):
    for w in (False, True):
        assert im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"].startswith(kernel)


def test_every_selected_fp32_instance_of_three_channel_layers_has_a_gpu_test():
    tested = {instance_name(shape[5], instance, w) for shape, instance in SHALLOW_SHAPES for w in (False, True)}
    rng, seen = random.Random(19), set()
    for _ in range(30000):
        f, s = rng.choice([(3, 1), (3, 2), (3, 3), (7, 1), (7, 2), (7, 3), (7, 8), (11, 1), (11, 2), (11, 3), (11, 4), (11, 8)])
        Hi, p = int(2 ** rng.uniform(2, 10.5)), rng.randint(0, 6)
        Wi = Hi if rng.random() < 0.5 else int(2 ** rng.uniform(2, 10.5))
        shape = (int(2 ** rng.uniform(0, 9)), 3, Hi, Wi, rng.choice([1, 24, 32, 33, 64, 65, 96, 97, 128, 200]), f, f, s, p)
        if Hi + 2 * p < f or Wi + 2 * p < f or shape[0] * max(shape[4], 3 * f) * (Hi + 2 * p) * (Wi + 2 * p) >= 2 ** 31:
            continue
        for w in (False, True):
            name = im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"]
            if name.startswith("conv_mfma_shallow_kernel<"):
                seen.add(name)
    assert seen == tested, (sorted(seen ^ tested))


def test_both_calls_of_large_layers():
    """The im2win tensor is up to Hf times the input: where only one of them is within 32-bit offsets, both calls turn the layer away."""
    rng, taken = random.Random(17), [0, 0]
    shapes = [(4, 3, 7000, 7000, 96, 11, 11, 4, 0), (6, 3, 7120, 4184, 32, 7, 7, 2, 3), (2, 3, 6000, 6000, 16, 7, 7, 2, 0)]
    while len(shapes) < 4000:
        f, s = rng.choice([(3, 1), (3, 2), (7, 2), (11, 4), (1, 1), (1, 2)])
        Hi, Wi, Ci = int(2 ** rng.uniform(9, 14)), int(2 ** rng.uniform(9, 14)), rng.choice([8, 64, 512]) if f == 1 else 3
        shape = (rng.randint(1, 12), Ci, Hi, Wi, rng.choice([16, 65, 96, 128]), f, f, s, rng.randint(0, f // 2))
        N, Ho, Wo = shape[0], (Hi + 2 * shape[8] - f) // s + 1, (Wi + 2 * shape[8] - f) // s + 1
        if max(N * Ci * Ho * f * (Wi + 2 * shape[8]), N * Ci * Hi * Wi, N * shape[4] * Ho * Wo) < 2 ** 31:
            shapes.append(shape)
    for shape in shapes:
        a, b = (im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"] for w in (False, True))
        assert a.startswith("conv_split") == b.startswith("conv_split"), (shape, a, b)
        if a.startswith("conv_split"):
            assert a.rsplit(", ", 1)[0] == b.rsplit(", ", 1)[0], (shape, a, b)
        taken[a.startswith("conv_split")] += 1
    assert min(taken) > 500, taken


def test_one_by_one_layers():
    """The piece kernel of 1x1 layers: both calls take it or neither does, and it keeps to the layers it can index."""
    rng, taken = random.Random(13), 0
    for _ in range(20000):
        Hi, s, p = int(2 ** rng.uniform(0, 8)), rng.choice([1, 1, 1, 2, 3]), rng.choice([0, 0, 0, 1])
        Wi = Hi if rng.random() < 0.5 else int(2 ** rng.uniform(0, 8))
        Ci, Co = rng.choice([8, 16, 60, 64, 250, 256, 520, 1024, rng.randint(1, 40), rng.randint(1, 40)]), rng.choice([1, 64, 65, 128, 130, 256, 1000])
        shape = (int(2 ** rng.uniform(0, 12)), Ci, Hi, Wi, Co, 1, 1, s, p)
        if shape[0] * max(Ci, Co) * (Hi + 2 * p) * (Wi + 2 * p) >= 2 ** 31:
            continue
        plans = [im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w) for w in (False, True)]
        split = [q["kernel"].startswith("conv_split_1x1") for q in plans]
        assert split[0] == split[1], (shape, plans)
        if split[0]:
            taken += 1
            assert p == 0 and Ci > 4 and plans[0]["grid"] == plans[1]["grid"] and plans[0]["lds_bytes"] <= 160 * 1024
            assert [q["kernel"].split(", ", 1)[1] for q in plans] == ["%s, %s>" % _tf(Ci % 8, w) for w in (False, True)], plans
        elif p == 0 and Ci > 16 and s <= 65536:
            # the fp32 1x1 kernel, or words out of reach of the pieces' offsets
            assert (Ci % 8 == 0 and Co % 4 == 0) or shape[0] * Ci * Hi * Wi >= 2 ** 29, (shape, plans)
    assert taken > 5000


# (layer, whether it runs in pieces): both sides of the lines where the fp32 1x1 kernel has no instance.  In us, generic kernel in two calls /
# workspace-free / pieces:
ONE_BY_ONE_LINES = [
    ((64, 4, 40, 40, 33, 1, 1, 1, 0), False),     # four channels
    ((37, 8, 63, 63, 6, 1, 1, 1, 0), False),      # 9.4 / 9.6 / 17.7
    ((60, 6, 163, 163, 3, 1, 1, 2, 0), False),    # 26 / 28 / 42
    ((121, 7, 102, 102, 2, 1, 1, 1, 0), False),   # 75 / 78 / 117
    ((156, 7, 184, 184, 19, 1, 1, 1, 0), False),  # 365 / 374 / 491
    ((102, 16, 77, 76, 9, 1, 1, 1, 0), False),    # 41 / 41 / 58
    ((128, 5, 224, 224, 1, 1, 1, 1, 0), False),
    ((233, 13, 1, 1, 28, 1, 1, 2, 0), True),      # 16 / 23 / 6.7
    ((84, 10, 1, 1, 10, 1, 1, 2, 0), True),       # 15 / 21 / 5.6
    ((3, 5, 16, 15, 20, 1, 1, 1, 0), True),
    ((152, 7, 197, 3, 10, 1, 1, 1, 0), True),     # 16 / 18 / 12: three pixels a row
    ((231, 8, 114, 114, 286, 1, 1, 2, 0), True),  # 330 / 335 / 237
    ((58, 33, 9, 5, 94, 1, 1, 2, 0), True),
]


@pytest.mark.parametrize("shape,pieces", ONE_BY_ONE_LINES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_lines_between_the_kernels_of_1x1_layers(shape, pieces):
    for w in (False, True):
        name = im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=w)["kernel"]
        assert name.startswith("conv_split_1x1_kernel<") == pieces, name
