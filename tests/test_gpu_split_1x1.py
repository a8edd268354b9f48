"""The bf16-piece kernel of 1x1 layers at ragged channel, pixel and plane counts through both calls, its error against the fp32 matrix
cores, the range of its operands, infinities and NaN."""
import pytest
import torch

import oracle
import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import workloads
from parity_util import assert_conv_close, check_any_alignment, check_second_pass, conv_errors
from test_gpu_split import _assert_like_basic
from test_gpu_split_stem import _run

pytestmark = pytest.mark.gpu

# (shape, runs of 128 pixels per tile: test_split_dispatch.py holds the dispatch to them)
SHAPES = [
    ((64, 256, 14, 15, 256, 1, 1, 1, 0), 1),     # whole tiles of channels
    ((17, 520, 19, 21, 500, 1, 1, 1, 0), 1),     # a last K block of one group, a last tile of 127 pixels
    ((300, 512, 7, 7, 130, 1, 1, 1, 0), 1),      # two channels past a tile, planes of 49 pixels
    ((33, 512, 29, 28, 257, 1, 1, 2, 0), 1),     # stride 2, one channel past a tile
    ((9000, 256, 2, 2, 256, 1, 1, 1, 0), 1),     # a tile spans 32 images
    ((60, 504, 31, 40, 395, 1, 1, 3, 0), 2),     # stride 3, 63 groups of channels
    ((67, 384, 20, 19, 385, 1, 1, 1, 0), 2),     # one channel past a tile
    ((21000, 256, 1, 1, 256, 1, 1, 1, 0), 2),    # a tile spans 256 images
    ((64, 128, 30, 33, 129, 1, 1, 1, 0), 2),     # several tiles per workgroup
    ((29, 43, 28, 30, 100, 1, 1, 1, 0), 1),      # channels that are no multiple of eight: 11 in the last K block, one tile of 128 channels
    ((3, 5, 16, 15, 20, 1, 1, 1, 0), 1),         # five channels
    ((58, 33, 9, 5, 94, 1, 1, 2, 0), 1),         # one channel in the last K block, stride 2
    ((40, 127, 57, 55, 200, 1, 1, 2, 0), 2),     # 31 of 32 in the last K block, stride 2
    ((64, 77, 40, 41, 33, 1, 1, 1, 0), 2),
    ((31, 72, 20, 21, 66, 1, 1, 1, 0), 1),       # output channels that are no multiple of four
]


@pytest.mark.parametrize("shape,runs", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_both_calls(shape, runs):
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(9950 + sum(shape), N, Ci, Hi, Wi, Co, Hf, Wf)
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    got, fp32 = _run(shape, I, F)
    assert_conv_close(got, O_ref, B_ref)
    l2, l2_32 = conv_errors(got, O_ref, B_ref)[1], conv_errors(fp32, O_ref, B_ref)[1]
    print("relative L2 error: pieces %.2e, fp32 %.2e" % (l2, l2_32))
    assert l2 <= l2_32


@pytest.mark.parametrize("shape", [SHAPES[2][0], SHAPES[8][0], SHAPES[9][0], SHAPES[12][0]], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("ei,ef", [(-118, 4), (4, -124), (-140, 20), (105, 0), (-120, 120), (60, 60)])
def test_no_operand_loses_bits(shape, ei, ef):
    """The 24 bits of an operand hold whatever its magnitude: against 64 bits no further off than the fp32 kernel."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(9960, N, Ci, Hi, Wi, Co, Hf, Wf)
    I, F = torch.ldexp(I.double(), torch.tensor(ei)).float(), torch.ldexp(F.double(), torch.tensor(ef)).float()
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    got, fp32 = _run(shape, I, F)
    assert conv_errors(got, O_ref, B_ref)[1] <= 1.1 * conv_errors(fp32, O_ref, B_ref)[1]


@pytest.mark.parametrize("shape", [SHAPES[i][0] for i in (2, 3, 5, 8, 9, 12)], ids=lambda v: "x".join(map(str, v)))
def test_buffers_of_any_alignment(shape):
    check_any_alignment(shape, 9985)


@pytest.mark.parametrize("shape", [SHAPES[1][0], SHAPES[2][0], SHAPES[5][0], SHAPES[8][0], SHAPES[9][0], SHAPES[12][0]], ids=lambda s: "x".join(map(str, s)))
def test_the_second_pass_writes_what_the_first_left(shape):
    check_second_pass(shape, 9980)


@pytest.mark.parametrize("shape", [(64, 256, 24, 31, 130, 1, 1, 1, 0), SHAPES[8][0]], ids=lambda s: "x".join(map(str, s)))
def test_infinities_nan_and_the_ends_of_the_range(shape):
    """As in plain fp32 (the one-thread-per-output kernel), in both calls."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    assert im2win.conv2d_im2win_fwd_launch_info(*shape)["kernel"].startswith("conv_split_1x1_kernel<")
    I, F = workloads.random_layer_inputs(9970, N, Ci, Hi, Wi, Co, Hf, Wf)
    I.abs_()
    I[0, 2, 10, 10], I[1, 1, 0, Wi - 1], I[2, 0, Hi - 1, 0] = float("inf"), float("-inf"), float("nan")
    I[3, 127, 20, 20] = 3.4028e38            # rounds to infinity in bf16
    I[4, 2, 5, 5], I[4, 9, 5, 5] = float("inf"), float("-inf")
    I[5, 2, 21, 17] = torch.finfo(torch.float32).min
    I[6, 1, 23, 30] = 2.0 ** 60
    F[:, 2] *= 0.25
    F[2, 2], F[3, 2], F[4, 1] = 0.0, 2.0 ** -140, 2.0 ** 50
    ref = _assert_like_basic(shape, I, F)
    assert torch.isnan(ref).any() and torch.isinf(ref).any()
