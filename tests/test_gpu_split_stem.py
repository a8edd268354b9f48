"""The bf16-piece kernel of three-channel layers: every instance the dispatch selects (test_split_dispatch.py holds the list to that) at
ragged sizes through both calls, its error against the fp32 matrix cores, the range of its operands, infinities and NaN."""
import pytest
import torch

import oracle
import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import workloads
from parity_util import assert_conv_close, check_any_alignment, check_second_pass, conv_errors, run_transform
from test_gpu_split import _assert_like_basic

pytestmark = pytest.mark.gpu

# (N, Ci, Hi, Wi, Co, Hf, Wf, s, p) and the instance: blocks of 32 channels, parts of K, runs of pixels per workgroup, blocks of 32
# pixels per run
SHAPES = [
    ((9, 3, 85, 91, 17, 7, 7, 2, 3), (1, 2, 4, 1)),      # odd widths, a last tile of a few pixels
    ((21, 3, 32, 32, 32, 7, 7, 2, 0), (1, 2, 4, 1)),     # 13 pixels a row: eleven rows to a tile
    ((9, 3, 91, 85, 33, 7, 7, 2, 3), (2, 2, 2, 1)),      # one channel past a block
    ((1, 3, 33, 36, 130, 7, 7, 2, 1), (2, 2, 2, 1)),     # three groups of channels, the last block of two
    ((41, 3, 139, 144, 64, 7, 7, 2, 3), (2, 1, 4, 1)),   # several tiles per workgroup
    ((60, 3, 118, 113, 50, 7, 7, 2, 8), (2, 1, 4, 1)),   # padding wider than the filter: windows of zeros
    ((33, 3, 31, 64, 96, 7, 7, 2, 3), (3, 2, 2, 1)),
    ((1, 3, 7, 47, 70, 7, 7, 2, 0), (3, 2, 2, 1)),       # one row, one tile
    ((16, 3, 227, 225, 20, 11, 11, 4, 0), (1, 4, 2, 1)),
    ((330, 3, 11, 530, 31, 11, 11, 4, 0), (1, 4, 2, 1)),  # one row per image: a tile may span two images
    ((1, 3, 60, 230, 5, 11, 11, 4, 5), (2, 4, 1, 1)),
    ((55, 3, 39, 40, 64, 11, 11, 4, 5), (2, 4, 1, 1)),   # eight pixels a row
    ((9, 3, 130, 127, 96, 11, 11, 4, 2), (3, 4, 1, 1)),
    ((7, 3, 63, 67, 131, 11, 11, 4, 0), (3, 4, 1, 1)),   # two groups of channels
    ((5, 3, 61, 64, 30, 3, 3, 2, 1), (1, 1, 4, 1)),
    ((3, 3, 47, 45, 65, 3, 3, 2, 0), (1, 1, 4, 1)),   # 22 pixels a row: seven rows to a tile
    ((9, 3, 64, 59, 50, 3, 3, 2, 1), (2, 1, 4, 1)),
    ((60, 3, 101, 102, 17, 3, 3, 1, 0), (1, 1, 4, 4)),   # 16-byte stores, 9900 pixels a plane
    ((54, 3, 99, 100, 67, 3, 3, 1, 1), (1, 1, 4, 4)),
]


def _plan(shape, workspace_free=False):
    return im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=workspace_free)["kernel"]


def _run(shape, I, F):
    """Output of both calls (with guards around each), and of the fp32 kernel."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    n = N * Co * Ho * Wo
    dW, dI, dF = run_transform(I, Hf, Wf, s, p), I.cuda(), F.cuda()
    buf = torch.full((4, n + 64), float("nan"), device="cuda")
    outs = [b[32:32 + n] for b in buf]
    print("stem pieces", shape, _plan(shape), flush=True)
    im2win.conv2d_im2win_fwd(dW, dF, outs[0], *shape)
    im2win.conv2d_im2win_fwd(dW, dF, outs[1], *shape)
    im2win.conv2d_im2win_implicit_fwd(dI, dF, outs[2], *shape)
    im2win.conv2d_im2win_fwd_variant(dW, dF, outs[3], *shape, im2win.VARIANT_NO_PIPELINE)
    torch.cuda.synchronize()
    assert torch.isnan(buf[:, :32]).all() and torch.isnan(buf[:, 32 + n:]).all()   # nothing written outside
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))       # no races on LDS
    assert torch.equal(outs[0].view(torch.int32), outs[2].view(torch.int32))       # same pieces, same order
    return outs[0].cpu().numpy().reshape(N, Co, Ho, Wo), outs[3].cpu().numpy().reshape(N, Co, Ho, Wo)


@pytest.mark.parametrize("shape,instance", SHAPES, ids=lambda v: "x".join(map(str, v)))
def test_both_calls(shape, instance):
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(9700 + sum(shape), N, Ci, Hi, Wi, Co, Hf, Wf)
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    got, fp32 = _run(shape, I, F)
    assert_conv_close(got, O_ref, B_ref)
    l2, l2_32 = conv_errors(got, O_ref, B_ref)[1], conv_errors(fp32, O_ref, B_ref)[1]
    print("relative L2 error: pieces %.2e, fp32 %.2e" % (l2, l2_32))
    assert l2 <= l2_32


@pytest.mark.parametrize("ei,ef", [(-118, 4), (4, -124), (-140, 20), (105, 0), (-120, 120), (60, 60)])
@pytest.mark.parametrize("shape", [SHAPES[4][0], SHAPES[6][0], SHAPES[12][0], SHAPES[17][0]], ids=lambda v: "x".join(map(str, v)))
def test_no_operand_loses_bits(shape, ei, ef):
    """The 24 bits of an operand hold whatever its magnitude: against 64 bits no further off than the fp32 kernel."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(9800, N, Ci, Hi, Wi, Co, Hf, Wf)
    I, F = torch.ldexp(I.double(), torch.tensor(ei)).float(), torch.ldexp(F.double(), torch.tensor(ef)).float()
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    got, fp32 = _run(shape, I, F)
    assert conv_errors(got, O_ref, B_ref)[1] <= 1.1 * conv_errors(fp32, O_ref, B_ref)[1]


@pytest.mark.parametrize("shape", [SHAPES[0][0], SHAPES[4][0], SHAPES[8][0], SHAPES[12][0], SHAPES[16][0], SHAPES[18][0]], ids=lambda v: "x".join(map(str, v)))
def test_infinities_nan_and_the_ends_of_the_range(shape):
    """As in plain fp32 (the one-thread-per-output kernel), in both calls: also beside windows (the padded parts of a chunk hold zeros)."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(9900, N, Ci, Hi, Wi, Co, Hf, Wf)
    I.abs_()                                 # (weights of 2^50 on both signs would cancel: 1e-4 of the result is not 1e-4 of the magnitudes)
    low = torch.finfo(torch.float32).min
    I[0, 2, 10, 10] = float("inf")
    I[1, 1, 0, Wi - 1] = float("-inf")
    I[2, 0, Hi - 1, 0] = float("nan")
    I[3, 1, 20, 20] = 3.4028e38              # rounds to infinity in bf16
    I[4, 2, 5, 5], I[4, 0, 6, 6] = float("inf"), float("-inf")
    I[5, 2, 31, 17] = low                    # a mask
    I[6, 1, 33, 40] = 2.0 ** 60
    I[7, 0, 12, 13] = torch.tensor([0x7F800001], dtype=torch.int32).view(torch.float32)[0]
    F[:, 2] *= 0.25
    F[2, 2] = 0.0                            # infinity and the mask times zero
    F[3, 2] = 2.0 ** -140
    F[4, 1] = 2.0 ** 50                      # a sum past 2^96
    ref = _assert_like_basic(shape, I, F)
    assert torch.isnan(ref).any() and torch.isinf(ref).any()


@pytest.mark.parametrize("shape", [SHAPES[i][0] for i in (0, 2, 4, 6, 8, 10, 12, 14, 16, 18)], ids=lambda v: "x".join(map(str, v)))
def test_buffers_of_any_alignment(shape):
    check_any_alignment(shape, 9945)


@pytest.mark.parametrize("shape", [q[0] for q in SHAPES], ids=lambda v: "x".join(map(str, v)))
def test_the_second_pass_writes_what_the_first_left(shape):
    check_second_pass(shape, 9940)


@pytest.mark.parametrize("shape", [SHAPES[17][0], SHAPES[18][0], (512, 3, 36, 36, 32, 3, 3, 1, 0), (300, 3, 42, 42, 16, 3, 3, 1, 1),
                                   (150, 3, 64, 59, 67, 3, 3, 1, 1)], ids=lambda v: "x".join(map(str, v)))
def test_an_output_off_16_byte_alignment(shape):
    """The same kernel whatever the alignment, so the same bits: on images that the stem kernel takes and on narrower ones, where its tile
    of 512 pixels has too many rows."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    assert _plan(shape).startswith("conv_split_stem_kernel<3, 1, 1, 4, 4" if Wo > 42 else "conv_mfma_shallow_kernel")
    assert Ho * Wo % 4 == 0 and N * Ho * Wo >= 2048 * 256
    I, F = workloads.random_layer_inputs(9990, N, Ci, Hi, Wi, Co, Hf, Wf)
    n = N * Co * Ho * Wo
    dI, dW, dF = I.cuda(), run_transform(I, Hf, Wf, s, p), F.cuda()
    buf = torch.full((3, n + 96), float("nan"), device="cuda")
    outs = [buf[a, 32 + a:][:n] for a in range(3)]
    assert (n + 96) % 4 == 0 and [o.data_ptr() % 16 for o in outs] == [0, 4, 8]
    for call, source in ((im2win.conv2d_im2win_fwd, dW), (im2win.conv2d_im2win_implicit_fwd, dI)):
        for o in outs:
            call(source, dF, o, *shape)
        torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all()
        for a, o in enumerate(outs):
            assert torch.equal(outs[0].view(torch.int32), o.view(torch.int32)), a
            assert torch.isnan(buf[a, :32 + a]).all() and torch.isnan(buf[a, 32 + a + n:]).all()   # nothing written outside
