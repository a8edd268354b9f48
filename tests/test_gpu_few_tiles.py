"""Layers of few tiles on the fp32 matrix cores: quarter tiles, and ragged channel counts in half tiles, at the edges of tiles, K blocks and
planes through both calls, against the oracle."""
import pytest
import torch

import oracle
import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import workloads
from parity_util import assert_conv_close, conv_errors, run_transform

pytestmark = pytest.mark.gpu

# (N, Ci, Hi, Wi, Co, Hf, Wf, s, p) and the kernel of the two-call path, which test_split_dispatch.py holds the dispatch to
SHAPES = [
    ((1, 64, 56, 56, 64, 3, 3, 1, 1), "conv_mfma_quarter_kernel<3, 3, 8, 1, false, false>"),
    ((1, 8, 40, 47, 97, 3, 3, 1, 0), "conv_mfma_quarter_kernel<3, 3, 8, 1, false, false>"),    # one K block; one channel and 14 pixels past a tile
    ((1, 9, 33, 33, 31, 3, 3, 1, 1), "conv_mfma_quarter_kernel<3, 3, 8, 1, false, true>"),     # one channel in the last K block, one channel short of a tile
    ((2, 31, 29, 30, 70, 3, 3, 1, 2), "conv_mfma_quarter_kernel<3, 3, 8, 1, false, true>"),    # a tile spans two images
    ((19, 23, 7, 6, 40, 3, 3, 1, 0), "conv_mfma_quarter_kernel<3, 3, 8, 2, false, true>"),     # planes of 20 pixels
    ((3, 24, 40, 33, 33, 3, 3, 2, 1), "conv_mfma_quarter_kernel<3, 3, 8, 2, false, false>"),   # stride 2: two strip words per thread
    ((1, 12, 7, 180, 20, 3, 3, 2, 0), "conv_mfma_quarter_kernel<3, 3, 8, 2, false, true>"),
    ((1, 48, 3, 3, 5, 3, 3, 1, 3), "conv_mfma_fast_kernel<3, 3, 8, 1, 4, 3, false, false, true, false, false>"),   # one tile: sixteenths
    ((1, 33, 3, 3, 5, 3, 3, 1, 3), "conv_mfma_quarter_kernel<3, 3, 8, 1, false, true>"),       # padding as wide as the filter: windows of zeros
    ((1, 3, 32, 32, 16, 3, 3, 1, 0), "conv_mfma_quarter_kernel<3, 3, 8, 1, false, true>"),     # less than a K block
    ((2, 1, 28, 27, 33, 3, 3, 1, 1), "conv_mfma_quarter_kernel<3, 3, 8, 1, false, true>"),
    ((1, 7, 31, 30, 20, 3, 3, 2, 1), "conv_mfma_quarter_kernel<3, 3, 8, 2, false, true>"),
    ((2, 10, 20, 33, 40, 5, 5, 1, 1), "conv_mfma_quarter_kernel<5, 5, 8, 2, false, true>"),    # two channels in the last K block
    ((1, 16, 19, 90, 33, 5, 5, 1, 4), "conv_mfma_quarter_kernel<5, 5, 8, 2, false, false>"),
    ((1, 17, 21, 90, 33, 5, 5, 1, 0), "conv_mfma_quarter_kernel<5, 5, 8, 2, false, true>"),
    ((2, 8, 24, 100, 40, 5, 5, 2, 2), "conv_mfma_quarter_kernel<5, 5, 8, 3, false, false>"),
    ((2, 31, 24, 50, 63, 5, 5, 2, 2), "conv_mfma_quarter_kernel<5, 5, 8, 3, false, true>"),
    ((1, 24, 30, 41, 65, 5, 5, 1, 2), "conv_mfma_quarter_kernel<5, 5, 8, 2, false, false>"),
    ((1, 9, 24, 21, 33, 4, 4, 1, 0), "conv_mfma_quarter_kernel<4, 4, 8, 2, false, true>"),
    ((1, 24, 27, 31, 70, 4, 4, 1, 3), "conv_mfma_quarter_kernel<4, 4, 8, 2, false, false>"),
    ((1, 16, 17, 60, 20, 4, 4, 2, 1), "conv_mfma_quarter_kernel<4, 4, 8, 3, false, false>"),
    ((3, 23, 17, 60, 20, 4, 4, 2, 1), "conv_mfma_quarter_kernel<4, 4, 8, 3, false, true>"),
    ((2, 100, 45, 45, 120, 3, 3, 1, 1), "conv_mfma_fast_kernel<3, 3, 8, 1, 4, 2, false, false, false, true, true>"),
    ((3, 13, 50, 47, 120, 3, 3, 2, 1), "conv_mfma_quarter_kernel<3, 3, 8, 2, false, true>"),
    ((5, 20, 63, 44, 70, 3, 3, 2, 1), "conv_mfma_fast_kernel<3, 3, 8, 2, 4, 2, false, false, false, true, true>"),
    ((3, 13, 28, 29, 100, 5, 5, 1, 2), "conv_mfma_fast_kernel<5, 5, 4, 2, 4, 2, false, false, false, true, true>"),
    ((2, 7, 41, 90, 66, 5, 5, 2, 0), "conv_mfma_fast_kernel<5, 5, 4, 3, 4, 2, false, false, false, true, true>"),
]


@pytest.mark.parametrize("shape,kernel", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_both_calls(shape, kernel):
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(8800 + sum(shape), N, Ci, Hi, Wi, Co, Hf, Wf)
    print("few tiles", shape, kernel, flush=True)
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    n = O_ref.size
    dW, dI, dF = run_transform(I, Hf, Wf, s, p), I.cuda(), F.cuda()
    buf = torch.full((4, n + 64), float("nan"), dtype=torch.float32, device="cuda")
    outs = [b[32:32 + n] for b in buf]
    im2win.conv2d_im2win_fwd(dW, dF, outs[0], *shape)
    im2win.conv2d_im2win_fwd(dW, dF, outs[1], *shape)
    im2win.conv2d_im2win_implicit_fwd(dI, dF, outs[2], *shape)
    im2win.conv2d_im2win_fwd_variant(dW, dF, outs[3], *shape, im2win.VARIANT_NO_PIPELINE)
    torch.cuda.synchronize()
    assert torch.isnan(buf[:, :32]).all() and torch.isnan(buf[:, 32 + n:]).all()   # nothing written outside
    got, whole = (o.cpu().numpy().reshape(O_ref.shape) for o in (outs[0], outs[3]))
    assert_conv_close(got, O_ref, B_ref)
    # partial sums of a half or a quarter of the channels: no further off than one chain over all of them
    assert conv_errors(got, O_ref, B_ref)[1] <= 1.05 * conv_errors(whole, O_ref, B_ref)[1]
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))   # no races on LDS
    assert torch.equal(outs[0].view(torch.int32), outs[2].view(torch.int32))   # same strips, same order


@pytest.mark.parametrize("shape", [SHAPES[0][0], SHAPES[3][0], (2, 3, 20, 21, 16, 3, 3, 1, 0)], ids=lambda v: "x".join(map(str, v)))
def test_words_beyond_the_channels_are_not_used(shape):
    """The planes and filter rows behind the last channel's are the next image's and the next output channel's: with NaN there, an image or a
    channel of ordinary data stays ordinary, and only its neighbours are NaN."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(8900, N, Ci, Hi, Wi, Co, Hf, Wf)
    F[1] = float("nan")
    if N > 1:
        I[1] = float("nan")
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    outs = torch.zeros((2, N, Co, Ho, Wo), device="cuda")
    im2win.conv2d_im2win_fwd(run_transform(I, Hf, Wf, s, p), F.cuda(), outs[0], *shape)
    im2win.conv2d_im2win_implicit_fwd(I.cuda(), F.cuda(), outs[1], *shape)
    torch.cuda.synchronize()
    for o in outs:
        assert torch.isfinite(o[0, 0]).all() and torch.isfinite(o[0, 2:]).all() and torch.isnan(o[0, 1]).all()


@pytest.mark.parametrize("shape", [SHAPES[2][0], SHAPES[5][0]], ids=lambda v: "x".join(map(str, v)))
def test_outputs_of_any_alignment(shape):
    """Sources and outputs at every multiple of four bytes (the filter, whose alignment chooses the kernel, stays)."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(8950, N, Ci, Hi, Wi, Co, Hf, Wf)
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    n, dF = N * Co * Ho * Wo, F.cuda()
    want = None
    for words in range(4):
        for call, src in ((im2win.conv2d_im2win_fwd, run_transform(I, Hf, Wf, s, p)), (im2win.conv2d_im2win_implicit_fwd, I.cuda())):
            buf = torch.full((src.numel() + words + 1,), float("nan"), device="cuda")
            buf[words:words + src.numel()] = src.flatten()
            out = torch.full((n + words + 1,), float("nan"), device="cuda")
            call(buf[words:words + src.numel()], dF, out[words:words + n], *shape)
            torch.cuda.synchronize()
            got = out[words:words + n].clone()
            want = got if want is None else want
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)) and torch.isnan(out[:words]).all() and torch.isnan(out[words + n:]).all()
