"""The filter-stationary fp32 kernel of three-channel layers: every instance the dispatch selects (test_split_dispatch.py holds the list to
that) at ragged sizes through both calls."""
import pytest
import torch

import oracle
import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import workloads
from parity_util import assert_conv_close, run_transform

pytestmark = pytest.mark.gpu

# (N, Ci, Hi, Wi, Co, Hf, Wf, s, p) and the instance: blocks of 32 channels, parts of K, strip words per thread, runs of 64 pixels per
# tile, 16-byte stores
SHAPES = [
    ((13, 3, 62, 42, 24, 7, 7, 1, 1), (1, 1, 8, 1, False)),
    ((1, 3, 113, 141, 20, 7, 7, 2, 3), (1, 1, 8, 1, False)),      # stride 2: small layers only
    ((3, 3, 115, 113, 33, 7, 7, 1, 1), (2, 1, 4, 1, False)),      # one channel past a block
    ((1, 3, 130, 99, 64, 7, 7, 2, 2), (2, 1, 4, 1, False)),
    ((2, 3, 61, 75, 97, 7, 7, 1, 3), (3, 1, 3, 1, False)),        # two groups of channels
    ((1, 3, 40, 260, 96, 7, 7, 1, 8), (3, 1, 3, 1, False)),       # padding wider than the filter
    ((4, 3, 60, 100, 20, 11, 11, 2, 3), (1, 2, 12, 1, False)),
    ((2, 3, 57, 85, 64, 11, 11, 1, 0), (2, 2, 6, 1, False)),
    ((3, 3, 53, 131, 97, 11, 11, 3, 4), (3, 2, 4, 1, False)),
    ((1, 3, 75, 135, 24, 3, 3, 1, 1), (1, 1, 2, 1, False)),
    ((3, 3, 84, 77, 64, 3, 3, 1, 1), (2, 1, 1, 1, False)),
    ((5, 3, 40, 67, 97, 3, 3, 1, 0), (3, 1, 1, 1, False)),
    ((60, 3, 103, 133, 20, 3, 3, 1, 0), (1, 1, 7, 4, False)),     # planes of an odd number of pixels
    ((48, 3, 130, 132, 97, 3, 3, 1, 0), (1, 1, 7, 4, True)),      # groups of one block, the last with one channel
    ((60, 3, 103, 133, 50, 3, 3, 1, 0), (2, 1, 4, 4, False)),
    ((48, 3, 130, 132, 64, 3, 3, 1, 0), (2, 1, 4, 4, True)),
]


def instance_name(Hf, instance, workspace_free):
    wm, ks, jx, g, wide = instance
    return "conv_mfma_shallow_kernel<%d, %d, 3, %d, %d, %d, %s, %d, %s>" % (
        Hf, Hf, wm, ks, jx, "true" if workspace_free else "false", g, "true" if wide else "false")


@pytest.mark.parametrize("shape,instance", SHAPES, ids=lambda v: "x".join(map(str, v)))
def test_both_calls(shape, instance):
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(9600 + sum(shape), N, Ci, Hi, Wi, Co, Hf, Wf)
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    n = N * Co * Ho * Wo
    dI, dW, dF = I.cuda(), run_transform(I, Hf, Wf, s, p), F.cuda()
    buf = torch.full((3, n + 64), float("nan"), device="cuda")
    outs = [b[32:32 + n] for b in buf]
    print("shallow", shape, instance, flush=True)
    im2win.conv2d_im2win_fwd(dW, dF, outs[0], *shape)
    im2win.conv2d_im2win_fwd(dW, dF, outs[1], *shape)
    im2win.conv2d_im2win_implicit_fwd(dI, dF, outs[2], *shape)
    torch.cuda.synchronize()
    assert torch.isnan(buf[:, :32]).all() and torch.isnan(buf[:, 32 + n:]).all()   # nothing written outside
    assert torch.isfinite(outs[0]).all()
    for o in outs[1:]:
        assert torch.equal(outs[0].view(torch.int32), o.view(torch.int32))         # no races on LDS; same order in both calls
    some = sorted({0, N // 2, N - 1})   # (images are independent: three of them go through the oracle)
    O_ref, B_ref = oracle.conv2d_direct(I[some].numpy(), F.numpy(), s, p)
    assert_conv_close(outs[0].reshape(N, Co, Ho, Wo)[some].cpu().numpy(), O_ref, B_ref)
