"""Shared helpers for the GPU parity tests: run the library through its C ABI
on device tensors and compare with the CPU oracle."""
import numpy as np
import torch

import oracle
import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import workloads

# Acceptance bar for the fp32 convolution (fp32 multiply/accumulate on the
# matrix cores, any summation order) against the fp64 oracle:
#   every element: |O_gpu - O_ref| <= 1e-4 * sum|x||w|   and   relative L2 <= 1e-5.
# The expected error is about sqrt(K)*2^-24 relative (3e-6 at K = 2304).
ELEM_TOL = 1e-4
L2_TOL = 1e-5

POISON = float("nan")


def run_transform(I, Hf, Wf, s, p):
    N, Ci, Hi, Wi = I.shape
    Ho, _ = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    dI = I.cuda()
    dW = torch.full((N, Ci, Ho, (Wi + 2 * p) * Hf), POISON, dtype=torch.float32, device="cuda")
    im2win.im2win_transform(dI, dW, N, Ci, Hi, Wi, Hf, Wf, s, p)
    torch.cuda.synchronize()
    return dW


def run_conv(dW, F, N, Ci, Hi, Wi, s, p, basic=False):
    Co, _, Hf, Wf = F.shape
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    dF = F.cuda()
    dO = torch.full((N, Co, Ho, Wo), POISON, dtype=torch.float32, device="cuda")
    fn = im2win.conv2d_im2win_fwd_basic if basic else im2win.conv2d_im2win_fwd
    fn(dW, dF, dO, N, Ci, Hi, Wi, Co, Hf, Wf, s, p)
    torch.cuda.synchronize()
    return dO


def assert_bitwise_equal(dW, W_ref):
    got = dW.cpu().numpy().view(np.uint32)
    want = np.ascontiguousarray(W_ref).view(np.uint32)
    assert got.shape == want.shape
    if not np.array_equal(got, want):
        bad = np.argwhere(got != want)
        raise AssertionError("im2win tensor differs at %d of %d words, first at %s"
                             % (len(bad), got.size, bad[0]))


def conv_errors(O_gpu, O_ref, B_ref):
    """(max |err| / sum|x||w|, relative L2 error); O_gpu fp32 array, references fp64."""
    got = np.asarray(O_gpu, dtype=np.float64)
    assert got.shape == O_ref.shape
    assert np.isfinite(got).all(), "output holds NaN/Inf (an element was never written?)"
    err = np.abs(got - O_ref)
    scale = np.where(B_ref > 0, B_ref, 1.0)
    elem = float((err / scale).max())
    # where the bound is zero every term is zero and the output must be exactly zero
    assert not err[B_ref == 0].any()
    l2 = float(np.sqrt((err ** 2).sum()) / max(np.sqrt((O_ref ** 2).sum()), 1e-300))
    return elem, l2


def assert_conv_close(O_gpu, O_ref, B_ref):
    elem, l2 = conv_errors(O_gpu, O_ref, B_ref)
    assert elem <= ELEM_TOL, "max |err|/sum|x||w| = %.3e" % elem
    assert l2 <= L2_TOL, "relative L2 error = %.3e" % l2
    return elem, l2


def check_layer(I, F, s, p, basic=False, twice=True):
    """Transform + convolution of one layer against the oracle; returns the error norms."""
    N, Ci, Hi, Wi = I.shape
    Co, _, Hf, Wf = F.shape
    In, Fn = I.numpy(), F.numpy()
    dW = run_transform(I, Hf, Wf, s, p)
    assert_bitwise_equal(dW, oracle.im2win(In, Hf, Wf, s, p))
    O_ref, B_ref = oracle.conv2d_direct(In, Fn, s, p)
    dO = run_conv(dW, F, N, Ci, Hi, Wi, s, p, basic=basic)
    res = assert_conv_close(dO.cpu().numpy(), O_ref, B_ref)
    if twice:   # a second run must reproduce the first bit for bit (no races on LDS)
        dO2 = run_conv(dW, F, N, Ci, Hi, Wi, s, p, basic=basic)
        assert torch.equal(dO.view(torch.int32), dO2.view(torch.int32))
    return res


def _both_calls(shape, I, F):
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    dW, dI, dF = run_transform(I, Hf, Wf, s, p), I.cuda(), F.cuda()
    outs = torch.full((2, N, Co, Ho, Wo), 7.0, device="cuda")
    im2win.conv2d_im2win_fwd(dW, dF, outs[0], *shape)
    im2win.conv2d_im2win_implicit_fwd(dI, dF, outs[1], *shape)
    torch.cuda.synchronize()
    return outs


def check_second_pass(shape, seed):
    """The second pass writes the outputs that the first left infinite or NaN, of all channels or of some, and no other.  Inputs times
    2^100 take every sum of order one through it: the pieces, the products and their sums are the same, so the bits are."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    I, F = workloads.random_layer_inputs(seed, N, Ci, Hi, Wi, Co, Hf, Wf)
    print("second pass", shape, im2win.conv2d_im2win_fwd_launch_info(*shape)["kernel"], flush=True)
    plain = _both_calls(shape, I, F)
    assert torch.isfinite(plain).all()
    large = _both_calls(shape, torch.ldexp(I, torch.tensor(100)), F)
    assert torch.equal(large, torch.ldexp(plain, torch.tensor(100, device="cuda")))
    I2, F2 = I.clone(), F.clone()
    I2[N // 2], F2[1::3, 0, 0, Wf - 1] = float("nan"), float("nan")   # one image, a third of the channels
    some = _both_calls(shape, I2, F2)
    want = plain.clone()
    want[:, N // 2] = float("nan")
    want[:, :, 1::3] = float("nan")
    if p >= Hf:   # windows of padding only
        want[:, N // 2] = torch.where(_touched(shape), want[:, N // 2], plain[:, N // 2])
        want[:, N // 2, 1::3] = float("nan")
    assert torch.equal(torch.isnan(some), torch.isnan(want))
    assert torch.equal(some[~torch.isnan(want)].view(torch.int32), plain[~torch.isnan(want)].view(torch.int32))


def _touched(shape):
    """Outputs whose window meets the image."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    ones = torch.nn.functional.conv2d(torch.ones(1, 1, Hi, Wi), torch.ones(1, 1, Hf, Wf), stride=s, padding=p)
    return (ones[0, 0] > 0).cuda()


def check_any_alignment(shape, seed):
    """Buffers at every multiple of four bytes give the bits of aligned ones, and nothing is written outside the output."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    n = N * Co * Ho * Wo
    I, F = workloads.random_layer_inputs(seed, N, Ci, Hi, Wi, Co, Hf, Wf)
    dI, dF, dW = I.cuda(), F.cuda(), run_transform(I, Hf, Wf, s, p)

    def shifted(t, words):
        buf = torch.full((t.numel() + words + 1,), float("nan"), device="cuda")   # (NaN around: a word from outside would show)
        buf[words:words + t.numel()] = t.flatten()
        assert buf.data_ptr() % 16 == 0
        return buf[words:words + t.numel()]

    print("alignment", shape, im2win.conv2d_im2win_fwd_launch_info(*shape)["kernel"], flush=True)
    for call, src in ((im2win.conv2d_im2win_fwd, dW), (im2win.conv2d_im2win_implicit_fwd, dI)):
        want = None
        for a, b, c in ((0, 0, 0), (1, 2, 3), (2, 3, 1), (3, 1, 2)):
            out = torch.full((n + 68,), 7.0, device="cuda")
            got = out[32 + c:32 + c + n]
            call(shifted(src, a), shifted(dF, b), got, *shape)
            torch.cuda.synchronize()
            assert (out[:32 + c] == 7.0).all() and (out[32 + c + n:] == 7.0).all()
            want = got.clone() if want is None else want
            assert torch.isfinite(got).all() and torch.equal(got.view(torch.int32), want.view(torch.int32)), (a, b, c)
