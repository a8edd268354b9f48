"""The bf16-piece kernels: every instance the dispatch selects (test_split_dispatch.py holds the list to that), at ragged
channel, row and pixel counts, through both calls; precision; infinities and NaN."""
import numpy as np
import pytest
import torch

import oracle
import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import workloads
from parity_util import assert_conv_close, check_any_alignment, check_second_pass, conv_errors, run_conv, run_transform

pytestmark = pytest.mark.gpu


def _split(shape, workspace_free=False):
    return im2win.conv2d_im2win_fwd_launch_info(*shape, workspace_free=workspace_free)["kernel"].startswith("conv_split_kernel<")


# (N, Ci, Hi, Wi, Co, Hf, Wf, s, p) and the configuration, which test_split_dispatch.py holds the dispatch to (0 / 1 / 4: long filter stages, tiles of 64 x 256 / 64 x 128 / 32 x 256; 2 and 3:
# 64 x 256 with larger patches): every instance at channel counts off its K block and tile, with padding, on short images (a tile spans several)
# and at the strides it takes
SHAPES = [
    ((54, 404, 61, 6, 100, 1, 3, 1, 0), 1),
    ((26, 283, 23, 16, 20, 1, 3, 1, 4), 1),
    ((99, 298, 7, 31, 20, 1, 3, 1, 0), 1),
    ((22, 100, 50, 59, 128, 1, 3, 1, 0), 3),
    ((68, 131, 8, 116, 20, 1, 3, 1, 0), 4),
    ((17, 100, 44, 39, 33, 1, 7, 1, 3), 0),
    ((78, 63, 6, 89, 20, 1, 7, 1, 0), 4),
    ((6, 128, 57, 51, 32, 1, 7, 1, 1), 4),
    ((66, 232, 9, 38, 20, 1, 7, 1, 0), 4),
    ((14, 128, 41, 60, 65, 1, 7, 2, 1), 1),   # a stride wider than the filter is high: rows between the windows
    ((114, 126, 7, 70, 20, 1, 7, 2, 1), 1),
    ((49, 109, 94, 6, 20, 1, 7, 1, 4), 4),
    ((83, 506, 7, 26, 20, 3, 1, 1, 2), 1),
    ((113, 252, 10, 7, 20, 3, 1, 1, 3), 1),
    ((41, 282, 9, 52, 33, 3, 1, 1, 1), 1),
    ((52, 303, 19, 6, 20, 3, 1, 1, 4), 1),
    ((13, 128, 52, 28, 65, 3, 1, 1, 2), 3),
    ((106, 93, 10, 65, 20, 3, 1, 1, 0), 4),
    ((16, 32, 43, 50, 65, 3, 3, 1, 0), 0),   # one channel past a tile, two K blocks
    ((17, 100, 56, 38, 33, 3, 3, 1, 2), 0),   # a last K block of 4 channels, padding
    ((22, 100, 44, 11, 65, 3, 3, 1, 3), 4),   # padding as wide as the filter: windows of zeros
    ((23, 128, 53, 21, 32, 3, 3, 1, 1), 4),
    ((22, 40, 16, 58, 65, 3, 3, 1, 3), 2),   # 8 channels at a time: an odd tap against zero pixels
    ((42, 40, 8, 119, 65, 3, 3, 1, 0), 2),
    ((24, 128, 21, 48, 65, 3, 3, 1, 0), 4),
    ((80, 44, 9, 76, 20, 3, 3, 1, 1), 4),
    ((23, 16, 46, 38, 33, 4, 4, 1, 4), 0),
    ((38, 38, 12, 124, 20, 4, 4, 1, 0), 4),
    ((11, 47, 32, 62, 20, 4, 4, 1, 2), 1),
    ((19, 64, 59, 51, 33, 4, 4, 2, 4), 1),
    ((65, 60, 14, 105, 20, 4, 4, 2, 0), 1),
    ((107, 48, 9, 44, 65, 4, 4, 2, 2), 1),
    ((64, 63, 56, 51, 20, 4, 4, 3, 2), 1),
    ((119, 75, 15, 68, 20, 4, 4, 3, 4), 1),
    ((24, 32, 48, 50, 65, 4, 4, 2, 4), 4),
    ((65, 24, 14, 113, 65, 4, 4, 2, 2), 3),
    ((1, 46, 98, 114, 130, 5, 5, 1, 4), 4),
    ((11, 32, 46, 32, 32, 5, 5, 1, 3), 4),
    ((54, 45, 9, 41, 33, 5, 5, 1, 2), 4),
    ((11, 40, 60, 36, 65, 5, 5, 1, 0), 4),
    ((21, 8, 59, 57, 65, 5, 5, 1, 4), 2),   # one K block per tile
    ((21, 16, 47, 38, 32, 5, 5, 1, 3), 4),
    ((65, 16, 7, 70, 20, 5, 5, 1, 3), 4),
    ((17, 42, 42, 78, 20, 7, 1, 1, 2), 4),
    ((19, 64, 31, 49, 33, 7, 1, 1, 4), 0),
    ((2, 139, 102, 80, 20, 7, 1, 1, 3), 4),
    ((26, 120, 9, 78, 20, 7, 1, 1, 3), 4),
    ((31, 144, 5, 51, 65, 7, 1, 1, 3), 1),
    ((21, 128, 60, 49, 32, 7, 1, 2, 2), 1),
    ((49, 107, 86, 23, 20, 7, 1, 2, 1), 1),
    ((10, 42, 75, 58, 20, 7, 1, 1, 4), 4),
    ((94, 43, 8, 66, 20, 7, 1, 1, 3), 4),
    ((19, 8, 55, 49, 32, 7, 7, 1, 1), 4),
    ((83, 14, 11, 60, 65, 7, 7, 1, 2), 4),
    ((20, 40, 52, 8, 65, 7, 7, 1, 3), 4),
    ((91, 16, 5, 53, 20, 7, 7, 1, 3), 4),
    ((21, 40, 55, 26, 65, 7, 7, 2, 4), 1),   # stride 2
    ((24, 16, 42, 43, 65, 7, 7, 2, 2), 1),
    ((58, 34, 87, 52, 20, 7, 7, 3, 1), 1),
    ((81, 8, 12, 100, 20, 7, 7, 1, 0), 4),
    ((48, 7, 39, 96, 33, 7, 7, 2, 4), 3),
    ((67, 18, 27, 81, 20, 7, 7, 2, 4), 3),
    # strips of unequal width, the last with fewer tiles than the others (5, 7 and 3 strips; 43 tiles of 49, 12 of 15, 28 of 31)
    ((38, 33, 22, 73, 65, 3, 3, 1, 1), 4),
    ((11, 18, 23, 102, 65, 5, 5, 1, 2), 2),
    ((22, 18, 49, 81, 65, 7, 7, 2, 3), 3),
    ((1, 9, 105, 121, 200, 5, 5, 1, 2), 0),
    ((1, 13, 97, 69, 300, 5, 5, 1, 2), 0),
    ((62, 120, 41, 21, 64, 1, 3, 1, 4), 1),
    ((65, 113, 12, 20, 33, 1, 3, 1, 1), 1),
    ((69, 128, 5, 90, 64, 1, 3, 1, 1), 3),
    ((15, 65, 70, 31, 65, 1, 7, 1, 0), 0),
    ((45, 68, 10, 36, 100, 1, 7, 1, 0), 1),
    ((39, 15, 50, 6, 130, 1, 7, 1, 4), 3),
    ((33, 35, 60, 14, 200, 1, 7, 1, 0), 3),
    ((2, 124, 5, 9, 100, 3, 1, 3, 0), 1),
    ((49, 239, 42, 13, 33, 3, 1, 1, 1), 1),
    ((37, 99, 26, 117, 33, 3, 1, 1, 2), 3),
    ((14, 184, 45, 46, 130, 3, 1, 1, 0), 3),
    ((40, 47, 42, 18, 64, 3, 3, 1, 0), 1),
    ((7, 78, 24, 30, 300, 3, 3, 1, 2), 1),
    ((6, 31, 8, 5, 65, 3, 3, 3, 1), 1),
    ((50, 10, 8, 50, 200, 3, 3, 1, 0), 3),
    ((43, 14, 16, 103, 64, 3, 3, 1, 0), 3),
    ((36, 65, 44, 12, 130, 3, 3, 1, 2), 4),
    ((2, 60, 6, 12, 20, 3, 3, 3, 0), 1),
    ((23, 30, 54, 18, 130, 4, 4, 1, 0), 0),
    ((51, 21, 19, 112, 200, 4, 4, 2, 2), 3),
    ((8, 24, 5, 39, 64, 4, 4, 3, 0), 1),
    ((9, 81, 60, 8, 100, 5, 5, 2, 4), 1),
    ((1, 15, 25, 6, 300, 5, 5, 3, 3), 4),
    ((11, 18, 41, 92, 33, 5, 5, 1, 4), 2),
    ((31, 11, 30, 31, 65, 5, 5, 1, 1), 3),
    ((43, 42, 27, 32, 33, 5, 5, 1, 2), 3),
    ((1, 30, 12, 9, 64, 5, 5, 2, 1), 4),
    ((26, 37, 39, 100, 64, 7, 1, 1, 2), 0),
    ((83, 47, 27, 26, 33, 7, 1, 1, 0), 3),
    ((9, 57, 47, 59, 65, 7, 1, 1, 1), 3),
    ((13, 7, 38, 64, 33, 7, 7, 1, 4), 0),
    ((83, 12, 12, 32, 65, 7, 7, 1, 2), 0),
    ((8, 95, 9, 57, 200, 7, 7, 2, 0), 3),
    ((54, 15, 37, 22, 200, 7, 7, 2, 1), 3),
    ((2, 8, 47, 11, 20, 7, 7, 3, 0), 4),
    ((1, 114, 17, 22, 200, 7, 7, 2, 3), 4),
]


OTHER_SHAPES = [(7, 78, 24, 30, 300, 3, 3, 1, 2), (43, 14, 16, 103, 64, 3, 3, 1, 0), (83, 47, 27, 26, 33, 7, 1, 1, 0)]   # narrow tiles, larger patches


@pytest.mark.parametrize("shape,cfg", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_both_calls(shape, cfg):
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    name = im2win.conv2d_im2win_fwd_launch_info(*shape)["kernel"]
    I, F = workloads.random_layer_inputs(9100 + sum(shape), N, Ci, Hi, Wi, Co, Hf, Wf)
    print("pieces", shape, name, flush=True)
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    n = O_ref.size
    dW, dI, dF = run_transform(I, Hf, Wf, s, p), I.cuda(), F.cuda()
    buf = torch.full((3, n + 64), float("nan"), dtype=torch.float32, device="cuda")
    outs = [b[32:32 + n] for b in buf]
    im2win.conv2d_im2win_fwd(dW, dF, outs[0], *shape)
    im2win.conv2d_im2win_fwd(dW, dF, outs[1], *shape)
    im2win.conv2d_im2win_implicit_fwd(dI, dF, outs[2], *shape)
    torch.cuda.synchronize()
    assert torch.isnan(buf[:, :32]).all() and torch.isnan(buf[:, 32 + n:]).all()   # nothing written outside
    assert_conv_close(outs[0].cpu().numpy().reshape(O_ref.shape), O_ref, B_ref)
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))   # no races on LDS
    assert torch.equal(outs[0].view(torch.int32), outs[2].view(torch.int32))   # same pieces, same order


def test_an_image_beyond_the_fp32_pipeline():
    """Strips of more than 4 GiB, which the fp32 pipeline turns away: both calls run the piece kernel; the first and last rows
    in full, sampled outputs elsewhere."""
    shape = N, Ci, Hi, Wi, Co, Hf, Wf, s, p = (1, 64, 1400, 1400, 33, 3, 3, 1, 0)
    assert _split(shape) and _split(shape, True)
    I, F = workloads.random_layer_inputs(9600, N, Ci, Hi, Wi, Co, Hf, Wf)
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    dO = run_conv(run_transform(I, Hf, Wf, s, p), F, N, Ci, Hi, Wi, s, p)
    dO2 = torch.full_like(dO, float("nan"))
    im2win.conv2d_im2win_implicit_fwd(I.cuda(), F.cuda(), dO2, *shape)
    torch.cuda.synchronize()
    assert torch.equal(dO.view(torch.int32), dO2.view(torch.int32)) and bool(torch.isfinite(dO).all())
    got = dO.cpu().numpy()
    for rows in (slice(0, 3), slice(Ho - 3, Ho)):
        O_ref, B_ref = oracle.conv2d_direct(np.ascontiguousarray(I[:, :, rows.start:rows.stop + Hf - 1].numpy()), F.numpy(), s, p)
        assert_conv_close(got[:, :, rows], O_ref, B_ref)
    rng = np.random.default_rng(9600)
    idx = np.stack([rng.integers(0, n, 20000) for n in (N, Co, Ho, Wo)], axis=1).astype(np.int32)
    O_s, B_s = oracle.conv2d_direct_at(I.numpy(), F.numpy(), s, p, idx)
    assert (np.abs(got[tuple(idx.T)].astype(np.float64) - O_s) <= 1e-4 * B_s).all()


@pytest.mark.parametrize("shape", [(16, 32, 43, 50, 65, 3, 3, 1, 0), (24, 128, 21, 48, 65, 3, 3, 1, 0), (11, 40, 60, 36, 65, 5, 5, 1, 0),
                                   (24, 16, 42, 43, 65, 7, 7, 2, 2), (19, 64, 59, 51, 33, 4, 4, 2, 4), (19, 64, 31, 49, 33, 7, 1, 1, 4)],
                         ids=lambda s: "x".join(map(str, s)))
def test_a_tensor_whose_copies_differ(shape):
    """im2win_transform writes an input word several times and the kernel reads one of the copies, always the same one: a tensor
    of other origin, whose copies differ, gives one result and not another on each call."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    assert _split(shape)
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    g = torch.Generator().manual_seed(9500 + sum(shape))
    dW, dF = torch.randn((N, Ci, Ho, (Wi + 2 * p) * Hf), generator=g).cuda(), torch.randn((Co, Ci, Hf, Wf), generator=g).cuda()
    print("differing copies", shape, flush=True)
    outs = torch.full((4, N, Co, Ho, Wo), float("nan"), device="cuda")
    for o in outs:
        im2win.conv2d_im2win_fwd(dW, dF, o, *shape)
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all()
    for o in outs[1:]:
        assert torch.equal(o.view(torch.int32), outs[0].view(torch.int32))


@pytest.mark.parametrize("shape", [(16, 32, 43, 50, 65, 3, 3, 1, 0), (23, 128, 53, 21, 32, 3, 3, 1, 1), (24, 16, 42, 43, 65, 7, 7, 2, 2)],
                         ids=lambda s: "x".join(map(str, s)))
def test_error_is_below_the_fp32_matrix_cores(shape):
    """Against the 64-bit oracle, with the same inputs, the pieces are no further off than the fp32 kernel."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    assert _split(shape)
    I, F = workloads.random_layer_inputs(9200 + sum(shape), N, Ci, Hi, Wi, Co, Hf, Wf)
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    dW = run_transform(I, Hf, Wf, s, p)
    dO = run_conv(dW, F, N, Ci, Hi, Wi, s, p)
    d32 = torch.full_like(dO, float("nan"))
    im2win.conv2d_im2win_fwd_variant(dW, F.cuda(), d32, *shape, im2win.VARIANT_NO_PIPELINE)
    torch.cuda.synchronize()
    (_, l2), (_, l2_32) = conv_errors(dO.cpu().numpy(), O_ref, B_ref), conv_errors(d32.cpu().numpy(), O_ref, B_ref)
    print("relative L2 error: pieces %.2e, fp32 %.2e" % (l2, l2_32))
    assert l2 <= l2_32


# powers of two on the input and on the filter: normal and subnormal fp32 words below the last bf16 piece, subnormal
# results, operands and sums near the top of the range
SCALES = [(-112, 0), (-118, 4), (-124, 10), (4, -124), (-140, 20), (-63, -63), (105, 0), (120, -120), (-120, 120), (60, 60)]


@pytest.mark.parametrize("ei,ef", SCALES)
def test_no_operand_loses_bits(ei, ef):
    """The 24 bits of an operand hold whatever its magnitude: against 64 bits no further off than the fp32 kernel."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape = (16, 32, 43, 50, 65, 3, 3, 1, 0)
    assert _split(shape) and _split(shape, True)
    I, F = workloads.random_layer_inputs(9400, N, Ci, Hi, Wi, Co, Hf, Wf)
    I, F = torch.ldexp(I.double(), torch.tensor(ei)).float(), torch.ldexp(F.double(), torch.tensor(ef)).float()
    O_ref, B_ref = oracle.conv2d_direct(I.numpy(), F.numpy(), s, p)
    dW, dI, dF = run_transform(I, Hf, Wf, s, p), I.cuda(), F.cuda()
    d32 = torch.full(O_ref.shape, float("nan"), dtype=torch.float32, device="cuda")
    got, got2 = torch.full_like(d32, float("nan")), torch.full_like(d32, float("nan"))
    im2win.conv2d_im2win_fwd_variant(dW, dF, d32, *shape, im2win.VARIANT_NO_PIPELINE)
    im2win.conv2d_im2win_fwd(dW, dF, got, *shape)
    im2win.conv2d_im2win_implicit_fwd(dI, dF, got2, *shape)
    torch.cuda.synchronize()
    l2 = [conv_errors(o.cpu().numpy(), O_ref, B_ref)[1] for o in (got, got2, d32)]
    print("2^%d x 2^%d: relative L2 error, pieces %.2e %.2e, fp32 %.2e" % (ei, ef, *l2))
    assert max(l2[:2]) <= 1.1 * l2[2]   # (where the fp32 fallback computes the outputs, both are fp32 chains of K products)


def _assert_like_basic(shape, I, F):
    """Both calls against the one-thread-per-output fp32 kernel: the same infinities and NaN, the same finite values."""
    N, Ci, Hi, Wi, Co, Hf, Wf, s, p = shape
    dW, dF = run_transform(I, Hf, Wf, s, p), F.cuda()
    Ho, Wo = im2win.im2win_out_shape(Hi, Wi, Hf, Wf, s, p)
    ref = torch.empty((N, Co, Ho, Wo), device="cuda")
    im2win.conv2d_im2win_fwd_basic(dW, dF, ref, *shape)
    got, got2 = torch.zeros_like(ref), torch.zeros_like(ref)
    im2win.conv2d_im2win_fwd(dW, dF, got, *shape)
    im2win.conv2d_im2win_implicit_fwd(I.cuda(), dF, got2, *shape)
    torch.cuda.synchronize()
    for o in (got, got2):
        assert torch.equal(torch.isnan(o), torch.isnan(ref))
        assert torch.equal(torch.isinf(o), torch.isinf(ref))
        assert torch.equal(o[torch.isinf(o)], ref[torch.isinf(ref)])
        fin = torch.isfinite(ref)
        a, b = o[fin].double(), ref[fin].double()
        assert bool(((a - b).abs() <= 1e-4 * b.abs().clamp(min=1.0)).all())   # (K = 288 sums of order one; 1e-4 of the sum of magnitudes)
    return ref


@pytest.mark.parametrize("shape", [SHAPES[i][0] for i in (9, 18, 20, 22, 24, 29)] + OTHER_SHAPES, ids=lambda v: "x".join(map(str, v)))
def test_buffers_of_any_alignment(shape):
    check_any_alignment(shape, 9315)


@pytest.mark.parametrize("shape", [SHAPES[i][0] for i in (9, 18, 20, 22, 24, 29)] + OTHER_SHAPES, ids=lambda v: "x".join(map(str, v)))
def test_the_second_pass_writes_what_the_first_left(shape):
    check_second_pass(shape, 9310)


def test_infinities_nan_and_the_largest_values():
    """An infinite or NaN input, and values whose rounded first piece is infinite, reach exactly the outputs that
    plain fp32 arithmetic gives them (the one-thread-per-output kernel), in both calls."""
    shape = N, Ci, Hi, Wi, Co, Hf, Wf, s, p = (22, 32, 29, 50, 65, 3, 3, 1, 1)
    assert _split(shape)
    I, F = workloads.random_layer_inputs(9300, N, Ci, Hi, Wi, Co, Hf, Wf)
    I[0, 3, 10, 10] = float("inf")
    I[1, 31, 0, 49] = float("-inf")
    I[2, 0, 28, 0] = float("nan")
    I[3, 7, 20, 20] = 3.4028e38              # rounds to infinity in bf16
    I[5, 2, 5, 5], I[5, 9, 6, 6] = float("inf"), float("-inf")
    F[:, 7] *= 0.25
    F[4, 3, 1, 1] = 0.0                      # infinity times zero
    F[64, 0, 0, 0] = float("inf")
    ref = _assert_like_basic(shape, I, F)
    assert torch.isnan(ref).any() and torch.isinf(ref).any()


def test_the_ends_of_the_range_meet():
    """The lowest fp32 value (masks) against zero, tiny and ordinary weights, infinity against a subnormal weight, a NaN
    whose payload is in the low bits only, sums that pass 2^127 on the way: as in the fp32 kernel."""
    shape = N, Ci, Hi, Wi, Co, Hf, Wf, s, p = (22, 32, 29, 50, 65, 3, 3, 1, 1)
    assert _split(shape)
    I, F = workloads.random_layer_inputs(9301, N, Ci, Hi, Wi, Co, Hf, Wf)
    low = torch.finfo(torch.float32).min
    I[0, 3, 10, 10] = low
    I[1, 3] = low                            # a whole masked channel
    F[:, 3] *= 0.1                           # (sums of nine stay finite)
    F[5, 3] = 0.0
    F[6, 3] = 2.0 ** -125
    F[7, 3] = 2.0 ** -140
    I[2, 4, 5, 5] = float("inf")
    F[8, 4] = 2.0 ** -140
    I[4, 5, 7, 7] = torch.tensor([0x7F800001], dtype=torch.int32).view(torch.float32)[0]
    I[6, 6, 20, 20:22] = 2.0 ** 126          # each product fits, the sum of two does not
    F[9, 6] = 2.5
    I[7, 9, 3, 3], F[10, 9] = 2.0 ** 60, 2.0 ** 50    # a sum past 2^96 of small operands
    ref = _assert_like_basic(shape, I, F)
    assert torch.isnan(ref[4]).any() and torch.isinf(ref[2, 8]).any() and torch.isinf(ref[6, 9]).any()
    assert torch.isfinite(ref[1, 5]).all() and (ref[1, 5].abs() < 2.0 ** 48).all()   # (settled by dot_fp32)


@pytest.mark.parametrize("data", ["NaN weight", "NaN image", "infinite pixel", "all NaN", "all 2^100"])
def test_time_on_data_that_is_not_finite(data):
    """Infinite and NaN outputs cost a second pass over their tiles, not a scalar sum each (which took 7 to 180 times as long)."""
    shape = N, Ci, Hi, Wi, Co, Hf, Wf, s, p = (20, 64, 56, 56, 64, 3, 3, 1, 1)
    assert _split(shape) and _split(shape, True)
    I, F = workloads.random_layer_inputs(9302, N, Ci, Hi, Wi, Co, Hf, Wf)
    dO = torch.empty((N, Co, Hi, Wi), device="cuda")

    def times(I, F):
        dW, dI, dF = run_transform(I, Hf, Wf, s, p), I.cuda(), F.cuda()
        out = []
        for call in (lambda: im2win.conv2d_im2win_fwd(dW, dF, dO, *shape), lambda: im2win.conv2d_im2win_implicit_fwd(dI, dF, dO, *shape)):
            best = float("inf")
            for _ in range(5):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(10):
                    call()
                b.record()
                b.synchronize()
                best = min(best, a.elapsed_time(b))
            out.append(best)
        return out

    plain = times(I, F)
    if data == "NaN weight":
        F[3, 5, 1, 1] = float("nan")
    elif data == "NaN image":
        I[3] = float("nan")
    elif data == "infinite pixel":
        I[3, 2, 20, 20] = float("inf")
    elif data == "all NaN":
        I[:] = float("nan")
    else:
        I = torch.ldexp(I.double(), torch.tensor(100)).float()
    odd = times(I, F)
    print("%s: %.1f -> %.1f us, %.1f -> %.1f" % (data, plain[0] * 100, odd[0] * 100, plain[1] * 100, odd[1] * 100))
    assert odd[0] <= 4 * plain[0] and odd[1] <= 4 * plain[1]   # (measured: 2.0 to 2.5)
