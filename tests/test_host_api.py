"""CPU-only checks of the C-ABI library: it loads, exports every symbol the
header declares, derives shapes as the oracle does, and turns every invalid
argument into an error code without launching anything."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

import oracle
import paper_2306_14316_amd as im2win
from paper_2306_14316_amd import binding, workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(im2win.lib_path()):
        from paper_2306_14316_amd import build
        build.build()
    return im2win.load_library()


def test_header_symbols_are_exported(lib):
    hdr = open(os.path.join(ROOT, "include", "im2win.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(im2win_\w+|conv2d_\w+|im2col_\w+)\s*\(", hdr))
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None
    probes = open(os.path.join(ROOT, "include", "im2win_probe.h")).read()
    probes = re.sub(r"/\*.*?\*/", "", probes, flags=re.S)
    declared = set(re.findall(r"\b(im2win_\w+)\s*\(", probes))
    assert declared == set(binding.PROBE_EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None


def test_shapes_and_footprints_match_oracle(lib, golden_dir):
    for L in workloads.LAYERS:
        assert im2win.im2win_out_shape(L.Hi, L.Wi, L.Hf, L.Wf, L.stride, L.pad) == \
            oracle.out_shape(L.Hi, L.Wi, L.Hf, L.Wf, L.stride, L.pad)
        a = (L.N, L.Ci, L.Hi, L.Wi, L.Hf, L.Wf, L.stride, L.pad)
        assert im2win.im2win_workspace_bytes(*a) == 4 * oracle.im2win_elems(*a)
        assert im2win.im2col_footprint_bytes(*a) == 4 * oracle.im2col_elems(*a)
    # the paper's worked example and Table 2
    assert im2win.im2win_workspace_bytes(1, 3, 3, 3, 2, 2, 1, 0) == 4 * 36
    assert im2win.im2col_footprint_bytes(1, 3, 3, 3, 2, 2, 1, 0) == 4 * 48
    for ln in open(os.path.join(golden_dir, "table2_layers.txt")):
        if ln.startswith("#") or not ln.strip():
            continue
        _, Ci, Hi, Wi, Co, Hf, Wf, s, Ho, Wo = ln.split()
        assert im2win.im2win_out_shape(int(Hi), int(Wi), int(Hf), int(Wf), int(s), 0) == (int(Ho), int(Wo))


def test_workspace_bytes_of_the_five_layers(lib):
    want = [34560, 79822848, 88080384, 276971520, 210946560]
    got = [im2win.im2win_workspace_bytes(L.N, L.Ci, L.Hi, L.Wi, L.Hf, L.Wf, L.stride, L.pad)
           for L in workloads.LAYERS]
    assert got == want


BAD_SHAPES = [
    dict(N=0), dict(Ci=0), dict(Hi=0), dict(Wi=-1), dict(Co=0), dict(Hf=0), dict(Wf=0),
    dict(stride=0), dict(pad=-1), dict(Hf=9), dict(Wf=9),
]


@pytest.mark.parametrize("bad", BAD_SHAPES)
def test_invalid_shapes_are_rejected_before_any_launch(lib, bad):
    a = dict(N=1, Ci=2, Hi=8, Wi=8, Co=3, Hf=3, Wf=3, stride=1, pad=0)
    a.update(bad)
    one = ctypes.c_void_p(16)   # non-NULL dummy: validation must fail before it is touched
    rc = lib.im2win_transform(one, one, a["N"], a["Ci"], a["Hi"], a["Wi"], a["Hf"], a["Wf"],
                              a["stride"], a["pad"], None)
    if "Co" not in bad:
        assert rc == -2
    for fn in (lib.conv2d_im2win_fwd, lib.conv2d_im2win_fwd_basic):
        assert fn(one, one, one, a["N"], a["Ci"], a["Hi"], a["Wi"], a["Co"], a["Hf"], a["Wf"],
                  a["stride"], a["pad"], None) == -2
    assert lib.conv2d_im2win_fwd_variant(one, one, one, a["N"], a["Ci"], a["Hi"], a["Wi"], a["Co"], a["Hf"],
                                         a["Wf"], a["stride"], a["pad"], 1, None) == -2


def test_null_pointers_and_overflow(lib):
    one = ctypes.c_void_p(16)
    assert lib.im2win_transform(None, one, 1, 1, 4, 4, 2, 2, 1, 0, None) == -1
    assert lib.im2win_transform(one, None, 1, 1, 4, 4, 2, 2, 1, 0, None) == -1
    assert lib.conv2d_im2win_fwd(one, None, one, 1, 1, 4, 4, 1, 2, 2, 1, 0, None) == -1
    assert lib.conv2d_im2win_fwd(one, one, None, 1, 1, 4, 4, 1, 2, 2, 1, 0, None) == -1
    assert lib.conv2d_im2win_fwd_basic(None, one, one, 1, 1, 4, 4, 1, 2, 2, 1, 0, None) == -1
    assert lib.im2win_out_shape(4, 4, 2, 2, 1, 0, None, None) == -1
    assert lib.conv2d_im2win_fwd_variant(one, one, None, 1, 1, 4, 4, 1, 2, 2, 1, 0, 0, None) == -1
    assert lib.conv2d_im2win_fwd_variant(one, one, one, 1, 1, 4, 4, 1, 2, 2, 1, 0, 7, None) == -4
    assert lib.conv2d_im2win_fwd_variant(one, one, one, 1, 1, 4, 4, 1, 2, 2, 1, 0, -1, None) == -4
    # 2^31 or more elements in the im2win tensor / the output
    assert lib.im2win_transform(one, one, 4096, 64, 224, 224, 7, 7, 2, 0, None) == -3
    assert lib.conv2d_im2win_fwd(one, one, one, 128, 3, 1024, 1024, 64, 1, 1, 1, 0, None) == -3
    # the baselines: NULL pointers, and an im2col matrix of 2^31 or more groups of four floats
    assert lib.conv2d_direct_fwd(one, None, one, 1, 1, 4, 4, 1, 2, 2, 1, 0, None) == -1
    assert lib.conv2d_im2win_implicit_fwd(None, one, one, 1, 8, 4, 4, 1, 3, 3, 1, 0, None) == -1
    assert lib.im2col_transform(one, None, 1, 1, 4, 4, 2, 2, 1, 0, None) == -1
    assert lib.conv2d_im2col_fwd(None, one, one, 1, 1, 4, 4, 1, 2, 2, 1, 0, None) == -1
    assert lib.im2col_transform(one, one, 512, 256, 112, 112, 3, 3, 1, 1, None) == -3
    assert lib.conv2d_im2col_fwd(one, one, one, 512, 256, 112, 112, 8, 3, 3, 1, 1, None) == -3
    b = ctypes.c_size_t()
    assert lib.im2win_workspace_bytes(4096, 64, 224, 224, 7, 7, 2, 0, ctypes.byref(b)) == -3
    for code in (0, -1, -2, -3, -4, -5, 77):
        assert im2win.status_str(code)


def test_filter_as_large_as_padded_input_is_valid(lib):
    assert im2win.im2win_out_shape(6, 6, 8, 8, 1, 1) == (1, 1)
    with pytest.raises(im2win.Im2winError):
        im2win.im2win_out_shape(6, 6, 9, 8, 1, 1)


def test_binding_rejects_host_tensors(lib):
    import torch
    x = torch.zeros(1, 1, 4, 4)
    w = torch.zeros(1, 1, 3, 8)
    with pytest.raises(TypeError):
        im2win.im2win_transform(x, w, 1, 1, 4, 4, 2, 2, 1, 0)


def test_launch_info_names_the_dispatch(lib):
    """The planning calls run the library's own dispatch and launch nothing (no GPU needed: the
    grid is then planned for 256 compute units)."""
    want = {1: "conv_mfma_quarter_kernel<3, 3, 8, 1, false, true>", 2: "conv_split_kernel<3, 3, 0, false>", 3: "conv_split_kernel<3, 3, 0, false>",
            4: "conv_split_stem_kernel<7, 2, 1, 4, 1, false>", 5: "conv_split_stem_kernel<11, 3, 4, 1, 1, false>"}
    for idx, prefix in want.items():
        L = workloads.layer(idx)
        info = im2win.conv2d_im2win_fwd_launch_info(*L.dims)
        assert info["kernel"].startswith(prefix), info
        assert info["grid"][0] >= 1 and info["block"] in (256, 512, 768)
        t = im2win.im2win_transform_launch_info(L.N, L.Ci, L.Hi, L.Wi, L.Hf, L.Wf, L.stride, L.pad)
        assert t["kernel"].startswith("transform_assemble_kernel<%d, %d, " % (L.Hf, L.stride)), t
        assert t["kernel"].endswith("true>" if idx in (1, 3) else "false>"), t   # small planes go in groups
    assert im2win.im2win_transform_launch_info(1, 1, 12, 1100, 9, 1, 1, 1)["kernel"] == "transform_kernel<4>"
    assert im2win.im2win_transform_launch_info(1, 1, 4, 3, 2, 2, 1, 0)["kernel"] == "transform_kernel<4>"
    for L in workloads.TABLE2:
        t = im2win.im2win_transform_launch_info(L.N, L.Ci, L.Hi, L.Wi, L.Hf, L.Wf, L.stride, L.pad)
        assert t["kernel"].startswith("transform_assemble_kernel<") and t["lds_bytes"] <= 24 * 1024 + 32, t
    L = workloads.layer(2)
    assert im2win.conv2d_im2win_fwd_launch_info(*L.dims, variant=im2win.VARIANT_NO_MFMA)["kernel"] == "conv_basic_kernel"
    assert im2win.conv2d_im2win_fwd_launch_info(*L.dims, variant=im2win.VARIANT_NO_PIPELINE)["kernel"] == "conv_mfma_kernel<9, false>"
    assert im2win.conv2d_im2win_fwd_launch_info(*L.dims, variant=im2win.VARIANT_VALU_MICROKERNEL)["kernel"] == "conv_mfma_kernel<9, true>"
    # other layers: the default kernel, whichever that is
    for shape in ((128, 96, 24, 24, 256, 5, 5, 1, 0), (64, 128, 28, 28, 128, 1, 3, 1, 1), (64, 256, 28, 28, 256, 1, 1, 1, 0),
                  (64, 64, 28, 28, 64, 1, 5, 1, 0), (128, 100, 28, 28, 64, 3, 3, 1, 1), (128, 3, 224, 224, 64, 3, 3, 1, 0)):
        plans = [im2win.conv2d_im2win_fwd_launch_info(*shape, variant=v) for v in
                 (im2win.VARIANT_DEFAULT, im2win.VARIANT_NARROW_LOADS, im2win.VARIANT_SCALAR_LOADS)]
        assert plans[0] == plans[1] == plans[2], (shape, plans)
    assert im2win.conv2d_im2win_fwd_launch_info(4, *L.dims[1:])["kernel"].startswith("conv_mfma_fast_kernel<3, 3, 8, 1, 4, 3,")   # few tiles
    for v, cw in ((im2win.VARIANT_NARROW_LOADS, 2), (im2win.VARIANT_SCALAR_LOADS, 1)):
        assert im2win.conv2d_im2win_fwd_launch_info(*L.dims, variant=v)["kernel"].startswith(
            "conv_mfma_fast_kernel<3, 3, 8, 1, %d, 3," % cw)
    assert im2win.conv2d_im2win_fwd_launch_info(*L.dims, workspace_free=True)["kernel"] == "conv_split_kernel<3, 3, 0, true>"
    assert im2win.conv2d_im2win_fwd_launch_info(128, 60, 56, 56, 64, 3, 3, 1, 1)["kernel"] == "conv_split_kernel<3, 3, 0, false>"
    # a channel count off the K block still takes the pipelined kernel (its ragged instance)
    assert im2win.conv2d_im2win_fwd_launch_info(4, 13, 60, 60, 96, 3, 3, 1, 0)["kernel"] == \
        "conv_mfma_fast_kernel<3, 3, 8, 1, 4, 3, false, false, false, false, true>"
    assert im2win.conv2d_im2win_fwd_launch_info(3, 13, 12, 12, 96, 3, 3, 1, 0)["kernel"] == "conv_mfma_quarter_kernel<3, 3, 8, 1, false, true>"   # few tiles
    assert im2win.conv2d_im2win_fwd_launch_info(8, 7, 56, 56, 64, 3, 3, 1, 1)["kernel"] == "conv_mfma_kernel<9, false>"
    # 1x1 layers: their own kernel; 1x7 / 7x1 / 1x3 / 3x1: instances of the pipelined kernel; other asymmetric filters:
    # the pipelined generic kernel, its single-stage form when two stages do not fit LDS
    assert im2win.conv2d_im2win_fwd_launch_info(64, 256, 28, 28, 256, 1, 1, 1, 0)["kernel"] == "conv_split_1x1_kernel<2, false, false>"
    assert im2win.conv2d_im2win_fwd_launch_info(8, 256, 28, 28, 256, 1, 1, 1, 0)["kernel"] == "conv_mfma_1x1_kernel<32, false, 2, 1>"   # few tiles
    assert im2win.conv2d_im2win_fwd_launch_info(8, 256, 28, 28, 256, 1, 1, 1, 0, workspace_free=True)["kernel"] == "conv_mfma_1x1_kernel<32, false, 2, 1>"
    assert im2win.conv2d_im2win_fwd_launch_info(8, 256, 28, 28, 256, 1, 1, 2, 0)["kernel"] == "conv_mfma_1x1_kernel<32, true, 2, 1>"   # strided
    assert im2win.conv2d_im2win_fwd_launch_info(64, 252, 28, 28, 256, 1, 1, 1, 0)["kernel"] == "conv_split_1x1_kernel<2, true, false>"
    assert im2win.conv2d_im2win_fwd_launch_info(64, 252, 28, 28, 256, 1, 1, 1, 1)["kernel"] == "conv_mfma_pipe_kernel<1, 1>"   # padded
    assert im2win.conv2d_im2win_fwd_launch_info(4, 64, 28, 28, 64, 1, 7, 1, 0)["kernel"].startswith("conv_mfma_fast_kernel<1, 7, 8, 1, 4, 3, false,")
    assert im2win.conv2d_im2win_fwd_launch_info(4, 64, 28, 28, 64, 7, 1, 1, 3, workspace_free=True)["kernel"].startswith("conv_mfma_fast_kernel<7, 1, 8, 2, 4, 2, true,")
    # three channels: the bf16-piece kernel at stride 2 (7x7) and at stride 4 (11x11), otherwise the fp32 matrix cores
    assert im2win.conv2d_im2win_fwd_launch_info(128, 3, 227, 227, 96, 11, 11, 4, 0, workspace_free=True)["kernel"] == "conv_split_stem_kernel<11, 3, 4, 1, 1, true>"
    assert im2win.conv2d_im2win_fwd_launch_info(32, 3, 227, 227, 96, 11, 11, 2, 0)["kernel"] == "conv_mfma_shallow_kernel<11, 11, 3, 3, 2, 4, false, 1, false>"
    assert im2win.conv2d_im2win_fwd_launch_info(1, 3, 224, 224, 64, 7, 7, 2, 3)["kernel"] == "conv_mfma_shallow_kernel<7, 7, 3, 2, 1, 4, false, 1, false>"
    assert im2win.conv2d_im2win_fwd_launch_info(64, 64, 28, 28, 64, 1, 5, 1, 0)["kernel"] == "conv_mfma_pipe_kernel<0, 0>"
    assert im2win.conv2d_im2win_fwd_launch_info(2, 3, 35, 35, 96, 11, 11, 3, 0)["kernel"] == "conv_mfma_kernel<121, false>"
    assert im2win.conv2d_im2win_fwd_launch_info(2, 10, 35, 35, 96, 9, 9, 2, 0)["kernel"] == "conv_mfma_pipe_kernel<0, 0>"
    assert im2win.conv2d_im2win_fwd_launch_info(1, 2, 40, 40, 8, 17, 17, 1, 0)["kernel"] == "conv_mfma_kernel<0, false>"
    assert im2win.conv2d_im2win_fwd_launch_info(8, 7, 56, 56, 64, 3, 3, 1, 1, workspace_free=True)["kernel"] == "conv_mfma_kernel<9, false>"
    # layers that no tiled kernel takes go to the one-thread-per-output kernels instead of failing
    assert im2win.conv2d_im2win_fwd_launch_info(1, 2, 30, 28, 6, 25, 25, 1, 0)["kernel"] == "conv_basic_kernel"
    assert im2win.conv2d_im2win_fwd_launch_info(1, 2, 30, 28, 6, 25, 25, 1, 0, workspace_free=True)["kernel"] == "conv_direct_kernel"
    # a stride far beyond the image, one output per image: the strips of a tile are 64 windows
    info = im2win.conv2d_im2win_fwd_launch_info(3, 8, 3, 3, 5, 3, 3, 1 << 26, 0)
    assert info["kernel"] == "conv_mfma_kernel<9, false>" and info["lds_bytes"] <= 160 * 1024
    # ... and with two outputs per row the window step no longer fits the tiled kernels' indices
    assert im2win.conv2d_im2win_fwd_launch_info(1, 1, 1, (1 << 28) + 1, 1, 1, 1, 1 << 28, 0)["kernel"] == "conv_basic_kernel"
    # errors as for the calls they describe
    info = binding.LaunchInfo()
    assert lib.conv2d_im2win_fwd_launch_info(1, 1, 4, 4, 1, 5, 5, 1, 0, 0, 0, ctypes.byref(info)) == -2
    assert lib.conv2d_im2win_fwd_launch_info(1, 1, 4, 4, 1, 2, 2, 1, 0, 9, 0, ctypes.byref(info)) == -4
    assert lib.conv2d_im2win_fwd_launch_info(1, 1, 4, 4, 1, 2, 2, 1, 0, 1, 1, ctypes.byref(info)) == -4
    assert lib.conv2d_im2win_fwd_launch_info(1, 1, 4, 4, 1, 2, 2, 1, 0, 0, 0, None) == -1
    assert lib.im2win_transform_launch_info(1, 1, 4, 4, 2, 2, 1, 0, None) == -1


def test_sizes_kept_from_earlier_calls_are_of_plain_ints_only(lib):
    """A number that can change or that is no integer is asked about again on each call: a size kept for it would let a call past
    the check of its buffers."""
    import torch
    n = torch.tensor(1)
    for elems in (binding._elems, lambda *d: (im2win.layer_sizes(*d)["window_elems"], im2win.layer_sizes(*d)["output_elems"])):
        n.fill_(1)
        first = elems(n, 3, 8, 8, 5, 3, 3, 1, 0)
        n += 1
        for N in (n, 2, n):
            again = elems(N, 3, 8, 8, 5, 3, 3, 1, 0)
            assert again[0] == 2 * first[0] and int(again[1]) == 2 * 5 * 6 * 6
    for bad in (2.0, [2]):
        with pytest.raises(ctypes.ArgumentError):
            im2win.layer_sizes(bad, 3, 8, 8, 5, 3, 3, 1, 0)
    for N in range(1, 3000):   # bounded
        binding._elems(N, 3, 8, 8, 5, 3, 3, 1, 0)
    assert len(binding._kept_elems) <= 1024


def test_the_current_stream_needs_no_private_call(monkeypatch):
    import torch
    from types import SimpleNamespace
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=1234))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    for name in ("_torch", "_raw_stream"):   # as at the first call; put back behind the test
        monkeypatch.setattr(binding, name, None, raising=False)
    assert binding._stream(None) == 1234
    assert binding._stream(SimpleNamespace(cuda_stream=77)) == 77


def test_probe_arguments_are_validated(lib):
    one = ctypes.c_void_p(16)
    fl = ctypes.c_double()
    assert lib.im2win_probe_mfma_f32(None, 64, ctypes.byref(fl), None) == -1
    assert lib.im2win_probe_mfma_f32(one, 2, ctypes.byref(fl), None) == -2
    assert lib.im2win_probe_stream(3, one, one, 1024, None) == -4
    assert lib.im2win_probe_stream(0, None, one, 1024, None) == -1
    assert lib.im2win_probe_stream(0, one, one, 1000, None) == -2
    assert lib.im2win_probe_stream(2, None, ctypes.c_void_p(20), 1024, None) == -2


def test_bench_traffic_constants_are_the_profiled_ones():
    """bench.py reports HBM traffic per launch from constants; they must be the figures of the
    kept rocprofv3 summary, not numbers from some other run."""
    import bench
    path = os.path.join(ROOT, "profiles", "all_layers_default_bench.md")
    got = {"conv": {}, "transform": {}}
    for ln in open(path):
        m = re.match(r"\s+TRAFFIC_BYTES (\w+) (\w+) (\d+)", ln)
        if m:
            got[m.group(1)][m.group(2)] = int(m.group(3))
    assert got["conv"] == bench.MEASURED_CONV_TRAFFIC_BYTES
    assert got["transform"] == bench.MEASURED_TRANSFORM_TRAFFIC_BYTES
    assert set(got["conv"]) == {L.name for L in workloads.LAYERS}


def test_the_library_is_loaded_after_torch():
    """A size query before the program's own `import torch`: one HIP runtime in the process, torch's."""
    code = ("import sys, paper_2306_14316_amd as im2win\n"
            "assert 'torch' not in sys.modules and im2win.im2win_out_shape(5, 5, 3, 3, 1, 0) == (3, 3)\n"
            "import torch\n"
            "print(len({l.split()[-1] for l in open('/proc/self/maps') if 'libamdhip64' in l}))")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=root)
    assert r.returncode == 0 and r.stdout.split() == ["1"], (r.stdout, r.stderr)
