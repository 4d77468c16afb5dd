"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments before any GPU work."""
import ctypes as C
import os
import re

import pytest

import paper_2003_10735_amd as st

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "shadowtutor_head.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(st_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = st.lib()
    names = declared_functions()
    assert set(st.EXPORTS) <= set(names)
    for n in names:
        assert hasattr(L, n), n


def good():
    return st.HeadDesc(1, 64, 16, 16, 64, 64, 9, st.ST_F32, st.ST_COMPUTE_F32)


def test_sizes():
    d = good()
    assert st.st_num_params(d) == 74441
    assert st.st_workspace_bytes(d) > 0
    d720 = st.HeadDesc(1, 256, 90, 160, 128, 128, 19)
    assert st.st_num_params(d720) == 445075
    lay = st.st_get_workspace_layout(d720)
    assert lay["total"] == st.st_workspace_bytes(d720) and lay["elem_size"] == 2
    assert st.st_version()


@pytest.mark.parametrize("field,value,status", [
    ("n", 0, st.ST_ERR_SHAPE), ("h", -1, st.ST_ERR_SHAPE), ("upscale", 4, st.ST_ERR_SHAPE),
    ("n_classes", 1, st.ST_ERR_SHAPE), ("n_classes", 33, st.ST_ERR_SHAPE),
    ("feat_dtype", 7, st.ST_ERR_ARG), ("compute", 2, st.ST_ERR_ARG), ("feat_layout", 2, st.ST_ERR_ARG),
    ("ignore_index", -2, st.ST_ERR_ARG), ("w", 1 << 24, st.ST_ERR_SHAPE),
])
def test_bad_descriptors_are_rejected_on_the_host(field, value, status):
    d = good()
    setattr(d, field, value)
    assert st.st_num_params(d) == 0 and st.st_workspace_bytes(d) == 0
    cd = d.c()
    dummy = C.c_void_p(256)       # never dereferenced: validation comes first
    L = st.lib()
    assert L.st_head_forward(C.byref(cd), dummy, dummy, None, None, dummy, None) == status
    assert L.st_partial_distill(C.byref(cd), dummy, dummy, dummy, 1, 0.1, None, None, dummy, None) == status


def test_grouped_descriptor_sizes_and_limits():
    """One head per frame: the per-head parameter count stays, the workspace holds n heads, and
    shapes off the matrix-core kernels are refused."""
    one = st.HeadDesc(4, 256, 90, 160, 128, 128, 19)
    grp = st.HeadDesc(4, 256, 90, 160, 128, 128, 19, grouped=1)
    assert st.st_num_params(grp) == st.st_num_params(one) == 445075
    extra = st.st_workspace_bytes(grp) - st.st_workspace_bytes(one)
    assert extra >= 3 * 445075 * 4 * 4            # theta, two state vectors, gradient copies of 3 more heads
    assert st.st_workspace_bytes(st.HeadDesc(1, 256, 90, 160, 128, 128, 19, grouped=1)) > 0
    # float32 compute, or channel counts the matrix-core kernels do not take
    assert st.st_workspace_bytes(st.HeadDesc(2, 64, 16, 16, 64, 64, 9, st.ST_F32, st.ST_COMPUTE_F32, grouped=1)) == 0
    assert st.st_workspace_bytes(st.HeadDesc(2, 20, 16, 16, 24, 16, 9, grouped=1)) == 0
    assert st.st_workspace_bytes(st.HeadDesc(2, 64, 16, 16, 64, 64, 9, grouped=2)) == 0


@pytest.mark.parametrize("kw,fits,too_large", [
    # 64 rows x 9 taps x channels of padded weights, at two bytes: below 2^31 bytes
    (dict(c_in=1, h=1, w=1, c1=1, c2=1), dict(c_in=1864128), dict(c_in=1864129)),
    (dict(c_in=1, h=1, w=1, c1=1, c2=1), dict(c1=1864128), dict(c1=1864129)),
    (dict(c_in=1, h=1, w=1, c1=1, c2=1), dict(c2=1864128), dict(c2=1864129)),
    # two kernel rows of a frame, 64 bytes a cell, in the weight-gradient kernel
    (dict(c_in=1, h=1, w=1, c1=1, c2=1), dict(w=16 * 10**6), dict(w=17 * 10**6)),
])
def test_sizes_beyond_the_32_bit_offsets_of_the_padded_buffers(kw, fits, too_large):
    """bfloat16 heads are padded to 64 channels inside: what the kernels' 32-bit byte offsets cannot reach is
    refused, the last size before that is not, and the float32 path (padded to eight) takes both."""
    def desc(extra, compute):
        return st.HeadDesc(**{**dict(n=1, n_classes=2, compute=compute, feat_dtype=compute), **kw, **extra})
    assert st.st_workspace_bytes(desc(fits, st.ST_COMPUTE_BF16)) > 0
    d = desc(too_large, st.ST_COMPUTE_BF16)
    assert st.st_workspace_bytes(d) == 0
    dummy, cd = C.c_void_p(256), d.c()
    assert st.lib().st_partial_distill(C.byref(cd), dummy, dummy, dummy, 1, 0.1, None, None, dummy, None) == st.ST_ERR_SHAPE
    assert st.st_workspace_bytes(desc(too_large, st.ST_COMPUTE_F32)) > 0


def test_null_and_argument_errors():
    L = st.lib()
    cd = good().c()
    dummy = C.c_void_p(256)
    assert L.st_head_forward(None, dummy, dummy, None, None, dummy, None) == st.ST_ERR_NULL
    assert L.st_head_forward(C.byref(cd), None, dummy, None, None, dummy, None) == st.ST_ERR_NULL
    assert L.st_head_forward(C.byref(cd), dummy, dummy, None, None, None, None) == st.ST_ERR_WORKSPACE
    assert L.st_head_forward(C.byref(cd), dummy, dummy, None, None, C.c_void_p(264), None) == st.ST_ERR_WORKSPACE
    pd = L.st_partial_distill
    assert pd(C.byref(cd), dummy, None, dummy, 1, 0.1, None, None, dummy, None) == st.ST_ERR_NULL
    assert pd(C.byref(cd), dummy, dummy, dummy, -1, 0.1, None, None, dummy, None) == st.ST_ERR_ARG
    assert pd(C.byref(cd), dummy, dummy, dummy, 1, float("nan"), None, None, dummy, None) == st.ST_ERR_ARG
    assert pd(C.byref(cd), dummy, dummy, dummy, 1, float("inf"), None, None, dummy, None) == st.ST_ERR_ARG
    opts = st.StDistillOpts(0.9, None, 0.0, 1, 0)
    assert pd(C.byref(cd), dummy, dummy, dummy, 1, 0.1, C.byref(opts), None, dummy, None) == st.ST_ERR_NULL
    opts = st.StDistillOpts(float("nan"), dummy, 0.0, 1, 0)
    assert pd(C.byref(cd), dummy, dummy, dummy, 1, 0.1, C.byref(opts), None, dummy, None) == st.ST_ERR_ARG
    # Adam: state arrays required, no momentum, constants in range
    def adam_opts(**kw):
        o = st.StDistillOpts(0.0, None, 0.0, 1, 0, st.ST_OPTIM_ADAM, 0.9, 0.999, 1e-8, dummy, dummy, 0)
        for k, v in kw.items():
            setattr(o, k, v)
        return o
    for kw, status in (({"adam_m": None}, st.ST_ERR_NULL), ({"adam_v": None}, st.ST_ERR_NULL),
                       ({"momentum": 0.5, "velocity": dummy}, st.ST_ERR_ARG), ({"beta1": 1.0}, st.ST_ERR_ARG),
                       ({"beta2": -0.1}, st.ST_ERR_ARG), ({"eps": 0.0}, st.ST_ERR_ARG),
                       ({"adam_t0": -1}, st.ST_ERR_ARG), ({"optimizer": 2}, st.ST_ERR_ARG)):
        o = adam_opts(**kw)
        assert pd(C.byref(cd), dummy, dummy, dummy, 1, 0.1, C.byref(o), None, dummy, None) == status, kw
    assert L.st_miou(None, dummy, 10, 3, -1, dummy, dummy, None) == st.ST_ERR_NULL
    assert L.st_miou(dummy, dummy, -1, 3, -1, dummy, dummy, None) == st.ST_ERR_SHAPE
    assert L.st_miou(None, None, 0, 3, -1, None, dummy, None) == st.ST_ERR_NULL
    assert L.st_miou(dummy, dummy, 10, 0, -1, dummy, dummy, None) == st.ST_ERR_SHAPE
    assert L.st_get_workspace_layout(C.byref(cd), None) == st.ST_ERR_NULL
    # the forward entry point on the built-in scratch validates in the same order, then the size
    na = L.st_head_forward_noalloc
    assert na(None, dummy, dummy, None, None, None) == st.ST_ERR_NULL
    assert na(C.byref(cd), None, dummy, None, None, None) == st.ST_ERR_NULL
    big = st.HeadDesc(1, 256, 135, 240, 128, 128, 19).c()
    assert na(C.byref(big), dummy, dummy, None, None, None) == st.ST_ERR_TOO_LARGE
    # the loss-weight map: shape, then value arguments, then pointers
    ow = L.st_object_weights
    assert ow(dummy, 0, 8, 8, 19, 0, -1, 4, 5, dummy, None) == st.ST_ERR_SHAPE
    assert ow(dummy, 1, 8, 0, 19, 0, -1, 4, 5, dummy, None) == st.ST_ERR_SHAPE
    assert ow(dummy, 70000, 8, 8, 19, 0, -1, 4, 5, dummy, None) == st.ST_ERR_SHAPE
    assert ow(dummy, 1, 8, 8, 0, 0, -1, 4, 5, dummy, None) == st.ST_ERR_SHAPE
    assert ow(dummy, 1, 8, 8, 19, 0, -1, -1, 5, dummy, None) == st.ST_ERR_ARG
    assert ow(dummy, 1, 8, 8, 19, 0, -1, st.ST_OBJECT_WEIGHTS_MAX_RADIUS + 1, 5, dummy, None) == st.ST_ERR_ARG
    assert ow(dummy, 1, 8, 8, 19, 0, -1, 4, 0, dummy, None) == st.ST_ERR_ARG
    assert ow(dummy, 1, 8, 8, 19, 0, -1, 4, 256, dummy, None) == st.ST_ERR_ARG
    assert ow(None, 1, 8, 8, 19, 0, -1, 4, 5, dummy, None) == st.ST_ERR_NULL
    assert ow(dummy, 1, 8, 8, 19, 0, -1, 4, 5, None, None) == st.ST_ERR_NULL
    for s in (0, -1, -2, -3, -4, -5, -6, -7, -99):
        assert L.st_strerror(s)


def test_product_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2003_10735_amd")
    for dirpath, _, files in os.walk(pkg):
        for fn in files:
            if fn.endswith((".py", ".hip", ".hpp", ".h", ".cpp")):
                text = open(os.path.join(dirpath, fn)).read()
                assert "oracle" not in text.replace("no CPU fallback", ""), os.path.join(dirpath, fn)


def test_bench_refuses_more_than_one_gpu():
    """The library runs on one GPU: asked for more, the benchmark says so and stops before it
    touches a device."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)


def test_missing_tensors_are_the_librarys_error():
    """A tensor that is not there is refused by the library (status of a null pointer), through every binding."""
    import types
    import torch
    d, stream = good(), types.SimpleNamespace(cuda_stream=0)
    t = torch.zeros(256)
    for call in (lambda: st.st_head_forward(d, None, t, workspace=t, stream=stream),
                 lambda: st.st_head_forward(d, t, None, workspace=t, stream=stream),
                 lambda: st.st_head_forward_noalloc(d, None, t, stream=stream),
                 lambda: st.st_partial_distill(d, None, t, t, 1, 0.1, workspace=t, stream=stream),
                 lambda: st.st_partial_distill(d, t, None, t, 1, 0.1, workspace=t, stream=stream),
                 lambda: st.st_miou(t, None, 9, confusion=t, miou=t, stream=stream)):
        with pytest.raises(st.StError) as e:
            call()
        assert e.value.status == st.ST_ERR_NULL


# (n, c_in, h, w, c1, c2, classes, compute): heads whose padded buffers, or all of a training call's, exceed the
# built-in scratch while the head's own activations do not; then an unpadded head, one column below and above the
# limit; last, float32 heads whose half fragments of input channels take no room, one row below and above it
@pytest.mark.parametrize("shape,fits", [
    ((1, 64, 160, 200, 64, 192, 21, "bf16"), True), ((1, 64, 200, 100, 64, 512, 21, "bf16"), True),
    ((1, 1, 810, 810, 1, 1, 2, "bf16"), True), ((32, 3, 511, 24, 6, 3, 4, "bf16"), True),
    ((2139, 8, 1, 187, 3, 1, 3, "bf16"), True), ((2, 54004, 4, 1, 2, 32, 28, "bf16"), True),
    ((1, 41037, 1, 2, 1, 2, 32, "f32"), True), ((8, 26386, 2, 4, 1, 5, 30, "f32"), True),
    ((1, 8, 6000, 5000, 8, 8, 2, "bf16"), False), ((1, 8, 6000, 5000, 8, 8, 2, "f32"), False),
    ((2, 256, 217, 33, 64, 256, 24, "bf16"), True), ((2, 256, 218, 33, 64, 256, 24, "bf16"), False),
    ((1, 24, 520, 300, 40, 200, 9, "f32"), True), ((1, 24, 521, 300, 40, 200, 9, "f32"), False),
    ((1, 40, 357, 300, 88, 128, 19, "f32"), True), ((1, 40, 358, 300, 88, 128, 19, "f32"), False),
    ((1, 8, 230, 300, 8, 512, 19, "f32"), True), ((1, 8, 231, 300, 8, 512, 19, "f32"), False)])
def test_what_the_built_in_scratch_takes(shape, fits):
    """st_head_forward_noalloc takes a head by what its forward pass needs at least.  (Without a GPU a call that
    passes the size check ends with ST_ERR_NO_DEVICE: nothing is launched, no pointer is followed.)"""
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch kernels on dummy pointers")
    n, c_in, h, w, c1, c2, classes, compute = shape
    code = st.ST_COMPUTE_BF16 if compute == "bf16" else st.ST_COMPUTE_F32
    d = st.HeadDesc(n, c_in, h, w, c1, c2, classes, compute=code, feat_dtype=code).c()
    dummy = C.c_void_p(256)
    assert st.lib().st_head_forward_noalloc(C.byref(d), dummy, dummy, None, None, None) == (st.ST_ERR_NO_DEVICE if fits else st.ST_ERR_TOO_LARGE)


# (n, c_in, h, w, c1, c2, classes, grouped): the last shape that fits, and the first that does not -- one cell row, one head or eight columns
# (the pitch of a row) more.  Those that fit do so by less than what their parameter vectors, rounded up to whole cache lines, would add.
@pytest.mark.parametrize("shape,more", [
    ((1, 256, 21, 1520, 64, 64, 7, 0), (1, 256, 21, 1528, 64, 64, 7, 0)), ((1, 128, 53, 889, 64, 64, 5, 0), (1, 128, 54, 889, 64, 64, 5, 0)),
    ((1, 128, 3, 3438, 256, 64, 22, 0), (1, 128, 3, 3446, 256, 64, 22, 0)), ((3, 128, 31, 208, 64, 256, 10, 1), (3, 128, 32, 208, 64, 256, 10, 1)),
    ((20, 64, 6, 11, 64, 256, 13, 1), (21, 64, 6, 11, 64, 256, 13, 1)), ((36, 64, 54, 2, 64, 64, 14, 1), (37, 64, 54, 2, 64, 64, 14, 1)),
    ((25, 64, 20, 1, 128, 64, 10, 1), (25, 64, 21, 1, 128, 64, 10, 1))])
def test_the_layout_of_training_does_not_move_the_scratch_limit(shape, more):
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch kernels on dummy pointers")
    dummy = C.c_void_p(256)
    for (n, c_in, h, w, c1, c2, classes, grouped), want in ((shape, st.ST_ERR_NO_DEVICE), (more, st.ST_ERR_TOO_LARGE)):
        d = st.HeadDesc(n, c_in, h, w, c1, c2, classes, compute=st.ST_COMPUTE_BF16, feat_dtype=st.ST_BF16, grouped=grouped).c()
        assert st.lib().st_head_forward_noalloc(C.byref(d), dummy, dummy, None, None, None) == want


def test_layout_names_no_buffer_that_nothing_writes():
    """d loss / d z is assembled on the float32 path only."""
    for compute in (st.ST_COMPUTE_F32, st.ST_COMPUTE_BF16):
        for c in (24, 64):
            lay = st.st_get_workspace_layout(st.HeadDesc(1, c, 12, 20, c, c, 9, compute=compute, feat_dtype=compute))
            assert (lay["g"] == 0) == (compute == st.ST_COMPUTE_BF16) and min(lay[k] for k in ("feat", "a1", "a2", "da1", "da2", "z")) > 0
