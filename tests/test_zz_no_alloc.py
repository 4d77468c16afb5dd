"""st_head_forward_noalloc -- the forward entry point for callers that cannot allocate -- against
st_head_forward on a caller's workspace: same kernels, so the low-resolution logits and the class
map must agree bit for bit.  Two calls in a row share the library's built-in scratch, the second
with a smaller input (it meets whatever the first one left there), then a float32 shape; heads whose
training buffers exceed the built-in scratch run on the forward pass's alone, bit for bit as well, and
those whose padded buffers exceed it on buffers of the head's own sizes (k_head_direct.hip), where the
sums have another order; a shape beyond that is refused before any GPU work."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2003_10735_amd as st
import workloads as WL
from gpu_util import to_dev_features

pytestmark = pytest.mark.gpu


def both_ways(wl, seed):
    desc = st.HeadDesc.of(wl)
    f = to_dev_features(wl, WL.make_features(wl, seed=seed))
    p = torch.from_numpy(WL.make_head_params(wl, seed=seed + 1)).cuda()
    shape_z, shape_p = (wl.n, wl.n_classes, wl.h, wl.w), (wl.n, wl.H, wl.W)
    z_ref = torch.full(shape_z, float("nan"), dtype=torch.float32, device="cuda")
    q_ref = torch.full(shape_p, 255, dtype=torch.uint8, device="cuda")
    st.st_head_forward(desc, f, p, logits_lowres=z_ref, pred=q_ref, workspace=st.new_workspace(desc))
    z = torch.full(shape_z, float("nan"), dtype=torch.float32, device="cuda")
    q = torch.full(shape_p, 255, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    st.st_head_forward_noalloc(desc, f, p, logits_lowres=z, pred=q)
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
    np.testing.assert_array_equal(z.cpu().numpy(), z_ref.cpu().numpy())
    np.testing.assert_array_equal(q.cpu().numpy(), q_ref.cpu().numpy())
    assert np.isfinite(z_ref.cpu().numpy()).all() and int(q_ref.max()) < wl.n_classes
    assert len(np.unique(q_ref.cpu().numpy())) > 1            # a class map worth comparing
    # the class map alone (logits not asked for)
    q2 = torch.full(shape_p, 255, dtype=torch.uint8, device="cuda")
    st.st_head_forward_noalloc(desc, f, p, pred=q2)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(q2.cpu().numpy(), q_ref.cpu().numpy())


def test_two_calls_in_a_row_the_second_smaller():
    big = WL.WORKLOADS["720p"]
    assert st.st_workspace_bytes(st.HeadDesc.of(big)) <= st.ST_NOALLOC_MAX_WORKSPACE_MIB << 20
    both_ways(big, seed=41)
    small = WL.small_variant(big, h=12, w=40, c_in=64, c1=64, c2=64, n_classes=7)
    both_ways(small, seed=43)
    ragged = WL.small_variant(big, n=2, h=9, w=21, c_in=128, c1=64, c2=128, n_classes=21)
    both_ways(ragged, seed=45)
    both_ways(WL.WORKLOADS["tiny"], seed=47)                  # float32
    both_ways(big, seed=49)                                   # and a large one again


def test_shapes_beyond_the_built_in_scratch_are_refused():
    wl = WL.WORKLOADS["1080p"]
    desc = st.HeadDesc.of(wl)
    assert st.st_workspace_bytes(desc) > st.ST_NOALLOC_MAX_WORKSPACE_MIB << 20
    d = desc.c()
    dummy = C.c_void_p(256)       # never dereferenced: the size check comes first
    assert st.lib().st_head_forward_noalloc(C.byref(d), dummy, dummy, None, None, None) == st.ST_ERR_TOO_LARGE
    assert b"scratch" in st.lib().st_strerror(st.ST_ERR_TOO_LARGE)


def large(shape):
    n, c_in, h, w, c1, c2, classes, compute, feat, nhwc = shape
    wl = WL.small_variant(WL.WORKLOADS["tiny"], n=n, h=h, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=classes, compute=compute, feat_dtype=feat,
                          n_sites=9)
    desc = st.HeadDesc.of(wl)
    desc.feat_layout = st.ST_NHWC if nhwc else st.ST_NCHW
    assert st.st_workspace_bytes(desc) > st.ST_NOALLOC_MAX_WORKSPACE_MIB << 20
    f = to_dev_features(wl, WL.make_features(wl))
    f = f.permute(0, 2, 3, 1).contiguous() if nhwc else f
    p = torch.from_numpy(WL.make_head_params(wl)).cuda()
    # (biases that tell the channels apart: the ones of a fresh head are zero)
    p += 0.05 * torch.sin(torch.arange(p.numel(), device="cuda", dtype=torch.float32))
    out = []
    for call in (lambda **kw: st.st_head_forward(desc, f, p, workspace=st.new_workspace(desc), **kw),
                 lambda **kw: st.st_head_forward_noalloc(desc, f, p, **kw)):
        z = torch.full((n, classes, h, w), float("nan"), dtype=torch.float32, device="cuda")
        q = torch.full((n, 8 * h, 8 * w), 255, dtype=torch.uint8, device="cuda")
        call(logits_lowres=z, pred=q)
        torch.cuda.synchronize()
        out.append((z.cpu().numpy(), q.cpu().numpy()))
    return out


# (n, c_in, h, w, c1, c2, classes, compute, features, channels last)
@pytest.mark.parametrize("shape", [(1, 96, 180, 320, 48, 48, 9, "bf16", "bf16", False), (2, 20, 150, 161, 96, 24, 5, "bf16", "f32", True),
                                   (1, 64, 160, 200, 64, 192, 21, "bf16", "bf16", False), (1, 24, 300, 401, 20, 40, 9, "f32", "f32", False)])
def test_heads_whose_forward_buffers_fit(shape):
    (z_ref, q_ref), (z, q) = large(shape)
    np.testing.assert_array_equal(z, z_ref)
    np.testing.assert_array_equal(q, q_ref)
    assert np.isfinite(z).all() and len(np.unique(q)) > 1


@pytest.mark.parametrize("shape", [(1, 1, 810, 810, 1, 1, 2, "bf16", "bf16", False), (32, 3, 511, 24, 6, 3, 4, "bf16", "f32", True),
                                   (1, 2, 600, 777, 3, 5, 7, "bf16", "f32", False), (2, 54004, 4, 1, 2, 32, 28, "bf16", "bf16", False),
                                   (8, 26386, 2, 4, 1, 5, 30, "f32", "f32", False)])
def test_heads_whose_padded_buffers_do_not_fit(shape):
    """The products and the rounding points are the same.  A sum of K terms in another order differs by some
    sqrt(K) 2^-24 of its size (K up to 486 036: 4e-5).  On the bfloat16 path that turns the rounding of one activation
    in a few thousand by 2^-8 of it, which moves a logit by at most that share of its size, and its neighbours'
    by nothing: the bulk of the logits agrees to float32 accuracy."""
    (z_ref, q_ref), (z, q) = large(shape)
    assert np.isfinite(z).all()
    scale = float(np.max(np.abs(z_ref)))
    diff = np.abs(z - z_ref) / scale
    assert diff.max() < (1e-4 if shape[7] == "f32" else 2 ** -7)
    assert np.quantile(diff, 0.9) < 1e-4
    assert np.mean(q != q_ref) < 1e-3       # (pixels whose two best classes tie to that accuracy)
