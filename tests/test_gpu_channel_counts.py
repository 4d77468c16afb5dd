"""Channel counts that are no multiple of a matrix-core tile, and counts beyond one block's run of
channels: every layer width around the edges of the padding, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2003_10735_amd as st
import workloads as WL
from gpu_util import check_staged_bit_exact, rel_err, run_gpu, run_oracle, to_dev_features, update_err
from test_gpu_parity import check_adam

pytestmark = pytest.mark.gpu

# (c_in, c1, c2, classes, h, w, frames)
SHAPES = [(1, 1, 1, 2, 3, 5, 1), (33, 31, 65, 9, 7, 19, 1), (64, 63, 64, 19, 5, 33, 2), (65, 96, 40, 21, 9, 8, 1),
          (7, 130, 192, 32, 6, 11, 1), (24, 16, 320, 5, 4, 9, 2), (16, 40, 384, 12, 5, 6, 1)]


@pytest.mark.parametrize("compute", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_channel_counts(shape, compute):
    c_in, c1, c2, classes, h, w, n = shape
    wl = WL.small_variant(WL.WORKLOADS["tiny"], n=n, h=h, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=classes, steps=2, lr=0.02,
                          momentum=0.9, compute=compute, feat_dtype=compute, n_sites=6)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    gpu = run_gpu(wl, f, lab, p)
    check_staged_bit_exact(wl, gpu, lab)
    ora = run_oracle(wl, f, lab, p, bf16_operands=compute == "bf16")
    tol, update_tol = (1e-4, 2e-3) if compute == "f32" else (5e-4, 3e-2)
    assert rel_err(gpu["losses"], ora["losses"]) < tol
    assert rel_err(gpu["params"], ora["params"]) < tol
    assert update_err(f"channels {shape} {compute}", gpu["params"] - p, ora["params"] - p) < update_tol
    # the loop with exits hands the metric over with the backward pass already queued behind it
    early = run_gpu(wl, f, lab, p, threshold=1.5)
    np.testing.assert_array_equal(early["params"], gpu["params"])
    np.testing.assert_array_equal(early["losses"], gpu["losses"])


# 40 x 60 cells make 84 position tiles: 336 tiles of a launch for 97 output channels (eight wavefronts
# each), 588 for 203 (four); SHAPES above all stay below 256 (sixteen)
@pytest.mark.parametrize("c_in,c1,c2", [(97, 97, 203), (203, 203, 97)])
def test_f32_convolutions_with_four_and_eight_wavefronts(c_in, c1, c2):
    """Every epilogue of the float32 convolution (layer 1, layer 2 with the classifier, both data gradients) with four and
    with eight wavefronts per tile.  Sums of up to 9 * 203 float32 products: 1e-4, as everywhere on this path."""
    wl = WL.small_variant(WL.WORKLOADS["tiny"], h=40, w=60, c_in=c_in, c1=c1, c2=c2, n_classes=11, steps=1, lr=1.0, n_sites=20)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    pt = torch.from_numpy(p).cuda()
    df = torch.zeros((wl.n, c_in, wl.h, wl.w), dtype=torch.float32, device="cuda")
    losses = torch.zeros(2, dtype=torch.float32, device="cuda")
    st.st_partial_distill(st.HeadDesc.of(wl), to_dev_features(wl, f), torch.from_numpy(lab).cuda(), pt, 1, 1.0, losses=losses, feature_grad=df)
    loss, grad, df_o = O.feature_grad(O.desc_of(wl), WL.features_as_f64(wl, f), lab, p.astype(np.float64))
    assert abs(float(losses[0]) - loss) < 1e-4 * loss
    step = p - pt.cpu().numpy()          # lr = 1: the gradient, rounded where the new weight is (2^-24 of it)
    for name, sl in WL.param_slices(wl).items():
        assert np.abs(step[sl] - grad[sl]).max() < 1e-4 * np.abs(grad[sl]).max() + 2 ** -23 * np.abs(p[sl]).max(), name
    assert rel_err(df.cpu().numpy(), df_o) < 1e-4


@pytest.mark.parametrize("feat", ["f32", "bf16"])
@pytest.mark.parametrize("c_in", [20, 40, 96, 128])
def test_channels_last_features_of_any_count(c_in, feat):
    """bfloat16 path, features [n, h, w, c_in]: counts that are no multiple of eight (element by element), that leave a
    64-channel tile partly filled, and that fill it; both element types give what [n, c_in, h, w] gives, bit for bit."""
    wl = WL.small_variant(WL.WORKLOADS["720p"], n=2, c_in=c_in, h=7, w=19, c1=40, c2=64, n_classes=6, steps=2, n_sites=9, feat_dtype=feat)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    fd, results = to_dev_features(wl, f), []
    for layout in (st.ST_NCHW, st.ST_NHWC):
        desc = st.HeadDesc.of(wl)
        desc.feat_layout = layout
        pt = torch.from_numpy(p).cuda()
        z = torch.empty((wl.n, wl.n_classes, wl.h, wl.w), dtype=torch.float32, device="cuda")
        feats = fd if layout == st.ST_NCHW else fd.permute(0, 2, 3, 1).contiguous()
        st.st_partial_distill(desc, feats, torch.from_numpy(lab).cuda(), pt, wl.steps, wl.lr)
        st.st_head_forward(desc, feats, pt, z, None)
        torch.cuda.synchronize()
        results.append((pt.cpu().numpy(), z.cpu().numpy()))
    for a, b in zip(*results):
        np.testing.assert_array_equal(a, b)
    ora = run_oracle(wl, f, lab, p, bf16_operands=True)
    assert rel_err(results[1][0], ora["params"]) < 5e-4


@pytest.mark.parametrize("compute", ["f32", "bf16"])
def test_padded_head_with_adam_weights_and_graph(compute):
    wl = WL.small_variant(WL.WORKLOADS["tiny"], n=2, h=9, w=35, c_in=20, c1=33, c2=24, n_classes=6, steps=3, lr=0.01, compute=compute,
                          feat_dtype=compute, n_sites=9)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    tol = (1e-4, 1e-3) if compute == "f32" else (2e-3, 2e-2)
    check_adam(wl, f, lab, p, 3, compute == "bf16", *tol, object_radius=3)
    # the same call through the launch graph, replayed with other work in between
    desc, fd, lt, stream = st.HeadDesc.of(wl), to_dev_features(wl, f), torch.from_numpy(lab).cuda(), torch.cuda.Stream()
    ws, wts = st.new_workspace(desc), st.st_object_weights(lt, wl.n_classes, 3)
    live, losses = torch.zeros((3, p.size), dtype=torch.float32, device="cuda"), torch.zeros(4, dtype=torch.float32, device="cuda")
    st.st_graph_cache_clear()

    def call(graph):
        live.zero_(); losses.zero_()
        live[0].copy_(torch.from_numpy(p))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            st.st_partial_distill(desc, fd, lt, live[0], 3, wl.lr, losses=losses, workspace=ws, adam=dict(m=live[1], v=live[2]), pixel_weights=wts,
                                  graph=graph, stream=stream)
        torch.cuda.synchronize()
        return live.cpu().numpy(), losses.cpu().numpy()
    want = call(False)
    for _ in range(3):
        for a, b in zip(call(True), want):
            np.testing.assert_array_equal(a, b)
    assert st.st_graph_cache_size() == 1
    st.st_graph_cache_clear()
