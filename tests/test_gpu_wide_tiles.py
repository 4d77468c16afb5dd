"""The wide-tile convolution (96 positions x 128 channels per block), which grids of more than one round of
small tiles run with: each epilogue, last tiles that reach behind the grid, channel tiles that are half filled, several heads; its
sums are those of the small tiles."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2003_10735_amd as st
import workloads as WL
from gpu_util import check_staged_bit_exact, rel_err, run_gpu, run_oracle, to_dev_features, update_err
from test_gpu_grouped import SGD, inputs, run_grouped

pytestmark = pytest.mark.gpu

# n, h, w, c_in, c1, c2, classes; positions per wide tile (0: small tiles) of layer 1 / layer 2 with the classifier / its data
# gradient / the data gradient of layer 1
SHAPES = [
    (2, 100, 178, 64, 256, 128, 21),     # 96 / 96 / 96 / 0
    (1, 120, 213, 64, 192, 192, 5),      # 96 / 0 / 0 / 0, every second channel tile half filled
    (3, 75, 161, 320, 192, 128, 32),     # 0 / 96 / 96 / 96, half filled
    (1, 101, 181, 192, 128, 128, 2),     # 96 / 96 / 96 / 0
    (1, 90, 160, 256, 128, 128, 19),     # 0 / 0 / 0 / 0
]


@pytest.mark.parametrize("shape", SHAPES)
def test_wide_tiles(shape):
    """One step and the feature gradient against the oracle with the same rounding points: losses and weights to the 5e-4
    of every bfloat16 test; the update to 1e-3 of its largest entry, as at the full sizes (an activation whose sign the order of
    a sum decides moves an entry by one position's share, and there are 14 400 positions and more); the feature
    gradient to 5e-3 in the 2-norm (its sums run over channels, so a mask that turns switches whole elements)."""
    n, h, w, c_in, c1, c2, classes = shape
    wl = WL.small_variant(WL.WORKLOADS["720p"], n=n, h=h, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=classes, steps=1, lr=0.05)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    gpu = run_gpu(wl, f, lab, p)
    check_staged_bit_exact(wl, gpu, lab)
    ora = run_oracle(wl, f, lab, p, bf16_operands=True)
    assert rel_err(gpu["losses"], ora["losses"]) < 5e-4
    assert rel_err(gpu["params"], ora["params"]) < 5e-4
    assert update_err(f"wide tiles {shape}", gpu["params"] - p, ora["params"] - p) < 1e-3
    pt = torch.from_numpy(p).cuda()
    df = torch.zeros((n, c_in, h, w), dtype=torch.float32, device="cuda")
    st.st_partial_distill(st.HeadDesc.of(wl), to_dev_features(wl, f), torch.from_numpy(lab).cuda(), pt, 1, 0.05, feature_grad=df)
    np.testing.assert_array_equal(pt.cpu().numpy(), gpu["params"])
    _, _, df_o = O.feature_grad(O.desc_of(wl, True), WL.features_as_f64(wl, f), lab, p.astype(np.float64))
    d = df.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(d - df_o) < 5e-3 * np.linalg.norm(df_o)


@pytest.mark.parametrize("n,h,w", [(5, 61, 90), (3, 62, 97)])      # no tile across two heads
def test_wide_tiles_of_several_heads(n, h, w):
    wl = WL.small_variant(WL.WORKLOADS["720p"], n=n, h=h, w=w, c_in=64, c1=128, c2=128, n_classes=9, steps=2, lr=0.05, momentum=0.9)
    f, lab, p = inputs(wl)
    g = run_grouped(wl, f, lab, p, 2)
    ora = O.partial_distill_grouped(O.desc_of(wl, True), WL.features_as_f64(wl, f), lab, p.astype(np.float64), 2, SGD(wl))
    for i in range(n):
        assert rel_err(g["losses"][:, i], ora["losses"][:, i]) < 5e-4, i
        assert rel_err(g["params"][i], ora["params"][i]) < 5e-4, i
        assert rel_err(g["params"][i] - p[i], ora["params"][i] - p[i]) < 2e-3, i     # (5 600 positions)


@pytest.mark.parametrize("h,w,c_in,c1,c2,classes", [(62, 97, 256, 256, 256, 21), (75, 110, 192, 192, 192, 32)])   # (half-filled tiles)
def test_a_frame_alone_and_in_a_batch(h, w, c_in, c1, c2, classes):
    """A frame alone runs on small tiles, four of it on wide ones, every layer and direction: logits and feature gradient are the same bit for
    bit (the latter times four, from the mean over four times the pixels)."""
    res = []
    for n in (1, 4):
        wl = WL.small_variant(WL.WORKLOADS["720p"], n=n, h=h, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=classes, steps=1, lr=0.0)
        wl1 = WL.small_variant(wl, n=1)
        f, lab = np.repeat(WL.make_features(wl1), n, axis=0), np.repeat(WL.make_labels(wl1), n, axis=0)
        d, fd, pd = st.HeadDesc.of(wl), to_dev_features(wl, f), torch.from_numpy(WL.make_head_params(wl1)).cuda()
        z = torch.empty((n, classes, h, w), dtype=torch.float32, device="cuda")
        st.st_head_forward(d, fd, pd, z, None)
        df = torch.zeros((n, c_in, h, w), dtype=torch.float32, device="cuda")
        st.st_partial_distill(d, fd, torch.from_numpy(lab).cuda(), pd, 1, 0.0, feature_grad=df)
        res.append((z.cpu().numpy(), n * df.cpu().numpy()))
    (z1, df1), (z4, df4) = res
    assert np.abs(z1).max() > 0 and np.abs(df1).max() > 0
    for i in range(4):
        np.testing.assert_array_equal(z4[i], z1[0])
        np.testing.assert_array_equal(df4[i], df1[0])
