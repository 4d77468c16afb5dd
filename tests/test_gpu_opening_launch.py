"""The launch that opens a call, where its tiles end: label blocks of 31 cells, packing tiles of 64 columns, padded channels.
The workspace starts as all ones (NaN as a float, 255 as a byte): what the launch ought to clear and does not shows up."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2003_10735_amd as st
import workloads as WL
from gpu_util import rel_err, to_dev_features

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("compute,c_in,c1,c2", [("bf16", 64, 64, 64), ("bf16", 128, 96, 40), ("f32", 24, 33, 20)])
@pytest.mark.parametrize("w", [1, 8, 30, 31, 32, 56, 62, 63, 64, 72, 93, 128])
def test_widths_around_the_tiles(w, compute, c_in, c1, c2):
    wl = WL.small_variant(WL.WORKLOADS["720p" if compute == "bf16" else "tiny"], n=2, h=3, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=7, steps=1,
                          lr=0.02, n_sites=7, compute=compute, feat_dtype=compute)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    rng = np.random.default_rng(w)
    lab[rng.random(lab.shape) < 0.1] = 255                       # (no class index: not counted)
    lab[:, ::5, ::3] = rng.integers(0, 7, lab[:, ::5, ::3].shape)    # many short runs down a column
    wts = rng.integers(0, 6, lab.shape).astype(np.uint8)
    desc, fd = st.HeadDesc.of(wl), to_dev_features(wl, f)
    ws = torch.full_like(st.new_workspace(desc), 255)
    pt, losses = torch.from_numpy(p).cuda(), torch.zeros(2, dtype=torch.float32, device="cuda")
    df = torch.zeros((2, c_in, 3, w), dtype=torch.float32, device="cuda")
    st.st_partial_distill(desc, fd, torch.from_numpy(lab).cuda(), pt, 1, wl.lr, losses=losses, workspace=ws,
                          pixel_weights=torch.from_numpy(wts).cuda(), feature_grad=df)
    loss, grad, *_ = O.loss_and_grad(O.with_pixel_weights(O.desc_of(wl, compute == "bf16"), wts), WL.features_as_f64(wl, f), lab,
                                     p.astype(np.float64))
    tol = 1e-4 if compute == "f32" else 5e-4                     # as everywhere on these paths
    assert abs(float(losses[0]) - loss) < tol * loss
    assert rel_err(pt.cpu().numpy(), p - wl.lr * grad) < tol
    assert np.isfinite(df.cpu().numpy()).all()
    z = torch.empty((2, 7, 3, w), dtype=torch.float32, device="cuda")
    zs = []
    for fill in (255, 0):                                        # the forward call opens with the same launch
        ws.fill_(fill)
        st.st_head_forward(desc, fd, pt, z, None, workspace=ws)
        zs.append(z.cpu().numpy().copy())
    np.testing.assert_array_equal(zs[0], zs[1])
    zo, _ = O.head_forward(O.desc_of(wl, compute == "bf16"), WL.features_as_f64(wl, f), pt.cpu().numpy().astype(np.float64), want_pred=False)
    # (2-norm: an activation that rounds the other way, one in some ten thousand, moves the logits of its cells by up to
    #  2^-8 of one of the 40 to 64 products they are sums of -- 2e-3 of such a logit, nothing of the others)
    assert np.linalg.norm(zs[0] - zo) < (1e-5 if compute == "f32" else 5e-4) * np.linalg.norm(zo)
