"""Gradient of the 1x1 classifier from its slots of 64 positions: eight runs of them per value, added 8, 16 or 32 at a time; how exactly
many of them add up."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2003_10735_amd as st
import workloads as WL
from gpu_util import to_dev_features

pytestmark = pytest.mark.gpu


# a run of 1, 8, 9, 16, 17, 32, 33, 49 and 58 slots; `short`: how many slots the last run has fewer
@pytest.mark.parametrize("short", [0, 5])
@pytest.mark.parametrize("per", [1, 8, 9, 16, 17, 32, 33, 49, 58])
def test_every_length_of_a_run(per, short):
    """64 positions of the padded grid are one of its rows here, so h + 2 rows are h + 2 slots.  A slot left out or added twice moves
    the gradient by 1 / 464 or more of its 2-norm; the float32 path is right to 1e-4 of it, as everywhere, and the new weight
    rounds by 2^-24 of itself."""
    h = 8 * per - 2 - short
    if h < 1:
        pytest.skip("no grid that small")
    wl = WL.small_variant(WL.WORKLOADS["tiny"], h=h, w=62, c_in=8, c1=16, c2=24, n_classes=3, steps=1, lr=1.0, n_sites=20)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    pt = torch.from_numpy(p).cuda()
    st.st_partial_distill(st.HeadDesc.of(wl), to_dev_features(wl, f), torch.from_numpy(lab).cuda(), pt, 1, 1.0)
    _, grad, *_ = O.loss_and_grad(O.desc_of(wl), WL.features_as_f64(wl, f), lab, p.astype(np.float64))
    step = p.astype(np.float64) - pt.cpu().numpy()
    for name in ("W3", "b3"):
        sl = WL.param_slices(wl)[name]
        assert np.linalg.norm(step[sl] - grad[sl]) < 1e-4 * np.linalg.norm(grad[sl]) + 2.0 ** -24 * np.linalg.norm(p[sl]), name


def test_many_slots_add_up_as_exactly_as_few():
    """W3's gradient over 964 slots where everything in front of the sum is exact but for a few roundings: both layers hand the features on
    (one tap of 1, multiples of 1 / 16), and the logits are zero.  A column keeps its
    class for 64 cells.  Against float64, 2-norm: 1.35e-7; 1.66e-7 with 16 runs of slots added one after the other, 2.03e-7 with eight."""
    h = 962
    wl = WL.small_variant(WL.WORKLOADS["tiny"], h=h, w=62, c_in=16, c1=16, c2=16, n_classes=31, steps=1, lr=1.0)
    sl, rng = WL.param_slices(wl), np.random.default_rng(5)
    f = (rng.integers(0, 100, (1, 16, h, 62)) / 16).astype(np.float32)
    cells = np.repeat(rng.integers(0, 31, (1, h // 64 + 1, 62)), 64, axis=1)[:, :h]
    lab = np.kron(cells, np.ones((8, 8))).astype(np.int32)
    p = np.zeros_like(WL.make_head_params(wl))
    tap = np.zeros((16, 16, 3, 3), dtype=p.dtype)
    tap[np.arange(16), np.arange(16), 1, 1] = 1
    p[sl["W1"]] = p[sl["W2"]] = tap.reshape(-1)
    pt = torch.from_numpy(p).cuda()
    st.st_partial_distill(st.HeadDesc.of(wl), torch.from_numpy(f).cuda(), torch.from_numpy(lab).cuda(), pt, 1, 1.0)
    _, grad, *_ = O.loss_and_grad(O.desc_of(wl), f.astype(np.float64), lab, p.astype(np.float64), want_metric=False)
    got, want = -pt.cpu().numpy()[sl["W3"]].astype(np.float64), grad[sl["W3"]]
    assert np.linalg.norm(got - want) < 1.7e-7 * np.linalg.norm(want)
