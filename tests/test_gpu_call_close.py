"""The launches that close a step and a call, where their work splits: parameters out and in again for channel counts that are no
multiple of anything, class counts around eight threads a class, and more tile losses than one trip of a thread takes."""
import numpy as np
import pytest

import workloads as WL
from gpu_util import check_staged_bit_exact, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("compute,c_in,c1,c2,classes,h,w", [
    ("f32", 1, 1, 2, 2, 3, 5), ("f32", 1, 3, 1, 2, 130, 500),        # (130 x 16 tiles: nine tile losses a thread)
    ("f32", 3, 1, 4, 31, 9, 33), ("f32", 5, 9, 7, 8, 20, 40), ("bf16", 64, 64, 64, 32, 33, 40), ("bf16", 96, 48, 40, 9, 17, 70)])
def test_round_trip_metric_and_loss(compute, c_in, c1, c2, classes, h, w):
    wl = WL.small_variant(WL.WORKLOADS["720p" if compute == "bf16" else "tiny"], n=1, h=h, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=classes,
                          steps=1, lr=0.0, momentum=0.5, n_sites=11, compute=compute, feat_dtype=compute)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    vel = np.random.default_rng(w).standard_normal(p.shape).astype(np.float32)
    gpu, ora = run_gpu(wl, f, lab, p, velocity=vel), run_oracle(wl, f, lab, p, bf16_operands=compute == "bf16", velocity=vel.astype(np.float64))
    np.testing.assert_array_equal(gpu["params"], p)               # (a step of length zero)
    tol = 1e-4 if compute == "f32" else 5e-4                      # as everywhere on these paths
    assert rel_err(gpu["velocity"], ora["velocity"]) < tol
    assert rel_err(gpu["losses"], ora["losses"]) < tol
    assert gpu["mious"][0, 0] == gpu["mious"][1, 0]               # (both passes see the same head; counts cleared between)
    check_staged_bit_exact(wl, gpu, lab)
