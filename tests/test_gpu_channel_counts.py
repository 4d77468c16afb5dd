"""Channel counts that are no multiple of a matrix-core tile, and counts beyond one block's run of
channels: every layer width around the edges of the padding, against the oracle."""
import numpy as np
import pytest

import workloads as WL
from gpu_util import check_staged_bit_exact, rel_err, run_gpu, run_oracle, update_err

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
