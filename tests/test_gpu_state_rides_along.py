"""The optimiser's state in and out with the first and the last launch of a call: every vector, every head, odd channel counts
(one parameter per thread), and vectors of the caller that overlap."""
import pytest
import torch

import paper_2003_10735_amd as st
import workloads as WL
from gpu_util import to_dev_features

pytestmark = pytest.mark.gpu


def _call(compute, n, c_in, c1, c2, grouped):
    wl = WL.small_variant(WL.WORKLOADS["720p" if compute == "bf16" else "tiny"], n=n, h=7, w=24, c_in=c_in, c1=c1, c2=c2, n_classes=5, steps=2,
                          lr=0.02, n_sites=7, compute=compute, feat_dtype=compute)
    desc = st.HeadDesc.of(wl)
    desc.grouped = int(grouped)
    one = torch.from_numpy(WL.make_head_params(wl)).cuda()
    p = torch.cat([one * (1 + 0.1 * k) for k in range(n)]) if grouped else one
    return desc, to_dev_features(wl, WL.make_features(wl)), torch.from_numpy(WL.make_labels(wl)).cuda(), p


CASES = [("bf16", 1, 64, 64, 64, False), ("bf16", 1, 48, 40, 24, False), ("f32", 1, 7, 9, 5, False), ("f32", 2, 24, 36, 20, False),
         ("bf16", 3, 64, 64, 64, True)]


@pytest.mark.parametrize("compute,n,c_in,c1,c2,grouped", CASES)
def test_no_step_hands_back_what_came_in(compute, n, c_in, c1, c2, grouped):
    """Zero steps: in and out again, bit for bit, momentum and Adam."""
    desc, f, lab, p = _call(compute, n, c_in, c1, c2, grouped)
    gen = torch.Generator(device="cuda").manual_seed(1)
    vecs = [torch.rand(p.shape, device="cuda", generator=gen) for _ in range(2)]
    for adam in (False, True):
        got = [p.clone(), vecs[0].clone(), vecs[1].clone()]
        opt = dict(adam=dict(m=got[1], v=got[2])) if adam else dict(momentum=0.9, velocity=got[1])
        st.st_partial_distill(desc, f, lab, got[0], 0, 0.01, **opt)
        for x, y in zip(got, [p] + vecs):
            assert torch.equal(x, y)


@pytest.mark.parametrize("compute,n,c_in,c1,c2,grouped", CASES)
def test_two_calls_of_one_step_are_one_call_of_two(compute, n, c_in, c1, c2, grouped):
    """The state travels out and in again between the calls: bit for bit the same."""
    desc, f, lab, p = _call(compute, n, c_in, c1, c2, grouped)
    for adam in (False, True):
        ends = []
        for parts in ((2,), (1, 1)):
            x, a, b, t = p.clone(), torch.zeros_like(p), torch.zeros_like(p), 0
            for k in parts:
                opt = dict(adam=dict(m=a, v=b, t0=t)) if adam else dict(momentum=0.9, velocity=a)
                st.st_partial_distill(desc, f, lab, x, k, 0.02, **opt)
                t += k
            ends.append((x, a, b))
        for u, v in zip(*ends):
            assert torch.equal(u, v)
        assert float(ends[0][1].abs().max()) > 0


def test_overlapping_state_vectors_keep_their_order():
    """One vector as both of Adam's moments: it comes back as the second moment, which is written last."""
    desc, f, lab, p = _call("bf16", 1, 64, 64, 64, False)
    x, y, both = p.clone(), p.clone(), torch.zeros_like(p)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    st.st_partial_distill(desc, f, lab, x, 2, 0.02, adam=dict(m=m, v=v))
    st.st_partial_distill(desc, f, lab, y, 2, 0.02, adam=dict(m=both, v=both))
    assert torch.equal(x, y) and torch.equal(both, v) and not torch.equal(m, v)
