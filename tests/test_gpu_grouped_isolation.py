"""Clients of a grouped call are apart: whatever one client's features or head hold, infinities and NaN included, every
other client's head, optimiser state, losses, metric and class map are bit for bit what they are beside a finite neighbour."""
import pytest

import paper_2003_10735_amd as st

pytestmark = pytest.mark.gpu

# n, h, w, c_in, c1, c2: odd and even rows (a head's last pair of rows ends inside or behind its frame), a pitch above and below the 64
# positions of a block of the classifier's backward launch, frames of less than one block, tile columns beside each other
SHAPES = [(3, 9, 35, 64, 64, 64), (3, 3, 5, 64, 128, 64), (3, 13, 31, 64, 64, 128), (2, 45, 80, 128, 64, 64), (3, 6, 10, 64, 64, 64), (2, 61, 107, 64, 64, 64),
          (2, 5, 300, 64, 64, 64)]


@pytest.mark.parametrize("what", ["first row of features", "all features", "first layer", "second layer"])
@pytest.mark.parametrize("n,h,w,c_in,c1,c2", SHAPES)
def test_a_client_does_not_reach_another(n, h, w, c_in, c1, c2, what):
    import torch
    C, steps = 7, 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(h * 1000 + w)
    d = st.HeadDesc(n, c_in, h, w, c1, c2, C, feat_dtype=st.ST_BF16, compute=st.ST_COMPUTE_BF16, grouped=1)
    f = torch.randn((n, c_in, h, w), generator=gen, device="cuda").clamp(min=0).bfloat16()
    lab = torch.randint(0, C, (n, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    heads = torch.stack([torch.cat([torch.randn(r * k, generator=gen, device="cuda") * (2.0 / k) ** 0.5
                                    for r, k in ((c1, 9 * c_in), (1, c1), (c2, 9 * c1), (1, c2), (C, c2), (1, C))]) for _ in range(n)])

    def run(bad):
        fs, ps, vel = f.clone(), heads.clone(), torch.zeros_like(heads)
        if bad is not None:
            if what == "first layer":      # (some of its activations, of the size of 1, run to infinity)
                ps[bad, :c1 * c_in * 9] *= 2e38
            elif what == "second layer":
                ps[bad, c1 * c_in * 9 + c1:c1 * c_in * 9 + c1 + c2 * c1 * 9] *= 2e38
            elif what == "all features":
                fs[bad] = float("nan")
            else:
                fs[bad, :, 0] = float("inf")
        losses = torch.zeros((steps + 1, n), device="cuda")
        mious = torch.zeros((steps + 1, n), dtype=torch.float64, device="cuda")
        pred = torch.zeros((n, 8 * h, 8 * w), dtype=torch.uint8, device="cuda")
        st.st_partial_distill(d, fs, lab, ps, steps, 0.01, momentum=0.9, velocity=vel, losses=losses, mious=mious, pred=pred)
        z = torch.empty((n, C, h, w), device="cuda")
        st.st_head_forward(d, fs, ps, logits_lowres=z)
        torch.cuda.synchronize()
        return dict(params=ps, velocity=vel, losses=losses.t(), mious=mious.t(), pred=pred, logits=z)

    clean = run(None)
    assert all(torch.isfinite(clean[k]).all() for k in ("params", "velocity", "losses", "logits"))
    for bad in range(n):
        got = run(bad)
        assert not torch.isfinite(got["params"][bad]).all()
        for k, v in got.items():
            for client in range(n):
                if client != bad:
                    assert torch.equal(v[client], clean[k][client]), (k, "of client", client, "beside", bad)
