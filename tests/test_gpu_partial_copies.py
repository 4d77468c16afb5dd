"""The optimiser launch adds the partial gradients of the 3x3 layers in ascending order, whatever their number: the gradient that a step
of momentum leaves as velocity is, bit for bit, that sum of the copies in the workspace."""
import pytest

import paper_2003_10735_amd as st

pytestmark = pytest.mark.gpu


# n, h, w, c_in, c1, c2, grouped -> copies of layer 1 and layer 2
@pytest.mark.parametrize("n,h,w,c_in,c1,c2,grouped,copies", [
    (1, 3, 5, 64, 64, 64, 0, (1, 1)), (2, 16, 24, 64, 64, 64, 0, (2, 2)), (4, 90, 160, 256, 128, 128, 1, (2, 4)), (2, 33, 57, 128, 128, 128, 1, (3, 3)),
    (1, 33, 57, 64, 64, 64, 0, (4, 4)), (2, 24, 40, 64, 64, 64, 0, (5, 5)), (2, 45, 80, 128, 64, 64, 1, (6, 6)), (2, 33, 57, 128, 128, 128, 0, (7, 7)),
    (1, 60, 107, 128, 128, 128, 0, (8, 8)), (1, 45, 80, 64, 64, 64, 0, (9, 9)), (2, 60, 107, 128, 64, 64, 1, (10, 10)), (1, 60, 107, 192, 64, 64, 0, (11, 11)),
    (2, 45, 80, 96, 48, 48, 0, (13, 13)), (1, 60, 107, 64, 64, 64, 0, (14, 14)), (2, 45, 80, 64, 64, 64, 0, (15, 15)), (1, 75, 100, 64, 64, 64, 0, (16, 16))])
def test_copies_are_added_in_ascending_order(n, h, w, c_in, c1, c2, grouped, copies):
    import torch
    C, heads = 5, n if grouped else 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(h * 1000 + w)
    d = st.HeadDesc(n, c_in, h, w, c1, c2, C, feat_dtype=st.ST_BF16, compute=st.ST_COMPUTE_BF16, grouped=grouped)
    lay = st.st_get_workspace_layout(d)
    assert tuple(lay["splits"][:2]) == copies
    f = torch.randn((n, c_in, h, w), generator=gen, device="cuda").clamp(min=0).bfloat16()
    lab = torch.randint(0, C, (n, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    blocks = ((c1, 9 * c_in), (1, c1), (c2, 9 * c1), (1, c2), (C, c2), (1, C))
    params = torch.stack([torch.cat([torch.randn(r * k, generator=gen, device="cuda") * (2.0 / k) ** 0.5 for r, k in blocks]) for _ in range(heads)])
    vel, ws = torch.zeros_like(params), st.new_workspace(d)
    st.st_partial_distill(d, f, lab, params, 1, 0.0, momentum=0.5, velocity=vel, workspace=ws)
    torch.cuda.synchronize()
    held, stride = lay["grad_copies"], lay["grad_stride"]
    grad = ws[lay["grad"]:lay["grad"] + heads * held * stride * 4].view(torch.float32).reshape(heads, held, stride)
    at = 0
    for co, ci, number in ((c1, c_in, copies[0]), (c2, c1, copies[1])):
        for size, weights in ((co * ci * 9, True), (co, False)):
            want = grad[:, 0, at:at + size].clone()
            for k in range(1, number):
                want += grad[:, k, at:at + size]
            if weights:                       # (kept with the input channels fastest)
                want = want.reshape(heads, co, 9, ci).transpose(2, 3).reshape(heads, -1)
            assert want.abs().max() > 0 and torch.equal(vel[:, at:at + size], want), (co, ci, weights)
            at += size
