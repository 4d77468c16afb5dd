"""Gradient of the classifier's weights and bias, a sum over the backward launch's blocks of 64 positions, for as many blocks as fewer than,
exactly and more than the eight runs they are dealt out in: against float64 products of the activations the kernel read and the gradient
of the very logits it left, and the gradient it handed on, zero wherever there is no cell."""
import pytest

import paper_2003_10735_amd as st

pytestmark = pytest.mark.gpu

# n, h, w, c2, grouped: 1, 1, 2, 7, 8, 9, 15, 17, 26 blocks; several heads of 2, 3 and 9
SHAPES = [(1, 1, 1, 64, 0), (1, 2, 14, 128, 0), (1, 3, 22, 64, 0), (1, 12, 30, 64, 0), (1, 14, 30, 192, 0), (2, 4, 46, 64, 0), (1, 13, 62, 256, 0),
          (1, 15, 62, 128, 0), (1, 24, 62, 320, 0), (3, 6, 13, 64, 1), (5, 6, 21, 128, 1), (3, 12, 38, 64, 1)]


@pytest.mark.parametrize("n,h,w,c2,grouped", SHAPES)
def test_classifier_gradient_is_the_sum_over_all_blocks(n, h, w, c2, grouped):
    import torch
    C, c_in, c1 = 7, 64, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(h * 1000 + w)
    d = st.HeadDesc(n, c_in, h, w, c1, c2, C, feat_dtype=st.ST_BF16, compute=st.ST_COMPUTE_BF16, grouped=grouped)
    heads = n if grouped else 1
    ws = torch.full((st.st_workspace_bytes(d),), 0xFF, dtype=torch.uint8, device="cuda")
    f = torch.randn((n, c_in, h, w), generator=gen, device="cuda").clamp(min=0).bfloat16()
    lab = torch.randint(0, C, (n, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    one = [torch.randn(r * k, generator=gen, device="cuda") * (2.0 / k) ** 0.5 if b == 0 else torch.zeros(r, device="cuda")
           for r, k in ((c1, 9 * c_in), (c2, 9 * c1), (C, c2)) for b in (0, 1)]
    before = torch.cat(one * heads)
    # no step: the logits that the step below starts from
    st.st_partial_distill(d, f, lab, before.clone(), 0, 0.0, workspace=ws)
    torch.cuda.synchronize()
    lay = st.st_get_workspace_layout(d)
    Wp, Hp = lay["row_pitch"], h + 2
    z = ws[lay["z"]:lay["z"] + n * C * h * w * 4].view(torch.float32).reshape(n, C, h, w).double().cpu().requires_grad_(True)
    up = torch.nn.functional.interpolate(z, scale_factor=8, mode="bilinear", align_corners=False)
    loss = torch.nn.functional.cross_entropy(up, lab.long().cpu(), reduction="sum") / (n // heads * 64 * h * w)
    g, = torch.autograd.grad(loss, z)
    lr = 1.0
    after = before.clone()
    st.st_partial_distill(d, f, lab, after, 1, lr, workspace=ws)
    torch.cuda.synchronize()
    # (the last forward pass of that call has overwritten a2: the step before it is repeated without an update)
    keep = before.clone()
    st.st_partial_distill(d, f, lab, keep, 1, 0.0, workspace=ws)
    torch.cuda.synchronize()
    k2 = (c2 + 63) // 64 * 64
    a2, da2 = (ws[lay[m]:lay[m] + n * Hp * Wp * k2 * 2].view(torch.bfloat16).reshape(n, Hp, Wp, k2).double().cpu() for m in ("a2", "da2"))
    border = torch.ones(Hp, Wp, dtype=torch.bool)
    border[1:h + 1, 1:w + 1] = False
    assert (da2[:, border] == 0).all() and da2.abs().max() > 0
    a2 = a2[:, 1:h + 1, 1:w + 1, :c2]
    size = before.numel() // heads
    # g enters the product rounded to bfloat16 (2^-9, and the float32 sums behind it far less); the new weight is rounded once
    for k in range(heads):
        gk, ak = (g[k:k + 1], a2[k:k + 1]) if heads > 1 else (g, a2)
        step = (before[k * size:(k + 1) * size].double() - after[k * size:(k + 1) * size].double()).cpu() / lr
        old = before[k * size:(k + 1) * size].double().cpu()
        gm, am = gk.permute(0, 2, 3, 1).reshape(-1, C), ak.reshape(-1, c2)
        at = size - C - C * c2
        want, scale = gm.t() @ am, gm.abs().t() @ am.abs()
        ulp = old.abs().max() * 2.0 ** -23
        assert ((step[at:at + C * c2].reshape(C, c2) - want).abs() <= 2.0 ** -8 * scale + ulp).all(), k
        assert ((step[size - C:] - gm.sum(0)).abs() <= 2.0 ** -8 * gm.abs().sum(0) + ulp).all(), k


# float32: n, h, w, c2, classes -- 1, 7, 9, 26, 60, 256 and 257 blocks; channels short of a run of eight, of a tile of 32 and of the sixteen runs that
# go ahead, as many as a block takes, and two and three blocks of them
F32_SHAPES = [(1, 1, 1, 32, 2), (1, 2, 14, 20, 7), (1, 12, 30, 100, 9), (2, 4, 46, 128, 19), (1, 24, 62, 136, 32), (1, 30, 118, 64, 12), (1, 126, 120, 24, 5), (1, 62, 250, 40, 9),
              (1, 255, 62, 8, 3), (1, 8, 9, 512, 4), (1, 8, 9, 560, 4), (1, 3, 9, 1100, 4)]


@pytest.mark.parametrize("n,h,w,c2,C", F32_SHAPES)
def test_float32_classifier_backward(n, h, w, c2, C):
    import torch
    c_in, c1 = 16, 24
    gen = torch.Generator(device="cuda")
    gen.manual_seed(h * 1000 + w)
    d = st.HeadDesc(n, c_in, h, w, c1, c2, C, feat_dtype=st.ST_F32, compute=st.ST_COMPUTE_F32)
    ws = torch.zeros(st.st_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    f = torch.randn((n, c_in, h, w), generator=gen, device="cuda").clamp(min=0)
    lab = torch.randint(0, C, (n, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    params = torch.cat([torch.randn(r * k, generator=gen, device="cuda") * (2.0 / k) ** 0.5 if b == 0 else torch.zeros(r, device="cuda")
                        for r, k in ((c1, 9 * c_in), (c2, 9 * c1), (C, c2)) for b in (0, 1)])
    # (a step of nothing: the passes before and behind it are the same, and what the backward pass read and left is there to look at)
    st.st_partial_distill(d, f, lab, params.clone(), 1, 0.0, workspace=ws)
    torch.cuda.synchronize()
    lay = st.st_get_workspace_layout(d)
    Wp, Hp, PP = lay["row_pitch"], h + 2, n * (h + 2) * lay["row_pitch"]
    g = ws[lay["g"]:lay["g"] + n * C * h * w * 4].view(torch.float32).reshape(n, C, h, w).double()

    def act(name):
        # runs of eight channels, each as long as the guard columns and the positions between them
        guard = (Wp + 2 + 256 + 7) // 8 * 8
        run = (guard + (PP + 15) // 16 * 16 + guard) * 8
        k = (c2 + 7) // 8
        first = lay[name] // 4
        whole = ws.view(torch.float32)
        return torch.stack([whole[first + r * run:first + r * run + PP * 8].reshape(n, Hp, Wp, 8) for r in range(k)], -2).reshape(n, Hp, Wp, k * 8)[..., :c2].double()
    a2, da2 = act("a2"), act("da2")
    border = torch.ones(Hp, Wp, dtype=torch.bool, device="cuda")
    border[1:h + 1, 1:w + 1] = False
    assert (da2[:, border] == 0).all()
    W3 = params[-C * c2 - C:-C].reshape(C, c2).double()
    inner = lambda x: x[:, 1:h + 1, 1:w + 1].reshape(-1, c2)
    gm = g.permute(0, 2, 3, 1).reshape(-1, C)
    mask = inner(a2) > 0
    # chains of at most C, and of 64 and then all blocks' terms, each rounded to float32
    want, size = (gm @ W3) * mask, (gm.abs() @ W3.abs()) * mask
    assert ((inner(da2) - want).abs() <= (C + 2) * 2.0 ** -24 * size + 1e-38).all()
    grad = ws[lay["grad"]:lay["grad"] + params.numel() * 4].view(torch.float32).double()
    eps = (64 + 64) * 2.0 ** -24
    w3, s3 = gm.t() @ inner(a2), gm.abs().t() @ inner(a2).abs()
    assert ((grad[-C * c2 - C:-C].reshape(C, c2) - w3).abs() <= eps * s3 + 1e-38).all()
    assert ((grad[-C:] - gm.sum(0)).abs() <= eps * gm.abs().sum(0) + 1e-38).all()


@pytest.mark.parametrize("n,h,w,c2,C", F32_SHAPES)
def test_float32_classifier_backward_writes_every_cell(n, h, w, c2, C):
    """Out of a workspace of NaNs: a border cell, a run of channels or a half of a tile that the launch left out would show (the call itself
    clears the guard columns in front of and behind the positions, and none of these)."""
    import torch
    c_in, c1 = 16, 24
    gen = torch.Generator(device="cuda")
    gen.manual_seed(h * 1000 + w)
    d = st.HeadDesc(n, c_in, h, w, c1, c2, C, feat_dtype=st.ST_F32, compute=st.ST_COMPUTE_F32)
    ws = torch.full((st.st_workspace_bytes(d),), 0xFF, dtype=torch.uint8, device="cuda")
    f = torch.randn((n, c_in, h, w), generator=gen, device="cuda").clamp(min=0)
    lab = torch.randint(0, C, (n, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    params = torch.cat([torch.randn(r * k, generator=gen, device="cuda") * (2.0 / k) ** 0.5 if b == 0 else torch.zeros(r, device="cuda")
                        for r, k in ((c1, 9 * c_in), (c2, 9 * c1), (C, c2)) for b in (0, 1)])
    st.st_partial_distill(d, f, lab, params.clone(), 1, 0.0, workspace=ws)
    torch.cuda.synchronize()
    lay = st.st_get_workspace_layout(d)
    Wp, Hp, PP = lay["row_pitch"], h + 2, n * (h + 2) * lay["row_pitch"]
    guard = (Wp + 2 + 256 + 7) // 8 * 8
    run = (guard + (PP + 15) // 16 * 16 + guard) * 8
    k = (c2 + 7) // 8
    first = lay["da2"] // 4
    whole = ws.view(torch.float32)
    da2 = torch.stack([whole[first + r * run:first + r * run + PP * 8].reshape(n, Hp, Wp, 8) for r in range(k)], -2).reshape(n, Hp, Wp, k * 8)
    assert torch.isfinite(da2).all() and da2[..., :c2].abs().max() > 0
    border = torch.ones(Hp, Wp, dtype=torch.bool, device="cuda")
    border[1:h + 1, 1:w + 1] = False
    assert (da2[:, border] == 0).all()
    assert (da2[..., c2:] == 0).all()
