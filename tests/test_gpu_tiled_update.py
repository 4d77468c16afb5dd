"""The optimiser's launch on tiles of 32 x 32 weights (heads of 256 tiles or more whose channel counts are multiples of 32): every parameter gets its own
gradient, once, and the products' copies of the weights are the ones that the next call's opening launch makes of the parameters."""
import pytest
import torch
import torch.nn.functional as F

import paper_2003_10735_amd as st

pytestmark = pytest.mark.gpu

# c_in, c1, c2, heads: rows of one tile, channel counts short of a fragment of 64, more output than input channels and the reverse, 270 tiles; and,
# for the same checks on the way by consecutive parameters, 252 tiles and a channel count that is no multiple of 32
SHAPES = [(32, 256, 256, 1), (256, 224, 32, 1), (352, 160, 32, 1), (160, 224, 96, 1), (256, 256, 256, 1), (64, 256, 256, 3), (224, 224, 32, 1), (128, 160, 64, 1),
          (256, 128, 128, 2), (128, 128, 96, 1), (264, 256, 64, 1)]


@pytest.mark.parametrize("c_in,c1,c2,n", SHAPES)
def test_tiled_update(c_in, c1, c2, n):
    h, w, C, lr = 7, 24, 5, 0.02
    gen = torch.Generator(device="cuda")
    gen.manual_seed(c_in * 1000 + c2)
    d = st.HeadDesc(n, c_in, h, w, c1, c2, C, feat_dtype=st.ST_BF16, compute=st.ST_COMPUTE_BF16, grouped=int(n > 1))
    f = torch.randn((n, c_in, h, w), generator=gen, device="cuda").clamp(min=0).bfloat16()
    lab = torch.randint(0, C, (n, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    shapes = [(c1, c_in, 3, 3), (c1,), (c2, c1, 3, 3), (c2,), (C, c2), (C,)]
    p = torch.cat([torch.randn(s, generator=gen, device="cuda").flatten() * ((2.0 / s[1:].numel()) ** 0.5 if len(s) > 1 else 0.1)
                   for _ in range(n) for s in map(torch.Size, shapes)])

    def run(parts, adam):
        x, a, b, t = p.clone(), torch.zeros_like(p), torch.zeros_like(p), 0
        for k in parts:
            st.st_partial_distill(d, f, lab, x, k, lr, **(dict(adam=dict(m=a, v=b, t0=t)) if adam else dict(momentum=0.9, velocity=a)))
            t += k
        return x, a, b

    # the second step reads the copies that the first one left, or those made of the parameters: bit for bit the same
    for adam in (False, True):
        for u, v in zip(run((2,), adam), run((1, 1), adam)):
            assert torch.equal(u, v)

    if n == 1:
        # with a look at the metric behind every step, which keeps the parameters before the update: the same, and the best ones are some step's
        y, a, best = p.clone(), torch.zeros_like(p), torch.empty_like(p)
        r = st.st_partial_distill(d, f, lab, y, 2, lr, momentum=0.9, velocity=a, threshold=0.9999, best_params=best)
        steps = [(p,), run((1,), False), run((2,), False)]
        assert r[0] == 2 and torch.equal(y, steps[2][0]) and torch.equal(a, steps[2][1])
        assert any(torch.equal(best, q[0]) for q in steps)

    x, g, _ = run((1,), False)
    # w - lr g in one rounding; 2^-23 of either covers that of the product here
    assert ((p.double() - lr * g.double() - x.double()).abs() <= 2.0 ** -23 * (p.abs() + lr * g.abs()).double()).all()
    size = p.numel() // n
    for k in range(n):
        parts, at = [], k * size
        for s in map(torch.Size, shapes):
            parts.append(p[at:at + s.numel()].reshape(s).cpu().requires_grad_(True))
            at += s.numel()
        W1, b1, W2, b2, W3, b3 = parts
        y = F.conv2d(f[k:k + 1].float().cpu(), W1, b1, padding=1).relu()
        y = F.conv2d(y, W2, b2, padding=1).relu()
        z = F.interpolate(F.conv2d(y, W3[:, :, None, None], b3), scale_factor=8, mode="bilinear", align_corners=False)
        F.cross_entropy(z, lab[k:k + 1].long().cpu()).backward()
        at = k * size
        for q in parts:
            got = g[at:at + q.numel()].reshape(q.shape).cpu()
            at += q.numel()
            error = got - q.grad
            # a weight's gradient carries some of the activations' bfloat16 roundings, a few parts of 2^-9, and what a ReLU on the other side
            # makes of them; a tile that is another's is off by more than its own size
            ratio = float(error.norm() / q.grad.norm())
            assert ratio <= 0.1, (k, tuple(q.shape))
            if q.dim() == 4 and q.shape[1] % 32 == 0:
                tiles = lambda t: t.reshape(t.shape[0] // 32, 32, t.shape[1] // 32, 32, 9).permute(0, 2, 4, 1, 3).flatten(3).norm(dim=-1)
                ratio = float((tiles(error) / tiles(q.grad)).max())
                assert ratio <= 0.25, (k, tuple(q.shape))


@pytest.mark.parametrize("c_in,c1,c2", [s[:3] for s in SHAPES if s[3] == 1])
def test_gradient_of_the_features_in_a_second_step(c_in, c1, c2):
    """Its product reads the mirrored copy of layer 1's weights that the first step left; a call of its own for the second step makes that copy
    of the parameters anew: bit for bit the same."""
    h, w, C, lr = 7, 24, 5, 0.02
    gen = torch.Generator(device="cuda")
    gen.manual_seed(c_in * 1000 + c2)
    d = st.HeadDesc(1, c_in, h, w, c1, c2, C, feat_dtype=st.ST_BF16, compute=st.ST_COMPUTE_BF16)
    f = torch.randn((1, c_in, h, w), generator=gen, device="cuda").clamp(min=0).bfloat16()
    lab = torch.randint(0, C, (1, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    p = torch.cat([torch.randn(r * k, generator=gen, device="cuda") * (2.0 / k) ** 0.5 if b == 0 else torch.zeros(r, device="cuda")
                   for r, k in ((c1, 9 * c_in), (c2, 9 * c1), (C, c2)) for b in (0, 1)])

    def run(parts, adam):
        x, a, b, t = p.clone(), torch.zeros_like(p), torch.zeros_like(p), 0
        grad = torch.zeros((1, c_in, h, w), device="cuda")
        for k in parts:
            st.st_partial_distill(d, f, lab, x, k, lr, feature_grad=grad, **(dict(adam=dict(m=a, v=b, t0=t)) if adam else dict(momentum=0.9, velocity=a)))
            t += k
        return x, a, b, grad

    for adam in (False, True):
        two, ones = run((2,), adam), run((1, 1), adam)
        assert all(torch.equal(u, v) for u, v in zip(two, ones))
        assert two[3].abs().max() > 0
