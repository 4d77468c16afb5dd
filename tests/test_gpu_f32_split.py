"""Float32 path, whose operands enter the matrix cores as three bfloat16 parts except on grids of few tiles: every number of position tiles per block, odd runs of
eight channels (half a fragment of sixteen), the ends of the float32 range, and what an infinite feature reaches; the weight gradients
by themselves."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2003_10735_amd as st
import workloads as WL
from gpu_util import to_dev_features

pytestmark = pytest.mark.gpu


# tiles of 32 positions per block for c1 / c2 output channels: 1 (64 input channels), 2, 3, 4, 5 in turn; then grids of few tiles, on the
# float32 instruction: wavefronts without an item, with one to three, and more than are on their way at once; 256 tiles and 260
@pytest.mark.parametrize("h,w,c_in,c1,c2", [(11, 29, 64, 64, 24), (60, 107, 24, 64, 40), (45, 80, 72, 128, 128), (60, 107, 16, 128, 104),
                                            (68, 120, 88, 128, 128),
                                            (11, 29, 8, 40, 24), (11, 29, 104, 128, 56), (62, 126, 24, 32, 32), (63, 126, 24, 32, 32)])
def test_split_products_are_as_good_as_float32(h, w, c_in, c1, c2):
    """Logits, gradient of every parameter block and feature gradient of one step against the oracle in float64, 2-norm.  Each sum
    adds up to 9 * 128 products that are right to 2^-24 (2^-27.5 in the mean) in float32: 1e-6 for the logits, three times what the float32
    instructions show.  Backward one activation in a million changes sign with the last bit, which moves a gradient by one
    position's share (1 / 319 of it at the smallest size) and elements of the feature gradient as a whole."""
    wl = WL.small_variant(WL.WORKLOADS["tiny"], h=h, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=9, steps=1, lr=1.0, n_sites=20)
    f, lab, p = WL.make_features(wl), WL.make_labels(wl), WL.make_head_params(wl)
    d, fd, f64 = st.HeadDesc.of(wl), to_dev_features(wl, f), WL.features_as_f64(wl, f)
    pt = torch.from_numpy(p).cuda()
    z = torch.empty((1, 9, h, w), dtype=torch.float32, device="cuda")
    st.st_head_forward(d, fd, pt, z, None)
    zo, _ = O.head_forward(O.desc_of(wl), f64, p.astype(np.float64), want_pred=False)
    assert np.linalg.norm(z.cpu().numpy() - zo) < 1e-6 * np.linalg.norm(zo)
    df = torch.zeros((1, c_in, h, w), dtype=torch.float32, device="cuda")
    st.st_partial_distill(d, fd, torch.from_numpy(lab).cuda(), pt, 1, 1.0, feature_grad=df)
    _, grad, df_o = O.feature_grad(O.desc_of(wl), f64, lab, p.astype(np.float64))
    step = p.astype(np.float64) - pt.cpu().numpy()               # lr = 1: the gradient, rounded where the new weight is
    for name, sl in WL.param_slices(wl).items():
        rounding = 2.0 ** -24 * np.linalg.norm(p[sl])
        assert np.linalg.norm(step[sl] - grad[sl]) < 1e-4 * np.linalg.norm(grad[sl]) + rounding, name
    assert np.linalg.norm(df.cpu().numpy() - df_o) < 1e-3 * np.linalg.norm(df_o)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_infinite_features_reach_what_they_reach_in_float32(value):
    """Two 3x3 layers see two cells in every direction: beyond them the logits are those of the finite frame, bit for bit; within,
    infinities and NaN lie where float32 arithmetic has them (a ReLU of NaN is 0; the second layer's weights are positive and the
    classifier's of one sign per class, so that infinities get through).  8 input channels: the other half of a fragment is the
    zeros in front of the buffer."""
    wl = WL.small_variant(WL.WORKLOADS["tiny"], h=12, w=40, c_in=8, c1=24, c2=40, n_classes=5, n_sites=9)
    f, p, sl = WL.make_features(wl), WL.make_head_params(wl), WL.param_slices(wl)
    p[sl["W2"]] = np.abs(p[sl["W2"]])
    p[sl["W3"]] = (np.abs(p[sl["W3"]]).reshape(5, 40) * np.array([1, -1, 1, -1, 1])[:, None]).reshape(-1)
    d, pd, zs = st.HeadDesc.of(wl), torch.from_numpy(p.astype(np.float32)).cuda(), []
    for bad in (False, True):
        if bad:
            f = f.copy()
            f[0, 3, 5, 17] = value
        z = torch.empty((1, 5, 12, 40), dtype=torch.float32, device="cuda")
        st.st_head_forward(d, torch.from_numpy(f).cuda(), pd, z, None)
        zs.append(z.cpu().numpy())
    near = np.zeros((12, 40), dtype=bool)
    near[3:8, 15:20] = True
    np.testing.assert_array_equal(zs[0][:, :, ~near], zs[1][:, :, ~near])
    x, shapes = f.astype(np.float64), (("W1", (24, 8, 3, 3)), ("W2", (40, 24, 3, 3)), ("W3", (5, 40, 1, 1)))
    with np.errstate(invalid="ignore"):
        for i, (name, shape) in enumerate(shapes):
            x = O.conv_fwd(x, p[sl[name]].astype(np.float64).reshape(shape), p[sl["b%d" % (i + 1)]].astype(np.float64))
            x = np.fmax(x, 0.0) if i < 2 else x
    np.testing.assert_array_equal(np.where(np.isfinite(zs[1]), 0, zs[1]), np.where(np.isfinite(x), 0, x))
    assert np.isinf(x).any() == (value == float("inf"))


# powers of two on the features, W1, W2 and W3; what they are compared with; whether the sums stay finite with their operands scaled,
# so that the result is the same bit for bit; blocks of the parameters rounded to multiples of 2^-16 (exact as subnormals)
ENDS = [((-112, 60, 52, 0), (0, 0, 0, 0), "z", ""),           # features whose last bits lie below 2^-133
        ((0, -100, 50, 50), (0, 0, 0, 0), "z", ""),           # weights of layer 1, activations behind it
        ((0, 0, 40, -95), (0, 0, 0, -40), "df", ""),          # gradients (the logits are nothing against the zero biases)
        ((126, -126, 0, 0), (0, 0, 0, 0), "", "W1"),          # features up to 3.4e38, beyond the largest bfloat16
        ((-110, 110, 0, 0), (0, 0, 0, 0), "", ""),            # weights
        ((0, 0, -126, 126), (0, 0, 0, 0), "", "W2")]          # gradients


@pytest.mark.parametrize("h,w,c_in,c1,c2", [(11, 29, 8, 40, 24), (11, 29, 64, 64, 24), (45, 80, 72, 128, 104)])
@pytest.mark.parametrize("powers,plain,same,rounded", ENDS)
def test_convolutions_at_the_ends_of_the_float32_range(powers, plain, same, rounded, h, w, c_in, c1, c2):
    """Powers of two on the operands are powers of two on the results, as in float32: bit for bit where no sum of scaled
    products overflows, else (those sums are formed by the float32 instruction, in another order) as far as float32 sums of
    9 * 128 terms lie apart, through the softmax for the feature gradient.  Parts cut off below 2^-133, or an operand taken for infinite,
    cost 2e-6 or everything."""
    wl = WL.small_variant(WL.WORKLOADS["tiny"], h=h, w=w, c_in=c_in, c1=c1, c2=c2, n_classes=9, steps=1, lr=0.0, n_sites=20)
    rng, sl = np.random.default_rng(h), WL.param_slices(wl)
    x = (rng.uniform(0.25, 3.9999, (1, c_in, h, w)) * (rng.random((1, c_in, h, w)) < 0.5)).astype(np.float32)
    lab, p0 = torch.from_numpy(WL.make_labels(wl)).cuda(), WL.make_head_params(wl).astype(np.float32)
    for b in ("b1", "b2", "b3"):
        p0[sl[b]] = 0.0
    p0[sl["W3"]] = np.clip(p0[sl["W3"]], -1, 1)
    if rounded:
        p0[sl[rounded]] = np.round(p0[sl[rounded]] * 2.0 ** 16) * 2.0 ** -16
    res = []
    for a, b, c, d in (plain, powers):
        p = p0.astype(np.float64)
        for block, e in (("W1", b), ("W2", c), ("W3", d)):
            p[sl[block]] *= 2.0 ** e
        fd, pd = torch.from_numpy((x * 2.0 ** float(a)).astype(np.float32)).cuda(), torch.from_numpy(p.astype(np.float32)).cuda()
        z = torch.empty((1, 9, h, w), dtype=torch.float32, device="cuda")
        st.st_head_forward(st.HeadDesc.of(wl), fd, pd, z, None)
        df = torch.zeros((1, c_in, h, w), dtype=torch.float32, device="cuda")
        st.st_partial_distill(st.HeadDesc.of(wl), fd, lab, pd, 1, 0.0, feature_grad=df)
        res.append((z.cpu().numpy() * 2.0 ** -(a + b + c + d), df.cpu().numpy() * 2.0 ** -(b + c + d)))
    (z0, df0), (z1, df1) = res
    assert np.linalg.norm(z0) > 0 and np.linalg.norm(df0) > 0
    if same == "z":
        np.testing.assert_array_equal(z1, z0)
    elif same == "df":
        np.testing.assert_array_equal(df1, df0)
    else:
        assert np.linalg.norm(z1 - z0) < 1e-6 * np.linalg.norm(z0)
    if powers[1] >= -100:      # (else the feature gradient is subnormal)
        assert np.linalg.norm(df1 - df0) < 1e-5 * np.linalg.norm(df0)


def _identity_layers(h, w, c, powers=(0, 0, 0, 0), one_sign=False):
    """One step whose 3x3 layers hand their input through, features and layers times powers of two that cancel in the logits: the feature
    gradient is then both layers' dY exactly, but for its power.  Returns features, dY and the weight gradients without their powers."""
    C = 2 if one_sign else 9
    wl = WL.small_variant(WL.WORKLOADS["tiny"], h=h, w=w, c_in=c, c1=c, c2=c, n_classes=C, steps=1, lr=0.0, n_sites=20)
    rng, sl = np.random.default_rng(h), WL.param_slices(wl)
    x = (rng.uniform(0.25, 3.9999, (1, c, h, w)) * (rng.random((1, c, h, w)) < 0.5)).astype(np.float32)
    lab = np.zeros((1, 8 * h, 8 * w), np.int32) if one_sign else WL.make_labels(wl)
    a, b1, b2, b3 = (2.0 ** float(e) for e in powers)
    p = np.zeros(WL.make_head_params(wl).size)
    eye = np.zeros((c, c, 9))
    eye[np.arange(c), np.arange(c), 4] = 1.0
    w3 = rng.normal(0, (2.0 / c) ** 0.5, (C, c)).astype(np.float32).astype(np.float64)
    if one_sign:
        w3 = np.abs(w3) * np.array([-1.0, 1.0])[:, None]
    p[sl["W1"]], p[sl["W2"]], p[sl["W3"]] = (eye * b1).reshape(-1), (eye * b2).reshape(-1), (w3 * b3).reshape(-1)
    fd, pd = torch.from_numpy((x * a).astype(np.float32)).cuda(), torch.from_numpy(p.astype(np.float32)).cuda()
    v, df = torch.zeros_like(pd), torch.zeros_like(fd)
    st.st_partial_distill(st.HeadDesc.of(wl), fd, torch.from_numpy(lab).cuda(), pd, 1, 0.0, momentum=0.9, velocity=v, feature_grad=df)
    v = v.cpu().numpy().astype(np.float64)
    return (x[0].astype(np.float64), df.cpu().numpy()[0].astype(np.float64) / (b3 * b2 * b1),
            v[sl["W1"]].reshape(c, c * 9) / (a * b2 * b3), v[sl["W2"]].reshape(c, c * 9) / (a * b1 * b3))


def _weight_gradient(x, dy):
    c = x.shape[0]
    return dy.reshape(c, -1) @ torch.nn.functional.unfold(torch.from_numpy(x)[None], 3, padding=1)[0].numpy().T


# float32 instruction: 11, 42 and 156 units of 8 positions, an odd number of a wavefront and wavefronts without any; split: 44, 259 and 560
# units of 16; channels that leave 8 of a tile's 32, half tiles and whole ones
@pytest.mark.parametrize("h,w,c", [(9, 6, 8), (12, 20, 104), (24, 40, 64), (20, 30, 168), (45, 80, 104), (68, 120, 40)])
def test_weight_gradients_alone_are_as_good_as_float32(h, w, c):
    """Against float64 sums of the same dY and features, 2-norm.  The float32 instructions show 6e-8 to 3e-7, one missing product of
    parts 1.2e-6 and more (test_split_products.py).  Sums do not shift to one side either: an MFMA that adds a product far below its
    accumulator cuts it off downwards, which showed as 1.4e-8 to 1.2e-7 of the elements' sum; rounded to nearest, the mean of 9 c^2 errors is
    two orders below their size."""
    x, dy, g1, g2 = _identity_layers(h, w, c)
    ref = _weight_gradient(x, dy)
    for got in (g1, g2):
        err = got - ref
        assert np.linalg.norm(err) < 6e-7 * np.linalg.norm(ref)
        if c >= 40:
            assert abs(err.sum()) < 6e-9 * np.abs(ref).sum()


# powers of two on the features, W1, W2 and W3, with sum 0; whether all sums stay finite with their operands scaled (bit for bit the same)
@pytest.mark.parametrize("powers,same", [((-112, 60, 52, 0), True),       # features whose last bits lie below 2^-133
                                         ((95, 0, 0, -95), True),         # gradients
                                         ((126, -63, 0, -63), False),     # features up to 3.4e38, beyond the largest bfloat16
                                         ((-115, 0, 0, 115), False)])     # gradients
@pytest.mark.parametrize("h,w,c", [(13, 21, 40), (34, 54, 104)])
def test_weight_gradients_at_the_ends_of_the_float32_range(powers, same, h, w, c):
    _, _, p1, p2 = _identity_layers(h, w, c)
    _, _, g1, g2 = _identity_layers(h, w, c, powers)
    for got, plain in ((g1, p1), (g2, p2)):
        if same:
            np.testing.assert_array_equal(got, plain)
        else:
            assert np.linalg.norm(got - plain) < 1e-6 * np.linalg.norm(plain)


@pytest.mark.parametrize("h,w,c", [(13, 21, 40), (34, 54, 104)])
def test_weight_gradients_beyond_the_float32_range_are_infinite(h, w, c):
    """Finite operands of one sign whose sums exceed the largest float32: infinite, as a float32 sum is, and not NaN."""
    powers = (100, -140, 20, 20)
    x, dy, g1, g2 = _identity_layers(h, w, c, powers, one_sign=True)
    ref = _weight_gradient(x, dy)
    beyond = ref * 2.0 ** 140 > 1.01 * float(np.finfo(np.float32).max)
    assert beyond.any() and np.all(np.isposinf(g1[beyond])) and not np.isnan(g1).any()
    assert np.linalg.norm(g2 - ref) < 6e-7 * np.linalg.norm(ref)
