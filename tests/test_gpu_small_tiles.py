"""Half and quarter tiles of the bfloat16 convolutions: a frame alone, whose layers run on tiles of 32 or 64 positions, gives bit for bit
what it gives in a batch of copies, as many as it takes for all layers to run on tiles of 128 positions or the wide ones -- logits, and the
gradient of the features, of which the batch has one n-th (one pixel count for all frames; n is a power of two, so that it is exact)."""
import pytest

import paper_2003_10735_amd as st

pytestmark = pytest.mark.gpu


def blocks(n, h, w, bm, cout):
    """Blocks of a launch on tiles of bm positions x 64 channels: the small tiles run where there are 256 or fewer."""
    return -(-n * (h + 2) * (-(-(w + 2) // 8) * 8) // bm) * -(-cout // 64)


# heads whose layers alone run tiles of 32 positions, of 64, and of both; one and a few tiles, ends inside a tile (1400 and 2480 positions are
# no multiple of 32), the fewest stages, padded channels; on tiles of 32, whose slabs rotate three stages at a time, one to seven turns
@pytest.mark.parametrize("h,w,c_in,c1,c2,C", [(1, 1, 64, 64, 64, 3), (33, 35, 64, 64, 64, 7), (29, 78, 64, 64, 128, 6), (33, 38, 64, 128, 64, 11), (2, 6, 64, 128, 64, 9), (2, 7, 128, 64, 128, 12), (6, 22, 192, 64, 64, 19),
                                              (16, 24, 64, 64, 64, 32), (30, 53, 256, 128, 128, 19), (45, 80, 256, 128, 128, 5),
                                              (60, 107, 96, 128, 128, 9), (68, 118, 64, 64, 128, 21), (9, 22, 320, 64, 64, 4), (5, 14, 448, 384, 64, 8)])
def test_a_frame_alone_is_a_frame_of_a_batch(h, w, c_in, c1, c2, C):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(h * 1000 + w)
    f = torch.randn((1, c_in, h, w), generator=gen, device="cuda").clamp(min=0).bfloat16()
    lab = torch.randint(0, C, (1, 8 * h, 8 * w), generator=gen, device="cuda", dtype=torch.int32)
    params = torch.cat([torch.randn(r * k, generator=gen, device="cuda") * (2.0 / k) ** 0.5
                        for r, k in ((c1, 9 * c_in), (1, c1), (c2, 9 * c1), (1, c2), (C, c2), (1, C))])
    copies = 8
    while blocks(copies, h, w, 64, 64) <= 256:
        copies *= 2
    assert any(blocks(1, h, w, bm, c) <= 256 for bm in (32, 64) for c in (c1, c2)) and blocks(copies, h, w, 64, min(c_in, c1, c2)) > 256
    out = []
    for n in (1, copies):
        d = st.HeadDesc(n, c_in, h, w, c1, c2, C, feat_dtype=st.ST_BF16, compute=st.ST_COMPUTE_BF16)
        ws = torch.zeros(st.st_workspace_bytes(d), dtype=torch.uint8, device="cuda")
        fs, ls = f.repeat(n, 1, 1, 1), lab.repeat(n, 1, 1)
        z = torch.empty((n, C, h, w), device="cuda")
        st.st_head_forward(d, fs, params, logits_lowres=z, workspace=ws)
        grad = torch.zeros((n, c_in, h, w), device="cuda")
        st.st_partial_distill(d, fs, ls, params.clone(), 1, 0.0, workspace=ws, feature_grad=grad)
        torch.cuda.synchronize()
        out.append((z, grad * n))
    assert out[0][1].abs().max() > 0
    for alone, batch in zip(*out):
        assert torch.equal(alone.expand_as(batch), batch)
