"""The decoder's three heads are independent: hidden units that overflow to
infinity in one change none of the bits of what the other two put out, nor of
the other heads' weight gradients."""
import pytest
import torch

from paper_2601_19489_amd import _lib, scenes
from paper_2601_19489_amd.anchors import ANCHOR_NAMES, MLP_NAMES, AnchorDecoder, to_device

pytestmark = pytest.mark.gpu

OF_HEAD = (('opacity_logits',), ('sh',), ('log_scales', 'quats'))  # opacity, colour, covariance
OUT_ROWS = ((0, 10), (10, 40), (40, 110))


@pytest.mark.parametrize('A', [1, 16, 333])
@pytest.mark.parametrize('head', [0, 1, 2])
def test_infinite_hidden_units_stay_in_their_head(head, A):
    a = to_device(scenes.anchor_cloud(A, seed=3), ANCHOR_NAMES)
    m = to_device(scenes.decoder_mlp(seed=4), MLP_NAMES)
    cam = _lib.camera(scenes.look_at_camera((0.5, -0.3, -4.0), (0, 0, 0), 320, 240))
    over = {k: v.clone() for k, v in m.items()}
    over['b1'][32 * head + 5:32 * head + 9] = 3.4e38       # infinite in BF16
    g = torch.Generator(device='cuda').manual_seed(A)
    res = []
    for w in (m, over):
        dec = AnchorDecoder(A)
        ch = dec.decode(a, w, cam)
        dch = {k: torch.randn(v.shape, generator=g.manual_seed(A), device='cuda')
               for k, v in ch.items()}
        da, dm = dec.backward(a, w, cam, dch)
        torch.cuda.synchronize()
        res.append((ch, da, dm))
    (ch0, da0, dm0), (ch1, da1, dm1) = res
    assert torch.equal(ch0['means'], ch1['means'])
    assert torch.equal(da0['offsets'], da1['offsets'])
    for h in range(3):
        if h == head:
            assert not torch.equal(ch0[OF_HEAD[h][0]], ch1[OF_HEAD[h][0]])
            continue
        for k in OF_HEAD[h]:
            assert torch.isfinite(ch0[k]).all()
            assert torch.equal(ch0[k], ch1[k]), k
        lo, hi = OUT_ROWS[h]
        for k, rows in (('w1', slice(32 * h, 32 * h + 32)), ('b1', slice(32 * h, 32 * h + 32)),
                        ('w2', slice(lo, hi)), ('b2', slice(lo, hi))):
            assert torch.equal(dm0[k][rows], dm1[k][rows]), k
