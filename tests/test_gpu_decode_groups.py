"""The anchor decoder's forward around the sizes of its groups (16 anchors to
a wavefront, 65536 to a round of the launch). Anchors do not depend on one
another, so decoding them in pieces of any sizes gives the same bits; a piece
of 1000 is compared with the oracle elsewhere."""
import pytest
import torch

from paper_2601_19489_amd import _lib, scenes
from paper_2601_19489_amd.anchors import ANCHOR_NAMES, CHILD_NAMES, MLP_NAMES, AnchorDecoder, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('cuts', [(15, 1, 16), (17, 15), (33, 4063), (65536, 1), (65521, 1000, 32)])
def test_pieces_decode_to_the_same_bits(cuts):
    A = sum(cuts)
    a = to_device(scenes.anchor_cloud(A, seed=A), ANCHOR_NAMES)
    m = to_device(scenes.decoder_mlp(seed=3), MLP_NAMES)
    cam = _lib.camera(scenes.look_at_camera((-0.4, 0.2, -3.5), (0, 0, 0), 320, 240))
    whole = AnchorDecoder(A)
    whole.decode(a, m, cam)
    lo = 0
    for n in cuts:
        part = AnchorDecoder(n)
        part.decode({k: v[:, lo:lo + n].contiguous() for k, v in a.items()}, m, cam)
        for k in CHILD_NAMES:
            w, p = whole.children[k], part.children[k]
            w = w.reshape(-1, _lib.ANCHOR_CHILDREN, A)[:, :, lo:lo + n]
            assert torch.isfinite(p).all()
            assert torch.equal(w, p.reshape(-1, _lib.ANCHOR_CHILDREN, n)), (k, lo, n)
        lo += n
