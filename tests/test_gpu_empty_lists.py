"""The backward where no pixel blends a splat: no list entry and no record is
read, so none has to be there, and the gradients are zero."""
import pytest
import torch

from paper_2601_19489_amd import _lib, scenes

pytestmark = pytest.mark.gpu

NAMES = ('means', 'log_scales', 'quats', 'opacity_logits', 'sh')


@pytest.mark.parametrize('batched', [False, True])
@pytest.mark.parametrize('order', [False, True])
@pytest.mark.parametrize('tile,px', [(8, 1), (16, 1), (16, 2), (16, 4), (32, 2), (32, 4)])
def test_backward_of_empty_lists_reads_no_records(tile, px, order, batched):
    n, W, H = 70, 5 * tile - 3, 3 * tile - 1
    cam = _lib.camera(scenes.look_at_camera((0, 0, -4), (0, 0, 0), W, H, tile=tile), tile)
    z = lambda *s, **k: torch.zeros(s, device='cuda', **k)
    p = dict(means=z(3, n), log_scales=z(3, n), quats=z(4, n), opacity_logits=z(n), sh=z(1, 3, n))
    p['quats'][0] = 1.0
    grads = {k: torch.full_like(v, 7.0) for k, v in p.items()}
    gp, gg = (_lib.gaussians(*(d[k] for k in NAMES)) for d in (p, grads))
    ranges, n_contrib = z(16, dtype=torch.int32), z(H, W, dtype=torch.int32)
    T_final, dI = torch.ones((H, W), device='cuda'), torch.ones((3, H, W), device='cuda')
    grad2d = torch.full((n, _lib.GRAD2D_COMPONENTS), 7.0, dtype=torch.float64, device='cuda')
    tile_order = z(2 * 15, dtype=torch.int32) if order else None
    keep = _lib.gs_get_tuning()
    _lib.gs_set_tuning(bwd_px=px)
    try:
        if batched:
            v = _lib.GsView()
            v.cam = cam
            for k, t in (('ranges', ranges), ('T_final', T_final), ('n_contrib', n_contrib),
                         ('dL_dimage', dI), ('grad2d', grad2d)):
                setattr(v, k, _lib._ptr(t))
            _lib.gs_render_bwd_batched(gp, n, 0, [v], (0, 0, 0), z(1, dtype=torch.int32), gg,
                                       tile_order=tile_order)
        else:
            _lib.gs_render_bwd(gp, n, 0, cam, None, None, ranges, (0, 0, 0), T_final, n_contrib,
                               dI, None, grad2d, gg, tile_order=tile_order)
        torch.cuda.synchronize()
    finally:
        _lib.gs_set_tuning(bwd_px=keep['bwd_px'])
    assert torch.count_nonzero(grad2d) == 0
    for k, v in grads.items():
        assert torch.count_nonzero(v) == 0, k
