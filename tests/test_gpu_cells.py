"""Cells that a splat does not reach, and the groups and batches of list
entries, in the forward and the backward.

The compositing kernels leave a splat out of the blocks of pixels it cannot
blend in and walk what is left a few entries at a time; long lists are
worked on by four wavefronts in the backward. Hand-built lists with lengths
around every one of those sizes (groups of 2 and 4, blocks of 32, batches of
64 and 256, the length above which a region goes to a whole workgroup), of splats from less than
a pixel wide to long and thin, many ending at a cell's edge, against the
oracle: n_contrib is equal wherever no stop test is near, the image is within
1e-4, the 2D gradients within 1e-3 (as for every parity test)."""
import numpy as np
import pytest
import torch

from oracle import densify as oden
from oracle import render as orender
from paper_2601_19489_amd import _lib, scenes

from _parity import assert_grads_close, exclusions, gpu_splat_fields

pytestmark = pytest.mark.gpu

LENGTHS = (0, 1, 2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257)


def _lists(tiles_x, tiles_y, tile, seed):
    rng = np.random.default_rng(seed)
    lens = [LENGTHS[i % len(LENGTHS)] if i % 7 == 0 else LENGTHS[i % 10]
            for i in range(tiles_x * tiles_y)]
    ranges = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint32)
    n = int(ranges[-1])
    tid = np.repeat(np.arange(len(lens)), lens)
    ox, oy = tid // tiles_y * tile, tid % tiles_y * tile
    o = rng.uniform(0.02, 0.25, n)
    t = 2.0 * np.log(255.0 * o)
    s1 = np.exp(rng.uniform(np.log(0.4), np.log(8.0), n))           # axes in pixels
    s2 = s1 * np.exp(-rng.uniform(0.0, 2.8, n))                     # condition number up to 270
    th = rng.uniform(0, np.pi, n)
    l1, l2 = 1.0 / (s1 * s1), 1.0 / (s2 * s2)
    a = l1 * np.cos(th) ** 2 + l2 * np.sin(th) ** 2
    c = l1 * np.sin(th) ** 2 + l2 * np.cos(th) ** 2
    b = (l1 - l2) * np.cos(th) * np.sin(th)
    u = ox + rng.uniform(-0.3 * tile, 1.3 * tile, n)
    v = oy + rng.uniform(-0.3 * tile, 1.3 * tile, n)
    # a third end within a hair of a pixel centre next to a cell's edge
    edge = rng.random(n) < 0.33
    reach = np.sqrt(t * a / (a * c - b * b))                        # half height of Q = t
    row = 4 * rng.integers(0, max(tile // 4, 1), n)
    v = np.where(edge, oy + row - 0.5 - reach + rng.uniform(-0.05, 0.05, n), v)
    rec = np.zeros((n, _lib.SPLAT_FLOATS), np.float32)
    for k, x in enumerate((u, v, a, b, c, t, o)):
        rec[:, k] = x
    rec[:, 7] = rng.uniform(2.0, 5.0, n)
    rec[:, 8:11] = rng.uniform(0.0, 1.0, (n, 3))
    # every list entry is its own Gaussian, in shuffled order
    order = rng.permutation(n)
    inv = np.empty(n, np.int64)
    inv[order] = np.arange(n)
    return rec[order], inv.astype(np.uint32), ranges


@pytest.mark.parametrize('tile,across,fwd_px,bwd_px', [
    (16, 24, 1, 4), (16, 24, 2, 2), (16, 24, 4, 1), (8, 24, 1, 1), (32, 12, 1, 4), (32, 12, 2, 2)])
def test_lists_around_every_batch_size(tile, across, fwd_px, bwd_px):
    W, H = across * tile - 3, across * tile - 5         # ragged last cells
    cam = scenes.look_at_camera((0, 0, -4), (0, 0, 0), W, H, tile=tile)
    ccam = _lib.camera(cam, tile)
    rec, vals, ranges = _lists(across, across, tile, seed=tile + fwd_px)
    n = len(rec)
    dev = lambda x: torch.as_tensor(x, device='cuda').contiguous()
    splats, dvals, dranges = dev(rec), dev(vals.view(np.int32)), dev(ranges.view(np.int32))
    image = torch.empty((3, H, W), device='cuda')
    depth, T_final = (torch.empty((H, W), device='cuda') for _ in range(2))
    n_contrib = torch.empty((H, W), dtype=torch.int32, device='cuda')
    rng = np.random.default_rng(tile)
    dI = (rng.standard_normal((3, H, W)) * 1e-2).astype(np.float32)
    dD = (rng.standard_normal((H, W)) * 1e-3).astype(np.float32)
    params = dict(means=torch.zeros((3, n), device='cuda'),
                  log_scales=torch.zeros((3, n), device='cuda'),
                  quats=torch.zeros((4, n), device='cuda'),
                  opacity_logits=torch.zeros(n, device='cuda'),
                  sh=torch.zeros((1, 3, n), device='cuda'))
    params['means'][2] = 3.0
    params['quats'][0] = 1.0
    grads = {k: torch.empty_like(x) for k, x in params.items()}
    names = ('means', 'log_scales', 'quats', 'opacity_logits', 'sh')
    order = torch.empty(2 * across * across, dtype=torch.int32, device='cuda')
    grad2d = torch.empty((n, _lib.GRAD2D_COMPONENTS), dtype=torch.float64, device='cuda')
    keep = _lib.gs_get_tuning()
    _lib.gs_set_tuning(fwd_px=fwd_px, bwd_px=bwd_px)
    try:
        _lib.gs_render_fwd(splats, n, dvals, dranges, ccam, (0, 0, 0), image, depth, T_final,
                           n_contrib)
        _lib.gs_render_bwd(_lib.gaussians(*(params[k] for k in names)), n, 0, ccam, splats, dvals,
                           dranges, (0, 0, 0), T_final, n_contrib, dev(dI), dev(dD), grad2d,
                           _lib.gaussians(*(grads[k] for k in names)), tile_order=order)
        torch.cuda.synchronize()
    finally:
        _lib.gs_set_tuning(fwd_px=keep['fwd_px'], bwd_px=keep['bwd_px'])
    sp = gpu_splat_fields(rec.astype(np.float64))
    sp['depth'] = sp['dval']
    out = orender.render(sp, cam, vals, ranges)
    calm = ~out['ambiguous']
    assert calm.mean() > 0.99
    got = n_contrib.cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got[calm], out['n_contrib'][calm])
    assert got.max() > 129
    assert np.abs(image.cpu().numpy() - out['image'])[:, calm].max() <= 1e-4
    want, clamp = orender.render_backward(sp, cam, vals, ranges, dI.astype(np.float64),
                                          dD.astype(np.float64))
    skip = exclusions(vals, ranges, cam, out, clamp, n)
    for k, nm in enumerate(orender.GRAD2D):
        assert_grads_close(grad2d.cpu().numpy().T[k], want[k], skip, 'grad2d.' + nm)


@pytest.mark.parametrize('tile,across', [(8, 24), (16, 24), (32, 12)])
def test_split_score_around_every_batch_size(tile, across):
    """Counts under a mask that leaves out whole cells, single pixels and
    (one column of tiles) everything: equal to the oracle's wherever no pixel's
    decision is uncertain, within that many pixels elsewhere."""
    W, H = across * tile - 3, across * tile - 5
    cam = scenes.look_at_camera((0, 0, -4), (0, 0, 0), W, H, tile=tile)
    rec, vals, ranges = _lists(across, across, tile, seed=3 + tile)
    n = len(rec)
    rng = np.random.default_rng(tile)
    mask = rng.random((H, W)) < 0.4
    cells = rng.random((-(-H // 8), -(-W // 8))) < 0.5
    mask &= np.kron(cells, np.ones((8, 8), bool))[:H, :W]
    mask[:, tile:2 * tile] = False
    dev = lambda x: torch.as_tensor(x, device='cuda').contiguous()
    score = torch.zeros(n, dtype=torch.int32, device='cuda')
    _lib.gs_split_score(dev(rec), n, dev(vals.view(np.int32)), dev(ranges.view(np.int32)),
                        _lib.camera(cam, tile), dev(mask.astype(np.uint8)), score)
    torch.cuda.synchronize()
    sp = gpu_splat_fields(rec.astype(np.float64))
    sp['depth'] = sp['dval']
    want, unc = oden.split_score(sp, cam, vals, ranges, mask)
    got = score.cpu().numpy().astype(np.int64)
    sure = unc == 0
    assert sure.mean() > 0.95 and want.sum() > 1000
    np.testing.assert_array_equal(got[sure], want[sure])
    assert np.all(np.abs(got[~sure] - want[~sure]) <= unc[~sure])
