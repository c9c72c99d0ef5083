"""The backward's walks of one region, at list lengths around every group and
batch size: one wavefront on its own (no tile order given), a workgroup of 8
(launches of up to 4096 regions) and one of 4 (more regions, and the batched
launch), against the oracle (relative 1e-3, as for every parity test) and
against each other.

Every list entry is its own Gaussian, and the three form a region's sums from
the same values in the same order. So with 16-pixel tiles, where a tile is one
region, the 2D gradients are the same bits; with 32-pixel tiles a Gaussian
takes up to four FP64 adds, in any order."""
import numpy as np
import pytest
import torch

from oracle import render as orender
from paper_2601_19489_amd import _lib, scenes

from _parity import assert_grads_close, exclusions, gpu_splat_fields
from test_gpu_cells import _lists

pytestmark = pytest.mark.gpu

NAMES = ('means', 'log_scales', 'quats', 'opacity_logits', 'sh')


def _walks(tile, across, depth, batched):
    W, H = across * tile - 3, across * tile - 5
    cam = scenes.look_at_camera((0, 0, -4), (0, 0, 0), W, H, tile=tile)
    ccam = _lib.camera(cam, tile)
    rec, vals, ranges = _lists(across, across, tile, seed=31 + tile)
    n = len(rec)
    dev = lambda x: torch.as_tensor(x, device='cuda').contiguous()
    splats, dvals, dranges = dev(rec), dev(vals.view(np.int32)), dev(ranges.view(np.int32))
    image = torch.empty((3, H, W), device='cuda')
    dep, T_final = (torch.empty((H, W), device='cuda') for _ in range(2))
    n_contrib = torch.empty((H, W), dtype=torch.int32, device='cuda')
    rng = np.random.default_rng(tile)
    dI = (rng.standard_normal((3, H, W)) * 1e-2).astype(np.float32)
    dD = (rng.standard_normal((H, W)) * 1e-3).astype(np.float32) if depth else None
    gI, gD = dev(dI), None if dD is None else dev(dD)
    z = lambda *s: torch.zeros(s, device='cuda')
    p = dict(means=z(3, n), log_scales=z(3, n), quats=z(4, n), opacity_logits=z(n), sh=z(1, 3, n))
    p['means'][2] = 3.0
    p['quats'][0] = 1.0
    grads = {k: torch.empty_like(x) for k, x in p.items()}
    gp, gg = (_lib.gaussians(*(d[k] for k in NAMES)) for d in (p, grads))
    _lib.gs_render_fwd(splats, n, dvals, dranges, ccam, (0, 0, 0), image, dep, T_final, n_contrib)
    res = {}
    for mode in ('one', 'order') + (('batched',) if batched else ()):
        g2 = torch.empty((n, _lib.GRAD2D_COMPONENTS), dtype=torch.float64, device='cuda')
        order = torch.empty(2 * across * across, dtype=torch.int32, device='cuda')
        if mode == 'batched':
            v = _lib.GsView()
            v.cam = ccam
            for k, t in (('splats', splats), ('vals', dvals), ('ranges', dranges),
                         ('T_final', T_final), ('n_contrib', n_contrib), ('dL_dimage', gI),
                         ('dL_ddepth', gD), ('grad2d', g2)):
                setattr(v, k, _lib._ptr(t))
            _lib.gs_render_bwd_batched(gp, n, 0, [v], (0, 0, 0),
                                       torch.zeros(1, dtype=torch.int32, device='cuda'), gg,
                                       tile_order=order)
        else:
            _lib.gs_render_bwd(gp, n, 0, ccam, splats, dvals, dranges, (0, 0, 0), T_final,
                               n_contrib, gI, gD, g2, gg,
                               tile_order=None if mode == 'one' else order)
        torch.cuda.synchronize()
        if mode != 'one':
            # regions longer than the rule's threshold, so the workgroups' walk runs
            work = np.sort(order[across * across:].cpu().numpy())[::-1]
            nt, regions = across * across, across * across * (tile // 16) ** 2
            limit = sum(int(work[nt * i // 8]) for i in (1, 3, 5, 7)) * regions // 12288
            assert (work > max(limit, 129)).any()
        res[mode] = g2
    return res, (rec, vals, ranges, cam, n, dI, dD)


def _same(res, tile):
    for mode, g2 in res.items():
        if tile == 16:
            assert torch.equal(g2, res['one']), mode
        else:
            torch.testing.assert_close(g2, res['one'], rtol=1e-13,
                                       atol=1e-13 * float(g2.abs().max()))


@pytest.mark.parametrize('depth', [True, False])
@pytest.mark.parametrize('tile,across', [(16, 24), (32, 12)])
def test_walks_match_the_oracle_and_each_other(tile, across, depth):
    res, (rec, vals, ranges, cam, n, dI, dD) = _walks(tile, across, depth, batched=True)
    _same(res, tile)
    sp = gpu_splat_fields(rec.astype(np.float64))
    sp['depth'] = sp['dval']
    out = orender.render(sp, cam, vals, ranges)
    want, clamp = orender.render_backward(sp, cam, vals, ranges, dI.astype(np.float64),
                                          None if dD is None else dD.astype(np.float64))
    skip = exclusions(vals, ranges, cam, out, clamp, n)
    for mode, g2 in res.items():
        for k, nm in enumerate(orender.GRAD2D):
            assert_grads_close(g2.cpu().numpy().T[k], want[k], skip, f'{mode} grad2d.{nm}')


@pytest.mark.parametrize('depth', [True, False])
@pytest.mark.parametrize('tile,across', [(16, 70), (32, 34)])
def test_four_wavefronts_to_a_workgroup(tile, across, depth):
    # 4900 and 4624 regions, more than 4096
    res, _ = _walks(tile, across, depth, batched=False)
    _same(res, tile)
