"""Splats whose colour or depth is not finite, in the compositing kernels.

A pixel's sums take a splat's colour and depth where the pixel blends it and
nowhere else, so a pixel that blends none of the odd splats has the bits that it
has without them, stopped pixels in front of one included; a pixel that blends
one is not finite. In the backward the odd splats reach, through the pixels that
blend them, the gradients of the splats that those pixels blend, and no other.

Hand-built lists; which pixels blend an odd splat comes from a render in which
those splats alone have colour, which splats a set of pixels blends from the
Eq. 4 counts of that mask."""
import numpy as np
import pytest
import torch

from paper_2601_19489_amd import _lib, scenes

from test_gpu_cells import _lists

pytestmark = pytest.mark.gpu

NAMES = ('means', 'log_scales', 'quats', 'opacity_logits', 'sh')
BG = (0.25, 0.5, 0.125)


class Scene:
    def __init__(self, tile, across, opaque=False):
        self.W, self.H = across * tile - 3, across * tile - 5
        self.cam = _lib.camera(scenes.look_at_camera((0, 0, -4), (0, 0, 0), self.W, self.H,
                                                     tile=tile), tile)
        rec, vals, ranges = _lists(across, across, tile, seed=5 + tile)
        rng = np.random.default_rng(17)
        self.n = len(rec)
        if opaque:  # pixels stop, and odd splats lie behind the stop
            o = rng.uniform(0.6, 0.95, self.n).astype(np.float32)
            rec[:, 6], rec[:, 5] = o, 2.0 * np.log(255.0 * o)
        dev = lambda x: torch.as_tensor(x, device='cuda').contiguous()
        self.rec, self.vals = dev(rec), dev(vals.view(np.int32))
        self.ranges = dev(ranges.view(np.int32))
        self.odd = dev(rng.random(self.n) < 0.03)
        bad = rng.choice([np.nan, np.inf, -np.inf], size=(self.n, 4)).astype(np.float32)
        bad[rng.random((self.n, 4)) < 0.4] = 0.5      # some components stay finite
        bad[:, 0] = np.nan
        self.bad = dev(bad)
        self.dI = dev((rng.standard_normal((3, self.H, self.W)) * 1e-2).astype(np.float32))
        self.dD = dev((rng.standard_normal((self.H, self.W)) * 1e-3).astype(np.float32))
        self.p = dict(means=torch.zeros((3, self.n), device='cuda'),
                      log_scales=torch.zeros((3, self.n), device='cuda'),
                      quats=torch.zeros((4, self.n), device='cuda'),
                      opacity_logits=torch.zeros(self.n, device='cuda'),
                      sh=torch.zeros((1, 3, self.n), device='cuda'))
        self.p['means'][2] = 3.0
        self.p['quats'][0] = 1.0
        self.n_tiles = across * across

    def colours(self, rgb, z, odd):
        """The records with the odd splats' colour and depth replaced."""
        r = self.rec.clone()
        r[self.odd, 8:11], r[self.odd, 7] = rgb, z
        if odd:
            r[self.odd, 8:11], r[self.odd, 7] = self.bad[self.odd, :3], self.bad[self.odd, 3]
        return r

    def images(self):
        return dict(image=torch.empty((3, self.H, self.W), device='cuda'),
                    depth=torch.empty((self.H, self.W), device='cuda'),
                    T_final=torch.empty((self.H, self.W), device='cuda'),
                    n_contrib=torch.empty((self.H, self.W), dtype=torch.int32, device='cuda'))

    def render(self, rec, bg=BG):
        out = self.images()
        _lib.gs_render_fwd(rec, self.n, self.vals, self.ranges, self.cam, bg, out['image'],
                           out['depth'], out['T_final'], out['n_contrib'])
        return out

    def tainted(self):
        """The pixels that blend an odd splat, and the splats that such a pixel blends."""
        r = self.rec.clone()
        r[:, 7:11] = 0.0
        r[self.odd, 8] = 1.0
        pixels = self.render(r, (0, 0, 0))['image'][0] > 0
        score = torch.zeros(self.n, dtype=torch.int32, device='cuda')
        _lib.gs_split_score(self.rec, self.n, self.vals, self.ranges, self.cam,
                            pixels.to(torch.uint8).contiguous(), score)
        return pixels, score > 0

    def backward(self, rec, out, order):
        g2 = torch.empty((self.n, _lib.GRAD2D_COMPONENTS), dtype=torch.float64, device='cuda')
        grads = {k: torch.empty_like(v) for k, v in self.p.items()}
        o = torch.empty(2 * self.n_tiles, dtype=torch.int32, device='cuda') if order else None
        _lib.gs_render_bwd(_lib.gaussians(*(self.p[k] for k in NAMES)), self.n, 0, self.cam, rec,
                           self.vals, self.ranges, BG, out['T_final'], out['n_contrib'], self.dI,
                           self.dD, g2, _lib.gaussians(*(grads[k] for k in NAMES)), tile_order=o)
        return g2


def _check_forward(sc, got, want, pixels):
    calm = ~pixels
    assert 0.05 < calm.float().mean() < 0.999 and pixels.any()
    for k in ('T_final', 'n_contrib'):
        assert torch.equal(got[k], want[k]), k
    for k in ('image', 'depth'):
        g, w = got[k], want[k]
        assert torch.equal(g[..., calm], w[..., calm]), k
    assert torch.isnan(got['image'][0][pixels]).all()   # every odd splat's red is NaN


@pytest.mark.parametrize('opaque', [False, True])
@pytest.mark.parametrize('tile,across,px', [(8, 24, 1), (16, 24, 1), (16, 24, 2), (16, 24, 4),
                                            (32, 12, 1), (32, 12, 2), (32, 12, 4)])
def test_forward_takes_odd_colours_where_they_are_blended(tile, across, px, opaque):
    sc = Scene(tile, across, opaque)
    keep = _lib.gs_get_tuning()
    _lib.gs_set_tuning(fwd_px=px)
    try:
        pixels, _ = sc.tainted()
        want = sc.render(sc.colours(0.5, 0.5, odd=False))
        got = sc.render(sc.colours(0.5, 0.5, odd=True))
        torch.cuda.synchronize()
    finally:
        _lib.gs_set_tuning(fwd_px=keep['fwd_px'])
    assert not opaque or (want['T_final'] < 0.01).any()
    _check_forward(sc, got, want, pixels)


def test_checkpointed_forward_takes_odd_colours_where_they_are_blended():
    sc = Scene(16, 24)
    pixels, _ = sc.tainted()
    nbk = 10                                            # 257 entries at most
    res = []
    for odd in (False, True):
        out = sc.images()
        ck = torch.zeros((sc.n_tiles, nbk, 5, 256), device='cuda')
        ovf = torch.zeros(1, dtype=torch.int32, device='cuda')
        _lib.gs_render_fwd_ckpt(sc.colours(0.5, 0.5, odd), sc.n, sc.vals, sc.ranges, sc.cam, BG,
                                out['image'], out['depth'], out['T_final'], out['n_contrib'], ck,
                                nbk, ovf)
        res.append((out, ck, int(ovf.item())))
    (want, ck0, o0), (got, ck1, o1) = res
    assert o0 == 0 and o1 == 0
    _check_forward(sc, got, want, pixels)
    assert torch.equal(ck0[:, :, 0], ck1[:, :, 0])      # the transmittances
    same = (ck0 == ck1) | ~torch.isfinite(ck1)
    assert same.all() and torch.isnan(ck1).any()


@pytest.mark.parametrize('order', [False, True])
@pytest.mark.parametrize('tile,across,px', [(8, 24, 1), (16, 24, 1), (16, 24, 2), (16, 24, 4),
                                            (16, 70, 4), (32, 12, 2), (32, 12, 4)])
def test_backward_takes_odd_colours_where_they_are_blended(tile, across, px, order):
    # with an order: the long walks by whole workgroups, of 8 wavefronts, and
    # of 4 with more than 4096 regions (70 x 70 tiles)
    sc = Scene(tile, across)
    keep = _lib.gs_get_tuning()
    _lib.gs_set_tuning(bwd_px=px)
    try:
        _, reached = sc.tainted()
        calm = sc.colours(0.5, 0.5, odd=False)
        out = sc.render(calm)
        want = sc.backward(calm, out, order)
        got = sc.backward(sc.colours(0.5, 0.5, odd=True), out, order)
        torch.cuda.synchronize()
    finally:
        _lib.gs_set_tuning(bwd_px=keep['bwd_px'])
    free = ~reached
    assert free.float().mean() > 0.05 and bool((sc.odd & reached).any())
    assert want[free].abs().max() > 0
    # a region's FP32 sums add exact zeros for the other pixels; the FP64 adds
    # across the tiles' regions come in any order (53 bits, a few adds)
    assert torch.isfinite(got[free]).all()
    torch.testing.assert_close(got[free], want[free], rtol=1e-13,
                               atol=1e-13 * float(want.abs().max()))
    assert torch.isnan(got[reached]).any()
